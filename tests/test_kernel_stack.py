"""The kernels need no stack: the runtime allocates device memory, per queue, for one that does, at its first launch."""
import os

import paper_1512_02595_amd


def test_no_kernel_needs_memory_of_its_own():
    built = os.path.join(os.path.dirname(paper_1512_02595_amd.__file__), "libctc_mi355x.so")
    with open(built, "rb") as f:
        code = f.read()
    # the kernels' metadata, a MessagePack map each: a string of 27 bytes, then a number that is one byte if below 128
    key = b"\xbb.private_segment_fixed_size"
    sizes = [part[0] for part in code.split(key)[1:]]
    assert len(sizes) > 20 and not any(sizes)
