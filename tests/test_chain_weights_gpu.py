"""Every planner orders utterances by the same weight (chain_weight in ctc_internal.h), computed here by a small program: the host's, the one in the softmax launch of narrow
alphabets and the planning launch of wide ones and of many utterances, for batches in which frames times wavefronts gives another order.  The orders are read from the workspace."""
import os
import subprocess

import numpy as np
import pytest

from paper_1512_02595_amd import harness

from test_block_edges_gpu import batch_of

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <cstdio>
#include "ctc_internal.h"
int main()
{
    int crowded, best, folded, frames, L, repeats;
    while (std::scanf("%d %d %d %d %d %d", &crowded, &best, &folded, &frames, &L, &repeats) == 6) {
        // (the softmax launch's setup has no time to count every utterance's repeats)
        const bool logs = frames > ctc::kLinearMaxFrames || ctc::tight_fit(frames, L, folded ? 0 : repeats);
        const ctc::ChainForm form = ctc::chain_form((logs ? ctc::kUttLogDomain : 0) | (ctc::linear_two_pairs(L, crowded != 0) ? ctc::kUttTwoPairs : 0), best != 0);
        const int waves = form == ctc::ChainForm::kTwoPairs ? ctc::linear_plan2(L, crowded != 0).waves : ctc::plan_waves(L, crowded != 0).waves;
        std::printf("%lld\n", static_cast<long long>(ctc::chain_weight(frames, waves, form, crowded != 0)));
    }
}
"""


@pytest.fixture(scope="module")
def weights(tmp_path_factory):
    d = tmp_path_factory.mktemp("weights")
    (d / "weights.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_1512_02595_amd", "csrc"),
                    str(d / "weights.cpp"), "-o", str(d / "weights")], check=True)

    def ask(batch, best, folded):
        at, text = 0, ""
        for frames, L in zip(batch.input_lengths, batch.label_lengths):
            label = batch.flat_labels[at:at + L]
            at += L
            text += f"0 {int(best)} {int(folded)} {frames} {L} {int((label[1:] == label[:-1]).sum())}\n"
        return np.array(subprocess.run([str(d / "weights")], input=text, capture_output=True, text=True, check=True).stdout.split(), dtype=np.int64)
    return ask


# (uncrowded all; 600 utterances: more than the softmax launch plans for)
@pytest.mark.parametrize("how,A,B,longest,T", [("host", 29, 40, 520, 900), ("host", 90, 40, 520, 900), ("align", 90, 40, 520, 900), ("device", 29, 40, 520, 900), ("device", 90, 40, 520, 900),
                                               ("device", 29, 600, 70, 150)])
def test_orders(weights, how, A, B, longest, T):
    rng = np.random.default_rng([B, A])
    labels = rng.integers(0, longest + 1, B)
    labels[0] = longest
    frames = np.minimum(T, labels + labels // 8 + rng.integers(20, T - longest, B))
    batch = batch_of(frames, labels, A, seed=B, T=T)
    if how == "device":
        db = harness.DeviceMetaBatch(T, B, A, longest, batch.blank)
        db.load(batch)
        db.run()
    else:
        db = harness.DeviceBatch(batch)
        db.run_best_path() if how == "align" else db.run()
    ws = db.ws.cpu().numpy()[db.ws_ptr - db.ws.data_ptr():]
    order = ws[(64 * B + 255) // 256 * 256:][:12 * B].view(np.int32)
    folded = how == "device" and A <= 64 and B <= 512
    weight = weights(batch, how == "align", folded)
    heaviest = np.lexsort((np.arange(B), -weight))
    assert order[2 * B:].tolist() == heaviest[::-1].tolist()
    if 2 * B <= 256:                                     # (blocks of 16 utterances, their forward chains and then their backward ones)
        chains = [2 * u + d for first in range(0, B, 16) for d in (0, 1) for u in heaviest[first:first + 16]]
        assert order[:2 * B].tolist() == chains
