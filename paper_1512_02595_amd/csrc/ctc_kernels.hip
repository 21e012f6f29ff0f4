// HIP kernels of the batched CTC cost + gradient for gfx950 (wave64, CDNA4).
//
// Pipeline of one call (appendix "GPU Implementation of CTC Loss Function"; cost of
// Section 3.3 Eq. (ctc); softmax of Section 3.1; most probable alignment of Section 5.1):
//   upload    the per-call metadata from pinned host memory into the workspace
//             (or plan: the same records built on the GPU from device-resident lengths and labels);
//             alphabets of at most 64 symbols and few utterances: done by the softmax launch itself
//   setup     per utterance: label positions grouped by symbol (the appendix's one-off
//             key-value sort, done by counting), degenerate costs; rides in the softmax launch
//   softmax   per frame row: log2-sum-exp2 of the scaled logits, the blank's probability and the
//             emissions (softmax outputs divided by it) of every label position, gathered once so that
//             the recursions read them coalesced (small alphabets: of every symbol),
//             in chunks of eight frames a column; larger alphabets: also the gradient but for the
//             label columns
//   lattice   alpha and beta recursions, both in one launch, a workgroup per utterance and direction
//             (cost only, and alignment with the max recursion and recorded choices: half of the
//             frames each, up to where they meet); small alphabets: also the gradient where that
//             is quicker than a launch of its own
//   gradient  softmax minus the normalised per-symbol occupancy, from both recursions run once more
//             between the states that the chains have stored; zero fill of padding
//             (alignment: the backtrace instead)
//
// The recursions run on probabilities, each lane's values in fp64 with an int32 exponent of
// the lane's own (its "frame"), relative to the blank's: no transcendentals and a
// fifth of the instructions of the log-space form (run_chain_linear, run_chain_linear2).
// alpha and beta span thousands of binary orders of magnitude over a 15 s utterance, and the
// states that carry the mass lie a thousand orders below the largest of their frame, so the
// exponent has to be per lane; fp64 then leaves room for the steps until it is looked after.
// Utterances with an emission below 2^kLinearMinLog2 (found by the softmax launch), launches
// of the barrier kernel and the maximum recursion use the log-space form instead
// (run_chain_log): base-2 logarithms in fp64 (v_exp_f32 / v_log_f32 are base 2, so no scaling
// multiplies; only the bounded differences that enter them are narrowed to fp32), log(0) a
// large finite negative number, which keeps every operation NaN-free.
// What either leaves for the gradient is described at "lattice storage".

#include <hip/hip_runtime.h>

#include <type_traits>

#include "ctc_internal.h"

namespace ctc {
// A load from a buffer whose four words are in scalar registers.  (The builtin takes a resource made from a pointer, and one that moves is made anew each time: two scalar
// instructions more than moving on the base in the words.)
typedef float FourFloats __attribute__((ext_vector_type(4)));
typedef int BufferWords __attribute__((ext_vector_type(4)));
__device__ FourFloats buffer_load(BufferWords buffer, int lane_offset, int offset, int policy) __asm("llvm.amdgcn.raw.buffer.load.v4f32");

namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr double kLn2 = 0.6931471805599453;
constexpr double kNeg = -1.0e30;
constexpr int kRowThreads = 256;

__device__ __forceinline__ float fast_exp2(float v) { return __builtin_amdgcn_exp2f(v); }
__device__ __forceinline__ float fast_log2(float v) { return __builtin_amdgcn_logf(v); }
// log2 of a softmax output from the logit, the row's largest logit and log2 of the row's sum of
// 2^((x - max) log2 e).  The difference comes first: formed as x log2 e - (max log2 e + log2 sum) the
// result would carry the rounding of the offset, 6e-8 of its size, and a row of logits of size 100 whose
// winner has probability 1 - 1e-6 would give that winner an emission wrong by 1e-5, frame after frame.
__device__ __forceinline__ float log2_softmax(float x, float row_max, float log2_sum)
{
    return fmaf(x - row_max, kLog2e, -log2_sum);
}
// ... and its numerator, 2^((x - max) log2 e).
__device__ __forceinline__ float exp2_from_max(float x, float row_max) { return fast_exp2((x - row_max) * kLog2e); }

// ---- element access for the two activation types -------------------------------------

struct bf16_t { uint16_t bits; };

__device__ __forceinline__ float load_elem(const float* p, size_t i) { return p[i]; }
__device__ __forceinline__ float load_elem(const bf16_t* p, size_t i)
{
    return __uint_as_float(static_cast<uint32_t>(p[i].bits) << 16);
}
__device__ __forceinline__ void store_elem(float* p, size_t i, float v) { p[i] = v; }
__device__ __forceinline__ uint16_t to_bf16_bits(float v)
{
    uint32_t u = __float_as_uint(v);
    u += 0x7FFFu + ((u >> 16) & 1u);           // round to nearest, ties to even
    return static_cast<uint16_t>(u >> 16);
}
__device__ __forceinline__ void store_elem(bf16_t* p, size_t i, float v) { p[i].bits = to_bf16_bits(v); }

// 16-byte vectors of activations: 4 floats or 8 bf16.
// Sixteen bytes of a row.
typedef uint32_t RawVec __attribute__((ext_vector_type(4)));
template <typename T> struct Vec;
template <> struct Vec<float> {
    static constexpr int N = 4;
    static __device__ __forceinline__ float get(const RawVec& r, int e) { return __uint_as_float(r[e]); }
    static __device__ __forceinline__ RawVec pack(const float (&v)[4])
    {
        return RawVec{__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3])};
    }
};
template <> struct Vec<bf16_t> {
    static constexpr int N = 8;
    static __device__ __forceinline__ float get(const RawVec& r, int e)
    {
        return __uint_as_float(e & 1 ? r[e >> 1] & 0xFFFF0000u : r[e >> 1] << 16);
    }
    static __device__ __forceinline__ RawVec pack(const float (&v)[8])
    {
        RawVec r;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            r[i] = static_cast<uint32_t>(to_bf16_bits(v[2 * i])) | (static_cast<uint32_t>(to_bf16_bits(v[2 * i + 1])) << 16);
        return r;
    }
};
// Streaming store: the gradient of a large alphabet is written once and not read again by this call except in the few
// label columns (measured 7 % faster than a plain store on the 6000-symbol workload, and the later fix-up of the label
// columns 20 % faster).
__device__ __forceinline__ void store_streaming(void* p, const RawVec& v) { __builtin_nontemporal_store(v, static_cast<RawVec*>(p)); }

// ---- workgroup reductions (256 threads = 4 wavefronts), fixed order => repeatable -------

// Lane permutations inside a row of 16 lanes, as DPP operands of the add / max itself (no trip
// through the LDS crossbar): neighbours, pairs, then the mirrored half-row and the mirrored row.
template <int kCtrl>
__device__ __forceinline__ float dpp_permute(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), kCtrl, 0xf, 0xf, true));
}
// Every lane receives the sum (maximum) over its row of 16 lanes.  All 16 lanes must be active.
__device__ __forceinline__ float row16_sum(float v)
{
    v += dpp_permute<0xB1>(v);      // quad_perm [1,0,3,2]
    v += dpp_permute<0x4E>(v);      // quad_perm [2,3,0,1]
    v += dpp_permute<0x141>(v);     // row_half_mirror
    v += dpp_permute<0x140>(v);     // row_mirror
    return v;
}
__device__ __forceinline__ float row16_max(float v)
{
    v = fmaxf(v, dpp_permute<0xB1>(v));
    v = fmaxf(v, dpp_permute<0x4E>(v));
    v = fmaxf(v, dpp_permute<0x141>(v));
    v = fmaxf(v, dpp_permute<0x140>(v));
    return v;
}
// The same over groups of 4 neighbouring lanes.
__device__ __forceinline__ float quad_sum(float v)
{
    v += dpp_permute<0xB1>(v);
    v += dpp_permute<0x4E>(v);
    return v;
}
__device__ __forceinline__ float quad_max(float v)
{
    v = fmaxf(v, dpp_permute<0xB1>(v));
    v = fmaxf(v, dpp_permute<0x4E>(v));
    return v;
}
__device__ __forceinline__ int quad_sum(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xf, 0xf, true);
    return v;
}
// Whole wavefront (all 64 lanes active); the four row results are combined in a fixed order.
__device__ __forceinline__ float wave_sum(float v)
{
    const int r = __float_as_int(row16_sum(v));
    return (__int_as_float(__builtin_amdgcn_readlane(r, 0)) + __int_as_float(__builtin_amdgcn_readlane(r, 16))) +
           (__int_as_float(__builtin_amdgcn_readlane(r, 32)) + __int_as_float(__builtin_amdgcn_readlane(r, 48)));
}
__device__ __forceinline__ float wave_max(float v)
{
    const int r = __float_as_int(row16_max(v));
    return fmaxf(fmaxf(__int_as_float(__builtin_amdgcn_readlane(r, 0)), __int_as_float(__builtin_amdgcn_readlane(r, 16))),
                 fmaxf(__int_as_float(__builtin_amdgcn_readlane(r, 32)), __int_as_float(__builtin_amdgcn_readlane(r, 48))));
}

// `slot` is 4 floats of LDS private to this reduction.
__device__ __forceinline__ float block_sum(float v, float* slot)
{
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) slot[threadIdx.x >> 6] = v;
    __syncthreads();
    return (slot[0] + slot[1]) + (slot[2] + slot[3]);
}
__device__ __forceinline__ float block_max(float v, float* slot)
{
    v = wave_max(v);
    if ((threadIdx.x & 63) == 0) slot[threadIdx.x >> 6] = v;
    __syncthreads();
    return fmaxf(fmaxf(slot[0], slot[1]), fmaxf(slot[2], slot[3]));
}

// ---- upload --------------------------------------------------------------------------------
// First launch of a call.  The per-call metadata (utterance records, run order, labels) was
// written by the host into pinned host memory; this kernel copies it word by word into the
// workspace, every read in flight at once, so that no stream-ordered copy-engine transfer
// (about 18 us of latency per call) sits between two calls.
// Where the image also holds the labels as bytes (alphabets of at most 256 symbols), the label words
// [labels_first, labels_end) are made from those: a quarter of the bytes over PCIe for what is most
// of the image (512 utterances of 29 symbols: 171 KB -> 67 KB, 8.7 -> 5.8 us).
__global__ __launch_bounds__(kRowThreads)
void ctc_upload_kernel(const int* __restrict__ host_image, int* __restrict__ ws, int words,
                       int labels_first, int labels_end, const unsigned char* __restrict__ labels8)
{
    const int i = blockIdx.x * kRowThreads + threadIdx.x;
    if (i >= words) return;
    if (labels8 && i >= labels_first && i < labels_end)
        ws[i] = labels8[i - labels_first];
    else
        ws[i] = host_image[i];
}

// ---- device-side planning -------------------------------------------------------------------
// The device-metadata entry point has no host image: lengths and labels are device arrays that
// the host never sees, so this kernel (one workgroup) does what the host launcher does
// otherwise.  Per utterance: range checks, the count of adjacent repeats (an alignment exists
// iff T_b >= L + repeats), the wavefront plan, and the offsets of its blocks, which are laid
// out with the strides of the largest utterance the caller allows (labels [B][max_label]; emissions, lattice and frames what
// gathered_emissions, lattice_words and padded_frames give for T and longest_aligned).  Then the run
// order: heaviest chains first (rank by chain_weight, ties by index), -1 for the rest.
constexpr int kPlanThreads = 1024;

__global__ __launch_bounds__(kPlanThreads)
void ctc_plan_kernel(const int* __restrict__ labels, const int* __restrict__ label_lengths,
                     const int* __restrict__ input_lengths, Utt* __restrict__ meta,
                     int* __restrict__ order, int* __restrict__ status,
                     int Tt, int B, int A, int blank, int max_label, int poll_budget, bool crowded,
                     bool log_domain)
{
    __shared__ long long weight[kMaxDeviceMetaB];     // chain_weight; -1: does not run
    __shared__ int repeats[kMaxDeviceMetaB];          // adjacent equal symbols; kBadLabel added for a bad symbol
    __shared__ int s_bad, s_running;
    constexpr int kBadLabel = 1 << 20;
    const int tid = threadIdx.x;
    if (tid == 0) {
        s_bad = 0;
        s_running = 0;
    }
    int* const s_len = reinterpret_cast<int*>(weight);       // label lengths, until the weights are written
    for (int i = tid; i < B; i += kPlanThreads) {
        order[2 * i] = -1;
        order[2 * i + 1] = -1;
        repeats[i] = 0;
        s_len[i] = label_lengths[i];
    }
    __syncthreads();
    // Every entry of the padded label matrix on its own, eight reads per thread in flight.
    const int cells = B * max_label;
    for (int i0 = tid; i0 < cells; i0 += 8 * kPlanThreads) {
        int c[8], before[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = i0 + u * kPlanThreads;
            c[u] = (i < cells) ? labels[i] : 0;
            before[u] = (i < cells && i > 0) ? labels[i - 1] : -1;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = i0 + u * kPlanThreads;
            if (i >= cells) continue;
            const int b = i / max_label, j = i - b * max_label;
            const int L = s_len[b];
            if (j < L && L <= max_label) {
                int add = (c[u] < 0 || c[u] >= A || c[u] == blank) ? kBadLabel : 0;
                if (j > 0 && c[u] == before[u]) ++add;
                if (add) atomicAdd(&repeats[b], add);
            }
        }
    }
    __syncthreads();
    for (int b = tid; b < B; b += kPlanThreads) {
        const int L = label_lengths[b], Tb = input_lengths[b];
        const int rep = repeats[b];
        const bool bad = L < 0 || L > max_label || Tb < 0 || Tb > Tt || rep >= kBadLabel;
        const bool runs = !bad && Tb > 0 && Tb >= L + rep;
        const WavePlan wp = plan_waves(bad ? 0 : L, crowded);
        Utt m;
        m.Tb = bad ? 0 : Tb;
        m.L = bad ? 0 : L;
        m.lab_off = b * max_label;
        m.flags = (runs ? kUttRuns : 0) | (bad ? kUttInvalid : 0) |
                  ((log_domain || Tb > kLinearMaxFrames || tight_fit(Tb, L, rep)) ? kUttLogDomain : 0) |
                  (!bad && linear_two_pairs(L, crowded) ? kUttTwoPairs : 0);
        const int padded = static_cast<int>(padded_frames(Tt)), longest = longest_aligned(Tt, max_label);
        m.f_off = static_cast<unsigned>(b) * padded;
        m.waves = wp.waves;
        m.halo = wp.halo;
        const WavePlan wp2 = linear_plan2(bad ? 0 : L, crowded);
        m.waves2 = wp2.waves;
        m.halo2 = wp2.halo;
        m.poll_budget = poll_budget;
        m.e_direct = emission_layout(A);
        m.rough = 0;
        m.steep = 0;
        m.e_cols = m.e_direct == kEmitSymbols ? A : m.L;
        m.e_off = b * (m.e_direct == kEmitSymbols ? static_cast<int64_t>(padded) * A : gathered_emissions(Tt, longest));
        m.ab_off = b * lattice_words(Tt, longest);
        meta[b] = m;
        weight[b] = runs ? chain_weight(m, false, crowded) : -1;
        if (bad) s_bad = 1;
        if (runs) atomicAdd(&s_running, 1);
    }
    __syncthreads();
    if (tid == 0) *status = s_bad ? CTC_STATUS_INVALID_VALUE : CTC_STATUS_SUCCESS;
    for (int i = tid; i < B; i += kPlanThreads) {
        const long long wi = weight[i];
        int rank = 0;
        for (int j = 0; j < B; ++j) {
            const long long wj = weight[j];
            rank += (wj > wi) || (wj == wi && j < i);
        }
        order[2 * B + B - 1 - rank] = i;                 // (the utterances by when their chains end)
        if (wi < 0) continue;
        // Heaviest first, in blocks of kChainBlock utterances: a block's forward chains, then its
        // backward chains (order_chains; the device planner does not balance the SIMDs' loads
        // beyond that).
        const int first = rank - rank % kChainBlock, in_block = min(kChainBlock, s_running - first);
        for (int d = 0; d < 2; ++d) order[first * 2 + d * in_block + rank % kChainBlock] = 2 * i + d;
    }
}

// ---- setup role ----------------------------------------------------------------------------
// Runs in one extra grid column of the softmax launch, one workgroup per utterance, beside
// the row work.  It groups the label positions by symbol, once per utterance, for every frame
// of the gradient to reuse -- the purpose of the appendix's one-off key-value sort of the
// label.  Word of label position j:
//   bits  0..9   its slot in the order (symbol ascending, then position ascending): the
//                positions of one symbol occupy consecutive slots
//   bits 12..21  how often its symbol occurs in the label
//   bit  31      set if j is the first occurrence of its symbol (its slot then starts the run)
// The gradient kernels write each state's mass share to its slot and let the first occurrence
// add up the run in slot order, so a symbol's occupancy has one writer and a fixed order of
// summation.  Also here: costs of utterances without a lattice, the per-utterance error
// flags, the two constants of the emission array.
constexpr int kLinkSlotMask = 0x3FF, kLinkCountShift = 12;
static_assert(CTC_MAX_LABEL_LENGTH <= kLinkSlotMask, "slot and count fields hold 10 bits");

// (The constants that lanes without a label state read as their emission, kZeroEmission and
// kLogZeroEmission, are laid out in the launcher's header, with the chains' fetch schedule.)

struct SetupArgs {
    int* links;
    float* costs;
    int* chain_err;
    int* done;            // per utterance (kDoneStride apart): kDoneWords words that its chains and those who wait for them
                          // share (finish_loss, announce_end, take_chain)
    float* log0;          // kEmissionConstants floats that lattice lanes without a label state read as their
                          // emission: probability 0 (linear-domain chains) and log 0 (log-domain chains)
    double* emit_blank64; // alignments: log2 of the blank's probability per frame (Layout::emit_blank64)
    int* host_flag;       // pinned host word: receives flag_value once the upload has been consumed
    int flag_value;
    bool plain_logs;      // emissions are stored as log2 probabilities throughout (most probable alignment)
    int parts;            // workgroups per utterance that share the setup role (grid columns beyond the rows)
};

// The grouping compares every pair of label positions; it is spread over `parts` workgroups per
// utterance (64 positions each at a time) and four lanes per position, each lane walking a quarter
// of the label, so that a label of 500 symbols costs 125 steps per lane instead of 1000.
constexpr int kSetupLabelSlots = CTC_MAX_LABEL_LENGTH + 5;     // the label and a quarter's padding

__device__ __forceinline__ void setup_words(const Utt m, const int b, const SetupArgs sa);
__device__ __forceinline__ void setup_role(const Utt m, const int b, const int* __restrict__ labels,
                                           const SetupArgs sa, int* s_lab, const int part, const int parts)
{
    const int tid = threadIdx.x;
    const int* lab = labels + m.lab_off;
    const int quarter_length = (m.L + 3) / 4;
    // padding: a symbol that is neither smaller than nor equal to any real one
    for (int j = tid; j < 4 * quarter_length; j += kRowThreads) s_lab[j] = j < m.L ? lab[j] : 0x7FFFFFFF;
    __syncthreads();
    const int quarter = tid & 3;
    const int* const mine = s_lab + quarter * quarter_length;
    const int first_i = quarter * quarter_length;
    for (int j = part * 64 + (tid >> 2); j < m.L; j += parts * 64) {
        const int c = s_lab[j];
        // Independent iterations keep the LDS reads in flight.
        int below = 0, before = 0, count = 0;
        for (int i = 0; i < quarter_length; ++i) {
            const int ci = mine[i];
            below += ci < c;
            count += ci == c;
            before += (ci == c) & (first_i + i < j);
        }
        below = quad_sum(below);
        count = quad_sum(count);
        before = quad_sum(before);
        if (quarter == 0)
            sa.links[m.lab_off + j] = (below + before) | (count << kLinkCountShift) |
                                      (before == 0 ? static_cast<int>(0x80000000u) : 0);
    }
    if (part == 0) setup_words(m, b, sa);
}

// The per-utterance words that every call starts from, the constants of the emission array, and the costs
// of utterances without a lattice.  By one workgroup per utterance.
__device__ __forceinline__ void setup_words(const Utt m, const int b, const SetupArgs sa)
{
    if (threadIdx.x == 0) {
        sa.chain_err[b] = 0;
        for (int i = 0; i < kDoneWords; ++i) sa.done[b * kDoneStride + i] = 0;
        if (b == 0) {
            for (int i = 0; i < kEmissionConstants; ++i) sa.log0[i] = i < kLogZeroEmission ? 0.0f : static_cast<float>(kNeg);
            // This launch follows the upload kernel on the stream, so the host may now reuse
            // the pinned image.
            if (sa.host_flag)
                __hip_atomic_store(sa.host_flag, sa.flag_value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
        // No frames: the empty product (cost 0) for an empty label.  Otherwise no alignment.
        if (m.flags & kUttInvalid) sa.costs[b] = __uint_as_float(0x7FC00000u);
        else if (!(m.flags & kUttRuns)) sa.costs[b] = (m.Tb == 0 && m.L == 0) ? 0.0f : __builtin_inff();
    }
}

// ---- emission coding -------------------------------------------------------------------------
// The recursions run on probabilities (linear domain, see run_chain_linear) relative to the blank's: every frame is divided
// by its blank's probability y_blank, its *norm*, so that a step has no multiplication for the blank states and a chain no
// blank emissions to fetch.  Shares alpha beta / p do not change (p is divided by the same product of norms), and the cost
// gets the norms back at the end (Norms).
//   label emission v >= 0: the ratio y / y_blank; v < 0: log2 of it, where y < 2^kLinearMinLog2
//   word of the frame c >= 0: the norm y_blank; c < 0: the norm is 1, y_blank is 2^(c + 1) (below 2^kLinearMinLog2) and the
//   frame's label emissions are y itself, or log2 y
// A ratio is the quotient of the two rounded probabilities to within an ulp, so what the norms give back is what was taken.
// A lane that stores a negative word raises the utterance's kUttLogDomain flag, and its chains then take logarithms.
// (The most probable alignment has no sums to speed up: its launches store plain logarithms.)
struct FrameNorm {
    float inverse_sum, log_blank, blank, inverse;        // of the row; log2 y_blank, y_blank, about 1 / y_blank
    bool small;                                          // the norm is 1
    // From the blank's logit, the row's largest one, and the sum of 2^((x - max) log2 e) and its logarithm.  Probabilities are products
    // with 1 / sum: where a frame is nearly certain of a symbol, the exponential of log2 y would be off by an ulp or two of 1, and
    // elsewhere it carries the rounding of a larger logarithm (see encode_emission).
    __device__ __forceinline__ FrameNorm(float x, float row_max, float sum, float log2_sum)
    {
        log_blank = log2_softmax(x, row_max, log2_sum);
        const float about = __builtin_amdgcn_rcpf(sum);
        inverse_sum = fmaf(fmaf(-sum, about, 1.0f), about, about);
        blank = exp2_from_max(x, row_max) * inverse_sum;
        inverse = __builtin_amdgcn_rcpf(blank);
        small = log_blank < kLinearMinLog2;
    }
    __device__ __forceinline__ float word() const { return small ? log_blank - 1.0f : blank; }
};
// The emission of a symbol whose log2 y is lp and whose 2^((x - max) log2 e) is e.  The gradient multiplies the ratio by the norm
// again, which costs y a rounding or two; as a product y has that much less to begin with.  2-norm of its error, symbols of no label,
// 29 symbols, logits N(0, 1), N(0, 2) and N(0, 6): 7.0e-8, 6.9e-8, 7.7e-8; from the exponential of lp 1.12e-7, 7.95e-8, 7.8e-8, and
// without ratio and norm between 1.10e-7, 7.6e-8, 7.3e-8.
__device__ __forceinline__ float encode_emission(float lp, float e, const FrameNorm& f)
{
    const float y = e * f.inverse_sum, q = y * f.inverse;
    const float ratio = fmaf(fmaf(-q, f.blank, y), f.inverse, q);
    return lp < kLinearMinLog2 ? (f.small ? lp : lp - f.log_blank) : (f.small ? y : ratio);
}
__device__ __forceinline__ float encode_blank(const FrameNorm& f) { return f.small ? f.log_blank : 1.0f; }
// From a frame's word.
__device__ __forceinline__ float frame_norm(float c) { return c < 0.0f ? 1.0f : c; }
__device__ __forceinline__ float blank_emission_log2(float c) { return c < 0.0f ? c + 1.0f : 0.0f; }
__device__ __forceinline__ float blank_softmax(float c) { return c < 0.0f ? fast_exp2(c + 1.0f) : c; }
// log2 of a coded emission in two floats whose sum it is: the binary exponent of a stored probability
// and the logarithm of its mantissa.  (As one float the logarithm of 2^-40 would be good to 4e-6 only,
// frame after frame; a chain of 400 steps then misses the gradient's bound.)
struct Log2Parts { float whole, part; };
__device__ __forceinline__ Log2Parts emission_log2_parts(float v)
{
    // (selected, not branched on: with a branch per frame and state a log-domain step took 161 ns in place of 135.  0: a label
    // of a virtual frame)
    const float whole = static_cast<float>(__builtin_amdgcn_frexp_expf(v));
    const float part = fmaxf(fast_log2(__builtin_amdgcn_frexp_mantf(v)), static_cast<float>(kNeg));
    return {v < 0.0f ? v : whole, v < 0.0f ? 0.0f : part};
}
__device__ __forceinline__ double emission_log2(float v)
{
    const Log2Parts p = emission_log2_parts(v);
    return static_cast<double>(p.whole) + static_cast<double>(p.part);
}
// A softmax output from its emission and the frame's norm.
__device__ __forceinline__ float emission_softmax(float v, float norm) { return (v < 0.0f ? fast_exp2(v) : v) * norm; }
// Emissions of virtual frames (emission_layout in the launcher's header): blank with probability 1, labels with 0.
__device__ __forceinline__ float virtual_emission(bool blank, bool plain_logs)
{
    return plain_logs ? (blank ? 0.0f : static_cast<float>(kNeg)) : (blank ? 1.0f : 0.0f);
}
// The blank's emission of one padded frame: the frame's word, or (plain_logs) log2 y_blank, which is wanted as fp64 scalars.
__device__ __forceinline__ void store_blank(float* __restrict__ emit_blank, double* __restrict__ emit_blank64, size_t frame, float e, bool plain_logs)
{
    if (plain_logs) emit_blank64[kBlankSlack + frame] = static_cast<double>(e);
    else emit_blank[kBlankSlack + frame] = e;
}
// Where the emission of column `column` in frame `t` of an utterance sits.
__device__ __forceinline__ size_t emission_at(int64_t e_off, int columns, int t, int column)
{
    return kLabelSlack + static_cast<size_t>(e_off) + (static_cast<size_t>(t / kChunk) * columns + column) * kChunk + t % kChunk;
}
// The virtual frames of an utterance of a wide alphabet, by the lanes (q of `lanes`) of its last frame.
__device__ __forceinline__ void store_virtual_frames(const Utt& m, float* __restrict__ emit_blank, double* __restrict__ emit_blank64,
                                                     float* __restrict__ emit_label, bool plain_logs, int q, int lanes)
{
    for (int t = m.Tb; t < static_cast<int>(padded_frames(m.Tb)); ++t) {
        if (q == 0) store_blank(emit_blank, emit_blank64, static_cast<size_t>(m.f_off) + t, virtual_emission(true, plain_logs), plain_logs);
        for (int j = q; j < m.L; j += lanes)
            emit_label[emission_at(m.e_off, m.L, t, j)] = virtual_emission(false, plain_logs);
    }
}
// The smallest log2 probability that a lane has seen decides how the utterance's chains run (lattice_body).
// `m`: the utterance's record as this launch found it.  Stores, and no atomics: nothing else in the words changes during the
// launch, so that all who raise a flag write the same.  (One atomic per lane that met such an emission, in 64 words for the
// whole launch: 64 x 500 rows of 750 symbols with steep logits 650 us; one per row 110; so 23.)
__device__ __forceinline__ void raise_flags(Utt* meta, int b, const Utt& m, float lowest)
{
    if (lowest < kGentleMinLog2) {
        meta[b].rough = 1;
        if (lowest < kRoughMinLog2) meta[b].steep = 1;
        if (lowest < kLinearMinLog2) meta[b].flags = m.flags | kUttLogDomain;
    }
}

// ---- softmax statistics + emission gather --------------------------------------------------
// Alphabets above kDirectMaxA symbols.  The gradient of a row is the softmax itself except in the columns whose symbol
// occurs in the label, so the launch that holds the row also writes it: y for valid rows, zeros for padding rows and for
// utterances without an alignment (skipped when no gradient is asked for: grads == nullptr).  The activations are
// then never read a second time; the label columns are corrected after the recursions (ctc_gradient_wide_kernel).
//
// Zero rows need nothing that is computed here: a share of them (those with t % 16 below `defer`) is left to the lattice
// launch, whose compute units without a chain have nothing else to do (fill_rows).

// kLanes lanes (16, a wavefront or the workgroup) hold a row of up to kPerLane kLanes symbols in registers between the
// maximum and the sum (kPerLane: the fewest that suffice, see row_lanes): it is read once, with 16-byte loads, and written with 16-byte stores.  A row that starts off a 16-byte
// boundary (an alphabet size that is no multiple of the vector, or a tensor that starts off one) has up to N - 1 symbols
// before its first whole vector and as many after its last; a lane takes one of them each.  Where the gradient starts at
// another place within 16 bytes than the activations, the vectors read are written element by element (750 symbols, f32:
// 87.6 us a call against 86.8 with vectors, 134 with the three passes of ctc_softmax_kernel; 6000 bf16: 119, 107 and 292).
// Bound by memory: with the 308 of 768 MB of zero rows that the lattice launch takes over counted in, 64 x 500 rows of
// 6000 symbols, of which 300 on average are valid, moved at 4.8 TB/s with consecutive rows on consecutive dies (bf16: 128.5 us
// with a load in each branch, 119 with all loads first and zero rows left over) and take a ninth less in runs (RowPlan).
// 27 x 333 rows of 4733 symbols (no multiple of a vector): 108 us with three passes of four-byte loads, 41 so.  64 x 500
// rows of 750 symbols: 41.5 us with the rows in LDS, 34.7 so.
// kStreaming: the rows are loaded past the caches (see row_plan).
// grid: plan.groups workgroups with rows, then sa.parts per utterance for the setup role.

// Which rows a workgroup takes.  Workgroup i runs on die i mod 8, and each die has a cache of its own.  With consecutive groups of
// rows on consecutive dies all eight work in the same few pages of memory, and an utterance's emissions, eight frames to 32 bytes,
// are written a word here and a word there.  So a die gets tiles of neighbouring groups instead: `frames` frames times
// `columns` groups, every other round of eight tiles the other way round (utterances end one after the other, so that the tiles
// of a round have ever less to do).  A tile of 0 frames: consecutive groups, one after the other.
// Everything divides by a number that the launcher knows: with the processor's own divisions, a reciprocal and its corrections each, a row
// began a microsecond later (214 x 171 x 4186 bf16, cost alone: 62.9 us a call, so 60.4).
struct RowPlan {
    int groups;               // workgroups, some of them without rows
    Divisor per_frame;        // groups of rows in a frame
    int frames;               // a tile's
    Divisor columns;          // ... groups
    Divisor round, across;    // workgroups of eight tiles; tiles side by side in a frame
};
struct RowPlace { int t, group; };
__device__ __forceinline__ RowPlace row_place(const RowPlan& plan, unsigned index, bool runs)
{
    constexpr int kDies = 8;
    auto in_order = [&](unsigned i) {
        const unsigned t = plan.per_frame.quotient(i);
        return RowPlace{static_cast<int>(t), static_cast<int>(i - t * plan.per_frame.by)};
    };
    if (plan.frames == 0) return in_order(index);
    const unsigned round = plan.round.quotient(index), in_round = index - round * plan.round.by;
    const unsigned die = in_round % kDies, within = in_round / kDies, place = round & 1 ? kDies - 1 - die : die;
    // a run of consecutive groups, across the ends of frames; what is left behind the last whole round lies as it comes
    if (runs) return in_order((round + 1) * plan.round.by <= static_cast<unsigned>(plan.groups) ? (round * kDies + place) * plan.columns.by + within : index);
    const unsigned tile = round * kDies + place, band = plan.across.quotient(tile), frame = plan.columns.quotient(within);
    return {static_cast<int>(band * plan.frames + frame), static_cast<int>((tile - band * plan.across.by) * plan.columns.by + within - frame * plan.columns.by)};
}

template <typename T, int kLanes, int kPerLane, bool kStreaming>
__global__ __launch_bounds__(kRowThreads)
void ctc_softmax_rows_kernel(const T* __restrict__ x, T* __restrict__ grads, Utt* __restrict__ meta,
                             const int* __restrict__ labels, float* __restrict__ emit_blank, float* __restrict__ emit_label,
                             const SetupArgs sa, int Tt, int B, int A, int blank, const RowPlan plan, int defer)
{
    constexpr int N = Vec<T>::N, kVecs = kPerLane / N, kRows = kRowThreads / kLanes;
    static_assert(kLanes == 16 || kLanes == 64 || kLanes == kRowThreads, "row reductions exist for these");
    __shared__ float red[8];
    __shared__ int s_lab[kSetupLabelSlots];
    const int tid = threadIdx.x;
    if (static_cast<int>(blockIdx.x) >= plan.groups) {
        const int index = static_cast<int>(blockIdx.x) - plan.groups, b = index / sa.parts;
        setup_role(meta[b], b, labels, sa, s_lab, index % sa.parts, sa.parts);
        return;
    }
    const RowPlace place = row_place(plan, blockIdx.x, kLanes == kRowThreads);
    const int t = place.t, q = tid % kLanes;
    const int b = place.group * kRows + (kRows > 1 ? tid / kLanes : 0);
    if (t >= Tt || place.group >= static_cast<int>(plan.per_frame.by) || b >= B) return;
    const Utt m = meta[b];
    const size_t row_off = (static_cast<size_t>(t) * B + b) * A;
    const T* const row = x + row_off;
    T* const grow = grads ? grads + row_off : nullptr;
    if (t >= m.Tb || !(m.flags & kUttRuns)) {
        if (grow && (t & 15) >= defer) {
            const int head = min(static_cast<int>((16 - (reinterpret_cast<uintptr_t>(grow) & 15)) & 15) / static_cast<int>(sizeof(T)), A);
            const int nvec = (A - head) / N, rest = A - nvec * N;
            for (int i = q; i < nvec; i += kLanes) store_streaming(grow + head + static_cast<size_t>(i) * N, RawVec{0, 0, 0, 0});
            if (q < rest) store_elem(grow, q < head ? q : nvec * N + q, 0.0f);
        }
        return;
    }
    const int head = min(static_cast<int>((16 - (reinterpret_cast<uintptr_t>(row) & 15)) & 15) / static_cast<int>(sizeof(T)), A);
    const int nvec = (A - head) / N, rest = A - nvec * N;
    const int single = q < rest ? (q < head ? q : nvec * N + q) : -1;          // this lane's symbol outside the vectors

    // All of the row and the labels' symbols are asked for before any of it is used: no conversion, and no lane left out,
    // between one load and the next (a vector past the end is the last one again, counted by nobody).
    RawVec raw[kVecs];
#pragma unroll
    for (int i = 0; i < kVecs; ++i) {
        const auto* const from = reinterpret_cast<const RawVec*>(row + head + static_cast<size_t>(min(q + i * kLanes, nvec - 1)) * N);
        raw[i] = kStreaming ? __builtin_nontemporal_load(from) : *from;
    }
    float alone = load_elem(row, single >= 0 ? single : 0);
    const int* const lab = labels + m.lab_off;
    const int c_first = q < m.L ? lab[q] : 0;
    float mx = single >= 0 ? alone : -__builtin_inff();
    // (the vector that some lanes see again changes no maximum)
#pragma unroll
    for (int i = 0; i < kVecs; ++i)
#pragma unroll
        for (int e = 0; e < N; ++e) mx = fmaxf(mx, Vec<T>::get(raw[i], e));
    mx = kLanes == 16 ? row16_max(mx) : (kLanes == 64 ? wave_max(mx) : block_max(mx, red));
    float sum = single >= 0 ? fast_exp2((alone - mx) * kLog2e) : 0.0f;
#pragma unroll
    for (int i = 0; i < kVecs; ++i)
        if (q + i * kLanes < nvec)
#pragma unroll
            for (int e = 0; e < N; ++e) sum += fast_exp2((Vec<T>::get(raw[i], e) - mx) * kLog2e);
    sum = kLanes == 16 ? row16_sum(sum) : (kLanes == 64 ? wave_sum(sum) : block_sum(sum, red + 4));
    // log2 y_k = (x_k - max) log2 e - log2 sum: the difference first, so that the error is relative to
    // log2 y_k itself and not to the row's offset (see log2_softmax)
    const float ls = fast_log2(sum);
    if (grow) {
        const bool together = ((reinterpret_cast<uintptr_t>(row) ^ reinterpret_cast<uintptr_t>(grow)) & 15) == 0;
#pragma unroll
        for (int i = 0; i < kVecs; ++i) {
            const int at = q + i * kLanes;
            if (at < nvec) {
                float y[N];
#pragma unroll
                for (int e = 0; e < N; ++e) y[e] = fast_exp2(log2_softmax(Vec<T>::get(raw[i], e), mx, ls));
                T* const out = grow + head + static_cast<size_t>(at) * N;
                if (together)
                    store_streaming(out, Vec<T>::pack(y));
                else
#pragma unroll
                    for (int e = 0; e < N; ++e) store_elem(out, e, y[e]);
            }
        }
        if (single >= 0) store_elem(grow, single, fast_exp2(log2_softmax(alone, mx, ls)));
    }

    // the emissions, out of the row that the caches still hold; wavefronts without a label position make room for other rows (214 x
    // 171 x 4186 bf16, cost alone: 90.1 us a call with all of them waiting for the blank's logit, 86.1 so)
    if (q > 0 && q >= m.L && t != m.Tb - 1) return;
    const float blank_logit = load_elem(row, blank), first_logit = load_elem(row, c_first);        // (both asked for before either is used)
    const FrameNorm norm(blank_logit, mx, sum, ls);
    float lowest = norm.log_blank;
    if (q == 0) store_blank(emit_blank, sa.emit_blank64, static_cast<size_t>(m.f_off) + t, sa.plain_logs ? norm.log_blank : norm.word(), sa.plain_logs);
    float* const erow = emit_label + emission_at(m.e_off, m.L, t, 0);
    for (int j = q; j < m.L; j += kLanes) {
        const float logit = j == q ? first_logit : load_elem(row, lab[j]), lp = log2_softmax(logit, mx, ls);
        erow[static_cast<size_t>(j) * kChunk] = sa.plain_logs ? lp : encode_emission(lp, exp2_from_max(logit, mx), norm);
        lowest = fminf(lowest, lp);
    }
    if (t == m.Tb - 1) store_virtual_frames(m, emit_blank, sa.emit_blank64, emit_label, sa.plain_logs, q, kLanes);
    raise_flags(meta, b, m, lowest);
}

// Alphabets beyond 8192 symbols: one workgroup per row, read three times (the row does not fit the registers).
// grid (T + 1, B): the extra column does the setup role.
template <typename T>
__global__ __launch_bounds__(kRowThreads)
void ctc_softmax_kernel(const T* __restrict__ x, T* __restrict__ grads,
                        Utt* __restrict__ meta,
                        const int* __restrict__ labels,
                        float* __restrict__ emit_blank, float* __restrict__ emit_label,
                        const SetupArgs sa, int Tt, int B, int A, int blank, int defer)
{
    __shared__ float red[8];
    __shared__ int s_lab[kSetupLabelSlots];
    const int t = blockIdx.x, b = blockIdx.y;
    const Utt m = meta[b];
    if (t == Tt) { setup_role(m, b, labels, sa, s_lab, 0, 1); return; }
    const size_t row_off = (static_cast<size_t>(t) * B + b) * A;
    T* grow = grads + row_off;
    const bool runs = (m.flags & kUttRuns) != 0;
    if (t >= m.Tb || !runs) {
        if (grads && (t & 15) >= defer)
            for (int k = threadIdx.x; k < A; k += kRowThreads) store_elem(grow, k, 0.0f);
        return;
    }
    const T* row = x + row_off;

    float mx = -__builtin_inff();
    for (int k = threadIdx.x; k < A; k += kRowThreads) mx = fmaxf(mx, load_elem(row, k));
    mx = block_max(mx, red);
    float sum = 0.0f;
    for (int k = threadIdx.x; k < A; k += kRowThreads)
        sum += fast_exp2((load_elem(row, k) - mx) * kLog2e);
    sum = block_sum(sum, red + 4);
    const float ls = fast_log2(sum);

    if (grads)
        for (int k = threadIdx.x; k < A; k += kRowThreads)
            store_elem(grow, k, fast_exp2(log2_softmax(load_elem(row, k), mx, ls)));
    const FrameNorm norm(load_elem(row, blank), mx, sum, ls);
    float lowest = norm.log_blank;
    if (threadIdx.x == 0) store_blank(emit_blank, sa.emit_blank64, static_cast<size_t>(m.f_off) + t, sa.plain_logs ? norm.log_blank : norm.word(), sa.plain_logs);
    if (t == m.Tb - 1) store_virtual_frames(m, emit_blank, sa.emit_blank64, emit_label, sa.plain_logs, threadIdx.x, kRowThreads);
    float* erow = emit_label + emission_at(m.e_off, m.L, t, 0);
    const int* lab = labels + m.lab_off;
    for (int j = threadIdx.x; j < m.L; j += kRowThreads) {
        const float logit = load_elem(row, lab[j]), lp = log2_softmax(logit, mx, ls);
        erow[static_cast<size_t>(j) * kChunk] = sa.plain_logs ? lp : encode_emission(lp, exp2_from_max(logit, mx), norm);
        lowest = fminf(lowest, lp);
    }
    raise_flags(meta, b, m, lowest);
}

// The zero rows that the softmax launch has left (t % 16 < defer): the last of them by the label columns' launch, the others by
// workgroups of the lattice launch that land on compute units without a chain.  Workgroup i runs on compute unit i mod n_cu (see order_chains), so those whose place in
// a round is a chain's leave at once.  (64 x 500 x 6000: 10 us less in the softmax launch, 6.5 more in this one.)
struct FillArgs {
    void* grads;
    int elem_bytes;
    int T, B, A;
    int first, defer;         // of every 16 frames, `defer` from `first` on; 0: nothing to fill
    int n_cu, n_chains, rounds;
};
// By a workgroup, a wavefront per row: every workers-th row from the wavefront's own on.
__device__ __forceinline__ void fill_rows(const FillArgs& f, const Utt* __restrict__ meta, int worker, int workers);
__device__ __forceinline__ void fill_rows_beside_chains(const FillArgs& f, const Utt* __restrict__ meta)
{
    const int place = static_cast<int>(blockIdx.x) % f.n_cu, round = static_cast<int>(blockIdx.x) / f.n_cu;
    if (place < f.n_chains) return;
    const int waves = blockDim.x >> 6, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int idle = f.n_cu - f.n_chains;
    fill_rows(f, meta, (round * idle + place - f.n_chains) * waves + wave, idle * f.rounds * waves);
}
__device__ __forceinline__ void fill_rows(const FillArgs& f, const Utt* __restrict__ meta, const int worker, const int workers)
{
    const int lane = threadIdx.x & 63;
    const int frames = f.T / 16 * f.defer + min(max(f.T % 16 - f.first, 0), f.defer);
    const int row_bytes = f.A * f.elem_bytes;
    for (int64_t i = worker; i < static_cast<int64_t>(frames) * f.B; i += workers) {
        const int k = static_cast<int>(i / f.B), b = static_cast<int>(i - static_cast<int64_t>(k) * f.B);
        const int t = k / f.defer * 16 + f.first + k % f.defer;
        const int frames_of_b = (meta[b].flags & kUttRuns) ? meta[b].Tb : 0;
        if (t < frames_of_b) continue;
        char* const row = static_cast<char*>(f.grads) + (static_cast<size_t>(t) * f.B + b) * row_bytes;
        const int head = min(static_cast<int>((16 - (reinterpret_cast<uintptr_t>(row) & 15)) & 15), row_bytes);
        const int vectors = (row_bytes - head) / 16, tail = row_bytes - head - vectors * 16;
        typedef uint32_t v4u __attribute__((ext_vector_type(4)));
        for (int n = lane; n < vectors; n += 64) __builtin_nontemporal_store(v4u{0, 0, 0, 0}, reinterpret_cast<v4u*>(row + head) + n);
        // (rows are whole elements of two or four bytes, and so are what lies before and after the vectors)
        if (2 * lane < head) *reinterpret_cast<uint16_t*>(row + 2 * lane) = 0;
        if (2 * lane < tail) *reinterpret_cast<uint16_t*>(row + head + vectors * 16 + 2 * lane) = 0;
    }
}

// The emissions of 64 frames of a narrow alphabet into lp[64][A], a quad of lanes per frame, and behind them the frames'
// words (log2 y_blank if plain_logs).  Returns the smallest log2 probability among this lane's.
// kPerLane of a row's symbols to a lane, in registers from their load to the emission: a row costs one memory latency and, with a
// fixed number of them, no loops around exponentials.  (Kept in LDS between the maximum, the sum and the emission, and stored a
// word at a time: 4 x 50 frames of 29 symbols 15.0 us a call, so 13.9; one utterance of 750 40.7, 39.4; 64 x 750 51.3, 49.7, of 64
// symbols 57.2, 52.7; 512 x 750 131.5, 128.9; with the label and the image asked for together, which is 0.3 of it.)
template <int kPerLane, typename T>
__device__ __forceinline__ float narrow_rows_of(const T* __restrict__ x, float* lp, int Tb, int b, int t0, int B, int A, int blank, bool plain_logs)
{
    constexpr int kPerRow = 4;
    const int tid = threadIdx.x;
    const int r = tid / kPerRow, q = tid % kPerRow, t = t0 + r;
    float lowest = 0.0f;
    if (t < Tb) {
        float* const lrow = lp + r * A;
        const T* const row = x + (static_cast<size_t>(t) * B + b) * A;
        const float blank_logit = load_elem(row, blank);
        float v[kPerLane];
#pragma unroll
        for (int u = 0; u < kPerLane; ++u) v[u] = load_elem(row, min(q + u * kPerRow, A - 1));
        float mx = -__builtin_inff();
#pragma unroll
        for (int u = 0; u < kPerLane; ++u) mx = fmaxf(mx, v[u]);         // (the last symbol again where there is none)
        mx = quad_max(mx);
        float from_max[kPerLane], sum = 0.0f;
#pragma unroll
        for (int u = 0; u < kPerLane; ++u) {
            from_max[u] = exp2_from_max(v[u], mx);
            sum += q + u * kPerRow < A ? from_max[u] : 0.0f;
        }
        sum = quad_sum(sum);
        const float ls = fast_log2(sum);
        const FrameNorm norm(blank_logit, mx, sum, ls);
        if (q == 0) lp[kFlagFrames * A + r] = plain_logs ? norm.log_blank : norm.word();
#pragma unroll
        for (int u = 0; u < kPerLane; ++u) {
            const int k = q + u * kPerRow;
            const float l = log2_softmax(v[u], mx, ls), e = plain_logs ? l : (k == blank ? encode_blank(norm) : encode_emission(l, from_max[u], norm));
            lowest = fminf(lowest, l);
            if (k < A) lrow[k] = e;
        }
    }
    return lowest;
}
template <typename T>
__device__ __forceinline__ float narrow_rows(const T* __restrict__ x, float* lp, int Tb, int b, int t0, int B, int A, int blank, bool plain_logs)
{
    static_assert(kDirectMaxA <= 64, "sixteen symbols to a lane");
    return A <= 32 ? narrow_rows_of<8>(x, lp, Tb, b, t0, B, A, blank, plain_logs) : narrow_rows_of<16>(x, lp, Tb, b, t0, B, A, blank, plain_logs);
}

// A workgroup's share of the emission block: kRows frames from t0 on whose coded rows sit in lp[kRows][A], virtual
// frames past the utterance's end.  kRows is a whole number of chunks.
template <int kRows>
__device__ __forceinline__ void store_symbol_chunks(const float* lp, int Tb, unsigned f_off, int64_t e_off, int t0, int A, int blank,
                                                    float* __restrict__ emit_blank, double* __restrict__ emit_blank64,
                                                    float* __restrict__ emit_label, bool plain_logs)
{
    const int tid = threadIdx.x, rows = min(kRows, Tb - t0), padded = min(kRows, static_cast<int>(padded_frames(Tb)) - t0);
    if (tid < padded)
        store_blank(emit_blank, emit_blank64, static_cast<size_t>(f_off) + t0 + tid, tid < rows ? lp[kRows * A + tid] : virtual_emission(true, plain_logs), plain_logs);
    // a wavefront per chunk: [symbol][frame], 8 A floats in a row
    float* const out = emit_label + kLabelSlack + e_off + static_cast<size_t>(t0) * A;
    for (int chunk = tid >> 6; chunk * kChunk < padded; chunk += kRowThreads / 64)
        for (int i = tid & 63; i < 2 * A; i += 64) {
            const int a = i >> 1, r = chunk * kChunk + 4 * (i & 1);
            float e[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) e[k] = lp[(r + k) * A + a];
#pragma unroll
            for (int k = 0; k < 4; ++k) e[k] = r + k < rows ? e[k] : virtual_emission(a == blank, plain_logs);
            *reinterpret_cast<float4*>(out + chunk * kChunk * A + 4 * i) = make_float4(e[0], e[1], e[2], e[3]);
        }
}

// Alphabets of at most kDirectMaxA symbols, more utterances than the narrow launch below takes: a workgroup takes 64
// consecutive frames of one utterance, four lanes per frame; the normalised rows sit in LDS (64 A floats, dynamic) and go
// out as the emission block.  grid (ceil(T / 64) + 1, B), the extra column does the setup role.
template <typename T>
__global__ __launch_bounds__(kRowThreads)
void ctc_softmax_symbols_kernel(const T* __restrict__ x, Utt* __restrict__ meta,
                                float* __restrict__ emit_blank, float* __restrict__ emit_label,
                                const SetupArgs sa, int B, int A, int blank)
{
    constexpr int kRows = 64;
    extern __shared__ float lp[];                          // [kRows][A], [kRows]
    const int b = blockIdx.y;
    const Utt m = meta[b];
    if (blockIdx.x == gridDim.x - 1) {
        setup_words(m, b, sa);
        return;
    }
    const int t0 = blockIdx.x * kRows;
    if (!(m.flags & kUttRuns) || t0 >= m.Tb) return;
    const float lowest = narrow_rows(x, lp, m.Tb, b, t0, B, A, blank, sa.plain_logs);
    raise_flags(meta, b, m, lowest);
    __syncthreads();
    store_symbol_chunks<kRows>(lp, m.Tb, m.f_off, m.e_off, t0, A, blank, emit_blank, sa.emit_blank64, emit_label, sa.plain_logs);

}

// The narrowest alphabets (at most kDirectMaxA symbols), host-resident metadata: the first launch of
// the call.  There is no upload launch before it: every workgroup reads its utterance's record out
// of the pinned host image itself (one PCIe round trip, which the upload launch cost as well, but
// no launch boundary after it), and the workgroups of the setup role, besides their own work, copy
// the image into the workspace for the launches that follow.  Nothing in this launch writes where
// another of its workgroups reads: instead of raising a flag in the utterance's record, a workgroup
// that meets an emission too small for the linear domain says so in a word of its own
// (row_flags: one per kFlagFrames frames of an utterance, written by every workgroup that has rows),
// which the chains gather when they start.
// A workgroup takes 64 frames of one utterance, four lanes per frame, so that it has several
// kilobytes under way; the normalised rows are the emission block (kEmitSymbols).
// grid (ceil(T / 64) + parts, B); dynamic LDS 64 * A floats.
struct NarrowImage {
    const int* words;         // the pinned image: meta, order, labels as they lie in the workspace, then the labels as bytes
    int labels_first, labels_end;   // the label strings' place in it (4-byte words): not copied, the setup role writes them
    int count;                // words to copy (up to the byte labels)
    size_t labels8_offset;    // of the byte labels (bytes)
    int* labels_out;          // the workspace's label strings
};
// What the workgroups with rows need to know of an utterance travels with the kernel's arguments
// (hundreds of small reads out of host memory at once were measured to take longer than the upload
// launch they replace): its frames, with kRowsRun set if its chains run, and the frames of all
// utterances before it (padded).  An utterance's emission block starts A times that many floats into the region.
constexpr int kRowsRun = 1 << 30;     // (a flag of the record that rides along)
struct NarrowRows {
    int frames[kNarrowMaxB];
    unsigned frames_before[kNarrowMaxB];
    int label_length[kNarrowMaxB];       // and, for the setup role, the label's length and the symbols before it
    int labels_before[kNarrowMaxB];
};
// Either that (host-resident metadata) or the wavefront plans by label length (device-resident
// metadata: see NarrowDevice), in the same 2 KB of kernel arguments.
union NarrowArgs {
    NarrowRows rows;
    PlanTable plans;
};

// Device-resident metadata (ctc_loss_and_grad_device): there is no image and there are no records
// yet.  The workgroups with rows derive what they need from the lengths themselves (blocks are laid
// out by the caller's bounds: see ctc_plan_kernel); the first setup workgroup of an utterance builds
// its record, as ctc_plan_kernel does for wider alphabets in a launch of its own, and finds the
// utterance's place in the run order by counting the utterances that weigh more (all utterances
// take part, those without an alignment too: their chains' workgroups leave at once).
struct NarrowDevice {
    const int* labels;            // [B][max_label]; nullptr: the metadata is the host's (NarrowImage, NarrowRows)
    const int* label_lengths;
    const int* input_lengths;
    Utt* meta;                    // records to build
    int* order;
    int* status_words;            // [B] nonzero: the utterance's lengths or labels are invalid
    int max_label, poll_budget;
    bool crowded, log_domain;
    int n_cu;                     // compute units of the device (a multiple of kChainBlock, or 0: keep the plain order)
};

// Weight of an utterance in the run order (chain_weight; 0: its lengths are out of range).  Every utterance's setup weighs all of them, by their lengths alone: tight fits that
// only repeated neighbours make weigh as if they ran on probabilities.
// (Few instructions: of a batch of short utterances the setup is the softmax launch's longest, and takes 5 clocks for each.  64 x 93 x 30, lengths from 11 on, that launch 5.05 us with frames times
// wavefronts, 5.4 with each form's time in branches, so 5.2.)
__device__ __forceinline__ long long weight_of(const PlanTable& plans, int L, int Tb, int Tt, int max_label, bool log_domain, bool crowded)
{
    const bool in_range = L >= 0 && L <= max_label && Tb >= 0 && Tb <= Tt;
    const int one = plans.one[in_range ? L : 0], two = plans.two[in_range ? L : 0];      // (both at once: one after the other took a trip to memory more)
    const bool logs = log_domain || Tb > kLinearMaxFrames || tight_fit(Tb, L, 0);
    const ChainForm form = chain_form((logs ? kUttLogDomain : 0) | ((one & 128) ? kUttTwoPairs : 0), false);
    return in_range ? chain_weight(Tb, ((form == ChainForm::kTwoPairs ? two : one) & 15) + 1, form, crowded) : 0;
}
// By the whole workgroup.  Returns the record (the same in every thread).
__device__ __forceinline__ Utt build_record(const NarrowDevice& dv, const PlanTable& plans, int b, int Tt, int B, int A,
                                            int blank)
{
    __shared__ int s_repeats, s_bad, s_rank;
    const int tid = threadIdx.x;
    const int L_in = dv.label_lengths[b], Tb_in = dv.input_lengths[b];
    const bool bad_length = L_in < 0 || L_in > dv.max_label || Tb_in < 0 || Tb_in > Tt;
    const int L = bad_length ? 0 : L_in;
    if (tid == 0) {
        s_repeats = 0;
        s_bad = 0;
        s_rank = 0;
    }
    __syncthreads();
    const int* lab = dv.labels + static_cast<size_t>(b) * dv.max_label;
    int repeats = 0, bad = 0;
    for (int j = tid; j < L; j += kRowThreads) {
        const int c = lab[j];
        bad |= (c < 0 || c >= A || c == blank) ? 1 : 0;
        repeats += (j > 0 && c == lab[j - 1]) ? 1 : 0;
    }
    if (repeats) atomicAdd(&s_repeats, repeats);
    if (bad) s_bad = 1;
    // the utterances that come before this one in the run order: heavier, or as heavy and earlier
    const long long mine = weight_of(plans, L_in, Tb_in, Tt, dv.max_label, dv.log_domain, dv.crowded);
    int before = 0;
    for (int j = tid; j < B; j += kRowThreads) {
        const int Lj = dv.label_lengths[j], Tj = dv.input_lengths[j];
        const long long w = weight_of(plans, Lj, Tj, Tt, dv.max_label, dv.log_domain, dv.crowded);
        before += (w > mine || (w == mine && j < b)) ? 1 : 0;
    }
    if (before) atomicAdd(&s_rank, before);
    __syncthreads();
    const bool invalid = bad_length || s_bad != 0;
    const int Tb = invalid ? 0 : Tb_in;
    const bool runs = !invalid && Tb > 0 && Tb >= L + s_repeats;
    const int Lp = invalid ? 0 : L;
    Utt m;
    m.Tb = Tb;
    m.L = Lp;
    m.lab_off = b * dv.max_label;
    m.flags = (runs ? kUttRuns : 0) | (invalid ? kUttInvalid : 0) |
              ((dv.log_domain || Tb > kLinearMaxFrames || tight_fit(Tb, L, s_repeats)) ? kUttLogDomain : 0) |
              (!invalid && plans.two_pairs(L) ? kUttTwoPairs : 0);
    const int padded = static_cast<int>(padded_frames(Tt)), longest = longest_aligned(Tt, dv.max_label);
    m.f_off = static_cast<unsigned>(b) * padded;
    m.waves = plans.waves1(Lp);
    m.halo = plans.halo1(Lp);
    m.waves2 = plans.waves2(Lp);
    m.halo2 = plans.halo2(Lp);
    m.poll_budget = dv.poll_budget;
    m.e_direct = emission_layout(A);
    m.rough = 0;
    m.steep = 0;
    m.e_cols = m.e_direct == kEmitSymbols ? A : m.L;
    m.e_off = b * (m.e_direct == kEmitSymbols ? static_cast<int64_t>(padded) * A : gathered_emissions(Tt, longest));
    m.ab_off = b * lattice_words(Tt, longest);
    if (tid == 0) {
        dv.meta[b] = m;
        dv.status_words[b] = invalid ? 1 : 0;
        // heaviest first, in blocks of kChainBlock utterances: a block's forward chains, then its backward chains
        // Launches of more chains than compute units: workgroup i shares its compute unit with workgroups
        // i +- n_cu, so every other round of n_cu chains runs lightest first, and a compute unit's chains
        // add up to about the same (the host's order_chains goes by the SIMDs' loads; this is its first-order part).
        int rank = s_rank;
        dv.order[2 * B + B - 1 - rank] = b;              // (the utterances by when their chains end)
        const int per_round = dv.n_cu / 2;
        if (per_round >= kChainBlock && B * 2 > dv.n_cu && ((rank / per_round) & 1)) {
            const int round_first = rank - rank % per_round, in_round = min(per_round, B - round_first);
            rank = round_first + (in_round - 1 - rank % per_round);
        }
        const int first = rank - rank % kChainBlock, in_block = min(kChainBlock, B - first);
        for (int d = 0; d < 2; ++d) dv.order[first * 2 + d * in_block + rank % kChainBlock] = 2 * b + d;
    }
    return m;
}

template <typename T>
__global__ __launch_bounds__(kRowThreads)
void ctc_softmax_narrow_kernel(const T* __restrict__ x, const NarrowImage image, int* __restrict__ workspace_words,
                               float* __restrict__ emit_blank,
                               float* __restrict__ emit_label, int* __restrict__ row_flags,
                               const SetupArgs sa, const NarrowArgs args, const NarrowDevice dv,
                               int Tt, int B, int A, int blank)
{
    constexpr int kRows = kFlagFrames;
    static_assert(kRows * 4 == kRowThreads, "a quad per frame (narrow_rows)");
    extern __shared__ float lp[];                          // [kRows][A], [kRows]
    __shared__ int s_flags;
    const int b = blockIdx.y, tid = threadIdx.x;
    const int row_blocks = static_cast<int>(gridDim.x) - sa.parts;
    if (static_cast<int>(blockIdx.x) >= row_blocks && dv.labels) {
        // device-resident metadata: this workgroup builds the record and writes what depends on it
        setup_words(build_record(dv, args.plans, b, Tt, B, A, blank), b, sa);
        return;
    }
    if (static_cast<int>(blockIdx.x) >= row_blocks) {
        // (what is used of the utterance's record comes with the arguments: no read of the record out of host memory,
        // so that its share of the image is the first and only thing this workgroup waits for from there)
        Utt m{};
        m.Tb = args.rows.frames[b] & (kRowsRun - 1);
        m.flags = (args.rows.frames[b] & kRowsRun) ? kUttRuns : 0;
        m.L = args.rows.label_length[b];
        m.lab_off = args.rows.labels_before[b];
        const int part = static_cast<int>(blockIdx.x) - row_blocks;
        // this workgroup's share of the image
        const int groups = B * sa.parts, group = b * sa.parts + part;
        const int share = (image.count + groups - 1) / groups;
        // its utterance's label, from the bytes; both asked for before either is used: each is a trip to host memory
        const unsigned char* const labels8 = reinterpret_cast<const unsigned char*>(image.words) + image.labels8_offset + m.lab_off;
        const int end = min((group + 1) * share, image.count), length = part == 0 ? m.L : 0;
        int i = group * share + tid, j = tid;
        do {
            // (the label strings' own words are not written by the host where there are bytes, and not asked for)
            const bool copied = i < end && (i < image.labels_first || i >= image.labels_end);
            const int word = copied ? image.words[i] : 0;
            const int symbol = j < length ? labels8[j] : 0;
            __builtin_amdgcn_sched_barrier(0);
            if (copied) workspace_words[i] = word;
            if (j < length) image.labels_out[m.lab_off + j] = symbol;
            i += kRowThreads;
            j += kRowThreads;
        } while (i - tid < end || j - tid < length);
        if (part == 0) setup_words(m, b, sa);
        return;
    }
    // (the fields of the utterance's record that the rows need)
    struct { int Tb, flags; unsigned f_off; int64_t e_off; } m;
    if (dv.labels) {
        // (whether an alignment exists is not known here: the rows of every utterance with frames are prepared)
        const int L = dv.label_lengths[b], Tb = dv.input_lengths[b];
        const bool bad_length = L < 0 || L > dv.max_label || Tb < 0 || Tb > Tt;
        m.Tb = bad_length ? 0 : Tb;
        m.flags = kUttRuns;
        m.f_off = static_cast<unsigned>(b) * static_cast<int>(padded_frames(Tt));
    } else {
        m.Tb = args.rows.frames[b] & (kRowsRun - 1);
        m.flags = (args.rows.frames[b] & kRowsRun) ? kUttRuns : 0;
        m.f_off = args.rows.frames_before[b];
    }
    m.e_off = static_cast<int64_t>(m.f_off) * A;
    const int t0 = blockIdx.x * kRows;
    if (t0 >= m.Tb || !(m.flags & kUttRuns)) return;
    if (tid == 0) s_flags = 0;
    const float lowest = narrow_rows(x, lp, m.Tb, b, t0, B, A, blank, sa.plain_logs);
    __syncthreads();
    store_symbol_chunks<kRows>(lp, m.Tb, m.f_off, m.e_off, t0, A, blank, emit_blank, sa.emit_blank64, emit_label, sa.plain_logs);
    if (__ballot(lowest < kGentleMinLog2) != 0) {
        // (once a wavefront: one lane after the other on one word takes longer than the rows where many have something to say)
        const int met = kRowsRough | (__ballot(lowest < kRoughMinLog2) != 0 ? kRowsSteep : 0) | (__ballot(lowest < kLinearMinLog2) != 0 ? kRowsSmall : 0);
        if ((tid & 63) == 0) atomicOr(&s_flags, met);
    }
    __syncthreads();
    if (tid == 0) row_flags[static_cast<size_t>(b) * row_blocks + blockIdx.x] = s_flags;
}

// What the narrow softmax launch has met in an utterance's frames: kRowsSmall, kRowsRough, kRowsSteep.  Asked by a whole wavefront; the same
// answer in every lane.
__device__ __forceinline__ int rows_flagged(const int* __restrict__ row_flags, int b, int blocks_per_utterance, int Tb)
{
    if (!row_flags) return 0;
    const int lane = threadIdx.x & 63, n = (Tb + kFlagFrames - 1) / kFlagFrames;
    int any = 0;
    for (int i = lane; i < n; i += 64) any |= row_flags[static_cast<size_t>(b) * blocks_per_utterance + i];
    if (__builtin_expect(__ballot(any != 0) == 0, 1)) return 0;
    auto met = [&](int which) { return __ballot(any & which) != 0 ? which : 0; };
    return met(kRowsSmall) | met(kRowsRough) | met(kRowsSteep);
}

// ---- lattice storage -------------------------------------------------------------------------
// What the recursions leave for the gradient.
//
// Linear-domain chains store their whole state once per block of kBlockFrames frames (a checkpoint); the gradient runs
// both recursions once more over the frames of a block, from the checkpoints at its two ends, and forms the shares from
// the values in its registers.  Storing the label states of every frame instead (4.5 bytes per state, frame and
// direction, written by the chains and read by the gradient) cost the chains a fifth of their time -- a store is three
// to four issue slots of a lone wavefront and the wavefronts of a compute unit share its memory pipeline -- and bound
// the gradient by the bytes it read; a checkpoint is 20 bytes per state and block, 1.25 per frame.
//   alpha, after frame 16 k + 15:  per label position j  (blank j, label j) as doubles, and their frame (int32)
//   beta, after frame 16 k:        per label position j  (blank j + 1, label j)
// (inclusive quantities, see the recursions), position j in column 1 + j.  Rows lie in the order in which the chain stores them, the
// last one, which nobody asks for, left out; a row's 16-byte states come first, those of even columns before those of odd ones, then its
// frames (CheckpointRow).  All of it in the first half of the direction's region.
// (Where a lane stores two columns next to each other, either store otherwise writes half of every 32 bytes, and past the die's cache nobody
// puts them together: 512 x 750 frames, 29 symbols, three minibatches in turn, gradient beside the chains, 134.2 us a call.)
//
// Log-domain chains (rare) store every frame, per label state a number m * 2^e, as
//   a value word (uint32): the high dword of the fp64 m (sign, exponent, top 20 mantissa bits),
//   an exponent word (int32): e,
// both in rows of lattice_pitch(L) words by frame, values and exponents in the two halves of the region.
// Twenty mantissa bits bound the relative error of a state's share alpha * beta / p by 2^-19, which is 2e-6 of a gradient
// entry at most.  Exponents stay above -2^30 so that the sum of two cannot wrap.
//
// Wavefronts of linear-domain chains that have gone on with an exponent to every state (finish_with_exponents) store checkpoints, and hand states up, with
// kLogs as their frame and logarithms in the values' places (coded_logs).
//
// The mass p of an utterance (its reciprocal) keeps both parts in one 8-byte word (pack_state).
struct alignas(16) CheckpointState { double blank, label; };
struct CheckpointRow {
    int64_t pitch;                                       // columns
    __device__ __forceinline__ int64_t half() const { return (pitch + 1) / 2; }
    __device__ __forceinline__ int slot(int column) const { return (column >> 1) + ((column & 1) ? static_cast<int>(half()) : 0); }
    // (whole pieces of 64 bytes, as the region begins: 64 * pitch of them are there for a row)
    __device__ __forceinline__ int64_t bytes() const { return (frames_at() + pitch * static_cast<int64_t>(sizeof(int)) + 63) / 64 * 64; }
    __device__ __forceinline__ int64_t frames_at() const { return 2 * half() * static_cast<int64_t>(sizeof(CheckpointState)); }
    // (a block has fewer than 2^31 bytes: make_layout)
    __device__ __forceinline__ unsigned at(int row) const { return static_cast<unsigned>(row) * static_cast<unsigned>(bytes()); }
    __device__ __forceinline__ const CheckpointState* states(const uint32_t* block, int row) const
    {
        return reinterpret_cast<const CheckpointState*>(reinterpret_cast<const char*>(block) + at(row));
    }
    __device__ __forceinline__ const int* frames(const uint32_t* block, int row) const
    {
        return reinterpret_cast<const int*>(reinterpret_cast<const char*>(block) + at(row) + frames_at());
    }
};
constexpr int kNoExponent = -(1 << 28);   // exponent of zero: below every real one, far from int32's ends
// No frame: the values are logarithms.  They are coded such that nobody who renews frames has to ask for it: a renewal that meets the frame, in its own lane
// or below it, finds the lane's first blank 2^1000 below its label, or below 2^kLogs, and so strained (kStrained).
constexpr int kLogs = 1 << 30;
constexpr double kLogOffset = 0x1p29, kLogZeroCode = 0x1p20, kBlankLogScale = 0x1p-1000;      // (fp64 keeps 23 bits behind the point)

__device__ __forceinline__ double pack_state(double in_frame, int frame)
{
    return __hiloint2double(__double2hiint(in_frame), frame);
}
// (the exponent below it is no part of the mantissa: a negative one would read as nearly another 2^-20)
__device__ __forceinline__ float packed_mantissa(double packed)
{
    return static_cast<float>(__hiloint2double(__double2hiint(packed), 0));
}
// A base-2 logarithm (log-domain chains) as value and exponent: m = 2^fraction in [1, 2), e = floor.
// log 0 (and anything as small) is stored as the number 0 with the exponent of zero.
__device__ __forceinline__ void split_log2(double w, uint32_t& value, int& exponent)
{
    const double whole = floor(w);
    const double m = static_cast<double>(fast_exp2(static_cast<float>(w - whole)));
    const bool real = w > -1.0e9 && w < 1.0e9;
    value = real ? static_cast<uint32_t>(__double2hiint(m)) : 0u;
    exponent = real ? static_cast<int>(whole) : kNoExponent;
}
__device__ __forceinline__ double pack_log2(double w)          // the same as one word (1 / p)
{
    uint32_t value;
    int exponent;
    split_log2(w, value, exponent);
    return __hiloint2double(static_cast<int>(value), exponent);
}

// ---- lattice recursions ------------------------------------------------------------------
// What the chains leave may be read by workgroups of the same launch, on other dies, once they know the chains to have
// ended (announce_end): both sides go past the dies' own caches.
__device__ __forceinline__ void publish(int* p, int v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void publish(double* p, double v)
{
    __hip_atomic_store(reinterpret_cast<long long*>(p), __double_as_longlong(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int published(const int* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ double published(const double* p)
{
    return __longlong_as_double(__hip_atomic_load(reinterpret_cast<const long long*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
__device__ __forceinline__ CheckpointState published(const CheckpointState* p) { return {published(&p->blank), published(&p->label)}; }

// Where a linear-domain chain's lane stores its states and frames, row after row.  Through a buffer resource, for three reasons.
// Stores with kPast go past the die's cache as publish() does, but sixteen bytes at a time, and the compiler goes on counting them among
// the memory operations in flight.  With plain stores a chain had to have its die's cache written back at its end, during which every
// chain on the die waited a microsecond for its emissions: 64 x 750 frames, 29 symbols, blocks of 16 frames that take 0.44 us took up to
// 1.5 us once the short utterances ended.  A lane that has nothing to store gets an offset beyond the buffer's end, where the
// hardware drops stores.  And so is the row after the last one dropped, for which the chain's end would have to wait.
constexpr int kPast = 16;                                // (cache policy: sc1)
struct CheckpointRows {
    static constexpr unsigned kNowhere = 0x80000000u;    // (a block has fewer bytes: make_layout)
    __amdgpu_buffer_rsrc_t block;
    unsigned state_at, next_state_at, frame_at;          // in the row, of this lane's column and the one after it
    int at, next_by, step;                               // of the row
    __device__ __forceinline__ CheckpointRows(uint32_t* out, CheckpointRow row, int rows, bool stores, int column)
        : block(__builtin_amdgcn_make_buffer_rsrc(out, 0, static_cast<int>(rows * row.bytes()), 0x00020000)),
          state_at(stores ? static_cast<unsigned>(row.slot(column) * sizeof(CheckpointState)) : kNowhere),
          next_state_at(stores ? static_cast<unsigned>(row.slot(column + 1) * sizeof(CheckpointState)) : kNowhere),
          frame_at(stores ? static_cast<unsigned>(row.frames_at() + column * sizeof(int)) : kNowhere),
          at(0), next_by(0), step(static_cast<int>(row.bytes()))
    {
    }
    __device__ __forceinline__ void drop() { state_at = next_state_at = frame_at = kNowhere; }
    typedef unsigned Words4 __attribute__((ext_vector_type(4)));
    typedef unsigned Words2 __attribute__((ext_vector_type(2)));
    template <int kPolicy>
    __device__ __forceinline__ void state(int column, const CheckpointState& s) const
    {
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(Words4, s), block, static_cast<int>(column == 0 ? state_at : next_state_at), at, kPolicy);
    }
    template <int kPolicy>
    __device__ __forceinline__ void frame(int f) const { __builtin_amdgcn_raw_buffer_store_b32(static_cast<unsigned>(f), block, static_cast<int>(frame_at), at, kPolicy); }
    // (the same in two neighbouring columns)
    template <int kPolicy>
    __device__ __forceinline__ void frames(int f) const
    {
        __builtin_amdgcn_raw_buffer_store_b64(Words2{static_cast<unsigned>(f), static_cast<unsigned>(f)}, block, static_cast<int>(frame_at), at, kPolicy);
    }
    // (a chain stores when it begins a block; what the first one stores in the first row, the second one stores over)
    __device__ __forceinline__ void next()
    {
        at += next_by;
        next_by = step;
    }
};

__device__ __forceinline__ CheckpointState coded_logs(double blank, double label)
{
    auto code = [](double w) { return w > -1.0e9 ? w + kLogOffset : kLogZeroCode; };
    return {code(blank) * kBlankLogScale, code(label)};
}
// log2 of a pair's states, from their values and frame.
__device__ __forceinline__ CheckpointState state_logs(const CheckpointState& s, int frame, double log0 = kNeg)
{
    auto decoded = [&](double v) { return v > 0x1p27 ? v - kLogOffset : log0; };
    auto log2_of = [&](double v) {
        const double log2 = static_cast<double>(frame + __builtin_amdgcn_frexp_exp(v)) + static_cast<double>(fast_log2(static_cast<float>(__builtin_amdgcn_frexp_mant(v))));
        return v > 0.0 ? log2 : log0;
    };
    return {frame == kLogs ? decoded(s.blank * 0x1p1000) : log2_of(s.blank), frame == kLogs ? decoded(s.label) : log2_of(s.label)};
}
// log2(2^a + 2^b) for fp64 a, b with the exponentials taken on the fp32 difference.
__device__ __forceinline__ double lse2(double a, double b)
{
    const double hi = fmax(a, b);
    const float d = static_cast<float>(a - b);
    return hi + static_cast<double>(fast_log2(1.0f + fast_exp2(-fabsf(d))));
}
// Lane i receives the value of lane i-1 (DPP wave_shr:1).  The shift writes nothing into lane 0,
// which therefore keeps what `into` held there: initialised once to log 0 and passed back in at
// every step, it needs no refill (two moves per step otherwise).
__device__ __forceinline__ double shift_up(double v, int& into_lo, int& into_hi)
{
    into_lo = __builtin_amdgcn_update_dpp(into_lo, __double2loint(v), 0x138, 0xf, 0xf, false);
    into_hi = __builtin_amdgcn_update_dpp(into_hi, __double2hiint(v), 0x138, 0xf, 0xf, false);
    return __hiloint2double(into_hi, into_lo);
}

// max(window of the lane below, mine) in one instruction, the DPP shift as an operand of the maximum.
// Lane 0 has no lane below: the instruction then leaves its register alone, and `window` starts out as
// the lanes' own values.  (s_nop 1: a DPP operand must be two wait states old.)
__device__ __forceinline__ int window_max_step(int window, int mine)
{
    asm("s_nop 1\n\tv_max_i32_dpp %0, %0, %1 wave_shr:1 row_mask:0xf bank_mask:0xf" : "+v"(window) : "v"(mine));
    return window;
}

// The same, and the lane above in place of the lane below (the gradient's backward recursion); lane 63 has none.
__device__ __forceinline__ int window_max_step_down(int window, int mine)
{
    asm("s_nop 1\n\tv_max_i32_dpp %0, %0, %1 wave_shl:1 row_mask:0xf bank_mask:0xf" : "+v"(window) : "v"(mine));
    return window;
}
// Lane i receives the value of lane i - 1 (kDown: i + 1), and a lane without such a neighbour zero.
template <bool kDown>
__device__ __forceinline__ double lane_shift(double v)
{
    constexpr int kCtrl = kDown ? 0x130 : 0x138;
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(v), kCtrl, 0xf, 0xf, true),
                            __builtin_amdgcn_update_dpp(0, __double2loint(v), kCtrl, 0xf, 0xf, true));
}

// What is kept of an utterance's mass p (of its frames divided by their norms), kMassWords doubles:
//   kMassInverse  1 / p for the gradient, mantissa and exponent in one word (pack_state)
//   kMassValue, kMassLog2  two numbers x and y with log2 p = log2 x + y, for the cost
//   kMassNorms  cost-only calls: log2 of the product of the norms
constexpr int kMassInverse = 0, kMassValue = 1, kMassLog2 = 2, kMassNorms = 3;
static_assert(kMassWords == 4, "four words");
__device__ __forceinline__ float cost_of_mass(double x, double y, double log2_norms)
{
    // (in double: once per utterance, and a cost near zero, p near 1, would keep few of a float logarithm's bits)
    return x > 0.0 ? static_cast<float>(-(::log2(x) + (y + log2_norms)) * kLn2) : __builtin_inff();
}
// The product of an utterance's norms, mantissa * 2^exponent.
struct Norms {
    double mantissa;                                     // [0.5, 1)
    int exponent;
    __device__ __forceinline__ Norms times(double other_mantissa, int other_exponent) const
    {
        const double product = mantissa * other_mantissa;
        return {__builtin_amdgcn_frexp_mant(product), exponent + other_exponent + __builtin_amdgcn_frexp_exp(product)};
    }
    __device__ __forceinline__ double log2() const { return static_cast<double>(exponent) + ::log2(mantissa); }
};
// A lane's part of it: frames lane, lane + 64, ...
__device__ __forceinline__ Norms norms_of_lane(const Utt& m, const float* __restrict__ emit_blank)
{
    const int lane = threadIdx.x & 63, frames = static_cast<int>(padded_frames(m.Tb));
    const float* const words = emit_blank + kBlankSlack + m.f_off;
    Norms product{0.5, 1};
    constexpr int kAhead = 12;
    for (int t0 = 0; t0 < frames; t0 += 64 * kAhead) {
        float c[kAhead];
#pragma unroll
        for (int i = 0; i < kAhead; ++i) c[i] = words[min(t0 + 64 * i + lane, frames - 1)];
#pragma unroll
        for (int i = 0; i < kAhead; ++i) {
            if (t0 + 64 * i >= frames) break;
            const double norm = t0 + 64 * i + lane < frames ? static_cast<double>(frame_norm(c[i])) : 1.0;
            product = product.times(norm, 0);
        }
    }
    return product;
}
// The parts of a wavefront's lanes (all of them active) put together: the same in every lane, and the same each time.
// (750 frames: 2.5 us for both together, most of it waiting for memory, so whoever has nothing else to do does it: the
// gradient's workgroups, which write the cost, or workgroups of their own in a cost-only call.)
template <int kCtrl>
__device__ __forceinline__ Norms norms_permuted(const Norms& n)
{
    auto move = [](int v) { return __builtin_amdgcn_update_dpp(0, v, kCtrl, 0xf, 0xf, true); };
    return {__hiloint2double(move(__double2hiint(n.mantissa)), move(__double2loint(n.mantissa))), move(n.exponent)};
}
__device__ __forceinline__ Norms norms_of_wave(Norms n)
{
    auto with = [](const Norms& a, const Norms& b) { return a.times(b.mantissa, b.exponent); };
    n = with(n, norms_permuted<0xB1>(n));                // (the patterns of row16_sum)
    n = with(n, norms_permuted<0x4E>(n));
    n = with(n, norms_permuted<0x141>(n));
    n = with(n, norms_permuted<0x140>(n));
    auto row = [&](int lane) {
        auto read = [&](int v) { return __builtin_amdgcn_readlane(v, lane); };
        return Norms{__hiloint2double(read(__double2hiint(n.mantissa)), read(__double2loint(n.mantissa))), read(n.exponent)};
    };
    return with(with(row(0), row(16)), with(row(32), row(48)));
}

constexpr int kHaloEntries = 64;      // 16-byte entries of one wavefront boundary's exchange buffer (2 x 32)

enum class Sync { kNone, kHalo, kBarrier };

static_assert(kChunk == 8, "fetch_chunk loads two float4");
template <bool kBackward>
__device__ __forceinline__ void fetch_chunk(const float*& p, int64_t step, float (&el)[kChunk])
{
    const float4 lo = *reinterpret_cast<const float4*>(p), hi = *reinterpret_cast<const float4*>(p + 4);
    constexpr int kFlip = kBackward ? kChunk - 1 : 0;
    el[0 ^ kFlip] = lo.x; el[1 ^ kFlip] = lo.y; el[2 ^ kFlip] = lo.z; el[3 ^ kFlip] = lo.w;
    el[4 ^ kFlip] = hi.x; el[5 ^ kFlip] = hi.y; el[6 ^ kFlip] = hi.z; el[7 ^ kFlip] = hi.w;
    p += step;
}
// Predecessor choices of a pair at one frame, as stored for the backtrace: three bits, the steps of a chunk in one word
// with the first step in the highest.  Bit 0: the blank state came from the label of the pair before (else it stayed).
// Bits 2 and 1, the label state: it came from the label of the pair before, skipping the blank; if not, it came from
// the pair's blank (else it stayed).  (A byte per frame and pair, stored at every step, took four issue slots of a step;
// a bit of the word is one, an addition with carry.)
constexpr int kChoiceBits = 3;
__device__ __forceinline__ unsigned append_bit(unsigned word, unsigned long long lanes)
{
    unsigned long long carry;
    asm("v_addc_co_u32_e64 %0, %1, %2, %2, %3" : "=v"(word), "=s"(carry) : "v"(word), "s"(lanes));
    return word;
}
// Every kSegment steps a chain also keeps, per state, which state the best way to it was in kSegment steps before (its
// origin), so that the backtrace walks all segments at once.
constexpr int kSegmentChunks = 4, kSegment = kSegmentChunks * kChunk;
// Words in the exponent block, after the last states: a segment's origins by pair, blank state's in the low half.
__host__ __device__ constexpr int64_t origin_word(int64_t pairs, int64_t segment) { return (4 + segment) * pairs; }


// LDS of a chain's workgroup (dynamic, sized by the launch for its widest chain): a header, then
// one block per wavefront that holds what that wavefront hands to the one above it.
struct HaloHeader {
    // Cost-only chains: the last wavefront to finish writes the cost (or NaN if any gave up).
    int finished;                     // wavefronts that have reached the end of the chain
    int gave_up;
    float cost;
    int left;                         // chains of a launch that writes the gradient too: see lattice_body
};
// Log-domain chains.
struct HaloWave {
    double2 data[kHaloEntries];
    int origins[kHaloEntries];        // Mode::kBest: blank state's in the low half
    int ready;                        // last generation this wavefront has published
    int done;                         // last generation this wavefront has taken from the one below
    int unused[2];
};

// Linear-domain chains: what a wavefront hands to the one above it at the end of a block, the states, frames and number of the hand-over of its upper lanes.
// kRing blocks: now and then a wavefront has a renewal to do that takes as long as a block, each at another time, and where one could only be two
// hand-overs ahead of the next, all of them waited for whoever was at it.
constexpr int kRing = 4;
template <int kPairs>
struct LinearWave {
    static constexpr int kLanes = 32 / kPairs;           // the widest halos (plan_waves, plan_waves2)
    struct alignas(16) Tag { int2 word; };               // (the lane's frame, number of the hand-over; as far apart as the states, so that one address serves)
    struct Slot {
        double2 states[kPairs][kLanes];
        Tag tag[kLanes];
    } slot[kRing];                                       // of a block's end, by the block's number
};
// How often the wavefronts of a chain hand over: never (there is one), at every block's end, at every second one's; or whichever of these it is (steep chains).
enum class Exchange { kNone, kBlock, kTwoBlocks, kAny };

// What a wavefront had when it left the recursion on probabilities (finish_with_exponents): a lane's states and frame (kLogs: they are logarithms).
// (In LDS, from where they are read again: as values that leave the loop from a dozen places they took more registers than there are.  So the wavefront goes
// on to the end of the loop's round, its stores going nowhere.)
struct StrainedWave {
    double2 states[2][64];
    int frame[64];
};
constexpr size_t kExchangeBytes = std::max({sizeof(HaloWave), sizeof(LinearWave<1>), sizeof(LinearWave<2>)});
constexpr size_t kHaloWaveBytes = kExchangeBytes + sizeof(StrainedWave);
static_assert(sizeof(HaloHeader) % 16 == 0 && kExchangeBytes % 16 == 0 && kHaloWaveBytes % 16 == 0, "the blocks hold 16-byte entries");
// Bytes of dynamic LDS of a lattice launch whose workgroups have `waves` wavefronts.
constexpr size_t halo_lds_bytes(int waves) { return sizeof(HaloHeader) + static_cast<size_t>(waves) * kHaloWaveBytes; }
template <typename Wave>
__device__ __forceinline__ Wave* halo_wave(void* lds, int wave)
{
    return reinterpret_cast<Wave*>(static_cast<char*>(lds) + sizeof(HaloHeader) + static_cast<size_t>(wave) * kHaloWaveBytes);
}
__device__ __forceinline__ StrainedWave* strained_wave(void* lds, int wave)
{
    return reinterpret_cast<StrainedWave*>(static_cast<char*>(lds) + sizeof(HaloHeader) + static_cast<size_t>(wave) * kHaloWaveBytes + kExchangeBytes);
}


// One chain = one direction of one utterance.  A lane owns the pair
//   forward : (blank state 2j,       label j        = state 2j+1)
//   backward: (blank state 2(L-j),   label L-1-j    = state 2(L-j)-1)
// so that in both directions the only value needed from a neighbour is the label entry of
// pair j-1 (one DPP shift), and both directions run the same recursion on the "inclusive"
// quantity
//   w_step(state) = E_frame(state) + log2 sum over predecessors of 2^w_{step-1}
// which is alpha going forward.  Going backward, the sum before E is added is the beta that
// excludes its own frame's emission, and that is what gets stored, so that
// log alpha + log beta is the log mass of alignments through a state.
//
// The gradient needs the label states' shares only and takes the blank's occupancy as 1 minus that of all label states
// (sum_s alpha_t(s) beta_t(s) = p at every frame).
//
// In the modes without a gradient the two chains of an utterance meet in the middle (chain_chunks): each runs over half
// of the frames and leaves its last state, which finish_loss (or the backtrace) combines.  (Log-domain chains of cost-only
// calls are too rare to be worth a second way of combining: there the forward chain runs all the way, alone.)
//
// A chain starts from the state "all mass in its first blank, before any frame" and takes whole chunks of the
// utterance's padded frames; virtual frames (emission_layout) leave the start state as it is, and a forward chain's
// virtual frames after the last real one only gather p in the last blank.
//
// A lone wavefront on its SIMD issues an instruction about every five clocks whatever its kind
// (a vector memory instruction counts for three), so the step is written for instruction count:
// pointers advance by adds, lanes without a pair write to a sink or nowhere, whole chunks run without a look
// at the step number.
//
// Labels of more than 63 symbols span several wavefronts.  Exchanging a value at every step
// costs more than a third of the step, so with Sync::kHalo each wavefront recomputes, in its
// first `halo` lanes, the last `halo` pairs of the wavefront below it:
//     pair of (wave, lane) = wave * (64 - halo) + lane
// (wavefront 0 has nothing below it: all its 64 lanes are exact, its lane 0 is pair 0).
// An error at lane 0 (whose neighbour is missing) moves up one lane per step, so the lanes
// from `halo` on stay exact for `halo` steps.  Every `halo` steps (a whole number of chunks)
// the lower wavefront hands
// over the exact state of those pairs through LDS.  No barrier; the wavefronts run skewed.  A wavefront waits for data only on lower
// ones and for space only on higher ones, wavefront 0 needs no data and the last one no space,
// so every wait ends; a poll budget bounds them regardless and raises chain_err when spent.
// (Here two counters guard a boundary's buffer: `ready` written by the producer after the data, `done` by the consumer after its read.  Linear-domain chains: HandOvers.)
template <bool kBackward, Sync kSync, Mode kMode>
__device__ __forceinline__ void run_chain_log(const Utt m, const int u, const int* __restrict__ labels,
                                          const float* __restrict__ emit_blank, const double* __restrict__ emit_blank64,
                                          const float* __restrict__ emit_label,
                                          uint32_t* __restrict__ out, int* __restrict__ out_exponents,
                                          double* __restrict__ mass,
                                          float* __restrict__ costs, int* __restrict__ chain_err,
                                          uint32_t* __restrict__ sink, void* lds)
{
    static_assert(kMode != Mode::kLoss || !kBackward, "see above");
    // Launches for the most probable alignment store plain logarithms, the others coded emissions.
    constexpr bool kCoded = kMode != Mode::kBest;
    const int L = m.L, P = L + 1, chunks = 2 * frame_blocks(m.Tb);
    const int count = kMode == Mode::kBest ? chain_chunks(m.Tb, kBackward) : chunks;     // chunks of this chain
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // (uniform: in a scalar register)
    const int halo = (kSync == Sync::kHalo) ? m.halo : 0;
    const int j = wave * (64 - halo) + lane;
    const int* lab = labels + m.lab_off;
    const bool has_label = j >= 0 && j < L;
    const bool active = (wave == 0 || lane >= halo) && j <= L;   // this lane stores pair j
    const int li = kBackward ? (L - 1 - j) : j;          // label index of this pair's label state
    // May the label state be entered from pair j-1's label?  (Not across equal symbols.)
    const bool skip_ok = has_label && j >= 1 && lab[li] != lab[kBackward ? (li + 1) : (li - 1)];
    const double skip_penalty = skip_ok ? 0.0 : kNeg;

    // Label emissions: a per-lane pointer that moves one chunk at a time.  A lane without a label
    // state reads a constant log 0 and stays there.
    const float* ep = emit_label + label_emission_offset(m, has_label, has_label ? lab[li] : 0, li,
                                                         chain_chunk(0, chunks, kBackward), kLogZeroEmission);
    const int64_t estep = label_emission_step(m, has_label, kBackward);
    // Blank emissions: lane i of a chunk's load takes the frame of the chunk's step i % kChunk.
    const float* const bp = emit_blank + (kBackward ? kChunk - 1 - (lane & (kChunk - 1)) : (lane & (kChunk - 1)));
    // Output: only the label state of each pair is kept (rows by frame, column = 1 + label index, in both directions).
    // Lanes that store nothing write to a sink instead.
    // With Mode::kBest the value block holds a word of choices per pair and chunk instead, rows in the chain's own
    // order, column = pair, pair L included: its blank state has a choice to record.
    const int64_t out_pitch = (kMode == Mode::kBest) ? P : lattice_pitch(L);
    const bool stores = (kMode == Mode::kBest) ? active : (active && has_label);
    const int64_t first_row = kBackward ? static_cast<int64_t>(chunks) * kChunk - 1 : 0;
    uint32_t* op = stores ? out + m.ab_off + (kMode == Mode::kBest ? j : first_row * out_pitch + li + 1) : sink;
    const int64_t ostride = stores ? (kBackward && kMode != Mode::kBest ? -out_pitch : out_pitch) : 0;
    int* xp = (stores && kMode == Mode::kGrad) ? out_exponents + m.ab_off + first_row * out_pitch + li + 1 : reinterpret_cast<int*>(sink);
    const int64_t xstride = (stores && kMode == Mode::kGrad) ? (kBackward ? -1 : 1) * out_pitch : 0;
    unsigned choices = 0;
    int blank_origin = 2 * j, label_origin = 2 * j + 1;
    uint32_t* origin_out = stores && kMode == Mode::kBest ? reinterpret_cast<uint32_t*>(out_exponents) + m.ab_off + origin_word(P, 0) + j : sink;
    auto store_state = [&](double w) {
        uint32_t value;
        int exponent;
        split_log2(w, value, exponent);
        *op = value;
        *xp = exponent;
        xp += xstride;
    };

    HaloHeader* const hl = static_cast<HaloHeader*>(lds);
    const int last_wave = m.waves - 1;
    HaloWave* const mine_lds = halo_wave<HaloWave>(lds, wave);
    HaloWave* const below_lds = halo_wave<HaloWave>(lds, wave > 0 ? wave - 1 : 0);
    HaloWave* const above_lds = halo_wave<HaloWave>(lds, wave < last_wave ? wave + 1 : wave);
    int budget = m.poll_budget;                          // polls left before this wavefront gives up waiting
    bool lost = false;                                   // it did give up: what it computed since is not to be trusted
    // Hand-overs fall on chunk boundaries (the halo is a multiple of kChunk), so the step
    // itself carries no countdown and the hand-over code exists once per chunk, not per step.
    const int chunks_per_hand_over = halo / kChunk;
    int until_hand_over = chunks_per_hand_over;          // chunks until the next hand-over
    int generation = 0;
    // Each boundary's buffer is used as two halves of 32 entries, alternating by generation
    // (halo <= 32), so a producer may run one hand-over ahead of its consumer.
    int half = 0;                                        // entry offset of the half in use: 0 or 32
    double2* const wr_base = (kSync == Sync::kHalo)
        ? &mine_lds->data[lane >= 64 - halo ? lane - (64 - halo) : 0] : nullptr;
    const double2* const rd_base = (kSync == Sync::kHalo)
        ? &below_lds->data[lane < halo ? lane : 0] : nullptr;
    int* const my_ready = &mine_lds->ready;
    int* const my_done = &mine_lds->done;
    int* const up_done = &above_lds->done;
    int* const low_ready = &below_lds->ready;

    double i_blank, i_label;
    double v_blank = (j == 0) ? 0.0 : kNeg, v_label = kNeg;

    auto counter = [&](int* p) {
        return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    auto uniform = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    int done_seen = 0;                                   // a (possibly old) reading of done[wave + 1]
    // After a step whose number is a multiple of `halo`: pass the exact state of the top `halo`
    // pairs up, take the exact state of the halo pairs from below.
    auto hand_over = [&]() {
        ++generation;
        half ^= 32;
        if (wave < last_wave) {
            // Space: the consumer must have taken generation - 2.  The reading from the last
            // hand-over usually shows that already.
            int seen = uniform(done_seen);
            if (__builtin_expect(seen < generation - 2, 0)) {
                while (seen < generation - 2 && budget > 0) {
                    --budget;
                    seen = uniform(counter(up_done));
                }
                lost = lost || seen < generation - 2;
            }
            if (lane >= 64 - halo) {
                wr_base[half] = make_double2(v_blank, v_label);
                if (kMode == Mode::kBest) mine_lds->origins[half + lane - (64 - halo)] = blank_origin | label_origin << 16;
            }
            // LDS operations of a wavefront complete in order: the counter follows the data.
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            if (lane == 63) __hip_atomic_store(my_ready, generation, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            done_seen = counter(up_done);                // consumed at the next hand-over
        }
        if (wave > 0) {
            // Counter and data are read back to back; the data count only if the counter,
            // read first, already showed this generation.
            const int* const rd_origin = &below_lds->origins[half + (lane < halo ? lane : 0)];
            int ready = counter(low_ready);
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            double2 v = rd_base[half];
            int origins = kMode == Mode::kBest ? *rd_origin : 0;
            ready = uniform(ready);
            if (__builtin_expect(ready < generation, 0)) {
                while (ready < generation && budget > 0) {
                    --budget;
                    ready = counter(low_ready);
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                    v = rd_base[half];
                    if (kMode == Mode::kBest) origins = *rd_origin;
                    ready = uniform(ready);
                }
                lost = lost || ready < generation;
            }
            if (lane < halo) {
                v_blank = v.x;
                v_label = v.y;
                if (kMode == Mode::kBest) {
                    blank_origin = origins & 0xFFFF;
                    label_origin = static_cast<int>(static_cast<unsigned>(origins) >> 16);
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            if (lane == 0) __hip_atomic_store(my_done, generation, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    };

    // Label value of pair j-1 after step s (log 0 for pair 0).  `mine` is this lane's.
    int prev_lo = __double2loint(kNeg), prev_hi = __double2hiint(kNeg);
    auto from_prev_pair = [&](double mine, int s) {
        double r = shift_up(mine, prev_lo, prev_hi);
        if (kSync == Sync::kBarrier) {
            double (*xch)[16] = static_cast<double (*)[16]>(lds);
            if (lane == 63) xch[s & 1][wave] = mine;
            __syncthreads();
            if (lane == 0 && wave > 0) r = xch[s & 1][wave - 1];
        }
        return r;
    };
    // ... and where the best way to it came from
    int prev_origin_lane = 0;
    auto origin_from_prev_pair = [&](int s) {
        prev_origin_lane = __builtin_amdgcn_update_dpp(prev_origin_lane, label_origin, 0x138, 0xf, 0xf, false);
        int r = prev_origin_lane;
        if (kSync == Sync::kBarrier) {
            int (*xch)[16] = reinterpret_cast<int (*)[16]>(static_cast<double*>(lds) + 32);
            if (lane == 63) xch[s & 1][wave] = label_origin;
            __syncthreads();
            if (lane == 0 && wave > 0) r = xch[s & 1][wave - 1];
        }
        return r;
    };

    auto finish_step = [&](double eb, float el) {
        v_blank = i_blank + eb;
        v_label = i_label + (kCoded ? emission_log2(el) : static_cast<double>(el));
        if (kMode == Mode::kGrad) {
            store_state(kBackward ? i_label : v_label);
            op += ostride;
        }
    };
    // After the last step of a chunk.
    auto end_chunk = [&]() {
        if (kSync == Sync::kHalo) {
            if (--until_hand_over == 0) {
                hand_over();
                until_hand_over = chunks_per_hand_over;
            }
        }
    };
    auto advance = [&](int step, double eb, float el) {
        const double prev = from_prev_pair(v_label, step);
        if (kMode == Mode::kBest) {
            // Of equally probable ways the one that stays highest in the label throughout: going forward that is the
            // shortest move, going backward the longest.
            auto better = [](double a, double b) { return kBackward ? a >= b : a > b; };
            const int prev_origin = origin_from_prev_pair(step);
            const double via_skip = prev + skip_penalty;
            const bool blank_moves = better(prev, v_blank), from_blank = better(v_blank, v_label);
            const double stay = fmax(v_blank, v_label);
            const bool skips = better(via_skip, stay);
            const int stay_origin = from_blank ? blank_origin : label_origin;
            i_blank = fmax(prev, v_blank);
            i_label = fmax(via_skip, stay);
            label_origin = skips ? prev_origin : stay_origin;
            blank_origin = blank_moves ? prev_origin : blank_origin;
            choices = append_bit(choices, __ballot(skips));
            choices = append_bit(choices, __ballot(from_blank));
            choices = append_bit(choices, __ballot(blank_moves));
        } else {
            // The blank state sums its own value and the label of the pair before; where the
            // label state may also be entered from that label (skip), its three-term sum is
            // its own value plus exactly the blank state's new sum, else plus the old blank:
            // two two-term sums per pair instead of a two- and a three-term one.
            i_blank = lse2(v_blank, prev);
            i_label = lse2(v_label, skip_ok ? i_blank : v_blank);
        }
        finish_step(eb, el);
    };
    auto readlane = [](float v, int l) {
        return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), l));
    };

    auto end_segment = [&]() {
        *origin_out = static_cast<uint32_t>(blank_origin | label_origin << 16);
        origin_out += ostride;
        blank_origin = 2 * j;
        label_origin = 2 * j + 1;
    };
    // (every lane starts from the exact state of its pair, halo lanes included)
    float el[4][kChunk], eb[2];                          // eb: the frames' words
    double blank_logs[2][kChunk] = {};                   // (Mode::kBest: as scalars, see run_chain_linear)
    const double* next_blanks = kMode == Mode::kBest ? emit_blank64 + blank_emission_offset(m, chain_chunk(0, chunks, kBackward)) : nullptr;
    auto fetch = [&](auto set, int i) {
        constexpr int k = decltype(set)::value;
        if (i >= kBlankAhead && kMode == Mode::kBest) {
            asm volatile("" : : "s"(blank_logs[(k + 1) & 1][0]), "s"(blank_logs[(k + 1) & 1][kChunk - 1]));
#pragma unroll
            for (int q = 0; q < kChunk; ++q) blank_logs[k & 1][q] = next_blanks[kBackward ? kChunk - 1 - q : q];
            next_blanks += kBackward ? -kChunk : kChunk;
        } else if (i >= kBlankAhead) {
            eb[k & 1] = bp[blank_emission_offset(m, chain_chunk(i - kBlankAhead, chunks, kBackward))];
        }
        fetch_chunk<kBackward>(ep, estep, el[k]);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto run = [&](auto set, int i) {
        constexpr int k = decltype(set)::value;
        const float blank = kCoded ? blank_emission_log2(eb[k & 1]) : 0.0f;
#pragma unroll
        for (int q = 0; q < kChunk; ++q)
            advance(i * kChunk + q,
                    kCoded ? static_cast<double>(readlane(blank, q)) : blank_logs[k & 1][q],
                    el[k][q]);
        end_chunk();
        if (kMode == Mode::kBest) {
            *op = choices;
            op += ostride;
            static_assert(kSegmentChunks == 4, "the sets of chain_schedule");
            if (k == 3) end_segment();
        }
    };
    chain_schedule(count, fetch, run);

    if (kMode == Mode::kBest) {
        if (count % kSegmentChunks) end_segment();
        // the backtrace looks for the best way through the frames where the chains meet
        if (active) reinterpret_cast<CheckpointState*>(out_exponents + m.ab_off)[j] = CheckpointState{v_blank, v_label};
        if (kSync == Sync::kHalo && lost && lane == 0) publish(&chain_err[u], 1);
        return;
    }
    if (!kBackward) {
        // p = alpha_{T-1}(2L) + alpha_{T-1}(2L-1): the blank of pair L and the label of pair L-1.
        // Pair L sits in an exact lane, and so does the lane below it or, if that is the last
        // halo lane, it is still exact: the error from lane 0 needs `halo` steps to get there,
        // and a hand-over that fell due after the last step has been done by end_chunk.
        const double prev = from_prev_pair(v_label, chunks * kChunk);
        if (kMode == Mode::kLoss) {
            const Norms norms = norms_of_wave(norms_of_lane(m, emit_blank));
            if (active && j == L) {
                const double lp = lse2(v_blank, prev);
                const float cost = cost_of_mass(lp < -1.0e29 ? 0.0 : 1.0, lp, norms.log2());
                if (kSync == Sync::kHalo) hl->cost = cost;
                else costs[u] = cost;
            }
        } else if (active && j == L) {
            const double lp = lse2(v_blank, prev);
            publish(&mass[u * kMassWords + kMassInverse], pack_log2(-lp));
            publish(&mass[u * kMassWords + kMassValue], lp < -1.0e29 ? 0.0 : 1.0);
            publish(&mass[u * kMassWords + kMassLog2], lp);
        }
    }
    if (kSync == Sync::kHalo && kMode == Mode::kLoss) {
        // No kernel follows that could turn a lost exchange into a NaN cost, so the cost is
        // written by whichever wavefront finishes last, once it has seen whether any gave up.
        // (One wavefront's LDS operations complete in order: flag and cost precede its count.)
        if (lost && lane == 0) hl->gave_up = 1;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        int before = 0;
        if (lane == 0)
            before = __hip_atomic_fetch_add(&hl->finished, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        before = __builtin_amdgcn_readfirstlane(before);
        if (before == m.waves - 1 && lane == 0) {
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const int lost = __hip_atomic_load(&hl->gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            const float cost = hl->cost;
            costs[u] = lost ? __uint_as_float(0x7FC00000u) : cost;
        }
    } else if (kSync == Sync::kHalo && lost && lane == 0) {
        publish(&chain_err[u], 1);
    }
}

// Where the chains of a launch leave their states: value and exponent blocks of both directions
// (see "lattice storage").  In the modes without a gradient: the state of every pair after a chain's last frame (cost
// only: one row of checkpoints in the value block), or the predecessor choices in the value block and
// the last states, base-2 logarithms, in the exponent block (Mode::kBest).
struct LatticeOut {
    uint32_t* alpha;
    int* alpha_exponents;
    uint32_t* beta;
    int* beta_exponents;
};

// What the chains' workgroups get besides.
struct LaunchWords {
    const int* row_flags;     // narrow softmax launch's words (rows_flagged), or nullptr: the records' flags say it all
    int flag_blocks;          // ... per utterance
    int* domain;              // per utterance and direction: did the chain run in the log domain
    int* done;                // per utterance, kDoneStride apart: see finish_loss, announce_end
    int late_percent;         // launch that writes the gradient too: this share of the chains' workgroups come late (tests)
    int* host_flag;           // pinned host word that receives host_flag_value: the image may be reused (or nullptr)
    int host_flag_value;
    const int* status_words;  // device-resident metadata built by the narrow softmax launch: per utterance, nonzero if
    int* status_out;          // invalid; gathered into the caller's status word by this launch (or nullptr)
    int status_count;
    int skip_directions;      // bit 0: leave the forward chains out, bit 1: the backward chains (measurements only)
    FillArgs fill;            // zero rows to write beside the chains
    int norm_groups, utterances;  // cost-only launches: the first workgroup that sees to the utterances' norms, and how many there are
};

// The arguments of a launch with chains as they lie in memory, in the kernels' order.
template <bool kFused>
struct ChainArgs {
    const Utt* meta;
    const int* order;
    const int* labels;
    const float* emit_blank;
    const double* emit_blank64;
    const float* emit_label;
    LatticeOut lat;
    double* mass;
    float* costs;
    int* chain_err;
    uint32_t* sink;
    LaunchWords wk;
};
template <>
struct ChainArgs<true> {
    const Utt* meta;
    const int* order;
    const int* labels;
    const float* emit_blank;
    const float* emit_label;
    LatticeOut lat;
    double* mass;
    float* costs;
    int* chain_err;
    uint32_t* sink;
    LaunchWords wk;
};
// Read again from there: nothing of it is kept in registers from before.
template <typename Args>
__device__ __forceinline__ const Args& args_again()
{
    typedef __attribute__((address_space(4))) const Args* ArgsPointer;
    ArgsPointer args = (ArgsPointer)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(args));
    return *(const Args*)args;
}

// The same chain on probabilities, each frame's divided by its blank's (FrameNorm), instead of their logarithms: a step is then
// two fused multiply-adds, an addition and a multiplication per pair, a fifth of the instructions of the
// log-domain step and no transcendentals.  What makes it safe is an exponent per lane:
//   true value = (v_blank, v_label) * 2^frame
// with fp64 values and an int32 `frame` that is looked after every n = kChunk steps (ChainFrames).  With probabilities of at least
// 2^-m (m = -kRoughMinLog2 = 79) ratios to the blank's are within 2^-m .. 2^m.  A renewal gives a lane
//   frame = largest binary exponent among its own pairs and the n pairs below it, its window,
// but no more than kFrameSlack above its own largest value, down to kFrameDrop below the window's top.  Mass moves up by at most
// one pair per step, so in the n steps that follow
//   - what arrives from the window is at most 2^kFrameDrop, and grows by 3 * 2^m a step at most: 2^(370 + 8 * 80.6) = 2^1015,
//   - a value of at least 2^-kFrameSlack shrinks by 2^-m a step at worst: 2^-(390 + 632) = 2^-1022,
// both inside fp64.  Utterances with smaller probabilities, down to 2^-100 (-kLinearMinLog2), are *steep*: n = kSteepSteps, 2^776 and
// 2^-790.  Their chains are a variant of their own, since a branch in the middle of a chunk would be two instructions more for the
// others (64 x 750 frames, 29 symbols, probabilities down to 2^-90: 55 us a call; in the log domain 123, and shares to 2^-19 only).
// Two neighbouring frames differ by at most kFrameSlack + kFrameDrop, which the factor between them (scale, constant between renewals
// and folded into the multiply-adds) can hold.
//
// The states of a lane share its frame.  One that lies 2^1022 below another further on in the label would be rounded to zero, and what
// would have gone on from it later be lost; symbols held against the blank for dozens of frames do that.  A wavefront that meets it (strains) leaves this
// recursion there and goes on with an exponent to every state (finish_with_exponents); so do those above it, once they are handed its logarithms.
// It suffices to look at a lane's first blank, when frames are renewed: a blank state loses nothing from step to step and gets at
// least what its pair's label gets, so but for the last steps' factors it is the least of the lane's states, and only a renewal makes values smaller.
//
// A pair further than 2^(kFrameSlack + kFrameDrop) below its window's top is rounded away.  Its neighbours have 2^760 times its
// mass and can still reach the end of the label (utterances with fewer than kTightFrames frames to spare, where they could
// not, run in the log domain from the start: tight_fit), each of their at most n extra moves costing 2^-m at worst: what is
// rounded away is below 2^-128 (steep: 2^-360) of the whole.  (With the window's top as the frame of every lane a pair 2^1000 below its
// neighbours was lost where it was all there is: an utterance with exactly as many frames as its label needs, logits spread
// over 40 nats, cost off by 0.03, gradient by 0.03.)
//
// Storage (Mode::kGrad): the whole state after every block (see "lattice storage").
//
// What a step costs (a lone wavefront of a chain issues an instruction every five clocks, whatever it is): 7 instructions and 35 clocks, 12 and 60
// where a lane owns two pairs; the rest is what a block's end adds.  Clocks a step (2.4 GHz; 1500 frames less 750, alone on the chip), labels of 40 / 127 / 190 / 240 /
// 420 symbols: 48 / 65 / 74 / 87 / 100 when a hand-over took 550 clocks, a look at the frames 100 and a checkpoint 110; so 45 / 56 / 62 / 78 / 85.  Logits doubled (rough
// utterances): 52 / 73 / 83 / 96 / 113, so 46 / 64 / 71 / 88 / 104.
constexpr int kFrameSlack = 390, kFrameDrop = 370;
__device__ __forceinline__ int lane_frame(int window_top, int own_top)
{
    return window_top - min(max(window_top - own_top - kFrameSlack, 0), kFrameDrop);
}
// A renewal (about 300 clocks, with what else is unusual at a block's end up to 900; a chunk's eight steps 300) is put off while it is not needed: every lane with
// mass has its largest value within [2^low, 2^high] of its frame, and no frame lies more than `smooth` a pair below the frame of the lane below it.  Until the next renewal can be
// had, n steps later with ratios within 2^-g .. 2^g, a value is at least 2^(low - n g), and at most 2^(high + n (smooth + g + 1.6)).  Each class of utterances has its own range:
//   gentle (all probabilities above 2^kGentleMinLog2, g = 32): kGentleLow, kGentleHigh, kGentleSmooth, looked at kLookAhead steps before a chunk ends, n = 9; a lane that takes
//     states handed up may have scaled them by 2^-kShiftDown to 2^kShiftUp since: 2^-1018 and 2^966.  (Looked at after blocks of 16 frames, what is admissible is so narrow that the
//     lanes above the front of the lattice renewed at every second block.)
//   rough (above 2^kRoughMinLog2, g = 79): kRoughLow, kRoughHigh, kSmoothFrames, looked at as early, n = 9: 2^-1021 and 2^1021
//   steep (g = 100): kEasyLow, kEasyHigh, kSteepSmoothFrames, looked at when kSteepSteps steps are done, n = 4: 2^-750 and 2^1005
// And after a renewal, n = 8 (steep: 4) steps: see above.
// (Rough ones, smooth / high: 28 / 44, 20 / 116 and 16 / 152 are as far as 24 / 80 goes; 64 x 750 x 29 of deviation 4 52.0, 51.6 and 52.8 us a call where this took 51.1.)
// Where a gentle one's renewal puts the largest value of a window: 2^kHeadroom below its frame, as values grow more often than they shrink.  (For rough ones, whose
// lanes hold states further apart, it made more of them strained: 64 x 750 frames, logits of deviation 6, 52 us a call, 81 with it.)
constexpr int kHeadroom = 100;
__device__ __forceinline__ int chain_frame(int window_top, int own_top, int headroom)
{
    return window_top + headroom - min(max(window_top - own_top - (kFrameSlack - headroom), 0), kFrameDrop + headroom);
}
constexpr int kLookAhead = 1;
constexpr int kEasyLow = -350, kEasyHigh = 99;
constexpr int kSmoothFrames = 24, kSteepSmoothFrames = 125;
// Gentle utterances.  States handed up are taken into the frames of the lanes that take them where those are no more than kShiftUp below and kShiftDown above the frames that they
// come in: a chunk later 2^-1018 and 2^966 at worst.  (In the frames that they come in, all factors between frames had to be made anew whenever a wavefront below had renewed its own.)
// That is for a lane's largest value.  A first blank, of which a renewal allows 2^kStrained, would be rounded by more than 2^-90.  It is not where the lane had mass when its frame was set:
// a blank never falls, so what that renewal found above 2^kStrained of the frame still is.  A lane without mass takes what has come up within the 32 frames since the last
// hand-over.  At the first look after it has, eight steps at most, its blank is 2^-714 of a frame that needs no renewal.  For less the largest of its window must have gained 2^600 on it
// since, and then hands that on to the next blank, which does not fall either; a path by the blank that is lost here can gain on those no more than 2^32 a frame, for half of the
// frames until the next hand-over puts it right, 2^512.  (kShiftDown of 90: half as many unusual block ends again to twice as many; 32 x 1500 x 29 111.1 us a call, 107.4 with 280.  Lanes
// left at 2^-710 instead: utterances that hold symbols for 60 frames at 6 nats 187, 177.  Replayed on the CPU, symbols held and dropped at 2^31 to their blank for 4 to 40 frames, none
// came below 2^-651.)
constexpr int kGentleLow = -450, kGentleHigh = 120, kGentleSmooth = 36;
constexpr int kRoughLow = -310, kRoughHigh = 80;
constexpr int kShiftUp = 220, kShiftDown = 280;
constexpr bool renewal_lasts(int steps, float min_log2) { return steps * min_log2 - kFrameSlack >= -1022 && kFrameDrop + steps * (1.6f - min_log2) < 1023; }
constexpr bool look_lasts(int steps, float min_log2, int smooth, int low, int high) { return low + steps * min_log2 >= -1022 && high + steps * (1.6f - min_log2 + smooth) < 1023; }
static_assert(renewal_lasts(kChunk, kGentleMinLog2) && look_lasts(kChunk + kLookAhead, kGentleMinLog2, kGentleSmooth, kGentleLow - kShiftDown, kGentleHigh + kShiftUp), "gentle");
static_assert(renewal_lasts(kChunk, kRoughMinLog2) && look_lasts(kChunk + kLookAhead, kRoughMinLog2, kSmoothFrames, kRoughLow, kRoughHigh), "rough");
static_assert(renewal_lasts(kSteepSteps, kLinearMinLog2) && look_lasts(kSteepSteps, kLinearMinLog2, kSteepSmoothFrames, kEasyLow, kEasyHigh), "steep");
// Does a renewal leave a lane's first blank below 2^kStrained of its new frame?  (`rise`: from the frame it had.  A lane without mass has a blank of 0, whose
// exponent reads 0.)  What is above keeps all its bits until the next renewal: 2^(kStrained + kLinearMinLog2) is above fp64's smallest normal number.
// (The look costs, with the gradient's, renew_pairs: 64 x 750 frames, 29 symbols 45.9 -> 46.3 us a call, cost only 28.2 -> 28.8, 512 x 750 114.2 -> 116.0, one
// utterance 38.8 -> 39.4: three to nine instructions more in a round of 290 to 390.  Ways out of the round itself, in place of a `count` that ends it, made the
// compiler keep what the chains hold in memory.
// 24 x 750 frames of symbols held for 60 frames at 14 nats take 184 us.  Redoing the whole utterance in the log domain took 663 us where this takes 52, random
// logits of deviation 4, which seldom strain a lane.)
constexpr int kStrained = -900;
static_assert(kStrained + kLinearMinLog2 >= -1022, "what a first blank of 2^kStrained gives its label");
static_assert(kGentleLow + kChunk * (kGentleMinLog2 - 1) - kShiftDown >= -1022, "what a shift leaves of a blank whose label has come up since the last look");
// (of_label: lanes behind the label's end hold nothing that anybody needs.)
__device__ __forceinline__ bool strains(double first, int rise, bool of_label) { return __ballot(of_label && __builtin_amdgcn_frexp_exp(first) + rise < kStrained) != 0; }
// The test, on the exponent of the largest value of a lane: one subtraction and one unsigned compare.  Lanes without mass pass it.
struct EasyRange {
    int low, width, smooth, headroom;                    // smooth: for a pair
    __device__ __forceinline__ EasyRange(bool gentle, bool steep)
        : low(gentle ? kGentleLow : (steep ? kEasyLow : kRoughLow)), width(gentle ? kGentleHigh - kGentleLow : (steep ? kEasyHigh - kEasyLow : kRoughHigh - kRoughLow)),
          smooth(gentle ? kGentleSmooth : (steep ? kSteepSmoothFrames : kSmoothFrames)), headroom(gentle ? kHeadroom : 0)
    {
    }
    __device__ __forceinline__ bool outside(double top) const
    {
        static_assert(kEasyLow < -1 && kEasyHigh > 0 && kRoughLow < -1 && kRoughHigh > 0 && kGentleLow < -1 && kGentleHigh > 0, "zero, whose exponent reads 0, is in it");
        return static_cast<unsigned>(__builtin_amdgcn_frexp_exp(top) - 1 - low) > static_cast<unsigned>(width);
    }
};

// A forward chain's end: p = value * 2^frame.
__device__ __forceinline__ void publish_mass(double* mass, double value, int frame)
{
    publish(&mass[kMassInverse], value > 0.0 ? pack_state(1.0 / __builtin_amdgcn_frexp_mant(value), -(frame + __builtin_amdgcn_frexp_exp(value))) : 0.0);
    publish(&mass[kMassValue], value);
    publish(&mass[kMassLog2], static_cast<double>(frame));
}

// How a wavefront of a linear-domain chain ends.
struct ChainEnd {
    int unit;                                            // nonzero: after so many half chunks it has left the recursion (finish_with_exponents)
    bool lost;                                           // it gave up a wait
};

// A chain's frames; kPairs pairs to a lane.
template <int kPairs, bool kSteep>
struct ChainFrames {
    static constexpr int kSteps = (kSteep ? kSteepSteps : kChunk) / kPairs;     // lanes that mass moves up in a chunk at worst
    const EasyRange easy;
    __device__ __forceinline__ explicit ChainFrames(bool gentle) : easy(gentle, kSteep) {}
    int frame = 0;
    double scale = 1.0;                                  // 2^(frame of the lane below - frame)
    unsigned long long rough = ~0ull;                    // lanes that may not put a renewal off: see rescale
    // The factors between the frames.  `massless`: lanes without mass.  A lane's frame may lie kSmooth below that of the
    // lane below it and no further, one without mass not above it either.
    __device__ __forceinline__ void rescale(unsigned long long massless)
    {
        const int down = __builtin_amdgcn_update_dpp(kNoExponent, frame, 0x138, 0xf, 0xf, false) - frame;
        // 2^1023 is the largest factor there is; a pair that far below its neighbour has been rounded away already.
        scale = __builtin_amdgcn_ldexp(1.0, min(max(down, -1100), 1023));
        const int smooth = kPairs * easy.smooth;
        rough = __ballot(down > smooth) | (__ballot(down < -smooth) & massless & ~1ull);       // (lane 0 has nothing below)
    }
    // The frames after a renewal; returns what the lane's values are to be scaled by.  `top`: the largest of them.  Lanes above the highest one with mass take that one's frame, so that the front of the lattice
    // passes through a wavefront like anything else; where no lane has mass, `reference`'s.
    __device__ __forceinline__ int renew(double top, int reference)
    {
        const bool has_mass = top > 0.0;
        const unsigned long long massive = __ballot(has_mass);
        const int mine = has_mass ? frame + __builtin_amdgcn_frexp_exp(top) : kNoExponent;
        int window = mine;
#pragma unroll
        for (int k = 0; k < kSteps; ++k) window = window_max_step(window, mine);
        int next = massive != 0 ? chain_frame(window, mine, easy.headroom) : frame;
        const int front = massive != 0 ? 63 - __builtin_clzll(massive) : reference;
        const int beyond = __builtin_amdgcn_readlane(next, front);
        next = static_cast<int>(threadIdx.x & 63) > front ? beyond : next;
        const int rise = frame - next;
        frame = next;
        rescale(~massive);
        return rise;
    }
    // Is a renewal due?  (A lane without mass is where it should be unless it is rough.)
    __device__ __forceinline__ bool renewal_due(double top) const { return (__ballot(easy.outside(top)) | rough) != 0; }
};

// The hand-overs of a linear-domain chain of several wavefronts (what they are for: see above run_chain_log), at the ends of blocks.  What decides their cost is how
// many instructions they take, as anywhere in a chain, and that nothing is waited for.  A wavefront asks for what the one below it has left some steps before its block
// ends, and compares before the last step: the halo's lanes whether they have read the number of this hand-over beside their states and whether the
// frame is near enough to theirs to take these by a shift, lane 63, in the tag of the wavefront above, whether what is about to be overwritten has been taken
// (a number is published when that hand-over has been taken from below as well).  Where any lane says no, or one is due for a renewal, the block's end is
// unusual: whoever has asked too early asks again until it is there, and then waits a little more, so as not to be early at every block from then on;
// frames are taken over from below; frames are renewed.  LDS operations of a wavefront complete in order: a tag is read before the states, and written after
// them.  (A hand-over took 550 clocks when it was asked for at the block's end, two counters one after the other, and made all factors between frames anew; now 180.
// Unusual ends, replayed on the CPU: 1 of 47 in the lowest wavefront of a label of 190 symbols, 5 in the others; of a rough utterance 11, and 37.)
constexpr int kSlack = 2;                                // (s_sleep: 64 clocks each)
constexpr int kAskAhead = 5, kAskAhead2 = 4;             // steps before the block's end, with one pair to a lane and with two
template <int kPairs>
struct HandOvers {
    static constexpr int kNever = 0x7FFFFFFF, kLeft = 1 << 30;
    typedef LinearWave<kPairs> Wave;
    typedef typename Wave::Slot Slot;
    const char *in, *out;                                // in the first slot: what this lane takes (its tag: looks at), what it hands up
    bool takes, hands;                                   // this lane is one of the halo's; of the ones above's
    int behind;                                          // by how much the tag that it reads may be behind the hand-over
    unsigned shift;                                      // ... and its frame differ, from shift_down below this lane's on
    int shift_down;
    int number = 2;                                      // of the coming hand-over, times two, and one more where states are due for a renewal (kLeft: the chain has been left)
    unsigned round = 0;                                  // the first slot of this round of blocks, in bytes
    int2 tag{};
    double2 states[kPairs] = {};
    unsigned long long late = 0, shifted = 0;
    __device__ __forceinline__ HandOvers(void* lds, int wave, int last_wave, int halo, bool every_block, bool gentle)
    {
        const int lane = threadIdx.x & 63, first = 64 - halo;
        takes = wave > 0 && lane < halo;
        hands = lane >= first;
        const bool looks_up = wave < last_wave && lane == 63;
        in = reinterpret_cast<const char*>(&halo_wave<Wave>(lds, looks_up ? wave + 1 : (wave > 0 ? wave - 1 : 0))->slot[0].states[0][takes ? lane : (looks_up ? halo - 1 : 0)]);
        out = reinterpret_cast<const char*>(&halo_wave<Wave>(lds, wave)->slot[0].states[0][hands ? lane - first : 0]);
        behind = takes ? 0 : (looks_up ? 2 * (every_block ? kRing : kRing / 2) : kNever);
        shift_down = gentle ? kShiftDown : 0;
        shift = takes ? (gentle ? kShiftDown + kShiftUp : 0) : ~0u;
        asm volatile("" : "+v"(number));                 // (in a vector register, from where it is stored)
    }
    // A lane's states and tag in the slot of this round's block `block`.
    __device__ __forceinline__ double2* states_at(const char* lane, int block, int pair) const
    {
        return const_cast<double2*>(reinterpret_cast<const double2*>(lane + round + block * sizeof(Slot) + pair * Wave::kLanes * sizeof(double2)));
    }
    __device__ __forceinline__ unsigned long long* tag_at(const char* lane, int block) const
    {
        return const_cast<unsigned long long*>(reinterpret_cast<const unsigned long long*>(lane + round + block * sizeof(Slot) + offsetof(Slot, tag)));
    }
    // (from then on nobody hears of this wavefront through here)
    __device__ __forceinline__ void leave()
    {
        number = kLeft;
        hands = false;
    }
    __device__ __forceinline__ void ask(int block)
    {
        const unsigned long long w = __hip_atomic_load(tag_at(in, block), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        tag = make_int2(static_cast<int>(w), static_cast<int>(w >> 32));
#pragma unroll
        for (int k = 0; k < kPairs; ++k) states[k] = *states_at(in, block, k);
    }
    // What has been asked for is there now.  (Else it would be waited for where it is used, and what has been stored since with it.)
    __device__ __forceinline__ void arrive()
    {
#pragma unroll
        for (int k = 0; k < kPairs; ++k) asm volatile("" : "+v"(states[k].x), "+v"(states[k].y));
    }
    // Lanes that have not read what the next hand-over needs, or take states that are due for a renewal (a tag further than this
    // hand-over's); lanes that take states in a frame far from their own.
    __device__ __forceinline__ void look(int frame)
    {
        late = __ballot(static_cast<unsigned>(number - tag.y) > static_cast<unsigned>(behind));
        shifted = __ballot(static_cast<unsigned>(tag.x - frame + shift_down) > shift);
        arrive();
    }
    // Where any are: waits for what is late, and gives the lanes that take states the frames of those.  due: so are the states handed up (whoever takes them
    // renews as well).
    __device__ __forceinline__ void prepare(int block, bool due, int& frame, int& budget, bool& lost)
    {
        if (__builtin_amdgcn_readfirstlane(number) >= kLeft) return;
        auto waits = [&]() { return __ballot(number - tag.y > behind) != 0; };
        if (waits()) {
            bool still = true;
            for (; still && budget > 0; --budget) {
                ask(block);
                still = waits();
            }
            arrive();
            lost = lost || still;
            __builtin_amdgcn_s_sleep(kSlack);
        }
        frame = takes ? tag.x : frame;
        number += due ? 1 : 0;
    }
    __device__ __forceinline__ void publish(int block, const double2 (&mine)[kPairs], int frame)
    {
        if (hands) {
#pragma unroll
            for (int k = 0; k < kPairs; ++k) *states_at(out, block, k) = mine[k];
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __hip_atomic_store(tag_at(out, block), (static_cast<unsigned long long>(static_cast<unsigned>(number)) << 32) | static_cast<unsigned>(frame),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        number += 2;
    }
    __device__ __forceinline__ void next_round() { round ^= 2 * sizeof(Slot); }
};
static_assert(kRing == 4, "two rounds of two blocks");

// Where a linear-domain chain is in its emissions: what moves is the same for all lanes, and so in scalar registers (a pointer and a step of each lane's own took a 64-bit
// addition of all lanes a chunk and pair).  They are read as from a buffer, and lanes without a label state past its end, where loads give 0 (emission_column): such states stay
// 0, and neither put a lane's frame where it is not needed nor call for a renewal.  (With what the label's last symbol has in their place: 32 x 1500 x 29 114.6 us a call, so 107.8; logits of
// deviation 4, one utterance of 750 frames 42.4 and 39.5, 512 x 750 x 29 109.5 and 106.6.)
template <bool kBackward>
struct ChainEmissions {
    BufferWords chunk;                                   // base (48 bits), bytes, format
    int64_t step;                                        // bytes
    __device__ __forceinline__ ChainEmissions(const Utt& m, const float* __restrict__ emit_label)
        : step(label_emission_step(m, m.L > 0, kBackward) * static_cast<int64_t>(sizeof(float)))
    {
        const float* const first = emit_label + label_emission_offset(m, m.L > 0, 0, 0, chain_chunk(0, 2 * frame_blocks(m.Tb), kBackward), kZeroEmission);
        const uint64_t base = reinterpret_cast<uint64_t>(first);
        chunk = BufferWords{static_cast<int>(base), static_cast<int>(base >> 32) & 0xFFFF, static_cast<int>(kNoColumn - 1), 0x00020000};
    }
    // The column of pair j, in bytes.
    __device__ __forceinline__ unsigned column(const Utt& m, const int* __restrict__ lab, int j) const
    {
        const int position = kBackward ? m.L - 1 - j : j;
        return emission_column(j, m.L, j < m.L && m.e_direct == kEmitSymbols ? lab[position] : position);
    }
    __device__ __forceinline__ void read(unsigned column, float (&el)[kChunk]) const
    {
        const FourFloats lo = buffer_load(chunk, static_cast<int>(column), 0, 0), hi = buffer_load(chunk, static_cast<int>(column), 16, 0);
        constexpr int kFlip = kBackward ? kChunk - 1 : 0;
#pragma unroll
        for (int q = 0; q < kChunk; ++q) el[q ^ kFlip] = q < 4 ? lo[q] : hi[q - 4];
    }
    __device__ __forceinline__ void next()
    {
        const uint64_t base = (static_cast<uint64_t>(static_cast<unsigned>(chunk[1])) << 32 | static_cast<unsigned>(chunk[0])) + static_cast<uint64_t>(step);
        chunk[0] = static_cast<int>(base);
        chunk[1] = static_cast<int>(base >> 32);
        asm volatile("" : "+s"(chunk));                  // (or a round's chunks are counted from its first)
    }
};

// kPolicy: of the checkpoints' stores, kPast where another workgroup of the launch reads them.
template <bool kBackward, Exchange kHandsOver, Mode kMode, bool kSteep, int kPolicy>
__device__ __forceinline__ ChainEnd run_chain_linear(const Utt m, const int u, const bool gentle, const int* __restrict__ labels,
                                                 const float* __restrict__ emit_label, uint32_t* __restrict__ out,
                                                 double* __restrict__ mass, int* __restrict__ chain_err, void* lds)
{
    static_assert(kMode != Mode::kBest, "the maximum recursion runs in the log domain");
    constexpr bool kExchange = kHandsOver != Exchange::kNone;
    const int L = m.L, chunks = 2 * frame_blocks(m.Tb);
    int count = kMode == Mode::kLoss ? chain_chunks(m.Tb, kBackward) : chunks;     // chunks of this chain; -unit once it has been left
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // (uniform: in a scalar register)
    const int halo = kExchange ? m.halo : 0;
    const int j = wave * (64 - halo) + lane;             // pair of this lane (see run_chain_log)
    const int* lab = labels + m.lab_off;
    const bool has_label = j >= 0 && j < L;
    const bool active = (wave == 0 || lane >= halo) && j <= L;
    const int li = kBackward ? (L - 1 - j) : j;
    const bool skip_ok = has_label && j >= 1 && lab[li] != lab[kBackward ? (li + 1) : (li - 1)];

    ChainEmissions<kBackward> emissions(m, emit_label);
    const unsigned column = emissions.column(m, lab, j);
    // Checkpoints.  (Cost only: one row, by pair, in the chain's own order.)
    CheckpointRows rows(out + m.ab_off, CheckpointRow{lattice_pitch(L)}, kMode == Mode::kGrad ? frame_blocks(m.Tb) - 1 : 1,
                        kMode == Mode::kGrad ? active && has_label : active, kMode == Mode::kGrad ? li + 1 : j);

    const int last_wave = m.waves - 1;
    int budget = m.poll_budget;
    bool lost = false;
    const bool every_block = kHandsOver == Exchange::kBlock || (kHandsOver == Exchange::kAny && halo < 2 * kBlockFrames);
    HandOvers<1> with(kExchange ? lds : nullptr, wave, last_wave, halo, every_block, gentle && !kSteep);
    const unsigned long long look = kSteep ? ~0ull : 0ull;      // after every chunk, whatever the frames

    double v_blank = (j == 0) ? 1.0 : 0.0, v_label = 0.0;
    ChainFrames<1, kSteep> f(gentle && !kSteep);
    double skip_scale = skip_ok ? 1.0 : 0.0;             // f.scale where the label may be entered from the label of the pair below

    // Label value of pair j-1 after the last step, in that pair's frame (0 for pair 0: the shift
    // leaves lane 0 what it had).
    int prev_lo = 0, prev_hi = 0;
    auto from_prev_pair = [&](double mine) __attribute__((always_inline)) { return shift_up(mine, prev_lo, prev_hi); };
    auto top_value = [&]() __attribute__((always_inline)) { return fmax(v_blank, v_label); };
    // Leaves the recursion after `unit` half chunks, with the states in `frame` (StrainedWave).
    auto leave = [&](int unit, int frame) __attribute__((always_inline)) {
        if (count < 0) return;
        count = -unit;
        StrainedWave* const w = strained_wave(lds, wave);
        w->states[0][lane] = make_double2(v_blank, v_label);
        w->frame[lane] = frame;
        rows.drop();
        with.leave();
    };
    auto renew_frames = [&](int unit) __attribute__((always_inline)) {
        const int rise = f.renew(top_value(), halo > 0 ? halo - 1 : 0);
        if (__builtin_expect(strains(v_blank, rise, j <= L), 0)) leave(unit, f.frame + rise);
        v_blank = __builtin_amdgcn_ldexp(v_blank, rise);
        v_label = __builtin_amdgcn_ldexp(v_label, rise);
        skip_scale = skip_ok ? f.scale : 0.0;
    };

    // After a block's first chunk (steep: and in the middle of every chunk), and after a block.
    static_assert(kChunk == 2 * kSteepSteps, "the middle of a chunk");
    auto renew_if_due = [&](int unit) __attribute__((always_inline)) {
        if (f.renewal_due(top_value())) renew_frames(unit);
    };
    // Before a block's last kLookAhead steps: may its end be the ordinary one?  (A comparison's result is on its way to a branch for some 20 clocks.)
    unsigned long long outside = 0;
    auto look_ahead = [&](bool exchange) __attribute__((always_inline)) {
        outside = __ballot(f.easy.outside(top_value()));
        if (exchange) with.look(f.frame);
    };
    // (With hand-overs nothing here is said to be unlikely: what is goes to the kernel's end, further away than a branch reaches, and rough utterances take it at every other block.  us a call
    // with it there, and so: 64 x 750 x 29 41.1 and 41.3, logits of deviation 4 51.3 and 49.3, of 6 55.0 and 52.7, cost only 25.7 and 25.6, 32.3 and 31.5, 33.4 and 32.8; 32 x 1500 x 29
    // 107.5 and 108.2, 122.4 and 120.8; one utterance of 750 frames 32.4 and 32.3, 40.6 and 38.6.  A wavefront by itself renews seldom, and it is unlikely there: cost only 25.6 and
    // 25.2 with it at the end.)
    auto seldom = [](bool unusual) __attribute__((always_inline)) { return kExchange ? unusual : static_cast<bool>(__builtin_expect(unusual, 0)); };
    auto end_block = [&](int block, bool exchange, int unit) __attribute__((always_inline)) {
        const bool unusual = (outside | f.rough | look | (exchange ? with.late | with.shifted : 0ull)) != 0;
        if (exchange && unusual) with.prepare(block, (outside | f.rough) != 0, f.frame, budget, lost);
        if (exchange) {
            const double2 mine[1] = {make_double2(v_blank, v_label)};
            with.publish(block, mine, f.frame);
            if (with.takes) {
                const int shift = with.tag.x - f.frame;
                v_blank = __builtin_amdgcn_ldexp(with.states[0].x, shift);
                v_label = __builtin_amdgcn_ldexp(with.states[0].y, shift);
                asm volatile("" : "+v"(v_blank), "+v"(v_label));      // (a mask, and not a choice for each)
            }
        }
        if (seldom(unusual)) {
            const double top = top_value();
            if (exchange) with.number &= ~1;
            bool renews = __ballot(f.easy.outside(top)) != 0;      // (then the factors between the frames are made there)
            if (!renews) {
                if (exchange) {
                    f.rescale(__ballot(!(top > 0.0)));
                    skip_scale = skip_ok ? f.scale : 0.0;
                }
                renews = f.rough != 0;
            }
            if (renews) renew_frames(unit);
        }
    };
    auto checkpoint = [&]() __attribute__((always_inline)) {
        rows.template state<kPolicy>(0, CheckpointState{v_blank, v_label});
        rows.template frame<kPolicy>(f.frame);
        rows.next();
    };
    // One step.  The blank state sums its own value and the label of the pair before; the label state
    // its own value, the old blank and, where the skip is allowed, that label too:
    //   label' = fma(previous label, skip, label + blank) * emission.
    // Seven instructions, issued one every five clocks in the order of the statements (pin keeps the compiler from moving them; one
    // that reads the result of the one before it waits another clock).  The shift needs its operand two instructions old.
    auto pin = []() { __builtin_amdgcn_sched_barrier(0); };
    auto advance = [&](double& el_d, float next_el) __attribute__((always_inline)) {
#pragma clang fp contract(off)                           // (a product stays a product: fused into the next step's sum it would tie the steps together)
        const double prev = from_prev_pair(v_label);
        pin();
        const double u = v_blank + v_label;
        pin();
        const double i_label = __builtin_fma(prev, skip_scale, u);
        pin();
        v_label = i_label * el_d;
        pin();
        v_blank = __builtin_fma(prev, f.scale, v_blank);
        pin();
        el_d = static_cast<double>(next_el);             // (and the wait that the next step's shift of v_label needs)
        asm volatile("" : "+v"(el_d));
        pin();
    };

    float el[4][kChunk];
    auto fetch = [&](auto set, int) __attribute__((always_inline)) {
        constexpr int k = decltype(set)::value;
        emissions.read(column, el[k]);
        emissions.next();
        __builtin_amdgcn_sched_barrier(0);
    };
    auto run = [&](auto set, int i) __attribute__((always_inline)) {
        constexpr int k = decltype(set)::value;
        constexpr bool kEnds = (k & 1) != 0;             // the chunk ends a block
        const bool here = kEnds && kExchange && (kHandsOver != Exchange::kAny || last_wave > 0) && (k == 3 || every_block);
        if (kMode == Mode::kGrad && !kEnds) checkpoint();
        double el_d = static_cast<double>(el[k][0]);
#pragma unroll
        for (int q = 0; q < kChunk; ++q) {
            advance(el_d, el[k][q + 1 < kChunk ? q + 1 : q]);
            if (kSteep && q == kSteepSteps - 1) renew_if_due(2 * i + 1);
            if (here && q == kChunk - 1 - kAskAhead) with.ask(k >> 1);
            if (q == kChunk - 1 - kLookAhead) look_ahead(here);
        }
        if (kEnds) end_block(k >> 1, here, 2 * i + 2);
        else if (seldom((outside | f.rough | look) != 0)) {
            if (kSteep) renew_if_due(2 * i + 2);
            else renew_frames(2 * i + 2);
        }
        if (kExchange && k == 3) with.next_round();
    };
    chain_schedule(count, fetch, run);
    if (__builtin_expect(count < 0, 0)) return {-count, lost};

    if (kMode == Mode::kLoss) {
        // the state of every pair, for finish_loss
        rows.template state<kPolicy>(0, CheckpointState{v_blank, v_label});
        rows.template frame<kPolicy>(f.frame);
        return {0, lost};
    }
    if (!kBackward) {
        // p = alpha_{T-1}(2L) + alpha_{T-1}(2L-1), from the lane of pair L (exact, as is the
        // lane below it: see run_chain_log).
        const double from_below = from_prev_pair(v_label) * f.scale;
        if (active && j == L) publish_mass(&mass[u * kMassWords], v_blank + from_below, f.frame);
    }
    if (kExchange && lost && lane == 0) publish(&chain_err[u], 1);
    return {0, lost};
}

// Linear-domain chains of more than 64 pairs: a lane owns two neighbouring pairs, A = 2q and
// B = 2q + 1 (q = wave * (64 - halo) + lane), so a wavefront covers 128 pairs and most labels need
// one or two wavefronts instead of two to four.  Pair A takes the label of pair B of the lane
// below (one DPP shift and `scale`, as in run_chain_linear), pair B the label of pair A of its own
// lane: the two recursions of a lane are independent within a step and fill each other's issue
// gaps.  Both pairs share the lane's frame; mass moves up half a lane per step, so the window
// of a renewal is this lane and the kChunk / 2 lanes below it, and a halo of h lanes stays exact
// for 2h steps.
// The two pairs of a lane are neighbours in the checkpoint's row; where pair B has no label state (the lane of the last
// pair) its part falls on one of the row's two unused columns.

template <bool kBackward, Exchange kHandsOver, Mode kMode, bool kSteep, int kPolicy>
__device__ __forceinline__ ChainEnd run_chain_linear2(const Utt m, const int u, const bool gentle, const int* __restrict__ labels,
                                                  const float* __restrict__ emit_label, uint32_t* __restrict__ out,
                                                  double* __restrict__ mass, int* __restrict__ chain_err, void* lds)
{
    static_assert(kMode != Mode::kBest, "the maximum recursion runs in the log domain");
    constexpr bool kExchange = kHandsOver != Exchange::kNone;
    const int L = m.L, chunks = 2 * frame_blocks(m.Tb);
    int count = kMode == Mode::kLoss ? chain_chunks(m.Tb, kBackward) : chunks;     // (see run_chain_linear)
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // (uniform: in a scalar register)
    const int halo = kExchange ? m.halo2 : 0;
    const int waves = m.waves2;
    const int q = wave * (64 - halo) + lane;
    const int ja = 2 * q, jb = 2 * q + 1;                // the lane's pairs, in the chain's own order
    const int* lab = labels + m.lab_off;
    const bool has_a = ja < L, has_b = jb < L;           // label states (pair L has a blank state only)
    const bool active = (wave == 0 || lane >= halo) && ja <= L;
    const int lia = kBackward ? (L - 1 - ja) : ja;       // label index of pair A's label state
    const int lib = kBackward ? (lia - 1) : (lia + 1);
    const int back = kBackward ? 1 : -1;                 // label index of the pair before = index + back
    const bool skip_a = has_a && ja >= 1 && lab[lia] != lab[lia + back];
    const bool skip_b = has_b && lab[lib] != lab[lib + back];

    ChainEmissions<kBackward> emissions(m, emit_label);
    const unsigned column_a = emissions.column(m, lab, ja), column_b = emissions.column(m, lab, jb);
    // Checkpoints: position i in column 1 + i, this lane's two are columns 1 + min(lia, lib) and the next one.  (has_a
    // false: nothing of this lane is kept.)  Cost only: one row, by pair, in the chain's own order; a lane without a pair B stores
    // what nobody reads in the row's last column.
    CheckpointRows rows(out + m.ab_off, CheckpointRow{lattice_pitch(L)}, kMode == Mode::kGrad ? frame_blocks(m.Tb) - 1 : 1,
                        kMode == Mode::kGrad ? active && has_a : active, kMode == Mode::kGrad ? 1 + (kBackward ? lib : lia) : ja);

    const int last_wave = waves - 1;
    int budget = m.poll_budget;
    bool lost = false;
    const bool every_block = kHandsOver == Exchange::kBlock || (kHandsOver == Exchange::kAny && 2 * halo < 2 * kBlockFrames);
    HandOvers<2> with(kExchange ? lds : nullptr, wave, last_wave, halo, every_block, gentle && !kSteep);
    const unsigned long long look = kSteep ? ~0ull : 0ull;      // after every chunk, whatever the frames

    double va_blank = (ja == 0) ? 1.0 : 0.0, va_label = 0.0, vb_blank = 0.0, vb_label = 0.0;
    ChainFrames<2, kSteep> f(gentle && !kSteep);
    double skip_a_scale = skip_a ? 1.0 : 0.0;
    const double skip_b_one = skip_b ? 1.0 : 0.0;

    int prev_lo = 0, prev_hi = 0;
    auto from_lane_below = [&](double mine) __attribute__((always_inline)) { return shift_up(mine, prev_lo, prev_hi); };
    auto top_value = [&]() __attribute__((always_inline)) { return fmax(fmax(va_blank, va_label), fmax(vb_blank, vb_label)); };
    auto leave = [&](int unit, int frame) __attribute__((always_inline)) {
        if (count < 0) return;
        count = -unit;
        StrainedWave* const w = strained_wave(lds, wave);
        w->states[0][lane] = make_double2(va_blank, va_label);
        w->states[1][lane] = make_double2(vb_blank, vb_label);
        w->frame[lane] = frame;
        rows.drop();
        with.leave();
    };
    auto renew_frames = [&](int unit) __attribute__((always_inline)) {
        const int rise = f.renew(top_value(), halo > 0 ? halo - 1 : 0);
        if (__builtin_expect(strains(va_blank, rise, ja <= L), 0)) leave(unit, f.frame + rise);
        va_blank = __builtin_amdgcn_ldexp(va_blank, rise);
        va_label = __builtin_amdgcn_ldexp(va_label, rise);
        vb_blank = __builtin_amdgcn_ldexp(vb_blank, rise);
        vb_label = __builtin_amdgcn_ldexp(vb_label, rise);
        skip_a_scale = skip_a ? f.scale : 0.0;
    };

    auto checkpoint = [&]() __attribute__((always_inline)) {
        const CheckpointState state_a{va_blank, va_label}, state_b{vb_blank, vb_label};
        rows.template state<kPolicy>(0, kBackward ? state_b : state_a);
        rows.template state<kPolicy>(1, kBackward ? state_a : state_b);
        rows.template frames<kPolicy>(f.frame);          // both pairs of the lane share its frame
        rows.next();
    };
    auto renew_if_due = [&](int unit) __attribute__((always_inline)) {
        if (f.renewal_due(top_value())) renew_frames(unit);
    };
    // Before a block's last kLookAhead steps: may its end be the ordinary one?  (A comparison's result is on its way to a branch for some 20 clocks.)
    unsigned long long outside = 0;
    auto look_ahead = [&](bool exchange) __attribute__((always_inline)) {
        outside = __ballot(f.easy.outside(top_value()));
        if (exchange) with.look(f.frame);
    };
    auto seldom = [](bool unusual) __attribute__((always_inline)) { return kExchange ? unusual : static_cast<bool>(__builtin_expect(unusual, 0)); };      // (see run_chain_linear)
    auto end_block = [&](int block, bool exchange, int unit) __attribute__((always_inline)) {
        const bool unusual = (outside | f.rough | look | (exchange ? with.late | with.shifted : 0ull)) != 0;
        if (exchange && unusual) with.prepare(block, (outside | f.rough) != 0, f.frame, budget, lost);
        if (exchange) {
            const double2 mine[2] = {make_double2(va_blank, va_label), make_double2(vb_blank, vb_label)};
            with.publish(block, mine, f.frame);
            if (with.takes) {
                const int shift = with.tag.x - f.frame;
                va_blank = __builtin_amdgcn_ldexp(with.states[0].x, shift);
                va_label = __builtin_amdgcn_ldexp(with.states[0].y, shift);
                vb_blank = __builtin_amdgcn_ldexp(with.states[1].x, shift);
                vb_label = __builtin_amdgcn_ldexp(with.states[1].y, shift);
                asm volatile("" : "+v"(va_blank), "+v"(va_label), "+v"(vb_blank), "+v"(vb_label));      // (a mask, and not a choice for each)
            }
        }
        if (seldom(unusual)) {
            const double top = top_value();
            if (exchange) with.number &= ~1;
            bool renews = __ballot(f.easy.outside(top)) != 0;      // (then the factors between the frames are made there)
            if (!renews) {
                if (exchange) {
                    f.rescale(__ballot(!(top > 0.0)));
                    skip_a_scale = skip_a ? f.scale : 0.0;
                }
                renews = f.rough != 0;
            }
            if (renews) renew_frames(unit);
        }
    };
    // One step (see run_chain_linear): the pairs' own sums fill the time that the shift takes.
    //   label' = (label + blank + skip * previous label) * emission, as fma(previous, skip, label + blank)
    auto pin = []() { __builtin_amdgcn_sched_barrier(0); };
    auto advance = [&](float ela, float elb) __attribute__((always_inline)) {
#pragma clang fp contract(off)                           // (a product stays a product: fusing it into the next step's sum would tie the steps together)
        const double prev = from_lane_below(vb_label);
        pin();
        const double ub = vb_blank + vb_label;
        pin();
        const double elb_d = static_cast<double>(elb);
        pin();
        const double ib_label = __builtin_fma(va_label, skip_b_one, ub);
        pin();
        vb_blank = vb_blank + va_label;
        pin();
        const double ua = va_blank + va_label;
        pin();
        vb_label = ib_label * elb_d;
        pin();
        const double ela_d = static_cast<double>(ela);
        pin();
        const double ia_label = __builtin_fma(prev, skip_a_scale, ua);
        pin();
        va_blank = __builtin_fma(prev, f.scale, va_blank);
        pin();
        va_label = ia_label * ela_d;
        pin();
    };

    float ela[4][kChunk], elb[4][kChunk];
    auto fetch = [&](auto set, int) __attribute__((always_inline)) {
        constexpr int k = decltype(set)::value;
        emissions.read(column_a, ela[k]);
        emissions.read(column_b, elb[k]);
        emissions.next();
        __builtin_amdgcn_sched_barrier(0);
    };
    auto run = [&](auto set, int i) __attribute__((always_inline)) {
        constexpr int k = decltype(set)::value;
        constexpr bool kEnds = (k & 1) != 0;             // the chunk ends a block
        const bool here = kEnds && kExchange && (kHandsOver != Exchange::kAny || last_wave > 0) && (k == 3 || every_block);
        if (kMode == Mode::kGrad && !kEnds) checkpoint();
#pragma unroll
        for (int q = 0; q < kChunk; ++q) {
            advance(ela[k][q], elb[k][q]);
            if (kSteep && q == kSteepSteps - 1) renew_if_due(2 * i + 1);
            if (here && q == kChunk - 1 - kAskAhead2) with.ask(k >> 1);
            if (q == kChunk - 1 - kLookAhead) look_ahead(here);
        }
        if (kEnds) end_block(k >> 1, here, 2 * i + 2);
        else if (seldom((outside | f.rough | look) != 0)) {
            if (kSteep) renew_if_due(2 * i + 2);
            else renew_frames(2 * i + 2);
        }
        if (kExchange && k == 3) with.next_round();
    };
    chain_schedule(count, fetch, run);
    if (__builtin_expect(count < 0, 0)) return {-count, lost};

    if (kMode == Mode::kLoss) {
        // the state of every pair, for finish_loss
        rows.template state<kPolicy>(0, CheckpointState{va_blank, va_label});
        rows.template state<kPolicy>(1, CheckpointState{vb_blank, vb_label});
        rows.template frames<kPolicy>(f.frame);
        return {0, lost};
    }
    if (!kBackward) {
        // p = alpha_{T-1}(2L) + alpha_{T-1}(2L-1): the blank of pair L and the label of pair L - 1.
        // L even: pair L is this lane's A, pair L - 1 the B of the lane below; L odd: pair L is B.
        const double from_below = from_lane_below(vb_label) * f.scale;
        if (active && (ja == L || jb == L)) publish_mass(&mass[u * kMassWords], ja == L ? va_blank + from_below : vb_blank + va_label, f.frame);
    }
    if (kExchange && lost && lane == 0) publish(&chain_err[u], 1);
    return {0, lost};
}

// A record whose fields the compiler knows to be the same in every lane, wherever it was read from.
__device__ __forceinline__ Utt uniform_record(const Utt& m)
{
    Utt u = m;
    auto uniform = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    auto uniform64 = [&](int64_t v) {
        return static_cast<int64_t>(static_cast<uint64_t>(static_cast<unsigned>(uniform(static_cast<int>(v)))) |
                                    (static_cast<uint64_t>(static_cast<unsigned>(uniform(static_cast<int>(v >> 32)))) << 32));
    };
    u.Tb = uniform(m.Tb);
    u.L = uniform(m.L);
    u.lab_off = uniform(m.lab_off);
    u.flags = uniform(m.flags);
    u.f_off = static_cast<unsigned>(uniform(static_cast<int>(m.f_off)));
    u.e_cols = uniform(m.e_cols);
    u.e_direct = static_cast<int16_t>(uniform(m.e_direct));
    u.waves = uniform(m.waves);
    u.halo = uniform(m.halo);
    u.waves2 = uniform(m.waves2);
    u.halo2 = uniform(m.halo2);
    u.poll_budget = uniform(m.poll_budget);
    u.e_off = uniform64(m.e_off);
    u.ab_off = uniform64(m.ab_off);
    return u;
}

// A state with an exponent of its own, mantissa * 2^exponent; zero: 0 and kNoExponent.
struct OwnExponent {
    double mantissa;
    int exponent;
    __device__ __forceinline__ OwnExponent plus(const OwnExponent& other) const
    {
        const int higher = max(exponent, other.exponent);
        const double v = __builtin_amdgcn_ldexp(mantissa, exponent - higher) + __builtin_amdgcn_ldexp(other.mantissa, other.exponent - higher);
        return {__builtin_amdgcn_frexp_mant(v), higher + __builtin_amdgcn_frexp_exp(v)};
    }
    __device__ __forceinline__ OwnExponent times(double factor) const
    {
        const double v = mantissa * factor;
        return {v, v > 0.0 ? exponent : kNoExponent};
    }
    __device__ __forceinline__ double log2() const
    {
        const double v = static_cast<double>(exponent + __builtin_amdgcn_frexp_exp(mantissa)) +
                         static_cast<double>(fast_log2(static_cast<float>(__builtin_amdgcn_frexp_mant(mantissa))));
        return mantissa > 0.0 ? v : kNeg;
    }
    static __device__ __forceinline__ OwnExponent of(double v, int frame) { return {__builtin_amdgcn_frexp_mant(v), v > 0.0 ? frame + __builtin_amdgcn_frexp_exp(v) : kNoExponent}; }
    static __device__ __forceinline__ OwnExponent of_log2(double w)
    {
        const double whole = floor(w);
        return w > -1.0e9 ? OwnExponent{static_cast<double>(fast_exp2(static_cast<float>(w - whole))), static_cast<int>(whole)} : OwnExponent{0.0, kNoExponent};
    }
};

// The rest of a chain whose wavefront has left the recursion after `unit` half chunks: the same with an exponent to every state, and with the
// checkpoints and the hand-overs of the chain it goes on from, in logarithms (coded_logs).  Returns whether it gave up a wait.
// (Rare, and written to cost the chains it stands behind nothing: every argument is read again.  In logarithms throughout, as in the log domain, rounding added
// up differently in the two directions of an utterance: 2^21 frames, gradient off by 6e-4.)
template <Sync kSync, Mode kMode, bool kFused>
__device__ __forceinline__ bool finish_with_exponents(int unit, bool lost, void* lds)
{
    // (one at a time: eight words of them loaded at once had to be kept in memory)
    auto args = []() -> const ChainArgs<kFused>& { return args_again<ChainArgs<kFused>>(); };
    const int chain = __builtin_amdgcn_readfirstlane(args().order[blockIdx.x]), u = chain >> 1;
    const bool backward = (chain & 1) != 0;
    const Utt m = uniform_record(args().meta[u]);
    const bool two = kSync == Sync::kHalo && (m.flags & kUttTwoPairs) != 0;
    const int L = m.L, chunks = 2 * frame_blocks(m.Tb), units = 2 * (kMode == Mode::kLoss ? chain_chunks(m.Tb, backward) : chunks);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int halo = two ? m.halo2 : (kSync == Sync::kHalo ? m.halo : 0), last_wave = (two ? m.waves2 : m.waves) - 1;
    const int first_pair = (two ? 2 : 1) * (wave * (64 - halo) + lane);
    const bool active = (wave == 0 || lane >= halo) && first_pair <= L;
    const int* const lab = args().labels + m.lab_off;
    // Pair 0 or 1 of the lane: its label's index (back: to the pair before), whether it has one, whether that may be entered from the pair before's.
    const int back = backward ? 1 : -1;
    auto position = [&](int k) { return backward ? L - 1 - (first_pair + k) : first_pair + k; };
    const bool has0 = first_pair < L, has1 = two && first_pair + 1 < L;
    const int symbol0 = has0 ? lab[position(0)] : 0, symbol1 = has1 ? lab[position(1)] : 0;
    const bool skip0 = has0 && first_pair >= 1 && symbol0 != lab[position(0) + back], skip1 = has1 && symbol1 != symbol0;
    const int first_chunk = chain_chunk(0, chunks, backward);
    const float* const emit_label = args().emit_label;
    const float* const at0 = emit_label + label_emission_offset(m, has0, symbol0, position(0), first_chunk, kZeroEmission);
    const float* const at1 = emit_label + label_emission_offset(m, has1, symbol1, position(1), first_chunk, kZeroEmission);
    const int64_t step0 = label_emission_step(m, has0, backward), step1 = label_emission_step(m, has1, backward);

    struct Pair { OwnExponent blank, label; };
    const OwnExponent zero{0.0, kNoExponent};
    Pair s0{zero, zero}, s1{zero, zero};
    auto pair_of = [](const double2& v, int frame) {
        const CheckpointState logs = state_logs(CheckpointState{v.x, v.y}, frame);
        return frame == kLogs ? Pair{OwnExponent::of_log2(logs.blank), OwnExponent::of_log2(logs.label)} : Pair{OwnExponent::of(v.x, frame), OwnExponent::of(v.y, frame)};
    };
    auto take = [&](const double2& v0, const double2& v1, int frame) {
        s0 = pair_of(v0, frame);
        if (two) s1 = pair_of(v1, frame);
    };
    auto coded = [](const Pair& s) {
        const CheckpointState c = coded_logs(s.blank.log2(), s.label.log2());
        return make_double2(c.blank, c.label);
    };
    const StrainedWave* const from = strained_wave(lds, wave);
    take(from->states[0][lane], from->states[1][lane], from->frame[lane]);

    constexpr bool kGrad = kMode == Mode::kGrad;
    CheckpointRows rows((backward ? args().lat.beta : args().lat.alpha) + m.ab_off, CheckpointRow{lattice_pitch(L)}, kGrad ? frame_blocks(m.Tb) - 1 : 1,
                        active && (has0 || !kGrad), !kGrad ? first_pair : 1 + position(two && backward ? 1 : 0));
    rows.next_by = rows.step;
    if (kGrad) rows.at = ((unit - 1) >> 2) * rows.step;  // (four units make a block)
    constexpr int kPolicy = kFused || !kGrad ? kPast : 0;
    auto store = [&]() {
        const double2 c0 = coded(s0), c1 = coded(s1);
        const CheckpointState a{c0.x, c0.y}, b{c1.x, c1.y};
        const bool swapped = kGrad && two && backward;
        rows.template state<kPolicy>(0, swapped ? b : a);
        rows.template frame<kPolicy>(kLogs);
        if (two) {
            rows.template state<kPolicy>(1, swapped ? a : b);
            rows.template frames<kPolicy>(kLogs);
        }
        rows.next();
    };

    // Hand-overs: as in the chain, one thing after the other.
    const bool exchanges = kSync == Sync::kHalo && last_wave > 0;
    const bool every_block = (two ? 2 : 1) * halo < 2 * kBlockFrames;
    int generation = every_block ? unit >> 2 : unit >> 3, budget = m.poll_budget;
    // At the end of `block`.
    auto hand_over = [&](int block) {
        ++generation;
        const int slot = block & (kRing - 1), first = 64 - halo, wr_slot = max(lane - first, 0), rd_slot = min(lane, halo - 1);
        auto data = [&](int w, int l, int k) {
            return two ? &halo_wave<LinearWave<2>>(lds, w)->slot[slot].states[k][l] : &halo_wave<LinearWave<1>>(lds, w)->slot[slot].states[0][l];
        };
        auto tag = [&](int w, int l) {
            return reinterpret_cast<unsigned long long*>(two ? &halo_wave<LinearWave<2>>(lds, w)->slot[slot].tag[l].word : &halo_wave<LinearWave<1>>(lds, w)->slot[slot].tag[l].word);
        };
        // Waits until wavefront w has published the number `until`, in this lane's tag.  (LDS operations of a wavefront complete in order.)
        auto wait = [&](int w, int until) {
            unsigned long long seen;
            auto early = [&]() {
                seen = __hip_atomic_load(tag(w, rd_slot), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                return __ballot(static_cast<int>(seen >> 32) < 2 * until) != 0;
            };
            bool waits = early();
            for (; waits && budget > 0; --budget) waits = early();
            lost = lost || waits;
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            return static_cast<int>(seen);
        };
        if (wave < last_wave) wait(wave + 1, generation - (every_block ? kRing : kRing / 2));
        if (lane >= first) {
            *data(wave, wr_slot, 0) = coded(s0);
            if (two) *data(wave, wr_slot, 1) = coded(s1);
        }
        if (wave > 0) {
            const int f = wait(wave - 1, generation);
            const double2 v0 = *data(wave - 1, rd_slot, 0), v1 = *data(wave - 1, rd_slot, two ? 1 : 0);
            if (lane < halo) take(v0, v1, f);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        if (lane >= first)
            __hip_atomic_store(tag(wave, wr_slot), (static_cast<unsigned long long>(static_cast<unsigned>(2 * generation)) << 32) | static_cast<unsigned>(kLogs),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };

    auto from_lane_below = [&]() {
        const OwnExponent last = two ? s1.label : s0.label;
        return OwnExponent{lane_shift<false>(last.mantissa), __builtin_amdgcn_update_dpp(kNoExponent, last.exponent, 0x138, 0xf, 0xf, false)};
    };
    static_assert(kSteepSteps == 4 && kBlockFrames == 4 * kSteepSteps, "units of four steps");
    // (a block that has just ended has handed over, but its checkpoint is to come)
    if (kGrad && (unit & 3) == 0) store();
#pragma unroll 1
    for (; unit < units; ++unit) {
        const int64_t in_chunk = (unit & 1) != (backward ? 1 : 0) ? kSteepSteps : 0;
        const float4 el0 = *reinterpret_cast<const float4*>(at0 + (unit >> 1) * step0 + in_chunk), el1 = *reinterpret_cast<const float4*>(at1 + (unit >> 1) * step1 + in_chunk);
#pragma unroll 1
        for (int q = 0; q < kSteepSteps; ++q) {
            const int frame = backward ? kSteepSteps - 1 - q : q;
            auto component = [&](const float4& v) { return frame == 0 ? v.x : frame == 1 ? v.y : frame == 2 ? v.z : v.w; };
            auto step = [&](Pair& s, const OwnExponent& before, bool skip, float emission) {
                const OwnExponent blank = s.blank.plus(before), label = s.label.plus(skip ? blank : s.blank);
                s = Pair{blank, label.times(static_cast<double>(emission))};
            };
            const OwnExponent prev = from_lane_below();
            if (two) step(s1, s0.label, skip1, component(el1));
            step(s0, prev, skip0, component(el0));
        }
        if ((unit & 3) == 3) {
            if (exchanges && (every_block || (unit & 4) != 0)) hand_over(unit >> 2);
            if (kGrad) store();
        }
    }
    if (!kGrad) {
        store();
        return lost;
    }
    if (!backward) {
        // (see run_chain_linear2)
        const OwnExponent below = from_lane_below();
        if (active && (first_pair == L || (two && first_pair + 1 == L))) {
            const OwnExponent p = first_pair == L ? s0.blank.plus(below) : s1.blank.plus(s0.label);
            publish_mass(&args().mass[u * kMassWords], p.mantissa, p.exponent);
        }
    }
    if (kSync == Sync::kHalo && lost && lane == 0) publish(&args().chain_err[u], 1);
    return lost;
}

// Cost-only calls: the mass of an utterance from the states that its two chains have left where they meet, alpha after
// the last of the forward chain's frames and beta (its frame included) at the first of the backward chain's:
//   p = sum over states s of  (sum of alpha over s and its predecessors) * beta(s).
// A wavefront that has ended counts itself in, and the utterance's last one does the sum, whichever it is: the order of
// the additions is that of the pairs.  The count carries how many wavefronts gave up waiting for a
// neighbour, from bit 16 on (then the cost is NaN), and, from bit 24 on, how many
// have left logarithms (finish_with_exponents).  `waves`: wavefronts of a chain.  One more wavefront counts itself in, which has nothing to do with
// the chains and leaves the norms (norms_of_utterance).
__device__ __forceinline__ void finish_loss(const Utt& m, const int u, const int* __restrict__ labels, const LatticeOut& lat,
                                            const double* __restrict__ mass, int* __restrict__ done, float* __restrict__ costs,
                                            const int waves, const bool lost, const bool in_logs)
{
    constexpr int kLost = 1 << 16, kInLogs = 1 << 24;    // (up to 33 wavefronts)
    const int lane = threadIdx.x & 63, expected = 2 * waves + 1;
    // (the chains may run on different dies; what has been published is past the die's cache once it is out)
    int before = 0;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (lane == 0)
        before = __hip_atomic_fetch_add(&done[u * kDoneStride], 1 + (lost ? kLost : 0) + (in_logs ? kInLogs : 0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    before = __builtin_amdgcn_readfirstlane(before);
    if ((before & (kLost - 1)) != expected - 1) return;
    const bool given_up = (before & (kInLogs - kLost)) != 0 || lost, some_logs = before >= kInLogs || in_logs;
    const int L = m.L;
    const CheckpointRow row{lattice_pitch(L)};
    const CheckpointState *const alpha = row.states(lat.alpha + m.ab_off, 0), *const beta = row.states(lat.beta + m.ab_off, 0);
    const int *const fa = row.frames(lat.alpha + m.ab_off, 0), *const fb = row.frames(lat.beta + m.ab_off, 0);
    const int* const lab = labels + m.lab_off;
    const double log2_norms = published(&mass[u * kMassWords + kMassNorms]);
    // A lane's sum as sum * 2^top.
    double sum = 0.0;
    int top = kNoExponent;
    auto add = [&](double a, int a_frame, double b, int b_frame) {
        if (!(a > 0.0 && b > 0.0)) return;
        const double v = __builtin_amdgcn_frexp_mant(a) * __builtin_amdgcn_frexp_mant(b);
        const int e = a_frame + b_frame + __builtin_amdgcn_frexp_exp(a) + __builtin_amdgcn_frexp_exp(b);
        const int higher = max(top, e);
        sum = __builtin_amdgcn_ldexp(sum, max(top - higher, -2000)) + __builtin_amdgcn_ldexp(v, max(e - higher, -2000));
        top = higher;
    };
    // pair j going forward: blank j and label j; the backward chain's pair i: blank L - i and label L - 1 - i.  (Past the cache each look
    // is a trip to memory: kAtOnce pairs' words travel together.)  logs: some are logarithms.
    auto add_pairs = [&](auto logs) __attribute__((always_inline)) {
        constexpr bool kSomeLogs = decltype(logs)::value;
        constexpr int kAtOnce = kSomeLogs ? 1 : 2;
        // (to a value and a frame of its own again)
        auto plain = [](double& v, int& frame, bool is_blank) {
            const double code = is_blank ? v * 0x1p1000 : v, w = code - kLogOffset, whole = floor(w);
            if (!kSomeLogs || frame != kLogs) return;
            frame = code > 0x1p27 ? static_cast<int>(whole) : 0;
            v = code > 0x1p27 ? static_cast<double>(fast_exp2(static_cast<float>(w - whole))) : 0.0;
        };
        for (int j0 = lane; j0 - lane <= L; j0 += 64 * kAtOnce) {
            CheckpointState a[kAtOnce];
            double before_label[kAtOnce], blank_b[kAtOnce], label_b[kAtOnce];
            int a_frame[kAtOnce], before_frame[kAtOnce], blank_frame[kAtOnce], label_frame[kAtOnce];
            bool skips[kAtOnce];
#pragma unroll
            for (int n = 0; n < kAtOnce; ++n) {
                const int j = min(j0 + 64 * n, L), before = max(j - 1, 0), after = max(L - 1 - j, 0);
                a[n] = published(&alpha[row.slot(j)]);
                a_frame[n] = published(&fa[j]);
                before_label[n] = published(&alpha[row.slot(before)].label);
                before_frame[n] = published(&fa[before]);
                blank_b[n] = published(&beta[row.slot(L - j)].blank);
                blank_frame[n] = published(&fb[L - j]);
                label_b[n] = published(&beta[row.slot(after)].label);
                label_frame[n] = published(&fb[after]);
                skips[n] = j > 0 && j < L && lab[j] != lab[j - 1];
            }
#pragma unroll
            for (int n = 0; n < kAtOnce; ++n) {
                const int j = j0 + 64 * n;
                if (j > L) continue;
                int a_blank_frame = a_frame[n];
                plain(a[n].blank, a_blank_frame, true);
                plain(a[n].label, a_frame[n], false);
                plain(before_label[n], before_frame[n], false);
                plain(blank_b[n], blank_frame[n], true);
                plain(label_b[n], label_frame[n], false);
                add(a[n].blank, a_blank_frame, blank_b[n], blank_frame[n]);
                if (j > 0) add(before_label[n], before_frame[n], blank_b[n], blank_frame[n]);
                if (j < L) {
                    add(a[n].label, a_frame[n], label_b[n], label_frame[n]);
                    add(a[n].blank, a_blank_frame, label_b[n], label_frame[n]);
                    if (skips[n]) add(before_label[n], before_frame[n], label_b[n], label_frame[n]);
                }
            }
        }
    };
    if (__builtin_expect(some_logs, 0)) add_pairs(std::true_type{});
    else add_pairs(std::false_type{});
    for (int d = 1; d < 64; d <<= 1) {
        const double other = __shfl_xor(sum, d);
        const int other_top = __shfl_xor(top, d), higher = max(top, other_top);
        sum = __builtin_amdgcn_ldexp(sum, max(top - higher, -2000)) + __builtin_amdgcn_ldexp(other, max(other_top - higher, -2000));
        top = higher;
    }
    if (lane == 0) costs[u] = given_up ? __uint_as_float(0x7FC00000u) : cost_of_mass(sum, top, log2_norms);
}

// The word that an utterance's chains and the workgroups that wait for them share: wavefronts that have ended, wavefronts
// there are (from bit 10), chains that have said how many (from bit 20), and whether a workgroup has given up waiting.
constexpr int kWavesShift = 10, kChainsShift = 20, kWaitGivenUp = 1 << 24;
__device__ __forceinline__ bool chains_ended(int done)
{
    constexpr int kField = (1 << kWavesShift) - 1;
    return ((done >> kChainsShift) & 3) == 2 && (done & kField) == ((done >> kWavesShift) & kField);
}
// A wavefront of a chain has ended, and everything it has published is out; `waves` of them make the chain, the first says
// so.  (What log-domain chains have stored the ordinary way must leave the die's cache before.)
__device__ __forceinline__ void announce_end(int* done, int waves)
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const int count = threadIdx.x < 64 ? 1 + (waves << kWavesShift) + (1 << kChainsShift) : 1;
    if ((threadIdx.x & 63) == 0) __hip_atomic_fetch_add(done, count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A launch that writes the gradient too: an utterance's second word says which of its chains have been taken, that is, have a
// workgroup that runs them (bits 0 and 1), and which of the gradient's workgroups have left their places because that took
// too long: the last one's number plus one (from bit 2), the one before it in that one's word of `left`, and so on.
constexpr int kBothTaken = 3, kLeftShift = 2;
__device__ __forceinline__ int take_chain(int* word, int direction)
{
    return __hip_atomic_fetch_or(word, 1 << direction, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// (tests: a chain's workgroup comes so late that places have been left; bounded, in case there are none)
__device__ __forceinline__ void wait_until_left(const int* word)
{
    for (int polls = 1 << 14; polls > 0 && published(word) >> kLeftShift == 0; --polls) __builtin_amdgcn_s_sleep(10);
}

// `chain`: utterance * 2 + direction.  kFused: the launch writes the gradient too; then the result, for the wavefronts that are
// still there, is the list of places that this workgroup is to take after its chain (take_chain), 0 where there are none.
template <Sync kSync, Mode kMode, bool kFused = false>
__device__ __forceinline__ int lattice_body(const int chain, const Utt* __restrict__ meta, const int* __restrict__ labels,
                                             const float* __restrict__ emit_blank, const double* __restrict__ emit_blank64,
                                             const float* __restrict__ emit_label,
                                             const LatticeOut lat,
                                             double* __restrict__ mass, float* __restrict__ costs,
                                             int* __restrict__ chain_err, uint32_t* __restrict__ sink,
                                             void* lds, const LaunchWords& wk)
{
    // The first workgroup of the launch tells the host that the pinned image of the call is free
    // again (calls whose softmax launch read the image itself: this launch follows it).
    if (blockIdx.x == 0 && threadIdx.x == 0 && wk.host_flag)
        __hip_atomic_store(wk.host_flag, wk.host_flag_value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    // ... and gathers the per-utterance verdicts of a softmax launch that built the records itself.
    if (blockIdx.x == 0 && threadIdx.x < 64 && wk.status_out) {
        bool bad = false;
        for (int i = threadIdx.x; i < wk.status_count; i += 64) bad = bad || wk.status_words[i] != 0;
        const bool any = __ballot(bad) != 0;
        if (threadIdx.x == 0) *wk.status_out = any ? CTC_STATUS_INVALID_VALUE : CTC_STATUS_SUCCESS;
    }
    if (chain < 0) return 0;      // device-planned batches launch a workgroup per utterance and direction, running or not
    // (measurements of the recursions one after the other: a launch that leaves one direction out)
    if (kMode == Mode::kGrad && ((wk.skip_directions >> (chain & 1)) & 1)) return 0;
    // Lanes of log-domain chains with nothing to store write to a sink: 64 bytes of it per wavefront of the launch.  (One
    // address for the whole launch was what a crowded launch waited for: every store instruction of
    // every chain carried a write to it, and they all met in one channel of each die's L2.  512
    // utterances of 20 symbols and 740 frames: 59 -> 40 us.  Writing to an unused column of the
    // chain's own rows instead was slower than either in launches that are not crowded.)
    sink += (static_cast<size_t>(kFused ? chain : blockIdx.x) * kSinkWaves + (threadIdx.x >> 6)) * (kSinkBytes / sizeof(uint32_t));
    const int u = chain >> 1;
    const bool forward = (chain & 1) == 0;
    // (asked for here, looked at once what else the chain starts from has come)
    int before = 0, left = 0;
    if (kFused && threadIdx.x == 0) {
        int* const word = &wk.done[u * kDoneStride + kTakenWord];
        if (static_cast<int>(blockIdx.x) * 37 % 100 < wk.late_percent) wait_until_left(word);
        before = take_chain(word, forward ? 0 : 1);
        // the second to take one: nobody leaves after this
        left = (before & kBothTaken) != 0 ? before >> kLeftShift : 0;
    }
    const Utt m = meta[u];
    if (!(m.flags & kUttRuns)) return 0;     // (a run order built on the device lists every utterance)
    // Which recursion: the barrier kernel and the maximum recursion have the log domain only;
    // otherwise the flag that the softmax launch may have raised decides.  A linear-domain chain
    // gives one pair or two to a lane as the launcher planned it (two_pairs_per_lane).
    const int met = rows_flagged(wk.row_flags, u, wk.flag_blocks, m.Tb);
    const bool in_log_domain = kSync == Sync::kBarrier || kMode == Mode::kBest || (m.flags & kUttLogDomain) != 0 || (met & kRowsSmall) != 0;
    const bool gentle = m.rough == 0 && (met & kRowsRough) == 0, steep = m.steep != 0 || (met & kRowsSteep) != 0;
    if (kMode == Mode::kLoss && in_log_domain && !forward) return 0;       // (the forward chain runs all the way)
    const bool two_pairs = kSync == Sync::kHalo && !in_log_domain && (m.flags & kUttTwoPairs) != 0;
    const int waves = two_pairs ? m.waves2 : m.waves;
    const bool idle = static_cast<int>(threadIdx.x >> 6) >= waves;
    if (kSync == Sync::kHalo) {
        // the exchange buffer in use starts with every counter and hand-over number at zero
        // (every wavefront of the workgroup clears its own block, whether it takes part or not)
        HaloHeader* hl = static_cast<HaloHeader*>(lds);
        if (in_log_domain) {
            HaloWave* w = halo_wave<HaloWave>(lds, threadIdx.x >> 6);
            w->ready = 0;
            w->done = 0;
        } else {
            auto clear = [&](auto* w) {
                constexpr int kLanes = std::remove_pointer_t<decltype(w)>::kLanes;
                for (int i = threadIdx.x & 63; i < kRing * kLanes; i += 64) w->slot[i / kLanes].tag[i % kLanes].word = make_int2(0, 0);
            };
            if (two_pairs) clear(halo_wave<LinearWave<2>>(lds, threadIdx.x >> 6));
            else clear(halo_wave<LinearWave<1>>(lds, threadIdx.x >> 6));
        }
        if (threadIdx.x == 0) {
            hl->finished = 0;
            hl->gave_up = 0;
            hl->left = left;
        }
        __syncthreads();
        if (kFused) left = __builtin_amdgcn_readfirstlane(hl->left);
        if (idle) return left;
    } else if (kSync == Sync::kBarrier) {
        if (idle) {
            // Nothing to compute, but keep meeting the barriers of the working wavefronts:
            // one per recursion step, plus the forward chain's final exchange.
            // (the maximum's: two, for the origin as well)
            const int barriers = kMode == Mode::kBest ? 2 * chain_chunks(m.Tb, !forward) * kChunk
                                                      : static_cast<int>(padded_frames(m.Tb)) + (forward ? 1 : 0);
            for (int i = 0; i < barriers; ++i) __syncthreads();
            return 0;
        }
    }
    if (kFused && kSync == Sync::kNone) {
        HaloHeader* const hl = static_cast<HaloHeader*>(lds);
        if (threadIdx.x == 0) hl->left = left;
        __syncthreads();
        left = __builtin_amdgcn_readfirstlane(hl->left);
        if (threadIdx.x >= 64) return left;
    }
    // (for the gradient, which must know what each chain has left: a word per direction)
    if (kMode == Mode::kGrad && threadIdx.x == 0) publish(&wk.domain[2 * u + (forward ? 0 : 1)], in_log_domain ? kDomainLog : (steep ? kDomainSteep : 0));
    if constexpr (kSync != Sync::kBarrier && kMode != Mode::kBest) {
        if (!in_log_domain) {
            ChainEnd end{0, false};
            auto run = [&](auto steep_ones) __attribute__((always_inline)) {
                constexpr bool kSteep = decltype(steep_ones)::value;
                constexpr int kPolicy = kFused || kMode == Mode::kLoss ? kPast : 0;
                auto of_direction = [&](auto backward, auto exchange) __attribute__((always_inline)) {
                    constexpr bool kBackward = decltype(backward)::value;
                    constexpr Exchange kExchange = decltype(exchange)::value;
                    // (read again: with the pointers of both directions held through either the kernel came out with room for them in memory)
                    const auto& again = args_again<ChainArgs<kFused>>();
                    uint32_t* const out = kBackward ? again.lat.beta : again.lat.alpha;
                    if (kSync == Sync::kHalo && two_pairs)
                        end = run_chain_linear2<kBackward, kExchange, kMode, kSteep, kPolicy>(m, u, gentle, again.labels, again.emit_label, out, again.mass, again.chain_err, lds);
                    else
                        end = run_chain_linear<kBackward, kExchange, kMode, kSteep, kPolicy>(m, u, gentle, again.labels, again.emit_label, out, again.mass, again.chain_err, lds);
                };
                auto handing_over = [&](auto exchange) __attribute__((always_inline)) {
                    if (forward) of_direction(std::false_type{}, exchange);
                    else of_direction(std::true_type{}, exchange);
                };
                // (a halo lasts as many frames as it has pairs.  Steep chains, which are rare, ask as they go: with a loop for each kind of theirs as well the largest of these kernels had
                // 324 KB, so 249, and the build took 2.6 minutes, so 1.7.  us a call: 64 x 750 x 29, logits of deviation 6, 55.7 and 55.0, cost only, of deviation 4, 32.9 and 32.3.)
                if (kSync == Sync::kNone || (waves == 1 && !kSteep)) handing_over(std::integral_constant<Exchange, Exchange::kNone>{});
                else if constexpr (kSync == Sync::kHalo) {
                    if constexpr (kSteep) handing_over(std::integral_constant<Exchange, Exchange::kAny>{});
                    else if ((two_pairs ? 2 * m.halo2 : m.halo) < 2 * kBlockFrames) handing_over(std::integral_constant<Exchange, Exchange::kBlock>{});
                    else handing_over(std::integral_constant<Exchange, Exchange::kTwoBlocks>{});
                }
            };
            if (__builtin_expect(steep, 0)) run(std::true_type{});
            else run(std::false_type{});
            if (__builtin_expect(end.unit != 0, 0)) end.lost = finish_with_exponents<kSync, kMode, kFused>(end.unit, end.lost, lds);
            if (kMode == Mode::kLoss) finish_loss(m, u, labels, lat, mass, wk.done, costs, waves, end.lost, end.unit != 0);
            if (kFused) announce_end(&wk.done[u * kDoneStride], waves);
            return left;
        }
    }
    if (forward)
        run_chain_log<false, kSync, kMode>(m, u, labels, emit_blank, emit_blank64, emit_label, lat.alpha, lat.alpha_exponents, mass, costs, chain_err, sink, lds);
    else if constexpr (kMode != Mode::kLoss)
        run_chain_log<true, kSync, kMode>(m, u, labels, emit_blank, emit_blank64, emit_label, lat.beta, lat.beta_exponents, mass, costs, chain_err, sink, lds);
    if (kFused) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        announce_end(&wk.done[u * kDoneStride], waves);
    }
    return left;
}

// Cost-only launches: a wavefront of the workgroups behind the chains' leaves an utterance's norms and counts itself in.  (As one
// wavefront more in the forward chain's workgroup it moved the workgroups after it to other SIMDs than order_chains means, and with a
// write-back of the die's cache of its own: 512 x 750 frames 72 -> 83 us a call, 500 x 60 29.6 -> 35.7; so 69.6 and 28.9.)
template <Sync kSync>
__device__ __forceinline__ void norms_of_utterance(const Utt* __restrict__ meta, const int* __restrict__ labels, const float* __restrict__ emit_blank,
                                                   const LatticeOut& lat, double* __restrict__ mass, float* __restrict__ costs, const LaunchWords& wk)
{
    const int u = (static_cast<int>(blockIdx.x) - wk.norm_groups) * static_cast<int>(blockDim.x >> 6) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (u >= wk.utterances) return;
    const Utt m = meta[u];
    if (!(m.flags & kUttRuns)) return;
    if ((m.flags & kUttLogDomain) != 0 || (rows_flagged(wk.row_flags, u, wk.flag_blocks, m.Tb) & kRowsSmall) != 0) return;      // (run_chain_log)
    const Norms norms = norms_of_wave(norms_of_lane(m, emit_blank));
    if ((threadIdx.x & 63) == 0) publish(&mass[u * kMassWords + kMassNorms], norms.log2());
    const bool two_pairs = kSync == Sync::kHalo && (m.flags & kUttTwoPairs) != 0;
    finish_loss(m, u, labels, lat, mass, wk.done, costs, two_pairs ? m.waves2 : m.waves, false, false);
}

// grid = one workgroup per entry of `order` (utterance * 2 + direction: 0 forward, 1 backward); cost-only launches: then those of
// norms_of_utterance, a wavefront per utterance.
// blockDim.x = 64 * (most wavefronts any utterance of the batch uses).
// Variant for batches whose labels all fit one wavefront: no exchange at all.
template <Mode kMode>
__global__ __launch_bounds__(64)
void ctc_lattice_kernel_w1(const Utt* __restrict__ meta, const int* __restrict__ order,
                           const int* __restrict__ labels, const float* __restrict__ emit_blank,
                           const double* __restrict__ emit_blank64,
                           const float* __restrict__ emit_label,
                           const LatticeOut lat,
                           double* __restrict__ mass, float* __restrict__ costs,
                           int* __restrict__ chain_err, uint32_t* __restrict__ sink, const LaunchWords wk)
{
    if (kMode == Mode::kGrad && static_cast<int>(blockIdx.x) >= wk.fill.n_chains && wk.fill.defer > 0) {
        fill_rows_beside_chains(wk.fill, meta);
        return;
    }
    if (kMode == Mode::kLoss && static_cast<int>(blockIdx.x) >= wk.norm_groups) {
        norms_of_utterance<Sync::kNone>(meta, labels, emit_blank, lat, mass, costs, wk);
        return;
    }
    __shared__ double2 lds[kMode == Mode::kBest ? 1 : halo_lds_bytes(1) / sizeof(double2)];
    lattice_body<Sync::kNone, kMode>(order[blockIdx.x], meta, labels, emit_blank, emit_blank64, emit_label, lat,
                                                                   mass, costs, chain_err, sink, lds, wk);
}

// Multi-wavefront chains with the halo exchange.
template <Mode kMode>
__global__ __launch_bounds__(1024)
void ctc_lattice_kernel(const Utt* __restrict__ meta, const int* __restrict__ order,
                        const int* __restrict__ labels, const float* __restrict__ emit_blank,
                        const double* __restrict__ emit_blank64,
                        const float* __restrict__ emit_label,
                        const LatticeOut lat,
                        double* __restrict__ mass, float* __restrict__ costs,
                        int* __restrict__ chain_err, uint32_t* __restrict__ sink, const LaunchWords wk)
{
    extern __shared__ double2 halo_lds[];                    // halo_lds_bytes(wavefronts of the workgroup)
    if (kMode == Mode::kGrad && static_cast<int>(blockIdx.x) >= wk.fill.n_chains && wk.fill.defer > 0) {
        fill_rows_beside_chains(wk.fill, meta);
        return;
    }
    if (kMode == Mode::kLoss && static_cast<int>(blockIdx.x) >= wk.norm_groups) {
        norms_of_utterance<Sync::kHalo>(meta, labels, emit_blank, lat, mass, costs, wk);
        return;
    }
    lattice_body<Sync::kHalo, kMode>(order[blockIdx.x], meta, labels, emit_blank, emit_blank64, emit_label, lat,
                                                                   mass, costs, chain_err, sink, halo_lds, wk);
}

// Labels too long to leave room for a halo (more than 16 * 63 pairs): 64 pairs per wavefront
// and one barrier per step.
template <Mode kMode>
__global__ __launch_bounds__(1024)
void ctc_lattice_kernel_barrier(const Utt* __restrict__ meta, const int* __restrict__ order,
                                const int* __restrict__ labels, const float* __restrict__ emit_blank,
                                const double* __restrict__ emit_blank64,
                                const float* __restrict__ emit_label,
                                const LatticeOut lat,
                                double* __restrict__ mass, float* __restrict__ costs,
                                int* __restrict__ chain_err, uint32_t* __restrict__ sink, const LaunchWords wk)
{
    __shared__ double xch[3][16];                            // (labels by step parity; their origins, two words each)
    lattice_body<Sync::kBarrier, kMode>(order[blockIdx.x], meta, labels, emit_blank, emit_blank64, emit_label, lat, mass,
                                               costs, chain_err, sink, &xch[0][0], wk);
}

// ---- after the chains of the most probable alignment ------------------------------------------
// The best way through the two frames where the chains meet, and from there a walk over the stored choices in either
// direction, forward chain's frames back to the first and backward chain's frames on to the last.  grid (utterances,
// 2), one wavefront each; alignment is [B][T] (utterance-major): the lattice state of each
// frame (index into the blank-interleaved label), -1 for frames past the utterance's end and
// for utterances without an alignment.  Both chains index their states in their own order (the backward chain's state s
// is the lattice's 2 L - s), so the two walks are the same code.
//
// A walk is serial, one dependent look-up per frame, so it is cut into the chains' segments: from the junction the origins
// lead from segment to segment, and each wavefront walks its own.  That walk is kept on the scalar unit: the choices of the
// segment are in registers, a word per chunk, lane = pair column.  Going back kSegment steps the walk moves down by at
// most kSegment - 1 pairs (one per frame), so the 64 columns up to the walk's position hold everything those steps can
// touch.  A step is then a v_readlane at the walk's column, a shift, a mask and a subtraction in scalar registers, and
// a v_writelane that files the state for the segment's one coalesced store.
// (64 utterances of up to 750 frames: 23.7 us in one walk of 375 steps at 45 ns, with the choices as bytes.)
constexpr int kBacktraceWaves = 16;
constexpr int kOriginWords = 12288;       // origins kept in LDS, if they fit

// grid (B, 2), up to kBacktraceWaves wavefronts; dynamic LDS `lds_words` words.
__global__ __launch_bounds__(64 * kBacktraceWaves)
void ctc_backtrace_kernel(const Utt* __restrict__ meta, const int* __restrict__ labels, const LatticeOut lat,
                          const int* __restrict__ chain_err, float* __restrict__ costs, int* __restrict__ alignment, int Tt, int lds_words)
{
    extern __shared__ uint32_t s_origins[];
    const int b = blockIdx.x, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int waves = blockDim.x >> 6;
    const bool backward = blockIdx.y != 0;
    const Utt m = meta[b];
    int* arow = alignment + static_cast<size_t>(b) * Tt;
    const bool runs = (m.flags & kUttRuns) != 0;
    const bool bad = runs && chain_err[b] != 0;
    if (bad && threadIdx.x == 0 && !backward) costs[b] = __uint_as_float(0x7FC00000u);
    const int valid = (runs && !bad) ? m.Tb : 0, L = m.L;
    if (backward)
        for (int t = valid + threadIdx.x; t < Tt; t += blockDim.x) arow[t] = -1;
    if (valid == 0) return;
    const int rows_all = chain_chunks(m.Tb, backward) * kChunk, P = L + 1, segments = (rows_all + kSegment - 1) / kSegment;
    const uint32_t* const origins = reinterpret_cast<const uint32_t*>(backward ? lat.beta_exponents : lat.alpha_exponents) + m.ab_off + origin_word(P, 0);
    const bool in_lds = segments * P <= lds_words;
    if (in_lds)
        for (int i = threadIdx.x; i < segments * P; i += blockDim.x) s_origins[i] = origins[i];

    // The junction: the state `to` of the backward chain's first frame and the best state `from` before it.  Per
    // pair the blank before the label, within a state the predecessor as in the forward chain (stay first); of equal ways
    // the highest state.
    const CheckpointState* const alpha = reinterpret_cast<const CheckpointState*>(lat.alpha_exponents + m.ab_off);
    const CheckpointState* const beta = reinterpret_cast<const CheckpointState*>(lat.beta_exponents + m.ab_off);
    const int* const lab = labels + m.lab_off;
    double best = -1.0e300;
    int from = 0, to = 0;
    for (int j = lane; j <= L; j += 64) {
        const CheckpointState a = alpha[j];
        const double before = j > 0 ? alpha[j - 1].label : kNeg;
        const double to_blank = fmax(a.blank, before) + beta[L - j].blank;
        if (to_blank >= best) {
            best = to_blank;
            to = 2 * j;
            from = before > a.blank ? 2 * j - 1 : 2 * j;
        }
        if (j < L) {
            double w = a.label;
            int s = 2 * j + 1;
            if (a.blank > w) { w = a.blank; s = 2 * j; }
            if (j > 0 && lab[j] != lab[j - 1] && before > w) { w = before; s = 2 * j - 1; }
            w += beta[L - 1 - j].label;
            if (w >= best) {
                best = w;
                to = 2 * j + 1;
                from = s;
            }
        }
    }
    for (int d = 1; d < 64; d <<= 1) {
        const double other = __shfl_xor(best, d);
        const int other_from = __shfl_xor(from, d), other_to = __shfl_xor(to, d);
        if (other > best || (other == best && other_to > to)) {
            best = other;
            from = other_from;
            to = other_to;
        }
    }
    if (threadIdx.x == 0 && !backward) costs[b] = (best < -1.0e29) ? __builtin_inff() : static_cast<float>(-best * kLn2);

    // this walk: frames in the chain's own order (frame_of), from the state it was in at its last one
    __syncthreads();
    const int padded = static_cast<int>(padded_frames(m.Tb));
    const uint32_t* const choices = (backward ? lat.beta : lat.alpha) + m.ab_off;
    auto frame_of = [&](int step) { return backward ? padded - 1 - step : step; };
    // (clamped so that no stored value can lead the reads astray)
    auto clamped = [&](int s) { return __builtin_amdgcn_readfirstlane(min(max(s, 0), 2 * L)); };
    int segment = segments - 1;
    int state = clamped(backward ? 2 * L - to : from);               // at the last step of `segment`
    for (int mine = segments - 1 - wave; mine >= 0; mine -= waves) {
        for (; segment > mine; --segment) {
            const int at = segment * P + (state >> 1);
            const uint32_t word = in_lds ? s_origins[at] : origins[at];
            state = clamped(static_cast<int>(state & 1 ? word >> 16 : word & 0xFFFFu));
        }
        const int first = mine * kSegment, rows = min(kSegment, rows_all - first);       // (whole chunks)
        const int pair_hi = state >> 1, pair_lo = max(pair_hi - 63, 0);                   // both states of a pair share its word
        const int col = min(pair_lo + lane, pair_hi);
        uint32_t word[kSegmentChunks];
#pragma unroll
        for (int c = 0; c < kSegmentChunks; ++c) word[c] = choices[static_cast<int64_t>(min(first / kChunk + c, rows_all / kChunk - 1)) * P + col];
        int filed = 0, at = state;
#pragma unroll
        for (int c = kSegmentChunks - 1; c >= 0; --c) {
            if (c * kChunk >= rows) continue;
#pragma unroll
            for (int q = kChunk - 1; q >= 0; --q) {
                // lane r of `filed` = state at step first + r
                asm volatile("v_writelane_b32 %0, %1, %2" : "+v"(filed) : "s"(at), "n"(c * kChunk + q));
                const unsigned w = __builtin_amdgcn_readlane(word[c], (at >> 1) - pair_lo);
                // how far down the state of this step came from: the upper two bits (3 is 2 as well) if it is a label
                // state (odd), the lowest if it is a blank
                const int odd = at & 1, bits = static_cast<int>(w >> ((kChunk - 1 - q) * kChoiceBits + odd)) & (1 + 2 * odd);
                at = max(at - min(bits, 2), 0);
            }
        }
        if (lane < rows) {
            const int t = frame_of(first + lane);
            if (t < m.Tb) arow[t] = backward ? 2 * L - filed : filed;
        }
    }
}

// ---- gradient ------------------------------------------------------------------------------
//   gamma_t(s) = alpha_t(s) * beta_t(s) / p                 mass share of state s
//   grad[k]    = y_t(k) - sum_{s: symbol(s) = k} gamma_t(s)
// Only the label states' gamma are computed; the blank column gets
// 1 - (sum over label states), which is the blank states' share because the shares of all
// states of a frame add up to 1.  Every row of the gradient therefore sums to zero.
//
// A wavefront takes one block of kBlockFrames frames of one utterance and runs both recursions over it once more, from
// the checkpoints that the chains left at the block's ends (or from the start state): alpha forward, keeping the label
// states' high dwords in registers, then beta backward, forming a frame's shares as it passes.  A lane owns two
// neighbouring label positions for both directions, so a share needs nothing from another lane:
//   alpha: (blank j, label j) as in the forward chain;  beta: (label j, blank j + 1), the backward chain's pair.
// 128 positions make a piece; longer labels take several, each recomputing the 16 positions at its inner edges that
// its neighbour owns (an error at the edge moves up one position per frame).
// A row of one value per lane in LDS; two blocks of a row per frame.  (Not padded: 16 rows' 16-byte reads meet in the same banks, up to eight of
// them a piece (share_product), and the counters show twice the conflicts, but both words of a frame are one instruction's offsets apart: 32 address additions a
// piece less.  With four words of padding, so: 64 x 750 frames, 29 symbols 45.4 us a call, 45.5; 512 x 750 118.4, 118.6; 256 x 500, 60
// symbols 61.2, 60.9; 400 x 400, 90 symbols 114.2, 113.6: within half a per cent either way, and 512 bytes of LDS a wavefront less.)
constexpr int kShareRow = kPiecePositions / 2, kShareInts = 2 * kBlockFrames * kShareRow;
constexpr int kNormInts = kBlockFrames;
static_assert(kPieceStep % 32 == 0, "pieces start at multiples of 32 positions (share_product)");

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef __fp16 half2_raw __attribute__((ext_vector_type(2)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef unsigned uint2v __attribute__((ext_vector_type(2)));
typedef unsigned uint4v __attribute__((ext_vector_type(4)));

// alpha * beta / p of one state (without the mantissa of 1 / p) from alpha's high dword and beta, `exponents` the sum of
// all exponents.  Either value may lie a thousand binary orders below or above the unit of its own frame (lane_frame)
// while the product is a share of order one: alpha takes all the exponents first.  A state of any mass has beta above
// 2^-1000 in its frame, so that alpha is then below 2^1000; the cap is for those without.
__device__ __forceinline__ double scaled_alpha(unsigned alpha, int exponents)
{
    return __builtin_amdgcn_ldexp(__hiloint2double(static_cast<int>(alpha), 0), exponents);
}
__device__ __forceinline__ float state_share(unsigned alpha, double beta, int exponents)
{
    return static_cast<float>(fmin(scaled_alpha(alpha, exponents), 0x1p1000) * beta);
}
// (the same from two stored words)
__device__ __forceinline__ float word_share(unsigned a, unsigned b, int exponents)
{
    return state_share(a, __hiloint2double(static_cast<int>(b), 0), exponents);
}
typedef float float2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ half2_raw nearest_halves(float x, float y)
{
    return __builtin_convertvector((float2v{x, y}), half2_raw);
}
// x - (one half of a pair of fp16), in one instruction.
__device__ __forceinline__ float minus_low_half(float x, half2_raw h)
{
    float r;
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]" : "=v"(r) : "v"(h), "v"(x));
    return r;
}
__device__ __forceinline__ float minus_high_half(float x, half2_raw h)
{
    float r;
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(h), "v"(x));
    return r;
}

// Two state pairs of a lane with a common frame (see run_chain_linear2).  Backward: the lane above takes the part of the
// lane below.
struct LanePairs {
    double blank0, label0, blank1, label1;
    int frame;
    double scale;                                        // 2^(neighbour's frame - frame)
};
// steep: the next renewal comes after kSteepSteps frames, otherwise after a chunk.  Returns by how many binary orders the lane's first blank, position p0's
// going forward, p1's going backward, lies above the lane's largest value (negative: below).  Under -kHeldGap the new frame, which that value is 2^-kFrameSlack of
// at least, does not hold it.  (Of the lane's largest exponent, which says that there is no mass, and not of the frame, since there frames without mass go anywhere.)
constexpr int kHeldGap = 600;
static_assert(-kFrameSlack - kHeldGap >= -1022, "normal numbers");
template <bool kBackward>
__device__ __forceinline__ int renew_pairs(LanePairs& s, int frame0, int frame1, bool steep)
{
    const double top0 = fmax(s.blank0, s.label0), top1 = fmax(s.blank1, s.label1);
    const int mine = max(top0 > 0.0 ? frame0 + __builtin_amdgcn_frexp_exp(top0) : kNoExponent,
                         top1 > 0.0 ? frame1 + __builtin_amdgcn_frexp_exp(top1) : kNoExponent);
    int window = mine;
    auto lanes = [&](int from, int to) __attribute__((always_inline)) {
#pragma unroll
        for (int k = from; k < to; ++k) window = kBackward ? window_max_step_down(window, mine) : window_max_step(window, mine);
    };
    lanes(0, kSteepSteps / 2);
    if (__builtin_expect(!steep, 1)) lanes(kSteepSteps / 2, kChunk / 2);
    window = lane_frame(window, mine);
    const int held = __builtin_amdgcn_frexp_exp(kBackward ? s.blank1 : s.blank0) + (kBackward ? frame1 : frame0) - mine;
    s.blank0 = __builtin_amdgcn_ldexp(s.blank0, frame0 - window);
    s.label0 = __builtin_amdgcn_ldexp(s.label0, frame0 - window);
    s.blank1 = __builtin_amdgcn_ldexp(s.blank1, frame1 - window);
    s.label1 = __builtin_amdgcn_ldexp(s.label1, frame1 - window);
    s.frame = window;
    const int neighbour = __builtin_amdgcn_update_dpp(kNoExponent, window, kBackward ? 0x130 : 0x138, 0xf, 0xf, false);
    s.scale = __builtin_amdgcn_ldexp(1.0, min(max(neighbour - window, -1100), 1023));
    return held;
}

// The thread's index, for parts of a tile's code that a loop goes through again (places that have been left): not known to be
// the same each time, so that nothing made from it is held in registers from one time to the next.  Without it in these two
// parts the kernel of 33 to 64 symbols is two registers short, which go to memory.
__device__ __forceinline__ int tile_thread()
{
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// What a lane knows of its two label positions: the symbols, and where a label may be entered from the one before.
struct LaneLabels {
    int p0, p1;
    bool has0, has1, skip0, skip1, skip2;                // skip2: from position p1 to the next lane's first
    int symbol0, symbol1;
    __device__ __forceinline__ LaneLabels(const int* __restrict__ lab, int L, int base)
    {
        p0 = base + 2 * static_cast<int>(threadIdx.x & 63);
        p1 = p0 + 1;
        has0 = p0 < L;
        has1 = p1 < L;
        // (positions off either end read the nearest one: no branches, so that all loads travel together)
        auto at = [&](int p) { return lab[min(max(p, 0), L - 1)]; };
        const int before = at(p0 - 1), after = at(p1 + 1);
        symbol0 = at(p0);
        symbol1 = at(p1);
        skip0 = p0 >= 1 && has0 && symbol0 != before;
        skip1 = has1 && symbol1 != symbol0;
        skip2 = p1 + 1 < L && after != symbol1;
    }
};

// The checkpoints at both ends of a block for a lane's two positions (position p in column 1 + p; lanes without a
// position read the last one's).  At an utterance's ends there is none: zeros, with frame 0.
struct BlockEnds {
    CheckpointState a0{}, a1{}, b0{}, b1{};
    int fa0 = 0, fa1 = 0, fb0 = 0, fb1 = 0;
    // kPublished: in the launch of the chains, which have just published them
    template <bool kPublished>
    static __device__ __forceinline__ BlockEnds load(const Utt& m, const LatticeOut& lat, int p0, int block)
    {
        BlockEnds e;
        const CheckpointRow row{lattice_pitch(m.L)};
        const int blocks = frame_blocks(m.Tb), column = 1 + min(p0, max(m.L, 1) - 1);
        const int slot0 = row.slot(column) * static_cast<int>(sizeof(CheckpointState)), slot1 = row.slot(column + 1) * static_cast<int>(sizeof(CheckpointState));
        const int frame_at = static_cast<int>(row.frames_at()) + column * static_cast<int>(sizeof(int));
        constexpr int kPolicy = kPublished ? kPast : 0;
        auto load_row = [&](const uint32_t* states, int r, CheckpointState& s0, CheckpointState& s1, int& f0, int& f1) __attribute__((always_inline)) {
            const auto block_row = __builtin_amdgcn_make_buffer_rsrc(const_cast<CheckpointState*>(row.states(states + m.ab_off, r)), 0, static_cast<int>(row.bytes()), 0x00020000);
            s0 = __builtin_bit_cast(CheckpointState, __builtin_amdgcn_raw_buffer_load_b128(block_row, slot0, 0, kPolicy));
            s1 = __builtin_bit_cast(CheckpointState, __builtin_amdgcn_raw_buffer_load_b128(block_row, slot1, 0, kPolicy));
            const auto f = __builtin_amdgcn_raw_buffer_load_b64(block_row, frame_at, 0, kPolicy);
            f0 = static_cast<int>(f[0]);
            f1 = static_cast<int>(f[1]);
        };
        if (block > 0) load_row(lat.alpha, block - 1, e.a0, e.a1, e.fa0, e.fa1);
        if (block + 1 < blocks) load_row(lat.beta, blocks - 2 - block, e.b0, e.b1, e.fb0, e.fb1);
        return e;
    }
};

// The shares of the label positions base .. base + 127 in block `block` of the utterance: file(row, share0, share1) for
// the lane's two positions, row = 0 .. 15 in some order, 0 outside [own_first, own_end).  Shares are without the
// mantissa of 1 / p and times 2^kScaleLog2.  emissions(i, el0, el1): the lane's label emissions in the block's chunk 0, 1 and 0
// again, for i = 0, 1 and 2 in turn.
// alpha's high dwords wait in LDS, s_alpha0 and s_alpha1 [row][kShareRow], each lane's in a slot of its own that is free
// again when file is called for the row.  (In registers they cost 32 of them, and the loops over the chunks had to be
// unrolled: code that runs once per wavefront comes out of memory no faster than data.)
// steep: the chains were steep ones, and so frames are renewed every kSteepSteps here too.  (A branch: as a variant of its own the code
// took 20 to 59 registers more; the branch 2 to 5, and no time that can be measured.)
// Returns false where a lane's frame does not hold its states, or a chain has left logarithms: block_shares_of_logs does such a block.  (Asked once, at the end, with
// the least of what the renewals have found: what such a block files before is filed again.  With a way out behind every renewal a piece's loops had 990
// instructions in place of 880 and 840 without the question: 4 x 50 frames, 29 symbols 13.9 us a call in place of 13.7, 512 x 750 117.5 and 116.0.)
template <int kScaleLog2, typename Emissions, typename File>
__device__ __forceinline__ bool block_shares(const Utt& m, const LaneLabels& at, const BlockEnds& ends,
                                             const double packed_inverse_p, const bool steep, const int block,
                                             const int own_first, const int own_end, unsigned* s_alpha0, unsigned* s_alpha1,
                                             Emissions&& emissions, File&& file)
{
    const int lane = threadIdx.x & 63;
    const int L = m.L, blocks = frame_blocks(m.Tb);
    const int p0 = at.p0, p1 = at.p1;
    const bool has0 = at.has0, has1 = at.has1;
    const double skip1_one = at.skip1 ? 1.0 : 0.0;       // (skip0 and skip2 stay masks: registers)
    float el0[kChunk], el1[kChunk];
    // The order of the statements is the order of issue (run_chain_linear2): left to itself the compiler put results and
    // their uses next to each other, and a block's recomputation took 3.0 us in place of 2.0.
    auto pin = []() { __builtin_amdgcn_sched_barrier(0); };

    int held;
    // alpha
    int alpha_frame0 = 0, alpha_frame1 = 0;              // of the block's two chunks
    int alpha_middle0 = 0, alpha_middle1 = 0;            // ... from their middle on
    {
        LanePairs s;
        s.blank0 = block > 0 ? (has0 ? ends.a0.blank : 0.0) : (p0 == 0 ? 1.0 : 0.0);
        s.label0 = block > 0 && has0 ? ends.a0.label : 0.0;
        s.blank1 = block > 0 && has1 ? ends.a1.blank : 0.0;
        s.label1 = block > 0 && has1 ? ends.a1.label : 0.0;
        held = renew_pairs<false>(s, ends.fa0, ends.fa1, steep);
        alpha_frame0 = alpha_middle0 = s.frame;
        emissions(0, el0, el1);
#pragma unroll 1
        for (int h = 0; h < 2; ++h) {
            if (h) {
                held = min(held, renew_pairs<false>(s, s.frame, s.frame, steep));
                alpha_frame1 = alpha_middle1 = s.frame;
                emissions(1, el0, el1);
            }
            double skip0_scale = at.skip0 ? s.scale : 0.0;
#pragma unroll
            for (int q = 0; q < kChunk; ++q) {
#pragma clang fp contract(off)
                if (q == kSteepSteps && __builtin_expect(steep, 0)) {
                    held = min(held, renew_pairs<false>(s, s.frame, s.frame, steep));
                    (h ? alpha_middle1 : alpha_middle0) = s.frame;
                    skip0_scale = at.skip0 ? s.scale : 0.0;
                }
                const double prev = lane_shift<false>(s.label1);
                pin();
                const double u1 = s.blank1 + s.label1;
                pin();
                const double u0 = s.blank0 + s.label0;
                pin();
                const double n_blank1 = s.blank1 + s.label0;
                pin();
                const double el0_d = static_cast<double>(el0[q]);
                pin();
                const double n_label1 = __builtin_fma(s.label0, skip1_one, u1);
                pin();
                const double n_label0 = __builtin_fma(prev, skip0_scale, u0);
                pin();
                const double n_blank0 = __builtin_fma(prev, s.scale, s.blank0);
                pin();
                const double el1_d = static_cast<double>(el1[q]);
                pin();
                s.label0 = n_label0 * el0_d;
                pin();
                s.label1 = n_label1 * el1_d;
                pin();
                s.blank0 = n_blank0;
                s.blank1 = n_blank1;
                s_alpha0[(h * kChunk + q) * kShareRow + lane] = static_cast<unsigned>(__double2hiint(s.label0));
                s_alpha1[(h * kChunk + q) * kShareRow + lane] = static_cast<unsigned>(__double2hiint(s.label1));
            }
        }
    }
    // beta, and the shares
    LanePairs s;
    const bool last = block + 1 == blocks;
    s.blank0 = last ? (p0 == L - 1 ? 1.0 : 0.0) : (has0 ? ends.b0.blank : 0.0);
    s.label0 = !last && has0 ? ends.b0.label : 0.0;
    // (without a position p1 the blank of p0 once more, for renew_pairs: nothing comes of it)
    s.blank1 = last && has1 ? (p1 == L - 1 ? 1.0 : 0.0) : (has1 ? ends.b1.blank : s.blank0);
    s.label1 = !last && has1 ? ends.b1.label : 0.0;
    const bool own0 = p0 >= own_first && p0 < own_end, own1 = p1 >= own_first && p1 < own_end;
    const int to_share = __double2loint(packed_inverse_p) + kScaleLog2;
    // A step's shares are formed during the step after it (before the first: of zeros, in a row that is filed again).
    double pending_alpha0 = 0.0, pending_alpha1 = 0.0, pending_beta0 = 0.0, pending_beta1 = 0.0;
    int pending_row = kBlockFrames - 1;
    held = min(held, renew_pairs<true>(s, ends.fb0, has1 ? ends.fb1 : ends.fb0, steep));
#pragma unroll 1
    for (int h = 1; h >= 0; --h) {
        if (h == 0) held = min(held, renew_pairs<true>(s, s.frame, s.frame, steep));
        int x0, x1;
        auto set_exponents = [&](int alpha_frame) __attribute__((always_inline)) {
            const int exponents = alpha_frame + s.frame + to_share;
            x0 = own0 ? exponents : kNoExponent;
            x1 = own1 ? exponents : kNoExponent;
        };
        set_exponents(h == 0 ? alpha_middle0 : alpha_middle1);
        double skip2_scale = at.skip2 ? s.scale : 0.0;
        if (h == 0) emissions(2, el0, el1);              // (chunk 1's are still there)
        unsigned alpha0[kChunk], alpha1[kChunk];
#pragma unroll
        for (int q = 0; q < kChunk; ++q) {
            alpha0[q] = s_alpha0[(h * kChunk + q) * kShareRow + lane];
            alpha1[q] = s_alpha1[(h * kChunk + q) * kShareRow + lane];
        }
#pragma unroll
        for (int q = kChunk - 1; q >= 0; --q) {
#pragma clang fp contract(off)
            if (q == kSteepSteps - 1 && __builtin_expect(steep, 0)) {
                held = min(held, renew_pairs<true>(s, s.frame, s.frame, steep));
                set_exponents(h == 0 ? alpha_frame0 : alpha_frame1);
                skip2_scale = at.skip2 ? s.scale : 0.0;
            }
            const double next = lane_shift<true>(s.label0);
            pin();
            const double share0 = pending_alpha0 * pending_beta0;
            pin();
            const double u0 = s.blank0 + s.label0;
            pin();
            const double share1 = pending_alpha1 * pending_beta1;
            pin();
            const double u1 = s.blank1 + s.label1;
            pin();
            const float f0 = static_cast<float>(share0);
            pin();
            const double n_blank0 = s.blank0 + s.label1;
            pin();
            const float f1 = static_cast<float>(share1);
            pin();
            const double n_label0 = __builtin_fma(s.label1, skip1_one, u0);
            pin();
            const double n_label1 = __builtin_fma(next, skip2_scale, u1);
            pin();
            const double el0_d = static_cast<double>(el0[q]);
            pin();
            file(pending_row, f0, f1);
            pin();
            const double n_blank1 = __builtin_fma(next, s.scale, s.blank1);
            pin();
            const double a0 = scaled_alpha(alpha0[q], x0);
            pin();
            const double el1_d = static_cast<double>(el1[q]);
            pin();
            const double a1 = scaled_alpha(alpha1[q], x1);
            pin();
            s.label0 = n_label0 * el0_d;
            pin();
            pending_alpha0 = fmin(a0, 0x1p1000);
            pin();
            s.label1 = n_label1 * el1_d;
            pin();
            pending_alpha1 = fmin(a1, 0x1p1000);
            pin();
            s.blank0 = n_blank0;
            s.blank1 = n_blank1;
            pending_beta0 = n_label0;
            pending_beta1 = n_label1;
            pending_row = h * kChunk + q;
        }
    }
    file(pending_row, static_cast<float>(pending_alpha0 * pending_beta0), static_cast<float>(pending_alpha1 * pending_beta1));
    return __ballot(held < -kHeldGap) == 0;
}
// The same in logarithms, from checkpoints of either kind.  Rare, and written to need few registers beside those of the tile: two frames at a time from
// the last ones on, alpha from the block's start each time.  (Utterances of the linear domain: a blank's emission is its norm, and its logarithm 0.)
template <int kScaleLog2, bool kPublished, typename File>
__device__ __forceinline__ void block_shares_of_logs(const Utt* __restrict__ meta, const int* __restrict__ labels, const float* __restrict__ emit_label,
                                                     const LatticeOut& lat, const double* __restrict__ mass, const int b, int block, int base,
                                                     const int own_first, const int own_end, File&& file)
{
    const Utt m = uniform_record(meta[b]);
    const int* const lab = labels + m.lab_off;
    const double packed_inverse_p = published(&mass[b * kMassWords + kMassInverse]);
    // (everything is read again: nothing is kept for it through block_shares, no constant either)
    int low, high;
    asm volatile("" : "+s"(block));
    asm volatile("" : "+s"(base));
    asm volatile("v_mov_b32 %0, 0\n\tv_mov_b32 %1, 0xc6300000" : "=v"(low), "=v"(high));
    const double log0 = __hiloint2double(high, low);     // -2^100, as good as kNeg
    const int L = m.L, p0 = base + 2 * static_cast<int>(tile_thread() & 63), p1 = p0 + 1;
    int symbol0, symbol1, flags;                         // (in one register, not as masks in scalar ones)
    constexpr int kHas0 = 1, kHas1 = 2, kSkip0 = 4, kSkip1 = 8, kSkip2 = 16, kOwn0 = 32, kOwn1 = 64;
    {
        const LaneLabels at(lab, L, base);
        symbol0 = at.symbol0;
        symbol1 = at.symbol1;
        flags = (at.has0 ? kHas0 : 0) | (at.has1 ? kHas1 : 0) | (at.skip0 ? kSkip0 : 0) | (at.skip1 ? kSkip1 : 0) | (at.skip2 ? kSkip2 : 0) |
                (p0 >= own_first && p0 < own_end ? kOwn0 : 0) | (p1 >= own_first && p1 < own_end ? kOwn1 : 0);
    }
    auto is = [&](int which) {
        asm volatile("" : "+v"(flags));
        return (flags & which) != 0;
    };
    constexpr int kFrames = 2, kGroups = kBlockFrames / kFrames, kChunkGroups = kChunk / kFrames;
    auto emissions = [&](int has, int symbol, int p, int group) {
        return *reinterpret_cast<const float2*>(emit_label + label_emission_offset(m, is(has), symbol, p, 2 * block + group / kChunkGroups, kLogZeroEmission) +
                                                group % kChunkGroups * kFrames);
    };
    // the neighbour's label, log 0 at the end
    auto from_below = [&](double v) {
        int lo = __double2loint(log0), hi = __double2hiint(log0);
        return shift_up(v, lo, hi);
    };
    auto from_above = [&](double v) {
        const double w = lane_shift<true>(v);
        return (tile_thread() & 63) == 63 ? log0 : w;
    };
    struct Logs { double b0, l0, b1, l1; };
    auto ends_of = [&](bool backward) {
        const BlockEnds ends = BlockEnds::load<kPublished>(m, lat, p0, block);
        const bool none = backward ? block + 1 == frame_blocks(m.Tb) : block == 0;
        const int first = backward ? L - 1 : 0;          // position that has the blank a recursion starts from
        const CheckpointState s0 = backward ? ends.b0 : ends.a0, s1 = backward ? ends.b1 : ends.a1;
        const int f0 = backward ? ends.fb0 : ends.fa0, f1 = backward ? ends.fb1 : ends.fa1;
        const CheckpointState w0 = state_logs(s0, f0, log0), w1 = state_logs(s1, f1, log0);
        return Logs{none ? (p0 == first ? 0.0 : log0) : (is(kHas0) ? w0.blank : log0), !none && is(kHas0) ? w0.label : log0,
                    none ? (p1 == first ? 0.0 : log0) : (is(kHas1) ? w1.blank : log0), !none && is(kHas1) ? w1.label : log0};
    };
    Logs beta = ends_of(true);
    const double to_share = static_cast<double>(__double2loint(packed_inverse_p) + kScaleLog2);
    auto share = [&](int own, double alpha_label, double beta_label) {
        return is(own) ? fast_exp2(static_cast<float>(fmax(alpha_label + beta_label + to_share, -1.0e4))) : 0.0f;
    };
#pragma unroll 1
    for (int group = kGroups - 1; group >= 0; --group) {
        double alpha0[kFrames], alpha1[kFrames];
        Logs alpha = ends_of(false);
#pragma unroll 1
        for (int g = 0; g <= group; ++g) {
            const float2 x0 = emissions(kHas0, symbol0, p0, g), x1 = emissions(kHas1, symbol1, p1, g);
#pragma unroll
            for (int q = 0; q < kFrames; ++q) {          // (unrolled: registers for alpha0 and alpha1)
                const double prev = from_below(alpha.l1);
                const double nb1 = lse2(alpha.b1, alpha.l0), nl1 = lse2(alpha.l1, is(kSkip1) ? nb1 : alpha.b1);
                const double nb0 = lse2(alpha.b0, prev), nl0 = lse2(alpha.l0, is(kSkip0) ? nb0 : alpha.b0);
                alpha = Logs{nb0, nl0 + emission_log2(q ? x0.y : x0.x), nb1, nl1 + emission_log2(q ? x1.y : x1.x)};
                alpha0[q] = alpha.l0;
                alpha1[q] = alpha.l1;
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        const float2 x0 = emissions(kHas0, symbol0, p0, group), x1 = emissions(kHas1, symbol1, p1, group);
#pragma unroll
        for (int q = kFrames - 1; q >= 0; --q) {
            const double next = from_above(beta.l0);
            const double nb0 = lse2(beta.b0, beta.l1), nl0 = lse2(beta.l0, is(kSkip1) ? nb0 : beta.b0);
            const double nb1 = lse2(beta.b1, next), nl1 = lse2(beta.l1, is(kSkip2) ? nb1 : beta.b1);
            file(group * kFrames + q, share(kOwn0, alpha0[q], nl0), share(kOwn1, alpha1[q], nl1));
            beta = Logs{nb0, nl0 + emission_log2(q ? x0.y : x0.x), nb1, nl1 + emission_log2(q ? x1.y : x1.x)};
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}
// The same from the words that log-domain chains have stored for every frame, kFrames of them at a time: two, or one
// where a second frame's registers would cost the linear domain (512 utterances 0.4 %).  512 utterances in the log domain:
// 427 us a call with four-byte loads, 379 with both positions' words in one.
template <int kScaleLog2, int kFrames, typename File>
__device__ __forceinline__ void block_shares_log(const Utt& m, const LatticeOut& lat, const double packed_inverse_p, const int block,
                                                 const int base, const int own_first, const int own_end, File&& file)
{
    const int p0 = base + 2 * static_cast<int>(threadIdx.x & 63), p1 = p0 + 1;
    const bool own0 = p0 >= own_first && p0 < own_end, own1 = p1 >= own_first && p1 < own_end;
    const int to_share = __double2loint(packed_inverse_p) + kScaleLog2;
    // Several frames' words on their way at once, both positions' in one load (a row has a column to spare after the last
    // position's; lanes without a position read the end of the row).
    typedef uint32_t Pair __attribute__((ext_vector_type(2), aligned(4)));
    const int pitch = static_cast<int>(lattice_pitch(m.L)), column = 1 + min(p0, m.L - 1);
    int64_t row = m.ab_off + static_cast<int64_t>(block) * kBlockFrames * pitch;
#pragma unroll 1
    for (int r0 = 0; r0 < kBlockFrames; r0 += kFrames, row += kFrames * pitch) {
        Pair alpha[kFrames], beta[kFrames], exponents[kFrames];
        auto pair = [&](const void* words, int r) { return *reinterpret_cast<const Pair*>(static_cast<const uint32_t*>(words) + row + r * pitch + column); };
#pragma unroll
        for (int r = 0; r < kFrames; ++r) {
            alpha[r] = pair(lat.alpha, r);
            beta[r] = pair(lat.beta, r);
            exponents[r] = pair(lat.alpha_exponents, r) + pair(lat.beta_exponents, r);
        }
#pragma unroll
        for (int r = 0; r < kFrames; ++r)
            file(r0 + r, own0 ? word_share(alpha[r][0], beta[r][0], static_cast<int>(exponents[r][0]) + to_share) : 0.0f,
                 own1 ? word_share(alpha[r][1], beta[r][1], static_cast<int>(exponents[r][1]) + to_share) : 0.0f);
    }
}
// What wavefront `first` of `step` takes of a label's pieces: for_piece(base, own_first, own_end).
template <typename F>
__device__ __forceinline__ void for_pieces(int L, int first, int step, F&& for_piece)
{
    const int pieces = label_pieces(L);
    for (int i = first; i < pieces; i += step) {
        const int base = i * kPieceStep;
        for_piece(base, i == 0 ? 0 : base + kPieceHalo, i == pieces - 1 ? L : base + kPieceStep + kPieceHalo);
    }
}
// Wavefronts that share a block in the narrow gradient kernel, one piece each up to four -- in launches of few blocks,
// which last as long as one block takes (English minibatch: 18.8 -> 16.7 us; 512 utterances: 69 -> 83 us).
constexpr int kShareBlocksMost = 8192;    // blocks times pieces: two rounds of what the chip holds
// In a lattice launch that has more, those of the utterances that end last (about; blocks_to_share).
inline int shared_utterances(const Launch& p, int blocks)
{
    return std::min(p.B, p.share_last / (blocks * std::max(1, label_pieces(p.max_label))));
}
__host__ __device__ constexpr int block_waves(int L) { return label_pieces(L) <= 1 ? 1 : (label_pieces(L) == 2 ? 2 : 4); }
// The domain of an utterance as its chains published it (a word per direction).
template <bool kPublished>
__device__ __forceinline__ int domain_of(const int* domain, int b)
{
    const int d = kPublished ? published(&domain[2 * b]) | published(&domain[2 * b + 1]) : domain[2 * b] | domain[2 * b + 1];
    return __builtin_amdgcn_readfirstlane(d);
}

// Alphabets of at most 64 symbols (the English one has 29): a wavefront per block, or two or four that share the label's
// pieces (block_waves).
// The occupancy of a symbol is the sum of the shares of the label positions that carry it: a product of
// the frames' shares [frame][position] with the label's zero-one matrix [position][symbol], and so work for
// the matrix cores:
//   - the shares go to LDS as [frame][position], in two halves whose products share one accumulator (fp32 sums in a fixed
//     order): the nearest fp16, and the nearest fp16 to what that leaves, at most an ulp of the fp32 share away from it.  They
//     are carried times 2^15, the most that a share of 1 allows, so that the second half of a share of 2^-27 is above fp16's
//     subnormals; the matrix holds 2 for one.  Measured against the double-precision oracle over alphabets of 22 to 63 symbols,
//     2-norm of the gradient's error: within 1 % of what three bf16 parts (the whole fp32 share) give, which cost the 512
//     utterances' gradient 1.6 % of the call; with both halves rounded toward zero it was 7 to 11 % more;
//   - A operand, per 32 positions: lane l holds frame l % 16, positions 8 (l / 16) .. + 7, one 16-byte
//     read out of LDS;
//   - B operand: lane l holds the same positions for symbol l % 16 (+ 16 per tile of symbols), made from the
//     label's bytes in LDS; the blank's column is 1 everywhere, so that it receives the sum of all shares, and
//     the blank's occupancy is what is left of 1.
constexpr int kShareScaleLog2 = 15;
// Bytes of a label staged in LDS: whole pieces of 32 positions, kNoSymbol past the label's end.
constexpr int kNoSymbol = 0x40;
__host__ __device__ constexpr int tile_label_ints(int L) { return (L + 31) / 32 * 8; }
// The block's emissions in LDS: [chunk][symbol][frame], a chunk of a symbol in a row of 12 floats (eight and padding:
// lanes that read different symbols meet in few banks), one more row of zeros for lanes without a position.
constexpr int kEmissionRow = 12;
__host__ __device__ constexpr int tile_emission_ints(int tiles) { return (2 * 16 * tiles + 1) * kEmissionRow; }
// LDS of one wavefront.  staged: with the block's emissions.
__host__ __device__ constexpr int tile_lds_ints(int Lmax, int tiles, bool staged)
{
    return kNormInts + kShareInts + (staged ? tile_emission_ints(tiles) : 0) + tile_label_ints(Lmax);
}
__device__ __forceinline__ void stage_label_bytes(unsigned* s_label, const int* __restrict__ labels, int L)
{
    for (int w = threadIdx.x & 63; w < tile_label_ints(L); w += 64) {
        unsigned c[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) c[i] = labels[min(4 * w + i, L - 1)];      // (no branch: the four travel together)
        unsigned word = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) word |= (4 * w + i < L ? c[i] : static_cast<unsigned>(kNoSymbol)) << (8 * i);
        s_label[w] = word;
    }
}

template <int kTiles>
__device__ __forceinline__ void share_product(float4v (&acc)[kTiles], const unsigned* s_hi, const unsigned* s_lo,
                                              const unsigned* s_label, int base, int L, int blank)
{
    const int lane = tile_thread() & 63, c = lane & 15, g = lane >> 4;
    // the symbol of this lane's column, per tile of symbols: label bytes are compared as (byte & mask) ^ symbol == 0
    unsigned symbol[kTiles], mask[kTiles];
#pragma unroll
    for (int n = 0; n < kTiles; ++n) {
        const int k = 16 * n + c;
        symbol[n] = k == blank ? 0u : static_cast<unsigned>(k) * 0x01010101u;
        mask[n] = k == blank ? static_cast<unsigned>(kNoSymbol) * 0x01010101u : 0x7F7F7F7Fu;
    }
    for (int k0 = base; k0 < min(L, base + kPiecePositions); k0 += 32) {
        const int at = c * kShareRow + (k0 - base) / 2 + 4 * g;
        const half8 hi = __builtin_bit_cast(half8, *reinterpret_cast<const uint4v*>(s_hi + at));
        const half8 lo = __builtin_bit_cast(half8, *reinterpret_cast<const uint4v*>(s_lo + at));
        const uint2v word = *reinterpret_cast<const uint2v*>(s_label + k0 / 4 + 2 * g);
#pragma unroll
        for (int n = 0; n < kTiles; ++n) {
            uint4v one;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const unsigned differs = ((word[h] & mask[n]) ^ symbol[n]) + 0x7F7F7F7Fu;      // bit 7 of a byte: not this symbol
                const unsigned match = (~differs & 0x80808080u) >> 1;                          // 0x40 where it is: the top byte of fp16 2.0
                one[2 * h] = __builtin_amdgcn_perm(match, 0u, 0x05000400u);                    // bytes 0 and 1 to the halves' top bytes
                one[2 * h + 1] = __builtin_amdgcn_perm(match, 0u, 0x07000600u);
            }
            acc[n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(hi, __builtin_bit_cast(half8, one), acc[n], 0, 0, 0);
            acc[n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(lo, __builtin_bit_cast(half8, one), acc[n], 0, 0, 0);
        }
    }
}

// What the gradient's workgroups get, in a launch of their own or in the lattice launch.
struct TileArgs {
    void* grads;
    bool bf16;
    const double* mass;
    const int* chain_err;
    float* costs;
    const int* domain;
    const int* links;             // wide
    int* done;                    // lattice launch: what to wait for
    int* left;                    // ... and, per workgroup, who has left before it (chains_taken)
    int end_polls;                // ... and how often to look before giving up
    const int* by_end;            // ... the utterances, those first whose chains end first (nullptr, a launch of its own: as they come)
    int T, B, A, blank, Lmax;
    // narrow: by_end's utterances in segments, those of one with as many workgroups each as its longest needs.  (With as many as the tensor's frames need, two in five had nothing
    // but zero rows to write, a microsecond or two in the place of another, and workgroups go out one after the other: 75 in a microsecond.  us a call: 512 x 60 x 29 29.7,
    // so 27.2; 512 x 750 x 29 115.6 and 115.1; 400 x 1500 x 29 300.0 and 298.5.)
    static constexpr int kSegments = 8;
    unsigned segment_tile[kSegments + 1];      // its first workgroup; the last entry: how many there are
    int segment_rank[kSegments], segment_groups[kSegments];
    int shared_from;              // from this utterance on, a segment's first one, several wavefronts share a block
    int waves, alpha_at;          // wide
    int groups;                   // wide: workgroups per utterance
    int first_group;              // lattice launch: the first one with a tile
};
// Which utterance (of by_end's) a workgroup works for, and which of its workgroups it is.
struct TilePlace {
    int rank, within, groups;
    bool shares;
    static __device__ __forceinline__ TilePlace of(const TileArgs& g, unsigned tile)
    {
        unsigned first = 0;
        int first_rank = 0, groups = g.segment_groups[0];
#pragma unroll
        for (int i = 1; i < TileArgs::kSegments; ++i) {
            const bool here = tile >= g.segment_tile[i];
            first = here ? g.segment_tile[i] : first;
            first_rank = here ? g.segment_rank[i] : first_rank;
            groups = here ? g.segment_groups[i] : groups;
        }
        const unsigned i = tile - first, utterance = i / static_cast<unsigned>(groups);
        const int rank = first_rank + static_cast<int>(utterance);
        return {rank, static_cast<int>(i - utterance * groups), groups, rank >= g.shared_from};
    }
};
__device__ __forceinline__ void store_gradient(const TileArgs& g, size_t i, float v)
{
    if (g.bf16) store_elem(static_cast<bf16_t*>(g.grads), i, v);
    else store_elem(static_cast<float*>(g.grads), i, v);
}
// By a wavefront: waits until utterance b's chains have ended.  The wait is bounded (TileArgs::end_polls and four polls a frame, a
// frame taking less than one): should it run out, the answer is kNotEnded, there is nothing to compute from, and the utterance's
// cost is to be NaN: whoever gives up says so in the utterance's word, where whoever does not finds it (kSomebodyGaveUp), since
// nobody gives up once the chains have ended.
constexpr int kNotEnded = 0, kEnded = 1, kSomebodyGaveUp = 2;
__device__ __forceinline__ int chains_awaited(const TileArgs& g, int b, int frames)
{
    int* const done = &g.done[b * kDoneStride];
    auto look = [&]() { return __builtin_amdgcn_readfirstlane(published(done)); };
    int64_t polls = g.end_polls > 0 ? g.end_polls + 4 * static_cast<int64_t>(frames) : 0;
    int word = look();
    for (; !chains_ended(word) && polls > 0; --polls) {
        __builtin_amdgcn_s_sleep(10);
        word = look();
    }
    if (!chains_ended(word)) {
        if ((tile_thread() & 63) == 0) word = __hip_atomic_fetch_or(done, kWaitGivenUp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        word = __builtin_amdgcn_readfirstlane(word);
    }
    return !chains_ended(word) ? kNotEnded : ((word & kWaitGivenUp) != 0 ? kSomebodyGaveUp : kEnded);
}
// The same by the whole workgroup; the same answer in every thread.
__device__ __forceinline__ bool wait_for_chains(const TileArgs& g, int b, int frames)
{
    __shared__ int s_ended;
    if (tile_thread() < 64) {
        const int ended = chains_awaited(g, b, frames);
        if (tile_thread() == 0) s_ended = ended;
    }
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(s_ended) != kNotEnded;
}
// The cost of utterance b, by a wavefront.
template <bool kWait>
__device__ __forceinline__ void utterance_cost(const TileArgs& g, const Utt* __restrict__ meta, const float* __restrict__ emit_blank, int b)
{
    const Utt m = uniform_record(meta[b]);
    if (!(m.flags & kUttRuns)) return;                   // (written by the setup role)
    const double log2_norms = norms_of_wave(norms_of_lane(m, emit_blank)).log2();
    const int ended = kWait ? chains_awaited(g, b, m.Tb) : kEnded;
    const double* const mass = &g.mass[b * kMassWords];
    const float cost = cost_of_mass(published(&mass[kMassValue]), published(&mass[kMassLog2]), log2_norms);
    if ((tile_thread() & 63) == 0) g.costs[b] = ended != kEnded || published(&g.chain_err[b]) != 0 ? __uint_as_float(0x7FC00000u) : cost;
}

// The arguments of the launches with tiles (args_again): of the chains' launch, and of launches of their own.
struct FusedArgs {
    ChainArgs<true> chains;
    TileArgs tiles;
};
struct GradientArgs {
    TileArgs tiles;
    const Utt* meta;
    const int* labels;
    const float* emit_blank;
    const float* emit_label;
    LatticeOut lat;
};

// Workgroup `group` of utterance b: kRowThreads / 64 wavefronts, ceil((blocks of T + 1) / (4 / wavefronts per block)) workgroups: the first
// wavefront behind the utterance's blocks writes its cost.  (With a workgroup of its own for that, 512 x 40 to 130 frames took 43.3 us a
// call in place of 37.2: places for workgroups are what such launches wait for.)
// LDS 4 tile_lds_ints(Lmax, kTiles, kStaged) ints.  kTiles: tiles of 16 symbols.
// kStaged: the block's emissions wait in LDS, where they are at once when the chains have ended.  Otherwise a lane takes its own from the
// die's cache when it needs them: without them (3 and 6 KB a wavefront, 32 and 64 symbols) four workgroups fit a compute unit in place of
// three and two, as many as 128 registers allow.  (What the launch lasts then: 512 x 300 frames, 50 symbols, 67.1 us a call staged, 61.4 not;
// 300 x 400, 40 symbols bf16, 62.2 and 58.4; 512 x 750, 29 symbols, no difference: it is bound by issue.)
// kLean: the lane's number is made anew where the rows are written (tile_thread), so that 128 registers suffice.
template <int kTiles, bool kWait, bool kStaged, bool kLean = false>
__device__ __forceinline__ void narrow_tile(const TileArgs& g_args, const Utt* __restrict__ meta, const int* __restrict__ labels,
                                            const float* __restrict__ emit_blank, const float* __restrict__ emit_label,
                                            const LatticeOut& lat, uint4v* tile_lds, const int b, const int group, const int groups, const bool shares)
{
    const int Tt = g_args.T, B = g_args.B, A = g_args.A, blank = g_args.blank, Lmax = g_args.Lmax;
    const int lane = kLean ? tile_thread() & 63 : threadIdx.x & 63, c = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const Utt m = uniform_record(meta[b]);
    const int L = m.L, sharing = shares ? block_waves(L) : 1, part = wave & (sharing - 1);
    const int first_block = group * (kRowThreads / 64 / sharing);
    const int block = first_block + wave / sharing, t0 = block * kBlockFrames;
    const bool runs = (m.flags & kUttRuns) != 0, has_rows = runs && t0 < m.Tb;
    auto zero_rows = [&]() {
#pragma unroll 4
        for (int r = 0; r < kBlockFrames; ++r)
            if (t0 + r < Tt && lane < A) store_gradient(g_args, (static_cast<size_t>(t0 + r) * B + b) * A + lane, 0.0f);
    };
    // The rows behind the utterance's last workgroup are divided among all of them.
    const int covered = min(groups * (kRowThreads / 64 / sharing) * kBlockFrames, Tt), each = (Tt - covered + groups - 1) / groups;
    const int from = covered + group * each, until = min(from + each, Tt);
#pragma unroll 4
    for (int t = from + wave; t < until; t += kRowThreads / 64)
        if (lane < A) store_gradient(g_args, (static_cast<size_t>(t) * B + b) * A + lane, 0.0f);
    if (!has_rows) {
        if (part == 0) zero_rows();                      // no lattice
        // (the barriers below)
        if (kWait && runs && first_block * kBlockFrames < m.Tb) __syncthreads();
        if (runs && part == 0 && block == frame_blocks(m.Tb)) utterance_cost<kWait>(g_args, meta, emit_blank, b);
        if (sharing > 1) __syncthreads();
        return;
    }
    unsigned* const s_hi = reinterpret_cast<unsigned*>(tile_lds) + wave * tile_lds_ints(Lmax, kTiles, kStaged);
    unsigned* const s_lo = s_hi + kBlockFrames * kShareRow;
    float* const s_emit = reinterpret_cast<float*>(s_hi + kShareInts);
    float* const s_norm = s_emit + (kStaged ? tile_emission_ints(kTiles) : 0);
    unsigned* const s_label = reinterpret_cast<unsigned*>(s_norm + kBlockFrames);
    static_assert((kShareInts + (kStaged ? tile_emission_ints(kTiles) : 0)) % 4 == 0 && kNormInts % 4 == 0, "16-byte reads");
    // Everything that comes from memory is asked for here, before any of it is used.
    const float4* const emit_in = reinterpret_cast<const float4*>(emit_label + emission_at(m.e_off, A, t0, 0));
    // (the block's 16 A emissions: up to 4 A vectors, 64 lanes; variables of their own, as the array went to scratch memory)
    auto emission_vector = [&](int i) { return emit_in[min(64 * i + lane, 4 * A - 1)]; };
    float4 emit0, emit1, emit2, emit3;
    if constexpr (kStaged) {
        emit0 = emission_vector(0);
        emit1 = emission_vector(1);
    }
    if constexpr (kStaged && kTiles > 2) {
        emit2 = emission_vector(2);
        emit3 = emission_vector(3);
    }
    const float norm_word = emit_blank[blank_emission_offset(m, 2 * block) + (lane & (kBlockFrames - 1))];
    // (an empty label has no string to look at, and the caller's array may be empty)
    const int first_base = part * kPieceStep;
    const LaneLabels first_labels(L > 0 ? labels + m.lab_off : &meta[b].L, max(L, 1), first_base);
    // Not staged: a lane's emissions of either chunk and position.
    struct ChunkEmissions { float4 v0, v1; };
    auto chunk_emissions = [&](bool has, int symbol, int h) __attribute__((always_inline)) {
        const float4* const p = reinterpret_cast<const float4*>(emit_label + label_emission_offset(m, has, symbol, 0, 2 * block + h, kZeroEmission));
        return ChunkEmissions{p[0], p[1]};
    };
    BlockEnds ends;
    bool log_domain = false, steep = false;
    double packed_inverse_p = 0.0;
    auto load_ends = [&]() {
        ends = BlockEnds::load<kWait>(m, lat, first_labels.p0, block);
        packed_inverse_p = kWait ? published(&g_args.mass[b * kMassWords + kMassInverse]) : g_args.mass[b * kMassWords + kMassInverse];
        const int domain = domain_of<kWait>(g_args.domain, b);
        if (kLean)                                       // (the same in every lane: two registers)
            packed_inverse_p = __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(packed_inverse_p)),
                                                __builtin_amdgcn_readfirstlane(__double2loint(packed_inverse_p)));
        log_domain = (domain & kDomainLog) != 0;
        steep = (domain & kDomainSteep) != 0;
    };
    if (!kWait) load_ends();
    __builtin_amdgcn_sched_barrier(0);
    stage_label_bytes(s_label, labels + m.lab_off, L);
    auto stage = [&](int i, const float4& e) {
        const int v = 64 * i + lane;                     // vector v: half v % 2 of row v / 2
        if (v < 4 * A) *reinterpret_cast<float4*>(s_emit + (v >> 1) * kEmissionRow + (v & 1) * 4) = e;
    };
    if constexpr (kStaged) {
        stage(0, emit0);
        stage(1, emit1);
        if constexpr (kTiles > 2) {
            stage(2, emit2);
            stage(3, emit3);
        }
        if (lane < 8) s_emit[2 * A * kEmissionRow + lane] = 0.0f;
    }
    if (lane < kBlockFrames) s_norm[lane] = frame_norm(norm_word);
    if (kWait) {
        if (!wait_for_chains(g_args, b, m.Tb)) {
            if (part == 0) zero_rows();
            if (sharing > 1) __syncthreads();            // (as many barriers as in the other ways out)
            return;
        }
        load_ends();
    }
    if (kWait && log_domain) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    float4v acc[kTiles];
#pragma unroll
    for (int n = 0; n < kTiles; ++n) acc[n] = float4v{0.0f, 0.0f, 0.0f, 0.0f};
    auto file = [&](int row, float x0, float x1) {
        const half2_raw hi = nearest_halves(x0, x1);
        const half2_raw lo = nearest_halves(minus_low_half(x0, hi), minus_high_half(x1, hi));
        s_hi[row * kShareRow + lane] = __builtin_bit_cast(unsigned, hi);
        s_lo[row * kShareRow + lane] = __builtin_bit_cast(unsigned, lo);
    };
    auto product = [&](int base) __attribute__((always_inline)) {
        // LDS operations of one wavefront complete in program order; the fences only keep the
        // compiler from moving them across.
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        share_product<kTiles>(acc, s_hi, s_lo, s_label, base, L, blank);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    };
    // (two loops: in one, what either recursion needs is held through the other, 20 registers)
    if (log_domain)
        for_pieces(L, part, sharing, [&](int base, int own_first, int own_end) {
            block_shares_log<kShareScaleLog2, 1>(m, lat, packed_inverse_p, block, base, own_first, own_end, file);
            product(base);
        });
    bool strained = false;
    if (!log_domain)
        for_pieces(L, part, sharing, [&](int base, int own_first, int own_end) {
            if (strained) return;
            LaneLabels at = first_labels;
            if (base != first_base) {
                at = LaneLabels(labels + m.lab_off, L, base);
                ends = BlockEnds::load<kWait>(m, lat, at.p0, block);
            }
            auto emissions = [&](int i, float (&el0)[kChunk], float (&el1)[kChunk]) __attribute__((always_inline)) {
                const int h = i & 1;
                auto row = [&](bool has, int symbol, float (&el)[kChunk]) __attribute__((always_inline)) {
                    float4 x, y;
                    if constexpr (kStaged) {
                        const float4* v = reinterpret_cast<const float4*>(s_emit + (has ? h * A + symbol : 2 * A) * kEmissionRow);
                        x = v[0];
                        y = v[1];
                    } else {
                        const ChunkEmissions e = chunk_emissions(has, symbol, h);
                        x = e.v0;
                        y = e.v1;
                    }
                    el[0] = x.x; el[1] = x.y; el[2] = x.z; el[3] = x.w;
                    el[4] = y.x; el[5] = y.y; el[6] = y.z; el[7] = y.w;
                };
                row(at.has0, at.symbol0, el0);
                row(at.has1, at.symbol1, el1);
            };
            strained = !block_shares<kShareScaleLog2>(m, at, ends, packed_inverse_p, steep, block, own_first, own_end, s_hi, s_lo, emissions, file);
            if (__builtin_expect(!strained, 1)) product(base);
        });
    if (__builtin_expect(strained, 0)) {
#pragma unroll
        for (int n = 0; n < kTiles; ++n) acc[n] = float4v{0.0f, 0.0f, 0.0f, 0.0f};
        for_pieces(L, part, sharing, [&](int base, int own_first, int own_end) {
            // (read again as well)
            if constexpr (kWait) {
                const FusedArgs& a = args_again<FusedArgs>();
                block_shares_of_logs<kShareScaleLog2, kWait>(a.chains.meta, a.chains.labels, a.chains.emit_label, a.chains.lat, a.tiles.mass, b, block, base, own_first, own_end, file);
            } else {
                const GradientArgs& a = args_again<GradientArgs>();
                block_shares_of_logs<kShareScaleLog2, kWait>(a.meta, a.labels, a.emit_label, a.lat, a.tiles.mass, b, block, base, own_first, own_end, file);
            }
            product(base);
        });
    }
    if (sharing > 1) {
        // the first of the wavefronts adds up what the others have, in their order
        float4v* const s_acc = reinterpret_cast<float4v*>(s_hi);
        static_assert(kTiles * 64 * 4 <= kShareInts, "the accumulators fit where the shares were");
        if (part > 0)
#pragma unroll
            for (int n = 0; n < kTiles; ++n) s_acc[n * 64 + lane] = acc[n];
        __syncthreads();
        if (part > 0) return;
        for (int i = 1; i < sharing; ++i) {
            const float4v* const theirs = reinterpret_cast<const float4v*>(s_hi + i * tile_lds_ints(Lmax, kTiles, kStaged));
#pragma unroll
            for (int n = 0; n < kTiles; ++n) acc[n] += theirs[n * 64 + lane];
        }
    }
    // Result: lane l holds symbol 16 n + l % 16 of frames 4 (l / 16) .. + 3; y is the emission.
    const int writer = kLean ? tile_thread() & 63 : 0, column = kLean ? writer & 15 : c, quad = kLean ? writer >> 4 : g;
    const int tr = t0 + 4 * quad;
    const float scale = packed_mantissa(packed_inverse_p) * (0.5f / (1 << kShareScaleLog2));
    auto write = [&](auto* grads) {
#pragma unroll
        for (int n = 0; n < kTiles; ++n) {
            const int k = 16 * n + column;
            if (k >= A) continue;
            auto* out = grads + (static_cast<size_t>(tr) * B + b) * A + k;
            const float4 y = kStaged ? *reinterpret_cast<const float4*>(s_emit + ((quad >> 1) * A + k) * kEmissionRow + (quad & 1) * 4)
                                     : emit_in[2 * ((quad >> 1) * A + k) + (quad & 1)];
            const float4 norm = *reinterpret_cast<const float4*>(s_norm + 4 * quad);
            const float yv[4] = {y.x, y.y, y.z, y.w}, norms[4] = {norm.x, norm.y, norm.z, norm.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float occupancy = acc[n][i] * scale;
                const float v = emission_softmax(yv[i], norms[i]) - (k == blank ? 1.0f - occupancy : occupancy);
                if (tr + i < Tt) store_elem(out, static_cast<size_t>(i) * B * A, tr + i < m.Tb ? v : 0.0f);
            }
        }
    };
    if (g_args.bf16) write(static_cast<bf16_t*>(g_args.grads));
    else write(static_cast<float*>(g_args.grads));
}

// Which of its utterance's workgroups the within-th one is: one further on from utterance to utterance.  Workgroup i runs on die i mod 8
// and, as long as places are free, on compute unit i mod 256, and of an utterance's workgroups the last ones often have nothing to do.
// With 16 workgroups to an utterance they all fell to the same halves of the dies: 122 utterances of up to 454 frames, 34 symbols, 62.0 us
// a call (before costs had a workgroup 50.9), so 48.5; 32 symbols 50.2 (49.0), 44.4.
__device__ __forceinline__ int rotated_group(int within, int utterance, int groups) { return (within + utterance) % groups; }

// Without by_end: grid (workgroups per utterance, B).  With it: a workgroup per tile, in as many rows of the grid as they take, those of the utterances that took longest first.
// (Which utterances have several wavefronts to a block is as it is beside the chains: the sums are in another order with them.)
template <int kTiles, bool kStaged>
__global__ __launch_bounds__(kRowThreads, kStaged ? 1 : 4)
void ctc_gradient_narrow_kernel(const TileArgs args, const Utt* __restrict__ meta, const int* __restrict__ labels,
                                const float* __restrict__ emit_blank, const float* __restrict__ emit_label,
                                const LatticeOut lat)
{
    extern __shared__ uint4v tile_lds[];
    TilePlace place{static_cast<int>(blockIdx.y), static_cast<int>(blockIdx.x), static_cast<int>(gridDim.x), args.shared_from == 0};
    int b = place.rank;
    if (args.by_end) {
        const unsigned back = blockIdx.y * gridDim.x + blockIdx.x, tiles = args.segment_tile[TileArgs::kSegments];
        if (back >= tiles) return;
        place = TilePlace::of(args, tiles - 1 - back);
        b = __builtin_amdgcn_readfirstlane(args.by_end[place.rank]);
    }
    narrow_tile<kTiles, false, kStaged, !kStaged>(args, meta, labels, emit_blank, emit_label, lat, tile_lds, b,
                                                  rotated_group(place.within, place.rank, place.groups), place.groups, place.shares);
}

// Larger alphabets: the softmax launch has written y (and zeros); here the columns of the label's symbols and the
// blank's are corrected.  A workgroup per block.  Its wavefronts take the label's pieces; the shares go to LDS in slot order
// (the positions of a symbol next to each other, setup_role), and the lane of a symbol and frame adds up its run: one writer
// per symbol and a fixed order.  The last wavefront, if it has no piece, lists the symbols meanwhile.  The launch waits for its
// slowest block and leaves the memory idle, so its first workgroups write zero rows (columns_frames).  grid B, fill.rounds + blocks of T (wide_rows);
// LDS: wide_lds_bytes.
// What bounds it: in launches of up to a block per SIMD (64 utterances of 500 frames: 1140) the time of the slowest block, beyond
// that the issue of the recomputation.  With a wavefront to a block a block took 7 to 25 us (loads 2, a piece 4.5, sums 1 to 10),
// and 171 registers left room for three wavefronts on a SIMD.  Two wavefronts share the sums, four the pieces too; a piece's
// operands have one set of registers, whichever piece it is, and take 2.9 us.  64 x 500 frames, 750
// symbols: 89.3 -> 82.7 us a call; 512 x 500, 300 symbols: 397 -> 346; 400 x 500, 80 symbols: 303 -> 260; 32 x 1400, labels of up to
// 500 symbols: 288 -> 248.  Registers are for five wavefronts on a SIMD (91; at 101, four, labels of up to 175 symbols needed a second round of
// workgroups): 64 x 500, 750 symbols 76.1 -> 74.3; 400 x 500, 80 symbols 158.0 -> 149.7; 128 x 400, 3000 symbols bf16 152.6 -> 150.9.
// Labels of one piece take two wavefronts (64 x 500, 6000 symbols, bf16: 161.0 us; with four 162.7).
// Neighbouring workgroups are different utterances, one further on from block to block to each: a compute unit gets every n-th
// workgroup, and with an utterance's blocks side by side some got first blocks only and others the last ones, which many utterances
// do not have (one wavefront per block, 512 x 500 frames: 397 us, so 364).
constexpr int kWideWaves = 4;
// Its LDS: the list of symbols, then the shares [slot][frame] and a slot for those that a wavefront forms for its neighbour's
// positions, then alpha for each wavefront with a piece.
constexpr int kSharePitch = kBlockFrames + 1;
constexpr int wide_alpha_at(int Lmax) { return (2 * Lmax + kSharePitch * (Lmax + 1) + 3) / 4 * 4; }
constexpr size_t wide_lds_bytes(int Lmax, int waves)
{
    return (static_cast<size_t>(wide_alpha_at(Lmax)) + std::min(waves, std::max(label_pieces(Lmax), 1)) * kShareInts) * sizeof(unsigned);
}
// kFill: (without, as a variant of its own: 0.5 % for calls that leave no rows to it)
template <bool kFill>
__global__ __launch_bounds__(64 * kWideWaves)
void ctc_gradient_wide_kernel(const TileArgs g, const Utt* __restrict__ meta, const int* __restrict__ labels,
                              const float* __restrict__ emit_blank, const float* __restrict__ emit_label, const LatticeOut lat,
                              const FillArgs fill)
{
    const int grid_row = static_cast<int>(blockIdx.z * gridDim.y + blockIdx.y);
    if (kFill && grid_row < fill.rounds) {
        const int waves = blockDim.x >> 6;
        fill_rows(fill, meta, static_cast<int>(grid_row * gridDim.x + blockIdx.x) * waves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6),
                  static_cast<int>(fill.rounds * gridDim.x) * waves);
        return;
    }
    __shared__ float s_word[kBlockFrames], s_sum[kWideWaves * kBlockFrames];
    __shared__ int s_symbols;
    extern __shared__ uint4v wide_lds[];
    const int B = g.B, A = g.A, blank = g.blank;
    const int lane = threadIdx.x & 63, block = grid_row - (kFill ? fill.rounds : 0), t0 = block * kBlockFrames;
    const int b = static_cast<int>((blockIdx.x + 3u * block) % static_cast<unsigned>(B));      // (three: neighbours change dies too)
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6;
    const Utt m = uniform_record(meta[b]);
    if (!(m.flags & kUttRuns) || t0 >= m.Tb) return;
    unsigned* const s_list = reinterpret_cast<unsigned*>(wide_lds);
    float* const s_share = reinterpret_cast<float*>(s_list + 2 * g.Lmax);
    unsigned* const s_alpha = s_list + g.alpha_at + wave * kShareInts;
    const int L = m.L;
    const int* const lab = L > 0 ? labels + m.lab_off : &meta[b].L;      // (an empty label has no string to look at)
    const int* const link_of = L > 0 ? g.links + m.lab_off : &meta[b].L;
    if (threadIdx.x < kBlockFrames) s_word[lane] = emit_blank[blank_emission_offset(m, 2 * block) + lane];
    const int pieces = label_pieces(L);
    if (wave < pieces) {
        // Everything that comes from memory for a piece is asked for at once, before any of it is used.
        LaneLabels at(lab, L, wave * kPieceStep);
        int link0, link1;
        struct ChunkEmissions { float4 v0, v1; };
        ChunkEmissions emit00, emit01, emit10, emit11;   // [position][chunk]
        BlockEnds ends;
        auto chunk_emissions = [&](bool has, int position, int h) {
            const float4* const p = reinterpret_cast<const float4*>(emit_label + label_emission_offset(m, has, 0, position, 2 * block + h, kZeroEmission));
            return ChunkEmissions{p[0], p[1]};
        };
        auto load = [&]() {
            link0 = link_of[min(at.p0, L - 1)];
            link1 = link_of[min(at.p1, L - 1)];
            emit00 = chunk_emissions(at.has0, at.p0, 0);
            emit10 = chunk_emissions(at.has1, at.p1, 0);
            emit01 = chunk_emissions(at.has0, at.p0, 1);
            emit11 = chunk_emissions(at.has1, at.p1, 1);
            ends = BlockEnds::load<false>(m, lat, at.p0, block);
        };
        load();
        const int domain = domain_of<false>(g.domain, b);
        const double packed_inverse_p = g.mass[b * kMassWords + kMassInverse];
        __builtin_amdgcn_sched_barrier(0);
        const float inverse_p = packed_mantissa(packed_inverse_p);
        for (int i = wave;;) {
            const int own_first = i == 0 ? 0 : i * kPieceStep + kPieceHalo, own_end = i == pieces - 1 ? L : (i + 1) * kPieceStep + kPieceHalo;
            const bool own0 = at.p0 >= own_first && at.p0 < own_end, own1 = at.p1 >= own_first && at.p1 < own_end;
            float* const share0 = s_share + (own0 ? link0 & kLinkSlotMask : L) * kSharePitch;
            float* const share1 = s_share + (own1 ? link1 & kLinkSlotMask : L) * kSharePitch;
            auto file = [&](int row, float x0, float x1) {
                share0[row] = x0 * inverse_p;
                share1[row] = x1 * inverse_p;
            };
            if (domain == kDomainLog) block_shares_log<0, 2>(m, lat, packed_inverse_p, block, i * kPieceStep, own_first, own_end, file);
            else {
                // (the first chunk's are read once more when they are needed again: a trip to the cache, and 16 registers)
                auto emissions = [&](int k, float (&el0)[kChunk], float (&el1)[kChunk]) __attribute__((always_inline)) {
                    auto get = [](const ChunkEmissions& e, float (&el)[kChunk]) {
                        el[0] = e.v0.x; el[1] = e.v0.y; el[2] = e.v0.z; el[3] = e.v0.w;
                        el[4] = e.v1.x; el[5] = e.v1.y; el[6] = e.v1.z; el[7] = e.v1.w;
                    };
                    get(k == 0 ? emit00 : k == 1 ? emit01 : chunk_emissions(at.has0, at.p0, 0), el0);
                    get(k == 0 ? emit10 : k == 1 ? emit11 : chunk_emissions(at.has1, at.p1, 0), el1);
                };
                if (__builtin_expect(!block_shares<0>(m, at, ends, packed_inverse_p, domain == kDomainSteep, block, own_first, own_end, s_alpha,
                                                      s_alpha + kBlockFrames * kShareRow, emissions, file), 0))
                {
                    const GradientArgs& a = args_again<GradientArgs>();
                    block_shares_of_logs<0, false>(a.meta, a.labels, a.emit_label, a.lat, a.tiles.mass, b, block, i * kPieceStep, own_first, own_end, file);
                }
            }
            i += waves;
            if (i >= pieces) break;
            at = LaneLabels(lab, L, i * kPieceStep);
            load();
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (wave == waves - 1) {
        // The label's symbols one after the other: the word of the first occurrence with the position put into its unused bits,
        // and the symbol.
        static_assert(CTC_MAX_LABEL_LENGTH < 1024, "a position is ten bits");
        int symbols = 0;
        for (int j0 = 0; j0 < L; j0 += 64) {
            const int j = j0 + lane, link = j < L ? link_of[j] : 0, symbol = j < L ? lab[j] : 0;
            const unsigned long long firsts = __ballot(link < 0);
            if (link < 0) {
                const int i = symbols + __builtin_amdgcn_mbcnt_hi(static_cast<unsigned>(firsts >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<unsigned>(firsts), 0));
                s_list[2 * i] = static_cast<unsigned>((link & (kLinkSlotMask | kLinkSlotMask << kLinkCountShift)) | (j & 3) << 10 | (j >> 2) << 22);
                s_list[2 * i + 1] = static_cast<unsigned>(symbol);
            }
            symbols += __popcll(firsts);
        }
        if (lane == 0) s_symbols = symbols;
        if (t0 == 0) {
            const double log2_norms = norms_of_wave(norms_of_lane(m, emit_blank)).log2();
            if (lane == 0)
                g.costs[b] = g.chain_err[b] != 0 ? __uint_as_float(0x7FC00000u)
                                                 : cost_of_mass(g.mass[b * kMassWords + kMassValue], g.mass[b * kMassWords + kMassLog2], log2_norms);
        }
    }
    __syncthreads();
    const int symbols = __builtin_amdgcn_readfirstlane(s_symbols);
    // A lane per frame and symbol adds up the run of its symbol's positions, four symbols to a wavefront side by side and
    // kAtOnce such rounds in flight.  (A lane per symbol took every frame in turn, and the wavefront as long as its most
    // frequent symbol 16 times over.)
    constexpr int kAtOnce = 4;
    const int rows = min(kBlockFrames, m.Tb - t0);
    const int row = lane & (kBlockFrames - 1), t = t0 + row;
    const bool has_row = row < rows;
    const float* const share = s_share + row;
    const size_t out = (static_cast<size_t>(t) * B + b) * A;
    const float* const y_row = emit_label + emission_at(m.e_off, L, min(t, m.Tb - 1), 0);
    const float word_of_frame = s_word[row], norm = frame_norm(word_of_frame);
    float sum = 0.0f;
    for (int i0 = 4 * wave + (lane >> 4); i0 - (lane >> 4) < symbols; i0 += 4 * kAtOnce * waves) {
        uint2v entry[kAtOnce];
        float y[kAtOnce];
#pragma unroll
        for (int n = 0; n < kAtOnce; ++n) {
            entry[n] = *reinterpret_cast<const uint2v*>(&s_list[2 * min(i0 + 4 * waves * n, symbols - 1)]);
            const int position = static_cast<int>(entry[n][0] >> 10 & 3) | static_cast<int>(entry[n][0] >> 22) << 2;
            y[n] = y_row[static_cast<size_t>(position) * kChunk];
        }
#pragma unroll
        for (int n = 0; n < kAtOnce; ++n) {
            const int slot = static_cast<int>(entry[n][0] & kLinkSlotMask), count = static_cast<int>(entry[n][0] >> kLinkCountShift & kLinkSlotMask);
            float o = share[slot * kSharePitch];
            for (int k = 1; k < count; ++k) o += share[(slot + k) * kSharePitch];
            if (i0 + 4 * waves * n < symbols && has_row) {
                store_gradient(g, out + entry[n][1], emission_softmax(y[n], norm) - o);
                sum += o;
            }
        }
    }
    // the blank: what the label states leave of 1
    sum += __shfl_xor(sum, 16);
    sum += __shfl_xor(sum, 32);
    if (lane < kBlockFrames) s_sum[wave * kBlockFrames + lane] = sum;
    __syncthreads();
    if (wave == 0 && has_row && lane < kBlockFrames) {
        for (int w = 1; w < waves; ++w) sum += s_sum[w * kBlockFrames + lane];
        store_gradient(g, out + blank, blank_softmax(word_of_frame) - (1.0f - sum));
    }
}

// ---- chains and gradient in one launch -------------------------------------------------------------
// Alphabets of at most kDirectMaxA symbols.  Chains first, one workgroup each; then the gradient's workgroups, the
// utterances whose chains end first before the others.  A gradient workgroup asks for everything that the softmax launch
// has left and waits for its utterance's two chains; by the time the longest chains end, only their own blocks are left to do.
//
// A workgroup waits for chains that are under way, never for one that has yet to be given a compute unit: the order of the
// workgroups says nothing about that.  Each die hands out its share of a launch by itself, and two such launches on two
// streams can fill one die with workgroups that wait for chains which the other launch's keep from the other die, and the
// other way round.  So a chain's workgroup says that it is there (take_chain), and one of the gradient looks for that first.
// If it takes too long, it leaves its place to the chains' workgroups and makes room: the second of them, which knows that
// nobody leaves any more, takes the places on the list when its own chain has ended.  It waits for the first one's chain, and
// that waits for nothing outside its workgroup, so it ends, and so does every wait.
// (Waiting workgroups that run such a chain themselves need its code a second time: inlined 1 to 5 us of 57 for everybody, in a
// function a stack, for which the runtime takes 92 MB of device memory and 280 MB more over further queues.  English minibatch:
// 56.6 us without the look at the word, which cannot be trusted, 56.7 with it.)
constexpr int kLeavePolls = 1 << 10;      // about a millisecond: a chain's workgroup is there within 5 us in a launch alone on the chip

// By each wavefront of a workgroup, alike: waits until both chains of utterance b have a workgroup.  False: that took too long,
// and the place, `tile`, has been left.  (Bits and list only ever grow, and nobody joins the list once both chains are taken: all
// wavefronts come to the same answer whenever they look.)
__device__ __forceinline__ bool chains_taken(const TileArgs& g, int b, int tile)
{
    int* const word = &g.done[b * kDoneStride + kTakenWord];
    for (int polls = kLeavePolls;; --polls) {
        const int now = __builtin_amdgcn_readfirstlane(published(word));
        for (int i = now >> kLeftShift; i != 0; i = __builtin_amdgcn_readfirstlane(published(&g.left[i - 1])))
            if (i - 1 == tile) return false;
        if ((now & kBothTaken) == kBothTaken) return true;
        if (polls <= 0 && threadIdx.x == 0) {
            publish(&g.left[tile], now >> kLeftShift);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            int expected = now;
            __hip_atomic_compare_exchange_strong(word, &expected, (now & kBothTaken) | (tile + 1) << kLeftShift, __ATOMIC_RELAXED,
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __builtin_amdgcn_s_sleep(10);
    }
}


// kLean: 128 registers, so that a compute unit holds two workgroups of more than four wavefronts and not one, while the blocks wait
// that the chains have left behind: for up to 32 symbols (more would need a stack) and workgroups of that size (32 x 1500 frames,
// labels of up to 540 symbols: 135.5 -> 131.0 us a call; up to four wavefronts 0.5 % slower so).  Launches of more chains than compute
// units have it too, and no emissions in LDS (kStaged), so that four workgroups of up to four wavefronts share a compute unit: up to four
// times as many chains as compute units start together.
template <Sync kSync, int kTiles, bool kLean, bool kStaged>
__global__ __launch_bounds__(64 * (kStaged ? kFusedWaves : kCrowdedFusedWaves), kLean ? 4 : 1)
void ctc_lattice_gradient_kernel(const Utt* __restrict__ meta, const int* __restrict__ order,
                                 const int* __restrict__ labels, const float* __restrict__ emit_blank, const float* __restrict__ emit_label,
                                 const LatticeOut lat, double* __restrict__ mass, float* __restrict__ costs,
                                 int* __restrict__ chain_err, uint32_t* __restrict__ sink, const LaunchWords wk, const TileArgs tiles)
{
    extern __shared__ uint4v fused_lds[];
    const int index = static_cast<int>(blockIdx.x);
    if (index < tiles.first_group) {
        __builtin_amdgcn_s_setprio(3);
        int left = lattice_body<kSync, Mode::kGrad, true>(order[index], meta, labels, emit_blank, nullptr, emit_label, lat, mass,
                                                          costs, chain_err, sink, fused_lds, wk);
        if (__builtin_expect(left == 0, 1) || threadIdx.x >= kRowThreads) return;
        __builtin_amdgcn_s_setprio(0);
        do {
            __syncthreads();
            const FusedArgs& args = args_again<FusedArgs>();
            const ChainArgs<true>& a = args.chains;
            const int tile = left - 1;
            const TilePlace place = TilePlace::of(args.tiles, tile);
            const int b = __builtin_amdgcn_readfirstlane(args.tiles.by_end[place.rank]);
            narrow_tile<kTiles, true, kStaged, kLean>(args.tiles, a.meta, a.labels, a.emit_blank, a.emit_label, a.lat, fused_lds, b,
                                             rotated_group(place.within, place.rank, place.groups), place.groups, place.shares);
            left = __builtin_amdgcn_readfirstlane(published(&args.tiles.left[tile]));
        } while (left != 0);
    } else {
        const int tile = index - tiles.first_group;
        const TilePlace place = TilePlace::of(tiles, tile);
        const int group = rotated_group(place.within, place.rank, place.groups), b = __builtin_amdgcn_readfirstlane(tiles.by_end[place.rank]);
        const int flags = __builtin_amdgcn_readfirstlane(meta[b].flags), frames = __builtin_amdgcn_readfirstlane(meta[b].Tb);
        const int sharing = place.shares ? block_waves(__builtin_amdgcn_readfirstlane(meta[b].L)) : 1;
        if (threadIdx.x >= kRowThreads) return;          // (workgroups as large as the longest label's chains)
        const bool waits = (flags & kUttRuns) && group * (kRowThreads / 64 / sharing) <= frame_blocks(frames);     // (narrow_tile: rows, or the cost)
        if (waits && !chains_taken(tiles, b, tile)) return;
        narrow_tile<kTiles, true, kStaged, kLean>(tiles, meta, labels, emit_blank, emit_label, lat, fused_lds, b, group, place.groups, place.shares);
    }
}

template <typename F>
int checked_launch(F&& f)
{
    f();
    return static_cast<int>(hipGetLastError());
}

}  // namespace

namespace {
// Symbols to a lane of ctc_softmax_rows_kernel: 12 (fp32: three vectors; bf16 vectors have eight symbols), 16, 24 or 32.  Vectors
// behind a row's end are asked for all the same and cost their instructions.  With 16 and 32 alone 27 x 333 x 4733 bf16 44.3 us a call, so
// 43.4, fp32 67.3 and 67.0; 64 x 500 x 6000 247.8 and 246.5, bf16 138.2 and 137.6.  With 16 in place of 12, fp32, 64 x 500 frames: 100 symbols 52.0, so 51.9; 600
// 65.5 and 65.2; 750 72.6 and 72.1; 2100 125.1 and 123.4; 2500 134.4 and 132.8; 3000 148.4 and 148.0.
template <typename T>
constexpr int kFewest = sizeof(T) == 4 ? 12 : 16;
// Lanes per row of ctc_softmax_rows_kernel; 0 where it does not apply: rows of more than 8192 symbols, more workgroups than a
// grid holds.
int row_lanes(const Launch& p)
{
    if (p.A > 32 * kRowThreads) return 0;
    const int lanes = p.A <= 32 * 16 ? 16 : (p.A <= 32 * 64 ? 64 : kRowThreads);
    const int rows = kRowThreads / lanes;
    const int64_t groups = static_cast<int64_t>(p.T) * ((p.B + rows - 1) / rows) + static_cast<int64_t>(p.B) * (CTC_MAX_LABEL_LENGTH / 64 + 1);
    return groups <= INT32_MAX / kRowThreads ? lanes : 0;
}

// The tiles of ctc_softmax_rows_kernel.
// Rows of a workgroup each: runs of 64 rows.  64 x 500 x 6000 288.9 -> 261.6 us a call (runs of 8, 16, 32, 128 and 192 rows: 279 with
// streaming loads, 269.8, 262.6, 261.6 and 266), in bf16 162.7 -> 145.5; 16 x 1000 x 8000 194.5 -> 181; 200 x 150 x 5000 212 -> 207;
// 100 x 800 x 4001 bf16 264 -> 251.  From 24 rounds of them on: a die of 27 x 333 x 4733 (17 rounds) has up to a run more to do than
// another, 68.9 us without tiles and 69.5 with.
// Several rows to a workgroup: the eight frames of a chunk of emissions, and of a frame all groups up to 32, beyond that about 16 at
// a time.  64 x 500 x 750 82.0 -> 79.0; 32 x 1500 x 2000 240 -> 226.5; 64 x 1000 x 1000 bf16 147 -> 139; 150 x 500 x 120 87.5 -> 83.2;
// 512 x 400 x 200 bf16 134.3 -> 132; 256 x 700 x 100 157 -> 156.4, 160 in runs of 64 groups, which write words of a chunk from four
// dies; of 24 shapes only 200 x 500 x 700 bf16 lost (123.5 -> 125.5).
constexpr int kRunRows = 64, kRunRounds = 24, kTileGroupsMost = 32, kTileGroups = 16;
RowPlan row_plan(const Launch& p, int lanes)
{
    const int rows = kRowThreads / lanes, per_frame = (p.B + rows - 1) / rows;
    auto plan = [&](int groups, int frames, int columns) {
        return RowPlan{groups, Divisor(per_frame), frames, Divisor(columns), Divisor(8 * std::max(frames, 1) * columns), Divisor((per_frame + columns - 1) / columns)};
    };
    // (nothing but emissions is written: consecutive frames of an utterance are better off on one die where that happens to be so;
    // 214 x 171 x 4186 bf16, cost alone: 84.5 us a call without tiles, 93.6 with)
    if (!p.grads) return plan(p.T * per_frame, 0, 1);
    if (lanes == kRowThreads) return plan(p.T * per_frame, static_cast<int64_t>(p.T) * per_frame >= 8 * kRunRows * kRunRounds ? 1 : 0, kRunRows);
    const int across = per_frame <= kTileGroupsMost ? 1 : (per_frame + kTileGroups - 1) / kTileGroups;
    const int columns = (per_frame + across - 1) / across;
    const int64_t tiles = static_cast<int64_t>((per_frame + columns - 1) / columns) * ((p.T + kChunk - 1) / kChunk);
    const int64_t groups = (tiles + 7) / 8 * 8 * kChunk * columns;
    // (fewer tiles than dies, or too many groups of rows for a launch once the ends of tiles are counted in: none)
    if (tiles < 8 || groups + static_cast<int64_t>(p.B) * (CTC_MAX_LABEL_LENGTH / 64 + 1) > INT32_MAX / kRowThreads) return plan(p.T * per_frame, 0, columns);
    return plan(static_cast<int>(groups), kChunk, columns);
}
// Loads past the caches: fp32 rows of a workgroup each that begin on 16 bytes, in tensors of twice the last-level cache and more.
// 64 x 500 x 6000 261.6 -> 253.5 us a call, 64 x 500 x 4096 180.8 -> 169, 16 x 1000 x 8000 181 -> 176, 200 x 150 x 5000 206.9 -> 205.5.
// Smaller tensors lose what the cache still holds of them (20 x 200 x 6000, 96 MB: 41.8 -> 46.6), rows that share lines of memory
// load those twice (100 x 800 x 4001 bf16 251 -> 258.6), and bf16 gains nothing (64 x 500 x 6000 145.5 -> 146.5).
constexpr int64_t kStreamedBytes = 512'000'000;
bool streamed_rows(const Launch& p, int lanes)
{
    return lanes == kRowThreads && p.dtype == CTC_DTYPE_F32 && p.A % 4 == 0 && reinterpret_cast<uintptr_t>(p.x) % 16 == 0 &&
           static_cast<int64_t>(p.T) * p.B * p.A * 4 >= kStreamedBytes;
}
}

// Values in the first half of a direction's region, exponents in the second.
static LatticeOut lattice_blocks(const Launch& p)
{
    auto* alpha = reinterpret_cast<uint32_t*>(p.ws + p.lay.alpha);
    auto* beta = reinterpret_cast<uint32_t*>(p.ws + p.lay.beta);
    return {alpha, reinterpret_cast<int*>(alpha + p.lay.ab_doubles), beta, reinterpret_cast<int*>(beta + p.lay.ab_doubles)};
}

int launch_setup(const Launch& p, void* stream)
{
    // (the byte labels after the words are read in place)
    const int words = static_cast<int>(p.lay.labels8 / 4);
    const unsigned char* labels8 = p.A <= kByteLabelsMaxA ? static_cast<const unsigned char*>(p.host_image) + p.lay.labels8 : nullptr;
    return checked_launch([&] {
        hipLaunchKernelGGL(ctc_upload_kernel, dim3((words + kRowThreads - 1) / kRowThreads), dim3(kRowThreads),
                           0, static_cast<hipStream_t>(stream), static_cast<const int*>(p.host_image),
                           reinterpret_cast<int*>(p.ws), words, static_cast<int>(p.lay.labels / 4),
                           static_cast<int>(p.lay.labels8 / 4), labels8);
    });
}

int launch_plan(const Launch& p, void* stream)
{
    return checked_launch([&] {
        hipLaunchKernelGGL(ctc_plan_kernel, dim3(1), dim3(kPlanThreads), 0, static_cast<hipStream_t>(stream),
                           p.labels, p.dev_label_lengths, p.dev_input_lengths,
                           reinterpret_cast<Utt*>(p.ws + p.lay.meta), reinterpret_cast<int*>(p.ws + p.lay.order),
                           p.dev_status, p.T, p.B, p.A, p.blank, p.max_label, p.poll_budget, p.crowded,
                           p.needs_barrier);
    });
}

int launch_softmax(const Launch& p, void* stream)
{
    auto* meta = reinterpret_cast<Utt*>(p.ws + p.lay.meta);
    const int* labels = p.labels;
    auto* emit_blank = reinterpret_cast<float*>(p.ws + p.lay.emit_blank);
    auto* emit_label = reinterpret_cast<float*>(p.ws + p.lay.emit_label);
    const SetupArgs sa{reinterpret_cast<int*>(p.ws + p.lay.links), p.costs,
                       reinterpret_cast<int*>(p.ws + p.lay.chain_err), reinterpret_cast<int*>(p.ws + p.lay.done),
                       emit_label,
                       reinterpret_cast<double*>(p.ws + p.lay.emit_blank64),
                       p.folded ? nullptr : p.host_flag, p.host_flag_value, p.mode == Mode::kBest,
                       // gathered emissions and few utterances: spread the grouping of each one's label positions over
                       // several workgroups (its latency counts); many: one workgroup each keeps the chip busy already
                       p.A <= kDirectMaxA || p.B >= 256 ? 1 : std::max(1, (p.max_label + 63) / 64)};
    const dim3 block(kRowThreads);
    auto s = static_cast<hipStream_t>(stream);
    const bool f32 = p.dtype == CTC_DTYPE_F32;
    return checked_launch([&] {
        if (p.A <= kDirectMaxA && p.folded) {
            // the smallest alphabets, host metadata: the launch reads the pinned image itself
            const dim3 grid((p.T + kFlagFrames - 1) / kFlagFrames + sa.parts, p.B);
            const size_t lds = static_cast<size_t>(kFlagFrames) * (p.A + 1) * sizeof(float);
            const NarrowImage image{static_cast<const int*>(p.host_image), static_cast<int>(p.lay.labels / 4),
                                    static_cast<int>(p.lay.labels8 / 4), static_cast<int>(p.lay.labels8 / 4), p.lay.labels8,
                                    reinterpret_cast<int*>(p.ws + p.lay.labels)};
            auto* row_flags = reinterpret_cast<int*>(p.ws + p.lay.row_flags);
            NarrowArgs args;
            NarrowRows& rows_of = args.rows;
            NarrowDevice dv{};
            if (p.dev_label_lengths) args.plans = plans().table[p.crowded];
            if (p.dev_label_lengths)
                dv = NarrowDevice{p.labels, p.dev_label_lengths, p.dev_input_lengths, meta, reinterpret_cast<int*>(p.ws + p.lay.order),
                                  reinterpret_cast<int*>(p.ws + p.lay.status), p.max_label, p.poll_budget,
                                  p.crowded, p.needs_barrier,
                                  p.n_cu % kChainBlock == 0 ? p.n_cu : 0};
            const Utt* records = static_cast<const Utt*>(p.host_image);      // (the host reads its own image)
            for (int b = 0; records && b < p.B; ++b) {
                rows_of.frames[b] = records[b].Tb | ((records[b].flags & kUttRuns) ? kRowsRun : 0);
                rows_of.frames_before[b] = records[b].f_off;
                rows_of.label_length[b] = records[b].L;
                rows_of.labels_before[b] = records[b].lab_off;
            }
            if (f32)
                hipLaunchKernelGGL(ctc_softmax_narrow_kernel<float>, grid, block, lds, s, static_cast<const float*>(p.x),
                                   image, reinterpret_cast<int*>(p.ws), emit_blank, emit_label, row_flags, sa,
                                   args, dv, p.T, p.B, p.A, p.blank);
            else
                hipLaunchKernelGGL(ctc_softmax_narrow_kernel<bf16_t>, grid, block, lds, s, static_cast<const bf16_t*>(p.x),
                                   image, reinterpret_cast<int*>(p.ws), emit_blank, emit_label, row_flags, sa,
                                   args, dv, p.T, p.B, p.A, p.blank);
        } else if (p.A <= kDirectMaxA) {
            const dim3 grid((p.T + 63) / 64 + 1, p.B);
            const size_t lds = static_cast<size_t>(64) * (p.A + 1) * sizeof(float);
            if (f32)
                hipLaunchKernelGGL(ctc_softmax_symbols_kernel<float>, grid, block, lds, s, static_cast<const float*>(p.x), meta,
                                   emit_blank, emit_label, sa, p.B, p.A, p.blank);
            else
                hipLaunchKernelGGL(ctc_softmax_symbols_kernel<bf16_t>, grid, block, lds, s, static_cast<const bf16_t*>(p.x), meta,
                                   emit_blank, emit_label, sa, p.B, p.A, p.blank);
        } else if (row_lanes(p) > 0) {
            const int lanes = row_lanes(p);
            const RowPlan plan = row_plan(p, lanes);
            const dim3 grid(plan.groups + sa.parts * p.B);
#define CTC_LAUNCH_ROWS_FROM(TYPE, LANES, PER_LANE, STREAMING)                                     \
    hipLaunchKernelGGL((ctc_softmax_rows_kernel<TYPE, LANES, PER_LANE, STREAMING>), grid, block, 0, s, \
                       static_cast<const TYPE*>(p.x), static_cast<TYPE*>(p.grads), meta, labels,   \
                       emit_blank, emit_label, sa, p.T, p.B, p.A, p.blank, plan, p.defer + p.defer_columns)
#define CTC_LAUNCH_ROWS_OF_LANES(TYPE, LANES, STREAMING)                                           \
    do {                                                                                           \
        if (p.A <= LANES * kFewest<TYPE>) CTC_LAUNCH_ROWS_FROM(TYPE, LANES, kFewest<TYPE>, STREAMING);     \
        else if (p.A <= LANES * 16) CTC_LAUNCH_ROWS_FROM(TYPE, LANES, 16, STREAMING);              \
        else if (p.A <= LANES * 24) CTC_LAUNCH_ROWS_FROM(TYPE, LANES, 24, STREAMING);              \
        else CTC_LAUNCH_ROWS_FROM(TYPE, LANES, 32, STREAMING);                                     \
    } while (0)
#define CTC_LAUNCH_ROWS_OF(TYPE)                                                                   \
    do {                                                                                           \
        if (lanes == 16) CTC_LAUNCH_ROWS_OF_LANES(TYPE, 16, false);                                \
        else if (lanes == 64) CTC_LAUNCH_ROWS_OF_LANES(TYPE, 64, false);                           \
        else CTC_LAUNCH_ROWS_OF_LANES(TYPE, kRowThreads, false);                                   \
    } while (0)
            if (streamed_rows(p, lanes)) {
                CTC_LAUNCH_ROWS_OF_LANES(float, kRowThreads, true);
            } else if (f32) CTC_LAUNCH_ROWS_OF(float);
            else CTC_LAUNCH_ROWS_OF(bf16_t);
#undef CTC_LAUNCH_ROWS_OF
#undef CTC_LAUNCH_ROWS_OF_LANES
#undef CTC_LAUNCH_ROWS_FROM
        } else {
            const dim3 grid(p.T + 1, p.B);
            if (f32)
                hipLaunchKernelGGL(ctc_softmax_kernel<float>, grid, block, 0, s,
                                   static_cast<const float*>(p.x), static_cast<float*>(p.grads), meta, labels, emit_blank,
                                   emit_label, sa, p.T, p.B, p.A, p.blank, p.defer + p.defer_columns);
            else
                hipLaunchKernelGGL(ctc_softmax_kernel<bf16_t>, grid, block, 0, s,
                                   static_cast<const bf16_t*>(p.x), static_cast<bf16_t*>(p.grads), meta, labels, emit_blank,
                                   emit_label, sa, p.T, p.B, p.A, p.blank, p.defer + p.defer_columns);
        }
    });
}

// Narrow alphabets: do several wavefronts share a block?
static bool shares_blocks(const Launch& p)
{
    return static_cast<int64_t>(p.B) * frame_blocks(p.T) * label_pieces(p.max_label) <= kShareBlocksMost;
}
// Narrow alphabets: do the gradient's workgroups hold their emissions in LDS (narrow_tile)?  Those that wait for their chains while
// compute units are free do: it is time that they have.  And in launches of their own those of few blocks, which last as long as a block
// takes (300 x 60 x 29 24.9 us a call, from the cache 25.7; 512 x 45 x 29 27.8 and 29.1).
static bool staged_emissions(const Launch& p) { return p.fused ? p.n_chains <= p.n_cu : shares_blocks(p); }
// The gradient's workgroups: what they get, how many there are (narrow: by segment, args.segment_groups; wide: args.groups per utterance) and their LDS.
static TileArgs tile_args(const Launch& p, size_t* lds)
{
    TileArgs g{};
    g.grads = p.grads;
    g.bf16 = p.dtype != CTC_DTYPE_F32;
    g.mass = reinterpret_cast<const double*>(p.ws + p.lay.mass);
    g.chain_err = reinterpret_cast<const int*>(p.ws + p.lay.chain_err);
    g.costs = p.costs;
    g.domain = reinterpret_cast<const int*>(p.ws + p.lay.domain);
    g.links = reinterpret_cast<const int*>(p.ws + p.lay.links);
    g.done = reinterpret_cast<int*>(p.ws + p.lay.done);
    g.left = reinterpret_cast<int*>(p.ws + p.lay.left);
    g.end_polls = p.end_polls;
    g.by_end = reinterpret_cast<const int*>(p.ws + p.lay.order) + 2 * p.B;
    g.T = p.T; g.B = p.B; g.A = p.A; g.blank = p.blank;
    g.Lmax = p.max_label;
    constexpr int kWaves = kRowThreads / 64;
    const int blocks = frame_blocks(p.T);
    if (p.A <= kDirectMaxA) {
        const int shared = shares_blocks(p) ? p.B : shared_utterances(p, blocks), segments = TileArgs::kSegments;
        g.shared_from = p.B - shared;
        // (those whose blocks are shared, where others' are not, are the last segment)
        const bool apart = shared > 0 && shared < p.B;
        const int even = apart ? segments - 1 : segments, ranks = apart ? g.shared_from : p.B;
        auto lay_out = [&](const int32_t* frames_by_end) {
            uint64_t tiles = 0;
            for (int i = 0; i < segments; ++i) {
                const int first = i < even ? static_cast<int>(static_cast<int64_t>(ranks) * i / even) : ranks;
                const int end = i < even ? static_cast<int>(static_cast<int64_t>(ranks) * (i + 1) / even) : p.B;
                int frames = frames_by_end ? 0 : p.T;
                for (int r = first; frames_by_end && r < end; ++r) frames = std::max(frames, frames_by_end[r]);
                // (an utterance's blocks, and a wavefront for its cost)
                const int per_group = kWaves / (first >= g.shared_from ? block_waves(p.max_label) : 1);
                g.segment_tile[i] = static_cast<unsigned>(tiles);
                g.segment_rank[i] = first;
                g.segment_groups[i] = (frame_blocks(frames) + 1 + per_group - 1) / per_group;
                tiles += static_cast<uint64_t>(end - first) * g.segment_groups[i];
            }
            g.segment_tile[segments] = static_cast<unsigned>(tiles);
            return tiles;
        };
        const uint64_t fewer = lay_out(p.frames_by_end);
        // (a launch of its own whose workgroups are nearly as many anyway does not wait for the order first: 512 x 100 x 29 31.4 us a call with it, 30.5 without)
        if (!p.fused && !apart) {
            TileArgs by_segment = g;
            if (4 * fewer <= 3 * lay_out(nullptr)) g = by_segment;
            else g.by_end = nullptr;
        }
        *lds = static_cast<size_t>(kWaves) * tile_lds_ints(p.max_label, p.A <= 32 ? 2 : 4, staged_emissions(p)) * 4;
    } else {
        g.groups = blocks;
        g.waves = label_pieces(p.max_label) > 1 ? kWideWaves : 2;
        g.alpha_at = wide_alpha_at(p.max_label);
        *lds = wide_lds_bytes(p.max_label, g.waves);
    }
    return g;
}

int launch_lattice(const Launch& p, void* stream)
{
    // (a call whose softmax launch read the pinned image itself needs this launch for the release, chains or not)
    if (p.n_run == 0 && !(p.folded && p.host_flag)) return 0;
    auto* meta = reinterpret_cast<const Utt*>(p.ws + p.lay.meta);
    auto* order = reinterpret_cast<const int*>(p.ws + p.lay.order);
    const int* labels = p.labels;
    auto* emit_blank = reinterpret_cast<const float*>(p.ws + p.lay.emit_blank);
    auto* emit_label = reinterpret_cast<const float*>(p.ws + p.lay.emit_label);
    auto* sink = reinterpret_cast<uint32_t*>(p.ws + p.lay.sink);
    const LatticeOut lat = lattice_blocks(p);
    auto* mass = reinterpret_cast<double*>(p.ws + p.lay.mass);
    auto* chain_err = reinterpret_cast<int*>(p.ws + p.lay.chain_err);
    const size_t lds_bytes = (p.max_waves > 1 && !p.needs_barrier) ? halo_lds_bytes(p.max_waves) : 0;
    int n_groups = std::max(p.n_chains, 1);
    LaunchWords wk{};
    wk.row_flags = p.folded ? reinterpret_cast<const int*>(p.ws + p.lay.row_flags) : nullptr;
    wk.flag_blocks = (p.T + kFlagFrames - 1) / kFlagFrames;
    wk.domain = reinterpret_cast<int*>(p.ws + p.lay.domain);
    wk.done = reinterpret_cast<int*>(p.ws + p.lay.done);
    wk.host_flag = p.folded ? p.host_flag : nullptr;
    wk.host_flag_value = p.host_flag_value;
    if (p.folded && p.dev_status) {
        wk.status_words = reinterpret_cast<const int*>(p.ws + p.lay.status);
        wk.status_out = p.dev_status;
        wk.status_count = p.B;
    }
    wk.fill.n_chains = n_groups;
    if (p.defer > 0) {
        // as many workgroups per compute unit without a chain as make eight wavefronts
        const int rounds = std::max(1, 8 / p.max_waves);
        wk.fill = FillArgs{p.grads, p.dtype == CTC_DTYPE_F32 ? 4 : 2, p.T, p.B, p.A, 0, p.defer, p.n_cu, p.n_chains, rounds};
        n_groups = p.n_cu * rounds;
    }
    auto s = static_cast<hipStream_t>(stream);
    if (p.fused) {
        size_t lds;
        TileArgs tiles = tile_args(p, &lds);
        const int waves = std::max(p.max_waves, kRowThreads / 64);
        lds = std::max(lds, halo_lds_bytes(waves));
        wk.late_percent = p.late_percent;
        tiles.first_group = n_groups;
        const dim3 grid(n_groups + tiles.segment_tile[TileArgs::kSegments]), block(64 * waves);
#define CTC_LAUNCH_FUSED(SYNC, TILES, LEAN, STAGED)                                                \
    hipLaunchKernelGGL((ctc_lattice_gradient_kernel<SYNC, TILES, LEAN, STAGED>), grid, block, lds, s, meta, order, labels, emit_blank,   \
                       emit_label, lat, mass, p.costs, chain_err, sink, wk, tiles)
#define CTC_LAUNCH_FUSED_TILES(SYNC, LEAN, STAGED)                                                 \
    do {                                                                                           \
        if (p.A <= 32) CTC_LAUNCH_FUSED(SYNC, 2, LEAN, STAGED);                                    \
        else CTC_LAUNCH_FUSED(SYNC, 4, LEAN, STAGED);                                              \
    } while (0)
        return checked_launch([&] {
            if (!staged_emissions(p) && p.max_waves == 1) CTC_LAUNCH_FUSED_TILES(Sync::kNone, true, false);
            else if (!staged_emissions(p)) CTC_LAUNCH_FUSED_TILES(Sync::kHalo, true, false);
            else if (p.max_waves > kRowThreads / 64 && p.A <= 32) CTC_LAUNCH_FUSED(Sync::kHalo, 2, true, true);
            else if (p.max_waves == 1) CTC_LAUNCH_FUSED_TILES(Sync::kNone, false, true);
            else CTC_LAUNCH_FUSED_TILES(Sync::kHalo, false, true);
        });
#undef CTC_LAUNCH_FUSED_TILES
#undef CTC_LAUNCH_FUSED
    }
    if (p.mode == Mode::kLoss && !p.needs_barrier) {
        wk.norm_groups = n_groups;
        wk.utterances = p.B;
        n_groups += (p.B + p.max_waves - 1) / p.max_waves;
    }
    const dim3 grid(n_groups), block(64 * p.max_waves);
#define CTC_LAUNCH_LATTICE(KERNEL)                                                                 \
    hipLaunchKernelGGL(KERNEL, grid, block, lds_bytes, s, meta, order, labels, emit_blank,                 \
                       reinterpret_cast<const double*>(p.ws + p.lay.emit_blank64), emit_label,            \
                       lat, mass, p.costs, chain_err, sink, wk)
#define CTC_LAUNCH_LATTICE_KERNEL(KERNEL)                                                           \
    do {                                                                                           \
        if (p.mode == Mode::kLoss) CTC_LAUNCH_LATTICE((KERNEL<Mode::kLoss>));                      \
        else if (p.mode == Mode::kBest) CTC_LAUNCH_LATTICE((KERNEL<Mode::kBest>));                 \
        else CTC_LAUNCH_LATTICE((KERNEL<Mode::kGrad>));                                            \
    } while (0)
    return checked_launch([&] {
        // (measurements: the two recursions one after the other, forward chains first, as two launches)
        for (int pass = 0; pass < (p.sequential_chains ? 2 : 1); ++pass) {
            wk.skip_directions = p.sequential_chains ? (pass == 0 ? 2 : 1) : 0;
            if (p.max_waves == 1) CTC_LAUNCH_LATTICE_KERNEL(ctc_lattice_kernel_w1);
            else if (!p.needs_barrier) CTC_LAUNCH_LATTICE_KERNEL(ctc_lattice_kernel);
            else CTC_LAUNCH_LATTICE_KERNEL(ctc_lattice_kernel_barrier);
        }
    });
#undef CTC_LAUNCH_LATTICE_KERNEL
#undef CTC_LAUNCH_LATTICE
}

int launch_backtrace(const Launch& p, void* stream)
{
    auto* meta = reinterpret_cast<const Utt*>(p.ws + p.lay.meta);
    auto* chain_err = reinterpret_cast<const int*>(p.ws + p.lay.chain_err);
    return checked_launch([&] {
        const int segments = std::max(1, (chain_chunks(p.max_frames, false) + kSegmentChunks - 1) / kSegmentChunks);
        const int64_t words = static_cast<int64_t>(segments) * (p.max_label + 1);
        const int lds_words = static_cast<int>(std::min<int64_t>(words, kOriginWords));
        hipLaunchKernelGGL(ctc_backtrace_kernel, dim3(p.B, 2), dim3(64 * std::min(segments, kBacktraceWaves)), lds_words * 4,
                           static_cast<hipStream_t>(stream), meta, p.labels, lattice_blocks(p), chain_err, p.costs, p.alignment, p.T, lds_words);
    });
}

int launch_gradient(const Launch& p, void* stream)
{
    auto* meta = reinterpret_cast<const Utt*>(p.ws + p.lay.meta);
    auto* emit_blank = reinterpret_cast<const float*>(p.ws + p.lay.emit_blank);
    auto* emit_label = reinterpret_cast<const float*>(p.ws + p.lay.emit_label);
    auto s = static_cast<hipStream_t>(stream);
    size_t lds;
    const TileArgs args = tile_args(p, &lds);
    FillArgs fill{};
    if (p.defer_columns > 0) {
        // (a workgroup to a compute unit; twice and four times as many 0.5 % slower)
        fill = FillArgs{p.grads, p.dtype == CTC_DTYPE_F32 ? 4 : 2, p.T, p.B, p.A, p.defer, p.defer_columns, p.n_cu, p.n_chains, std::max(1, p.n_cu / p.B)};
    }
#define CTC_LAUNCH_NARROW(STAGED)                                                                  \
    do {                                                                                           \
        if (p.A <= 32)                                                                             \
            hipLaunchKernelGGL((ctc_gradient_narrow_kernel<2, STAGED>), grid, block, lds, s, args, meta, p.labels, emit_blank, emit_label, lattice_blocks(p)); \
        else                                                                                       \
            hipLaunchKernelGGL((ctc_gradient_narrow_kernel<4, STAGED>), grid, block, lds, s, args, meta, p.labels, emit_blank, emit_label, lattice_blocks(p)); \
    } while (0)
    const WideRows rows = p.A > kDirectMaxA ? wide_rows(args.groups + fill.rounds) : WideRows{1, 1};
    const unsigned tiles = args.segment_tile[TileArgs::kSegments], across = std::min(std::max(tiles, 1u), 1u << 20);
    const dim3 narrow = args.by_end ? dim3(across, (tiles + across - 1) / across) : dim3(args.segment_groups[0], p.B);
    const dim3 grid = p.A > kDirectMaxA ? dim3(p.B, rows.y, rows.z) : narrow, block(p.A > kDirectMaxA ? 64 * args.waves : kRowThreads);
    return checked_launch([&] {
        if (p.A > kDirectMaxA && p.defer_columns > 0)
            hipLaunchKernelGGL(ctc_gradient_wide_kernel<true>, grid, block, lds, s, args, meta, p.labels, emit_blank, emit_label,
                               lattice_blocks(p), fill);
        else if (p.A > kDirectMaxA)
            hipLaunchKernelGGL(ctc_gradient_wide_kernel<false>, grid, block, lds, s, args, meta, p.labels, emit_blank, emit_label,
                               lattice_blocks(p), fill);
        else if (staged_emissions(p)) CTC_LAUNCH_NARROW(true);
        else CTC_LAUNCH_NARROW(false);
    });
#undef CTC_LAUNCH_NARROW
}

}  // namespace ctc
