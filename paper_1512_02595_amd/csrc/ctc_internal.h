// Internal interfaces between the host launcher and the HIP kernels of the CTC library.
// Not part of the public ABI (that is include/ctc_mi355x.h).
#pragma once

#include <cstddef>
#include <algorithm>
#include <cstdint>
#include <type_traits>
#include <vector>

#include "ctc_mi355x.h"

namespace ctc {

// Per-utterance record, identical on host and device (64 bytes).
struct Utt {
    int32_t Tb;        // frames of this utterance (input_lengths[b])
    int32_t L;         // label length
    int32_t lab_off;   // offset of its label string in the flat label array
    int32_t flags;     // bit 0: the lattice runs (Tb > 0 and an alignment exists);
                       // bit 1: lengths or labels failed the device-side checks (cost NaN)
    uint32_t f_off;    // padded frames (padded_frames) of all earlier utterances: offset of its blank emissions
    int32_t waves;     // wavefronts its lattice chains use when a lane owns one state pair (log-domain
                       // chains, and linear-domain chains of at most 64 pairs)
    int32_t halo;      // lanes per wavefront that recompute the wavefront below (0: none)
    int32_t poll_budget; // LDS polls a wavefront of its chains may spend waiting on a neighbour before it gives up
    int64_t e_off;     // offset (floats) of its label emissions [chunk][e_cols][kChunk]
    int64_t ab_off;    // offset (8-byte words) of its alpha/beta blocks, lattice_words of them
    int32_t e_cols;    // columns of its emission block: a column per symbol, or one per label position
    int16_t e_direct;  // which of the two: kEmitGathered or kEmitSymbols (emission_layout)
    int8_t rough;      // set by the softmax launch when some probability is below 2^kGentleMinLog2
    int8_t steep;      // ... below 2^kRoughMinLog2
    int32_t waves2;    // the same plan for linear-domain chains of more than 64 pairs, whose lanes own
    int32_t halo2;     // two neighbouring pairs each (plan_waves2)
};
static_assert(sizeof(Utt) == 64, "Utt is copied word by word and read with scalar loads: keep it 8-byte sized");

// Alphabets up to this size skip the emission gather: a frame's normalised row is as small as
// the gathered emissions would be, and the rows themselves are the emission block (emission_layout).
constexpr int kDirectMaxA = 64;
constexpr int kByteLabelsMaxA = 256;  // alphabets up to this size: the labels travel to the GPU as bytes
constexpr int kDeviceFoldMaxB = 512;  // device-resident metadata: utterances up to which the narrow softmax launch builds the records
constexpr int kNarrowMaxB = 128;      // utterances whose frame counts travel in the narrow softmax launch's arguments
constexpr int kFlagFrames = 64;       // frames per word of Layout::row_flags = frames per workgroup of the narrow softmax launch

#if defined(__HIPCC__)
#define CTC_HOST_DEVICE __host__ __device__
#else
#define CTC_HOST_DEVICE
#endif

constexpr int kChunkSteps = 8;        // = kChunk (below): steps between two possible hand-overs

// How the L+1 state pairs of a chain are spread over wavefronts.
struct WavePlan {
    int waves;
    int halo;
    bool barrier;      // too long for a halo: 64 pairs per wavefront, one barrier per step
};

// Wavefronts and halo width for a label of this length.  Fitted to log-domain chains on gfx950: with one
// wavefront per SIMD (up to 4) a step costs about 210 clocks and a hand-over about 500; with
// several per SIMD the vector ALU is the limit (about 170 clocks per wavefront-step) and part
// of a hand-over's latency hides behind the other wavefronts (about 350).  (The linear domain's steps, which share the plans, take 35 to 60
// clocks at most a wavefront to a SIMD, 45 to 85 with all that comes at the ends of blocks: its plans have not been fitted to that.)
// (Host and device: the launcher plans on the host, the device-metadata entry point on the GPU.)
// `crowded`: the launch has more wavefronts than the chip runs side by side at one per SIMD, so
// what counts is the total work (wavefront-steps plus hand-overs), not one chain's latency.
CTC_HOST_DEVICE inline WavePlan plan_waves(int label_length, bool crowded = false)
{
    const int pairs = label_length + 1;
    if (pairs <= 64) return {1, 0, false};
    // Hand-overs happen on chunk boundaries: the halo is a multiple of kChunk (8 .. 32), and
    // the lanes handed up must themselves be exact ones (halo <= 64 - halo).
    WavePlan best{16, 0, true};
    float best_cost = 1e30f;
    const int w0 = (pairs - 8 + 55) / 56;       // fewest wavefronts with a halo of 8: w * 56 + 8 >= pairs
    for (int w = w0; w <= 16 && w <= w0 + 4; ++w) {
        // w * (64 - halo) + halo >= pairs
        int halo = (64 * w - pairs) / (w - 1);
        if (halo > 32) halo = 32;
        halo -= halo % 8;
        if (halo < 8) continue;
        const int per_simd = (w + 3) / 4;
        // the last term prefers fewer wavefronts when the estimates are close
        const float cost = crowded ? w * (170.0f + 350.0f / halo)
                                   : ((per_simd == 1) ? 210.0f + 500.0f / halo : per_simd * 170.0f + 350.0f / halo) + 4.0f * w;
        if (cost < best_cost) {
            best_cost = cost;
            best = {w, halo, false};
        }
    }
    return best;
}

// The same for chains whose lanes own two neighbouring state pairs each (linear domain, more than
// 64 pairs).  A wavefront then covers 128 pairs, an error at lane 0 needs two steps per lane to
// move up, so a halo of h lanes lasts 2h steps: h is a multiple of 4 (hand-overs on chunk
// boundaries), at most 16 (the exchange buffer).  Sixteen wavefronts hold any supported label.
// Fitted when a step took about 150 clocks with one wavefront per SIMD and a hand-over 600 (they take about 75, 35 ns, now).
CTC_HOST_DEVICE inline WavePlan plan_waves2(int label_length, bool crowded = false)
{
    const int lanes = (label_length + 2) / 2;          // ceil((L + 1) / 2)
    if (lanes <= 64) return {1, 0, false};
    WavePlan best{16, 4, false};
    float best_cost = 1e30f;
    // Fewest wavefronts with a halo of 4: w * 60 + 4 >= lanes.  The halo reaches its cap of 16 within
    // three more wavefronts (lanes / 48 against lanes / 60, lanes <= 512), and beyond that a further
    // wavefront only costs: no need to look further (the device-side planners run this per utterance).
    const int w_first = (lanes - 4 + 59) / 60 > 2 ? (lanes - 4 + 59) / 60 : 2;
    for (int w = w_first; w <= 16 && w <= w_first + 3; ++w) {
        // w * (64 - halo) + halo >= lanes
        int halo = (64 * w - lanes) / (w - 1);
        if (halo > 16) halo = 16;
        halo -= halo % 4;
        if (halo < 4) continue;
        const int per_simd = (w + 3) / 4;
        const float cost = crowded ? w * (110.0f + 300.0f / halo)
                                   : ((per_simd == 1) ? 150.0f : per_simd * 110.0f) + 300.0f / halo + 4.0f * w;
        if (cost < best_cost) {
            best_cost = cost;
            best = {w, halo, false};
        }
    }
    return best;
}

// Which of the two plans a linear-domain chain uses.  A step of a two-pair lane takes half as long again as one of a one-pair lane (180
// clocks against 120 when this was fitted, 12 instructions against 7 now), so while a
// label's one-pair plan keeps to one wavefront per SIMD (at most 4) it is the faster one; beyond
// that, and in crowded launches, where wavefront-steps count and not one chain's latency, the
// two-pair plan with half the wavefronts wins.  Where the emission block holds the symbols' rows
// (kEmitSymbols) a two-pair lane's fetches are cheap, and the two-pair plan also wins against
// a one-pair plan that hands over every chunk (halo 8): 64 utterances of 600 frames, lattice
// launch for labels of 215 symbols 52.1 -> 46.5 us, of 230 symbols 52.9 -> 50.1 us; up to 207
// symbols (halo 16 or more) the one-pair plan stays ahead by up to 4 us.
CTC_HOST_DEVICE inline bool two_pairs_per_lane(int label_length, bool crowded, bool symbol_major = false)
{
    if (label_length + 1 <= 64) return false;
    const WavePlan one = plan_waves(label_length, crowded);
    return crowded || one.barrier || one.waves > 4 || (symbol_major && one.halo < 2 * kChunkSteps);
}

// Linear-domain chains hand over at the ends of blocks of 16 frames.  A two-pair plan whose halo lasts for 8 frames only takes
// one more wavefront; of the one-pair plans, those are never chosen (linear_two_pairs).
CTC_HOST_DEVICE inline WavePlan linear_plan2(int label_length, bool crowded)
{
    WavePlan p = plan_waves2(label_length, crowded);
    if (p.waves > 1 && p.halo < kChunkSteps) {
        const int lanes = (label_length + 2) / 2, halo = (64 * (p.waves + 1) - lanes) / p.waves;
        p.halo = halo > 16 ? 16 : halo - halo % 4;
        p.waves += 1;
    }
    return p;
}
CTC_HOST_DEVICE inline bool linear_two_pairs(int label_length, bool crowded) { return two_pairs_per_lane(label_length, crowded, true); }

// The plans of every label length, packed: what a launch that builds its utterance records on the
// GPU carries in its arguments instead of evaluating plan_waves per utterance there.
//   one[L]: bits 0..3 wavefronts - 1, bits 4..6 halo / 8 (plan_waves), bit 7 two_pairs_per_lane
//   two[L]: bits 0..3 wavefronts - 1, bits 4..6 halo / 4 (plan_waves2)
struct PlanTable {
    uint8_t one[CTC_MAX_LABEL_LENGTH + 1];
    uint8_t two[CTC_MAX_LABEL_LENGTH + 1];
    CTC_HOST_DEVICE int waves1(int L) const { return (one[L] & 15) + 1; }
    CTC_HOST_DEVICE int halo1(int L) const { return ((one[L] >> 4) & 7) * 8; }
    CTC_HOST_DEVICE bool two_pairs(int L) const { return (one[L] & 128) != 0; }
    CTC_HOST_DEVICE int waves2(int L) const { return (two[L] & 15) + 1; }
    CTC_HOST_DEVICE int halo2(int L) const { return (two[L] >> 4) * 4; }
};
// The plans of every supported label length, evaluated once per process: a call looks its utterances up
// (evaluating plan_waves and plan_waves2 for each utterance of a 512-utterance minibatch was most of the
// launcher's 130 us).
struct Plans {
    PlanTable table[2];                                         // [crowded]
    uint8_t latency_waves[CTC_MAX_LABEL_LENGTH + 1];            // wavefronts of a linear-domain chain planned for latency
    int latency_waves_up_to[CTC_MAX_LABEL_LENGTH + 1];          // ... summed over all lengths up to this one
    uint8_t most_waves[2][CTC_MAX_LABEL_LENGTH + 1];            // [crowded]: most wavefronts of any plan for a label up to this length
    bool barrier[CTC_MAX_LABEL_LENGTH + 1];                     // WavePlan::barrier
};
const Plans& plans();

// How a launch's label emissions are laid out: [chunk][column][frame of the chunk], kChunk frames of a column side
// by side, so that a lane fetches what it needs of a chunk in two 16-byte loads.  The columns (Utt::e_direct) are
//   kEmitGathered: the label's positions (alphabets above kDirectMaxA): neighbouring lanes read neighbouring columns;
//   kEmitSymbols:  the symbols: the normalised rows themselves; a chunk of 29 symbols is 928 bytes, eight lines for the
//                  64 lanes of a fetch to meet in.  (With a row per symbol over all frames every lane asked for a line
//                  of its own, and the wavefronts of a compute unit queued for its L1.)
// Blocks cover whole blocks of kBlockFrames frames.  Past an utterance's last frame they hold virtual frames in which
// blank has probability 1 and every label 0: the start state of either recursion (its first blank has all the mass)
// goes through them unchanged, and after its last frame the forward recursion merely gathers p in the last blank.
// Chains thus consist of whole chunks on one grid in both directions.
constexpr int kEmitGathered = 0, kEmitSymbols = 1;
CTC_HOST_DEVICE inline int emission_layout(int A) { return A <= kDirectMaxA ? kEmitSymbols : kEmitGathered; }

// Frames between two states that a chain stores for the gradient (checkpoints): see block_shares.
constexpr int kBlockFrames = 2 * kChunkSteps;
CTC_HOST_DEVICE inline int frame_blocks(int frames) { return (frames + kBlockFrames - 1) / kBlockFrames; }
CTC_HOST_DEVICE inline int64_t padded_frames(int frames) { return static_cast<int64_t>(frame_blocks(frames)) * kBlockFrames; }

// Alphabets above kDirectMaxA: of every 16 frames, how many leave their zero rows (padding, utterances without an
// alignment) to the lattice launch, whose compute units without a chain would idle: as many as fit in the time of
// its longest chain.  `zero_bytes`: of all zero rows.
constexpr double kFillBytesPerUs = 3.0e6;      // what the idle half of the chip writes beside the chains
constexpr double kChainUsPerFrame = 0.045;     // the quickest chains when this was fitted (one wavefront; 0.018 now)
inline int deferred_frames(double zero_bytes, int longest, int n_chains, int n_cu)
{
    if (n_chains + n_cu / 4 > n_cu || zero_bytes <= 0) return 0;
    const double fits = kFillBytesPerUs * kChainUsPerFrame * longest * (n_cu - n_chains) / (n_cu / 2);
    return static_cast<int>(std::min(16.0, 16.0 * fits / zero_bytes));
}

// ... and how many more leave theirs to the label columns' launch, which moves little and waits for its slowest block: about
// kFillBesideColumns bytes.  (us a call without, with 1, 2, 3, 4 and 6 sixteenths of the frames: 64 x 500 x 6000, 308 MB of zero rows,
// 253.4 / 252.4 / 250.2 / 253.0 / 253.2 / 252.9; bf16 145.2 / 145.2 / 144.6 / 143.6 / 143.5 / 146.9; 64 x 500 x 4096
// 167.9 / 167.6 / 165.1 / 163.2 / 163.6 / 166.8; 200 x 150 x 5000 204.8 / 203.1 / 201.5 / 200.1 / 199.8 / 201.7.)
// Tensors with less than kFillBesideColumnsFrom of them leave none: us a call without / with, 42 MB (176 x 68 x 2051) 44.4 / 50.2, 40 (100 x
// 100 x 5000 bf16) 44.0 / 47.7, 54 (64 x 160 x 3000) 47.3 / 47.1, 61 (64 x 180 x 3000) 51.1 / 51.6, 69 (64 x 200 x 3000) 56.4 / 53.7, 77 (64 x
// 250 x 3000) 68.8 / 65.1, 79 (33 x 200 x 7999) 71.4 / 68.7, 80 (100 x 100 x 5000) 68.4 / 66.5.
constexpr double kFillBesideColumns = 40.0e6, kFillBesideColumnsFrom = 60.0e6;
// Rows of 2048 symbols and less take a wavefront of its own too long for that (512 x 300 x 100: 102.8 us without, 126.6 with).
constexpr int kFillBesideColumnsMinA = 2048;
inline int columns_frames(double zero_bytes, int A, int deferred)
{
    if (zero_bytes < kFillBesideColumnsFrom || A <= kFillBesideColumnsMinA) return 0;
    return static_cast<int>(std::min(16.0 - deferred, 16.0 * kFillBesideColumns / zero_bytes + 0.5));
}

// A number that the GPU divides by, up to 2^31, and what makes its quotients of numbers below 2^31 a product, a sum and a shift: with
// s = ceil(log2 by) and m = floor(2^32 (2^s - by) / by) + 1, n / by = (floor(n m / 2^32) + n) >> s.
struct Divisor {
    unsigned by, magic, shift;
    explicit Divisor(int divisor) : by(static_cast<unsigned>(divisor)), magic(0), shift(0)
    {
        while ((uint64_t(1) << shift) < by) ++shift;
        magic = static_cast<unsigned>((((uint64_t(1) << shift) - by) << 32) / by + 1);
    }
    CTC_HOST_DEVICE unsigned quotient(unsigned n) const { return (static_cast<unsigned>((static_cast<uint64_t>(n) * magic) >> 32) + n) >> shift; }
};

// That launch has the utterances in its grid's first dimension and `rows`, as many as an utterance of a million and more frames has
// blocks, in the other two, which take kMaxGridRows each.
constexpr int kMaxGridRows = 65535;
struct WideRows { int y, z; };
inline WideRows wide_rows(int rows)
{
    const int z = (rows + kMaxGridRows - 1) / kMaxGridRows;
    return {(rows + z - 1) / z, z};
}

// The gradient's recomputation takes a label in pieces of 128 positions, one to a wavefront, whose inner edges overlap by the
// frames of a block on either side.
constexpr int kPiecePositions = 128, kPieceHalo = kBlockFrames, kPieceStep = kPiecePositions - 2 * kPieceHalo;
CTC_HOST_DEVICE constexpr int label_pieces(int L)
{
    return L <= kPiecePositions ? (L > 0 ? 1 : 0) : (L - kPiecePositions + kPieceStep - 1) / kPieceStep + 1;
}

// The gradient of an utterance may be written by workgroups of the lattice launch that wait for its chains (Launch::fused).
// Chains that need more wavefronts than a workgroup of that launch has keep a launch of their own: with sixteen, 128 registers
// a lane remain, and labels of up to 900 symbols, which would need them, ran up to 60 % longer beside their chains than apart
// (64 utterances of 2000 frames); with eight, labels of 470 symbols and more could not use what it saves for 32 utterances of
// 1500 frames (540 symbols: 169.4 us apart, 157.6 beside).
constexpr int kFusedWaves = 12;
constexpr int kCrowdedFusedWaves = 8;    // ... where there are more chains than compute units
// The workgroups of that launch, all in the grid's first dimension, have fewer than 2^32 threads together; a gradient launch of its own has
// the utterances in the second.  (At worst a workgroup to a block of frames and one more to an utterance: from 512 utterances of 524 000 frames on,
// with labels of up to four wavefronts, the launches are apart.)
constexpr bool fused_grid_fits(int T, int B, int max_waves, int n_chains)
{
    const int64_t workgroups = n_chains + (static_cast<int64_t>(T) / kBlockFrames + 2) * B;
    return workgroups * 64 * std::max(max_waves, 4) < int64_t(1) << 32;
}
constexpr bool can_fuse_gradient(int A, int max_waves, int n_chains, int n_cu, int T, int B)
{
    return A <= kDirectMaxA && max_waves <= (n_chains <= n_cu ? kFusedWaves : kCrowdedFusedWaves) && fused_grid_fits(T, B, max_waves, n_chains);
}
// Whether that pays where a chain has more than eight wavefronts and a compute unit of its own.  Beside the chains, the compute units without one write
// the gradient of the utterances that end before the longest (`early`; `late`: whose chains end in the last 15 % of the time) and a launch boundary is
// saved.  But what is left at the end is written by fewer workgroups at a time than in a launch of its own, since they are as large as the chains' ones:
// one or two to a compute unit.  `early` and `late` are blocks of frames
// times pieces of the label, a third of a microsecond on the whole chip for every compute unit; `chain_us`: the longest chain.
// Fitted, before the chains' checkpoints went past the caches, to batches of 32 to 128 utterances with labels of up to 660 symbols: 128
// utterances of 1275 to 1500 frames, labels of 400 to 660, 294 us a call apart and 468 beside; 64 of 300 to 1500, labels of 360 to 600, 182 and 155; 32 of
// 1500 frames, labels of up to 540, 169.6 and 157.6.
inline bool gradient_beside_long_chains(double early, double late, double chain_us, int n_chains, int n_cu)
{
    const double busy = static_cast<double>(n_chains) / n_cu, saved = std::min(std::max(chain_us / 8, 2.0), 10.0);
    return 1.5 * late / n_cu + 18.0 * busy <= saved + 0.4 * early / n_cu * (1.0 - busy);
}
// What a chain of this many wavefronts took for a frame, in microseconds, when the rule above was fitted (up to four run on a SIMD each).
// The steps of a linear-domain chain take about half of that now, 0.019, 0.023 to 0.035 and 0.055; the rule divides by these.
inline double chain_us_per_frame(int waves) { return waves == 1 ? 0.045 : (waves <= 4 ? 0.06 : 0.088); }

// The rule that launches follow.  Random batches, three of a kind in turn:
// Up to a chain per compute unit, up to eight wavefronts: beside (87 batches: 0.79 to 0.97 of the time apart; 128 x 454 x 29 36.3 us a
// call apart, 32.3 beside; 64 x 750 x 60, lengths from 600 on, 72.0 and 65.4).
// More chains than compute units, up to four wavefronts: beside while all of them start together, four workgroups to a compute unit (51 batches: 0.83 to
// 1.01 of the time apart, in the mean 0.93; 512 x 750 x 29 127.3 apart, 115.5 beside).  Beyond it 51 batches took 0.85 to 1.18, in the mean 1.02.
// More wavefronts, two workgroups to a compute unit: up to 2.75 chains to one, and at least half of the work early (11 batches: 0.88 to 1.00,
// in the mean 0.95; seven others 0.87 to 1.08, 1.01).
// Chains of up to 100 frames keep to the launch apart: blocks that wait for them are most of such a launch (22 batches: 0.91 to 1.11, in the
// mean 0.98).
constexpr int kCrowdedBesideFrames = 100;
// Does the answer depend on `early`, `late` and `chain_us`?  (Adding them up takes the host a microsecond for 512 utterances.)
inline bool beside_by_work(int max_waves, int n_chains, int n_cu) { return max_waves > (n_chains > n_cu ? 4 : 8); }
inline bool gradient_in_lattice_launch(double early, double late, double chain_us, int max_frames, int max_waves, int n_chains, int n_cu)
{
    if (n_chains > n_cu)
        return max_frames > kCrowdedBesideFrames && (beside_by_work(max_waves, n_chains, n_cu) ? 4 * n_chains <= 11 * n_cu && late <= early : n_chains <= 4 * n_cu);
    return !beside_by_work(max_waves, n_chains, n_cu) || gradient_beside_long_chains(early, late, chain_us, n_chains, n_cu);
}

// Narrow alphabets, gradients whose blocks are not all shared by several wavefronts: of how many blocks times pieces, at most, those are which are, in the utterances that end last.
// By then compute units are free, and a label of five pieces keeps one wavefront to a block for 18 us after its chains have ended: us a call with none / 1024 / 2048 / 4096 / 8192,
// 32 x 1500 x 29 122.1 / 118.7 / 109.9 / 109.8 / 109.5 (logits tripled: 2048 563, 8192 526); the same, lengths from 400 on, 119.3 / 107.5 / 108.2 / 107.7 / 108.0; 128 x 750 x 29 48.5 / 45.7 /
// 45.1 / 44.7 / 44.8; 128 x 768 x 29 with 0.3 symbols a frame 56.2 / 50.2 / 49.5 / 51.5 / 53.9.  With four tiles of symbols in place of two a shared block has twice as much to add up:
// 32 x 1500 x 60 134.6 / 134.1 / 129.4 / 137.1 / 148.7; 128 x 750 x 40 52.1 / 50.9 / 52.4 / 53.1 / 55.1; 128 x 768 x 37 with 0.3 symbols a frame 59.3 / 56.0 / 58.3 / 61.9 / 69.1.
// None where those that end in the last 15 % of the time have more than the chip has places for wavefronts (`late`, in blocks times pieces; the batches above have up to 3000): then a shared block
// only costs more places.  64 utterances of 750 frames and 225 symbols 61.8 / 62.5 / 64.3 / 67.3 / 72.3, 128 of them 82.1 / 81.9 / 84.3 / 86.6 / 92.6, 32 of 1500 frames and 540 symbols 152.7 /
// 157.1 / 157.3 / 166.8 / 166.1 (48 of 1500 and 400 116.5 / 116.6 / 116.4 / 118.0 / 119.9; 64 of 900 and 400 94.5 / 88.6 / 88.8 / 90.5 / 91.0).
// With more chains than compute units, whose blocks are still under way: 512 x 750 x 29 105.7 / 104.8 / 104.6 / 106.0 / 107.0; where lengths are not known here (late < 0):
// 100 x 1000 x 29 67.7 / 64.8 / 61.2 / 61.9 / 66.5, 64 x 750 with labels of up to 270 symbols 68.0 / 66.9 / 66.9 / 70.5 / 70.5.
constexpr int kShareLast = 4096, kShareSome = 2048, kLateFillsChip = 4096;
inline int blocks_to_share(int64_t late, int A, int n_chains, int n_cu)
{
    if (n_chains > n_cu || late < 0) return kShareSome;
    return late > kLateFillsChip ? 0 : (A <= 32 ? kShareLast : kShareSome);
}

constexpr int kDoneStride = 16;      // words between two utterances' words: a line each for those who poll
constexpr int kTakenWord = 1;        // which of them says that the chains have a workgroup (take_chain; the first is the counter)
constexpr int kDoneWords = 2;
constexpr int kMassWords = 4;        // doubles per utterance that its forward chain leaves (see the kernels)

// The sink of a lattice launch: for each of its up to 2 B chain workgroups, kSinkBytes for each of the
// up to kSinkWaves wavefronts.
constexpr int kSinkWaves = 16, kSinkBytes = 64;

constexpr int kUttRuns = 1;
constexpr int kUttInvalid = 2;
// Set by the softmax launch when some emission of the utterance is too improbable for the
// linear-domain recursion (below 2^kLinearMinLog2): its chains then run in the log domain.
// (Also set for every utterance of a launch that uses the one-barrier-per-step kernel.)
constexpr int kUttLogDomain = 4;
// Linear-domain chains of this utterance give two neighbouring state pairs to every lane
// (plan_waves2) instead of one (plan_waves): see two_pairs_per_lane.
constexpr int kUttTwoPairs = 8;
constexpr float kLinearMinLog2 = -100.0f;
// Chains of the linear domain look after their lanes' exponents once a chunk of 8 frames where all probabilities of the utterance
// are above the second of these, in a wider range where they are above the first, and every kSteepSteps frames otherwise.
constexpr float kGentleMinLog2 = -32.0f, kRoughMinLog2 = -79.0f;
constexpr int kSteepSteps = 4;
constexpr int kRowsSmall = 1, kRowsRough = 2, kRowsSteep = 4;    // bits of Layout::row_flags: one below kLinearMinLog2, kGentleMinLog2, kRoughMinLog2
// What an utterance's chains publish (Layout::domain): words for every frame, or checkpoints, whose blocks are recomputed with a look at
// the exponents every kSteepSteps frames or every chunk.
constexpr int kDomainLog = 1, kDomainSteep = 2;
// Utterances of more frames than this run the log domain whatever their emissions: the lanes'
// exponents, which fall or rise by up to 100 per frame, must stay clear of kNoExponent and of int32's end.
constexpr int kLinearMaxFrames = 1 << 21;
// Utterances with fewer than this many frames to spare (frames - symbols - repeated neighbours) run the log
// domain too.  Where hardly a frame is to spare the alignments run along the front of the lattice, and the
// states behind the front, whose mass can no longer reach the end, may outweigh it by more than the lanes'
// frames of the linear domain hold (lane_frame in the kernels: 2^760 within nine state pairs, or five); with this
// many frames to spare every state that near the front can still reach the end.  Measured before the rule:
// 138 frames, 91 symbols, 47 repeats, emissions down to 2^-95: the front 2^1900 below its neighbours, the
// linear domain's cost +inf.
constexpr int kTightFrames = 16;
CTC_HOST_DEVICE inline bool tight_fit(int frames, int label_length, int repeats)
{
    return frames - label_length - repeats < kTightFrames;
}
// Where pair j of a linear-domain chain finds its label state's emissions, in bytes from the chunk's first (`column`: the symbol, or the position where they are gathered).  Pairs
// from L on have none: past the end of the buffer, whose loads give 0 there.
constexpr unsigned kNoColumn = 0x80000000u;
CTC_HOST_DEVICE inline unsigned emission_column(int j, int L, int column)
{
    return j < L ? static_cast<unsigned>(column) * static_cast<unsigned>(kChunkSteps * sizeof(float)) : kNoColumn;
}

// Lattice wavefronts of one launch beyond which chains are planned for total work: two per SIMD
// of the 256 compute units.
constexpr int kCrowdedWaves = 2 * 4 * 256;
// How an utterance's chains run, for its weight: on probabilities with a pair to a lane or two, on logarithms, or as the best alignment's.
enum class ChainForm { kOnePair, kTwoPairs, kLogs, kBest };
CTC_HOST_DEVICE inline ChainForm chain_form(int flags, bool best)
{
    if (best) return ChainForm::kBest;
    return (flags & kUttLogDomain) ? ChainForm::kLogs : ((flags & kUttTwoPairs) ? ChainForm::kTwoPairs : ChainForm::kOnePair);
}
// What an utterance weighs in the orders of chains and of ends: how long its chains take, a frame's time in ns (the difference between 1500 frames and 750, alone on the chip),
// where a chain has SIMDs of its own; in crowded launches, where what counts is how much they keep SIMDs busy, frames times wavefronts.  (By frames times wavefronts throughout,
// an utterance of two wavefronts with two pairs to a lane, which lasts longest, was taken to end early.)  Measured with 1 / 2 / 3 / 4 / 5 and 6 / 7 and 8 / 10 to 12 wavefronts:
// one pair 20 / 23 / 22 / 22 to 26 (rough utterances 20 / 25 / 25 / 28 to 30); two pairs - / 31 / 31 / 31 / 55; logarithms 101 / 109 / 111 / 115 / 197 / 196 / 287; alignments 51 / 59 / 60 / 65 / 87 / 89 / 120.
CTC_HOST_DEVICE inline int64_t chain_weight(int frames, int waves, ChainForm form, bool crowded)
{
    const int up_to_four = waves < 4 ? waves : 4, per_simd = (waves + 3) / 4;
    int per_frame = (0x1A171714 >> (8 * up_to_four - 8)) & 255;        // 20, 23, 23, 26
    if (form == ChainForm::kTwoPairs) per_frame = waves <= 4 ? 31 : 55;
    if (form == ChainForm::kLogs) per_frame = 97 * per_simd + (waves <= 4 ? 4 * waves : 0);
    if (form == ChainForm::kBest) per_frame = waves <= 4 ? 47 + 5 * waves : 20 + 34 * per_simd;
    return static_cast<int64_t>(frames) * (crowded ? waves : per_frame);
}
CTC_HOST_DEVICE inline int64_t chain_weight(const Utt& m, bool best, bool crowded)
{
    const ChainForm form = chain_form(m.flags, best);
    return chain_weight(m.Tb, form == ChainForm::kTwoPairs ? m.waves2 : m.waves, form, crowded);
}
// The order in which the lattice launch takes its chains (entry = utterance * 2 + direction).
// `utt`: the utterances whose lattice runs, heaviest (chain_weight) first; `dirs`: 2 when
// the backward chains run too.  Up to `n_cu` chains (one per compute unit) keep that order.
// Beyond that, chains share compute units, and the launch lasts as long as the busiest SIMD:
// a chain's wavefront nearly fills the SIMD it runs on, so two on one SIMD take the sum of
// their times.  The workgroup dispatcher, as observed on gfx950, hands workgroup i to compute
// unit i mod n_cu and, on a compute unit, starts each further workgroup one SIMD later than
// the one before it.  The order is therefore built in rounds of n_cu workgroups that follow
// the SIMDs' loads under that model: a round whose wavefronts land on SIMDs busier than the
// compute units' average takes the lightest chains left, any other the heaviest, and within
// a round the lightest chain goes to the compute unit whose landing SIMD is the busiest.
// (Should the dispatcher place workgroups otherwise, the order is merely not the best one.)
constexpr int kXcds = 8;     // accelerator dies of an MI355X, each with its own L2
constexpr int kChainBlock = 2 * kXcds;

inline void order_chains(const int32_t* utt, const int32_t* frames, const int32_t* waves, int n, int dirs,
                         int n_cu, int32_t* order)
{
    struct Chain { int32_t entry, frames, waves; };
    const int total = n * dirs;
    std::vector<Chain> chains(static_cast<size_t>(total));
    // Workgroup i runs on die (XCD) i mod kXcds.  The two chains of an utterance read the same
    // emissions; kChainBlock forward chains followed by the backward chains of the same
    // utterances puts the two a multiple of kXcds entries apart, on one die and its L2.
    for (int i0 = 0, at = 0; i0 < n; i0 += kChainBlock)
        for (int d = 0; d < dirs; ++d)
            for (int i = i0; i < std::min(n, i0 + kChainBlock); ++i) chains[at++] = {utt[i] * 2 + d, frames[i], waves[i]};
    if (n_cu < 1 || total <= n_cu) {
        for (int i = 0; i < total; ++i) order[i] = chains[i].entry;
        return;
    }
    std::vector<int64_t> load(static_cast<size_t>(n_cu) * 4, 0);
    std::vector<int> cus(static_cast<size_t>(n_cu));
    int lo = 0, hi = total, pos = 0;
    for (int round = 0; lo < hi; ++round) {
        const int k = std::min(n_cu, hi - lo), s = round & 3;
        int64_t landing = 0, all = 0, least = INT64_MAX, most = 0;
        for (int c = 0; c < k; ++c) {
            const int64_t l = load[static_cast<size_t>(c) * 4 + s];
            landing += l;
            least = std::min(least, l);
            most = std::max(most, l);
            for (int q = 0; q < 4; ++q) all += load[static_cast<size_t>(c) * 4 + q];
        }
        const bool lightest = landing * 4 > all;
        const int first = lightest ? hi - k : lo;      // chains[first .. first + k): heaviest first
        if (lightest) hi -= k; else lo += k;
        for (int c = 0; c < k; ++c) cus[c] = c;
        if (least != most)                              // busiest landing SIMD first; it gets the lightest chain
            std::stable_sort(cus.begin(), cus.begin() + k, [&](int a, int b) {
                return load[static_cast<size_t>(a) * 4 + s] > load[static_cast<size_t>(b) * 4 + s];
            });
        for (int j = 0; j < k; ++j) {
            const Chain& ch = (least != most) ? chains[first + k - 1 - j] : chains[first + j];
            const int c = cus[j];
            order[pos + c] = ch.entry;
            for (int w = 0; w < ch.waves; ++w) load[static_cast<size_t>(c) * 4 + ((s + w) & 3)] += ch.frames;
        }
        pos += k;
    }
}

constexpr int kDefaultPollBudget = 1 << 22;   // enough for seconds of waiting: only a stuck neighbour exhausts it
constexpr int kDefaultEndPolls = 1 << 22;     // the same for the workgroups that wait for chains in the lattice launch
constexpr int kMaxBatch = 65535;         // utterances index the second grid dimension of the row kernels
constexpr int kMaxDeviceMetaB = 4096;   // utterances the device-side planner ranks in LDS

// The lattice kernel reads emissions ahead of the recursion without bounds checks: a chunk's label emissions are
// requested three chunks before their use (chain_schedule), so up to three chunks past either end of an utterance's
// block (past the end going forward, before the start going backward).  These margins keep such reads inside the
// workspace; the values read there are never used.
constexpr int kChunk = kChunkSteps;   // steps whose emissions are fetched together (plan_waves: halo % 8 == 0)
constexpr int kOverFetchRows = 3 * kChunk;
constexpr int kBlankSlack = kOverFetchRows + kChunk;                          // floats, each side
constexpr int kLabelSlack = kOverFetchRows * (CTC_MAX_LABEL_LENGTH + 1);      // floats, each side

// Constants that lanes without a label state read as their emission, at the start of the
// label-emission region (inside its front slack): a chunk of probability 0, then one of log 0.
constexpr int kZeroEmission = 0, kLogZeroEmission = kChunk, kEmissionConstants = 2 * kChunk;
static_assert(kEmissionConstants <= kLabelSlack, "constants sit inside the front slack");

// ---- where and when a chain reads its emissions -------------------------------------------------
// Shared by the lattice kernels and by the host-side replay that checks every read against the
// regions' bounds (ctc_debug_replay_emission_fetches): the kernels fetch ahead without bounds
// checks, so what they may touch is defined here, once.  Offsets are in floats from the start of
// the region (Layout::emit_label, Layout::emit_blank).

// Where a lane's label emissions of chunk `chunk` (in frame order) start; kChunk floats in frame order, a backward
// chain uses them last to first.  `symbol` is the lane's label state's symbol, `li` its label position; a lane without
// a label state reads `constant` whatever the chunk.
CTC_HOST_DEVICE inline int64_t label_emission_offset(const Utt& m, bool has_label, int symbol, int li, int chunk, int constant)
{
    if (!has_label) return constant;
    return kLabelSlack + m.e_off + (static_cast<int64_t>(chunk) * m.e_cols + (m.e_direct == kEmitSymbols ? symbol : li)) * kChunk;
}
// From one chunk to the next of the chain.
CTC_HOST_DEVICE inline int64_t label_emission_step(const Utt& m, bool has_label, bool backward)
{
    return has_label ? (backward ? -1 : 1) * static_cast<int64_t>(m.e_cols) * kChunk : 0;
}
// What a chunk's frames have in common, one value per frame, in frame order: the frames' words as floats (FrameNorm), or, in launches for
// the most probable alignment, the blank's logarithms as doubles, which its chains take as scalars, a chunk in one load.
CTC_HOST_DEVICE inline int64_t blank_emission_offset(const Utt& m, int chunk)
{
    return kBlankSlack + m.f_off + static_cast<int64_t>(chunk) * kChunk;
}
// Chunk that a chain takes as its i-th one.
CTC_HOST_DEVICE inline int chain_chunk(int i, int chunks, bool backward) { return backward ? chunks - 1 - i : i; }

// How many of an utterance's chunks a chain takes when the two meet in the middle: whole blocks, the odd one forward.
CTC_HOST_DEVICE inline int chain_chunks(int frames, bool backward)
{
    const int blocks = frame_blocks(frames), forward = (blocks + 1) / 2;
    return 2 * (backward ? blocks - forward : forward);
}

// The order in which a chain requests (fetch) and consumes (run) the emissions of its chunks, an even number, in
// four register sets: set i mod 4 holds chunk i.  fetch(set, i) requests the label emissions of the chain's i-th chunk
// and, in chains that have blank emissions, the blank's of the one kBlankAhead before it; run(set, i) runs its eight steps.  The
// sets' numbers are compile-time constants (std::integral_constant).  A chunk takes 130 ns and more, a request out of the
// die's L2 about 300: hence three chunks ahead (two: 1 ns a step more); the blank's scalars go out one chunk ahead, two sets
// of 16 scalar registers being all there is room for.
// There is no branch inside a round: the compiler's count of the memory operations in flight stays exact, and a
// wavefront waits for the emissions it is about to use only, not for stores.
constexpr int kBlankAhead = 2;
// run may make `chunks` less than 0: the round is then the last one.
template <typename Fetch, typename Run>
CTC_HOST_DEVICE inline void chain_schedule(const int& chunks, Fetch&& fetch, Run&& run)
{
    const std::integral_constant<int, 0> a{};
    const std::integral_constant<int, 1> b{};
    const std::integral_constant<int, 2> c{};
    const std::integral_constant<int, 3> d{};
    fetch(a, 0);
    fetch(b, 1);
    fetch(c, 2);
    int i = 0;
    for (; i + 4 <= chunks; i += 4) {
        fetch(d, i + 3);
        run(a, i);
        fetch(a, i + 4);
        run(b, i + 1);
        fetch(b, i + 5);
        run(c, i + 2);
        fetch(c, i + 6);
        run(d, i + 3);
    }
    if (i < chunks) {
        fetch(d, i + 3);                                 // (for the blank's of the last chunk)
        run(a, i);
        run(b, i + 1);
    }
}

// Row pitch of an utterance's lattice blocks: column 1 + i holds label position i.
CTC_HOST_DEVICE inline int64_t lattice_pitch(int64_t L) { return L + 2; }
// What an utterance gets of either direction's region, in 8-byte words, and of the gathered emissions, in floats.  One with
// more symbols than frames has no alignment and needs neither; where only bounds are known, every utterance gets what the
// longest label with an alignment needs (longest_aligned).
CTC_HOST_DEVICE inline int64_t lattice_words(int frames, int64_t L) { return L <= frames ? padded_frames(frames) * lattice_pitch(L) : 0; }
CTC_HOST_DEVICE inline int64_t gathered_emissions(int frames, int64_t L) { return L <= frames ? padded_frames(frames) * L : 0; }
CTC_HOST_DEVICE inline int longest_aligned(int frames, int max_label) { return max_label < frames ? max_label : frames; }

// Byte offsets of the workspace regions, all multiples of 256.
struct Layout {
    size_t meta = 0;      // Utt[B]
    size_t order = 0;     // int32[2B]    the lattice launch's chains, one per workgroup: utterance * 2 + direction
                          //              (0 forward, 1 backward), -1 for a workgroup without one (order_chains);
                          // int32[B]     and all utterances, those first whose chains end first (about)
    size_t labels = 0;    // int32[sumL]
    size_t labels8 = 0;   // uint8[sumL]  the label strings once more, a byte per symbol (image only; narrow alphabets)
    size_t links = 0;     // int32[sumL]  grouping of the label positions by symbol (slot, count, first)
    size_t mass = 0;      // double[kMassWords B]  the alignments' mass of each utterance
    size_t sink = 0;      // what lanes with nothing to store scribble on: kSinkBytes per wavefront of a lattice launch
    size_t chain_err = 0; // int32[B]     set when a lattice wavefront gave up waiting for its neighbour
    size_t done = 0;      // int32[B * kDoneStride]  how far the utterance's chains are: cost-only calls (finish_loss)
                          //              and gradients written beside the chains (announce_end, take_chain)
    size_t left = 0;      // int32[B * (frame_blocks(T) + 1)]  narrow alphabets, gradient beside the chains: the list of workgroups that
                          //              have left their places (chains_taken)
    size_t domain = 0;    // int32[2 B]   per utterance and direction, nonzero: that chain ran in the log domain (published by
                          //              the chain for the gradient, which must know what it has stored)
    size_t row_flags = 0; // int32[B * ceil(T / 64)]  narrow alphabets: per 64 frames of an utterance, nonzero if one of
                          //              their emissions is too small for the linear domain (written by the softmax
                          //              launch, one word per workgroup, so that nothing needs clearing beforehand)
    size_t status = 0;    // int32[B]     device-resident metadata, records built by the narrow softmax launch: nonzero
                          //              if the utterance's lengths or labels are invalid
    size_t emit_blank = 0; // float[slack + sum padded_frames(Tb) + slack]  a word per frame: its norm, the blank's probability, which the
                           // label emissions are divided by (FrameNorm in the kernels)
    size_t emit_blank64 = 0; // double[slack + sum padded_frames(Tb) + slack]  launches for the most probable alignment: the blank's
                             // log2 probability per frame, for scalar loads
    size_t emit_label = 0; // float[slack + sum gathered_emissions + slack]  emission of each label position, the ratio of
                           // its probability to the blank's (encode_emission)
                           // (padded_frames(Tb)*A for small alphabets: emission_layout); the front slack starts with
                           // the constants that lanes without a label state read: probability 0 and log 0
    size_t alpha = 0;      // 8-byte words [sum lattice_words] (lattice storage, see the kernels)
    size_t beta = 0;
    size_t total = 0;
    size_t upload_bytes = 0;   // meta..labels are contiguous: the image the host prepares per call
    int64_t sumL = 0;
    int64_t frames = 0;
    int64_t emit_floats = 0;
    int64_t ab_doubles = 0;
};

// Fills `lay` from the batch shape. Returns a status (argument checks on sizes and lengths).
ctc_status_t make_layout(int T, int B, int A, const int32_t* label_lengths,
                         const int32_t* input_lengths, ctc_dtype_t dtype, Layout* lay);

// What a call computes, and so what its chains are run for:
//   kGrad  sum over alignments, label states of every frame stored (cost and gradient)
//   kLoss  sum over alignments, nothing stored (cost only; the chains meet in the middle)
//   kBest  maximum over alignments, predecessor choices stored per state pair and
//          frame (most probable alignment; the chains meet in the middle)
enum class Mode { kGrad, kLoss, kBest };

// The same for the device-metadata entry point: sized for B utterances of T frames and
// max_label symbols each.
ctc_status_t make_layout_bounds(int T, int B, int A, int max_label, ctc_dtype_t dtype, Layout* lay);

// Kernel launch parameters shared by all stages.
struct Launch {
    Mode mode;
    int T, B, A, blank;
    ctc_dtype_t dtype;
    int n_run;          // utterances whose lattice runs
    int n_chains;       // workgroups of the lattice launch (entries of the order array)
    int max_waves;      // wavefronts per lattice block
    int max_frames;     // longest utterance among those whose lattice runs
    int max_label;      // longest label of the batch
    int share_last;     // narrow alphabets: blocks_to_share
    const int32_t* frames_by_end = nullptr;   // host metadata: frames of the utterances (0: there is no lattice), those first whose chains end first; for this call only
    bool needs_barrier; // some utterance's label leaves no room for a halo
    const void* x;
    void* grads;        // nullptr unless mode == kGrad
    int32_t* alignment; // [B][T], mode == kBest only
    float* costs;
    char* ws;           // workspace base
    const int32_t* labels;    // device: the label strings, addressed by Utt::lab_off (inside the workspace
                              // for the host-metadata entry points, the caller's array otherwise)
    const void* host_image;   // pinned host copy of the meta/order/labels regions (device-readable)
    int* host_flag;           // pinned host word the device sets to host_flag_value when the image is free;
                              // nullptr when there is no image
    int host_flag_value;
    // device-metadata entry point only
    const int32_t* dev_label_lengths;
    const int32_t* dev_input_lengths;
    int32_t* dev_status;
    int poll_budget;          // copied into every Utt record
    bool crowded;             // plan the chains for total work rather than latency (device planner)
    int n_cu;                 // compute units of the device
    bool fused;               // the lattice launch writes the gradient too (ctc_lattice_gradient_kernel)
    int late_percent;         // ... and this share of the chains' workgroups come late (tests)
    int end_polls;            // ... and how often its workgroups look for the end of their chains (wait_for_chains)
    int defer;                // of every 16 frames, those whose zero rows the lattice launch writes (deferred_frames)
    int defer_columns;        // ... and the ones after those, whose zero rows the label columns' launch writes
    // Narrow alphabets, host metadata: there is no upload launch; the softmax launch reads the pinned image
    // itself and copies it into the workspace for the launches after it, and the lattice launch releases it.
    bool folded;
    bool sequential_chains = false;   // measurements: forward and backward chains in two launches, one after the other
    Layout lay;
};

// Each returns a hipError_t as int (0 = success). `stream` is a hipStream_t.
int launch_setup(const Launch& p, void* stream);       // host metadata: copies the image
int launch_plan(const Launch& p, void* stream);        // device metadata: builds meta and order on the GPU
int launch_softmax(const Launch& p, void* stream);
int launch_lattice(const Launch& p, void* stream);
int launch_gradient(const Launch& p, void* stream);   // kGrad
int launch_backtrace(const Launch& p, void* stream);   // kBest

}  // namespace ctc
