// Host side of the CTC library: argument validation, workspace layout, the per-call plan
// (which utterances run, in which order, how wide the lattice workgroups are) and the
// enqueueing of the kernels (upload, softmax, lattice, then gradient or backtrace).  No device memory is allocated here or anywhere else in
// the library (Section 4.3: allocation is kept off the training step; the caller hands in
// one workspace and this file carves it).

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstring>
#include <mutex>
#include <vector>

#include "ctc_internal.h"

// Workspace of ctc_loss_and_grad_device_static: device memory that belongs to the library's code
// object, one copy per GPU, so that the entry point needs no allocation by anybody.  In host code
// this name is only a handle for hipGetSymbolAddress; the kernels get the address it returns.
static __device__ __align__(256) unsigned char scratch[CTC_STATIC_WORKSPACE_BYTES];

namespace ctc {

namespace {

thread_local int g_last_hip_error = 0;
std::atomic<int> g_poll_budget{kDefaultPollBudget};
std::atomic<int> g_end_polls{kDefaultEndPolls};
std::atomic<int> g_sequential_chains{0};
std::atomic<int> g_overlap{-1};          // 0: the gradient in a launch of its own; 1..100: Launch::late_percent; more: beside the chains wherever it can be

constexpr size_t kAlign = 256;
inline size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

inline bool record(int err)
{
    if (err != 0) g_last_hip_error = err;
    return err == 0;
}

}  // namespace

namespace {
// Compute units of the current device (asked once per device).
int compute_units()
{
    static std::atomic<int> cached[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    int n = cached[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1) n = 256;
        cached[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

// Region offsets from the batch totals (label symbols, label emissions, frames, lattice pairs).
void carve(int T, int B, bool narrow, int64_t sumL, int64_t emit, int64_t frames, int64_t ab, Layout* lay)
{
    Layout l;
    l.sumL = sumL;
    l.emit_floats = emit;
    l.frames = frames;
    l.ab_doubles = ab;
    size_t off = 0;
    l.meta = off;   off += static_cast<size_t>(B) * sizeof(Utt);            // 64 B each: stays 8-byte aligned
    l.order = off;  off += static_cast<size_t>(B) * 3 * sizeof(int32_t);
    l.labels = off; off += static_cast<size_t>(sumL) * sizeof(int32_t);
    l.labels8 = off; off += (static_cast<size_t>(sumL) + 3) / 4 * 4;
    l.upload_bytes = off;
    off = align_up(off);
    l.links = off;  off = align_up(off + static_cast<size_t>(sumL) * sizeof(int32_t));
    l.mass = off;   off = align_up(off + static_cast<size_t>(B) * kMassWords * sizeof(double));
    l.sink = off;   off = align_up(off + static_cast<size_t>(B) * 2 * kSinkWaves * kSinkBytes);
    l.chain_err = off; off = align_up(off + static_cast<size_t>(B) * sizeof(int32_t));
    l.done = off;   off = align_up(off + static_cast<size_t>(B) * kDoneStride * sizeof(int32_t));
    l.left = off;   off = align_up(off + (narrow ? static_cast<size_t>(B) * (frame_blocks(T) + 1) * sizeof(int32_t) : 0));
    l.domain = off; off = align_up(off + static_cast<size_t>(B) * 2 * sizeof(int32_t));
    l.row_flags = off;
    off = align_up(off + static_cast<size_t>(B) * ((T + kFlagFrames - 1) / kFlagFrames) * sizeof(int32_t));
    l.status = off; off = align_up(off + static_cast<size_t>(B) * sizeof(int32_t));
    l.emit_blank = off;
    off = align_up(off + (static_cast<size_t>(frames) + 2 * kBlankSlack) * sizeof(float));
    l.emit_blank64 = off;
    off = align_up(off + (static_cast<size_t>(frames) + 2 * kBlankSlack) * sizeof(double));
    l.emit_label = off;
    off = align_up(off + (static_cast<size_t>(emit) + 2 * kLabelSlack) * sizeof(float));
    l.alpha = off;  off = align_up(off + static_cast<size_t>(ab) * sizeof(double));
    l.beta = off;   off = align_up(off + static_cast<size_t>(ab) * sizeof(double));
    l.total = off;
    *lay = l;
}
}  // namespace

const Plans& plans()
{
    static const Plans* const all = [] {
        Plans* p = new Plans();
        for (int crowded = 0; crowded < 2; ++crowded)
            for (int L = 0; L <= CTC_MAX_LABEL_LENGTH; ++L) {
                const WavePlan one = plan_waves(L, crowded), two = linear_plan2(L, crowded);
                const bool pairs = linear_two_pairs(L, crowded);
                PlanTable& t = p->table[crowded];
                t.one[L] = static_cast<uint8_t>((one.waves - 1) | ((one.halo / 8) << 4) | (pairs ? 128 : 0));
                t.two[L] = static_cast<uint8_t>((two.waves - 1) | ((two.halo / 4) << 4));
                if (!crowded) {
                    p->latency_waves[L] = static_cast<uint8_t>(pairs ? two.waves : one.waves);
                    p->latency_waves_up_to[L] = (L > 0 ? p->latency_waves_up_to[L - 1] : 0) + p->latency_waves[L];
                }
                p->most_waves[crowded][L] =
                    static_cast<uint8_t>(std::max({L > 0 ? static_cast<int>(p->most_waves[crowded][L - 1]) : 1, one.waves, two.waves}));
                p->barrier[L] = one.barrier;
            }
        return p;
    }();
    return *all;
}

ctc_status_t make_layout(int T, int B, int A, const int32_t* label_lengths,
                         const int32_t* input_lengths, ctc_dtype_t dtype, Layout* lay)
{
    if (!label_lengths || !input_lengths || !lay) return CTC_STATUS_INVALID_VALUE;
    if (T < 1 || B < 1 || A < 1) return CTC_STATUS_INVALID_VALUE;
    if (dtype != CTC_DTYPE_F32 && dtype != CTC_DTYPE_BF16) return CTC_STATUS_INVALID_VALUE;
    int64_t sumL = 0, emit = 0, ab = 0, frames = 0, padded_sum = 0;
    bool too_long = false;
    for (int b = 0; b < B; ++b) {
        const int64_t L = label_lengths[b], Tb = input_lengths[b];
        if (L < 0 || Tb < 0 || Tb > T) return CTC_STATUS_INVALID_VALUE;
        if (L > CTC_MAX_LABEL_LENGTH) too_long = true;
        sumL += L;
        const int64_t padded = padded_frames(input_lengths[b]);
        emit += A <= kDirectMaxA ? padded * A : gathered_emissions(input_lengths[b], L);
        padded_sum += padded;
        frames += Tb;
        // (the limits are on frames as the caller counts them)
        if (Tb * lattice_pitch(L) * 8 > INT32_MAX) too_long = true;
        ab += lattice_words(input_lengths[b], L);
    }
    if (too_long) return CTC_STATUS_UNSUPPORTED;
    if (sumL > INT32_MAX || frames > INT32_MAX) return CTC_STATUS_UNSUPPORTED;
    if (B > kMaxBatch) return CTC_STATUS_UNSUPPORTED;
    carve(T, B, A <= kDirectMaxA, sumL, emit, padded_sum, ab, lay);
    return CTC_STATUS_SUCCESS;
}

// Layout for the device-metadata entry point: every utterance gets the room of the largest one
// the caller allows (T frames, max_label symbols), so that offsets need no lengths.
ctc_status_t make_layout_bounds(int T, int B, int A, int max_label, ctc_dtype_t dtype, Layout* lay)
{
    if (!lay || T < 1 || B < 1 || A < 1 || max_label < 0) return CTC_STATUS_INVALID_VALUE;
    if (dtype != CTC_DTYPE_F32 && dtype != CTC_DTYPE_BF16) return CTC_STATUS_INVALID_VALUE;
    if (max_label > CTC_MAX_LABEL_LENGTH || B > kMaxDeviceMetaB) return CTC_STATUS_UNSUPPORTED;
    const int64_t Tl = T, Bl = B, Ll = max_label, padded = padded_frames(T);
    if (Tl * lattice_pitch(Ll) * 8 > INT32_MAX || Bl * Ll > INT32_MAX || Bl * Tl > INT32_MAX) return CTC_STATUS_UNSUPPORTED;
    const int longest = longest_aligned(T, max_label);
    carve(T, B, A <= kDirectMaxA, Bl * Ll, Bl * (A <= kDirectMaxA ? padded * A : gathered_emissions(T, longest)), Bl * padded, Bl * lattice_words(T, longest), lay);
    return CTC_STATUS_SUCCESS;
}

namespace {

// Pinned host buffers for the per-call metadata image.  The upload kernel reads the image
// straight from host memory, so a slot may be rewritten only after that kernel has run: the
// launch that follows it on the stream stores the slot's generation number into a pinned flag
// word in front of the image, which the host checks before it reuses the slot (no event, so no
// marker packet sits between two kernels of a call).
//
// All slots of a device come from one allocation, made at the first call on that device
// (kInitialSlots slots of at least kMinSlotBytes each), so that no later call allocates -- the
// point of Section 4.3.  The host never waits for a slot: when every slot is still in flight
// (the caller has enqueued that many calls ahead of the GPU), or when a batch's image outgrows
// the slots, a further pool with twice the slots, or larger ones, is allocated and used from
// then on (earlier pools serve when the last one is full); pools of one device stop growing at
// kMaxStagingBytes, the last one with the slots that still fit, and a call that finds every slot
// in flight then returns CTC_STATUS_NOT_READY at once.  (512 utterances of 95 symbols: about 400 calls
// ahead of the GPU.  When only the last pool served, and pools doubled or not at all, it was 128, which a
// caller that enqueues one in 45 us of what takes the GPU 145 reached after 190 calls.)
constexpr int kInitialSlots = 8;
constexpr size_t kMinSlotBytes = size_t(256) << 10;
constexpr size_t kMaxStagingBytes = size_t(256) << 20;
constexpr size_t kSpareStagingBytes = kMaxStagingBytes / 8;    // of these, left for images larger than any before
constexpr size_t kFlagBytes = 64;            // the flag word sits in front of the image

struct StagingSlot {
    char* host = nullptr;                    // kFlagBytes of flag, then the image
    int generation = 0;                      // value the device stores once the image is free
    bool in_flight = false;
    int* flag() const { return reinterpret_cast<int*>(host); }
    char* image() const { return host + kFlagBytes; }
    // Has the device released the image?  (A plain read of pinned memory; never waits.)
    bool released() const { return *static_cast<volatile int*>(flag()) == generation; }
};

struct StagingPool {
    char* base = nullptr;
    size_t slot_bytes = 0;                   // of the image part of each slot
    std::vector<StagingSlot> slots;
    int next = 0;
};

struct DeviceStaging {
    int device = -1;
    size_t total_bytes = 0;
    std::vector<StagingPool*> pools;         // the last one serves new calls
    std::atomic<long> allocations{0};
};

std::mutex g_staging_mutex;
std::vector<DeviceStaging*> g_staging;

DeviceStaging* staging_of(int dev)
{
    for (DeviceStaging* d : g_staging)
        if (d->device == dev) return d;
    DeviceStaging* d = new DeviceStaging();
    d->device = dev;
    g_staging.push_back(d);
    return d;
}

// A new pool of `slots` slots of `slot_bytes` each, or of as many as `most` bytes in all leave room for.  nullptr: none
// (status_out = NOT_READY) or the allocation failed (HIP_ERROR).
StagingPool* add_pool(DeviceStaging* d, int slots, size_t slot_bytes, size_t most, ctc_status_t* status_out)
{
    const size_t stride = kFlagBytes + slot_bytes, room = most - std::min(most, d->total_bytes);
    slots = static_cast<int>(std::min(static_cast<size_t>(slots), room / stride));
    if (slots == 0) {
        *status_out = CTC_STATUS_NOT_READY;
        return nullptr;
    }
    const size_t bytes = stride * static_cast<size_t>(slots);
    void* mem = nullptr;
    if (!record(hipHostMalloc(&mem, bytes, hipHostMallocDefault))) {
        *status_out = CTC_STATUS_HIP_ERROR;
        return nullptr;
    }
    StagingPool* pool = new StagingPool();
    pool->base = static_cast<char*>(mem);
    pool->slot_bytes = slot_bytes;
    pool->slots.resize(static_cast<size_t>(slots));
    for (int i = 0; i < slots; ++i) {
        pool->slots[static_cast<size_t>(i)].host = pool->base + stride * static_cast<size_t>(i);
        *pool->slots[static_cast<size_t>(i)].flag() = 0;
    }
    d->pools.push_back(pool);
    d->total_bytes += bytes;
    d->allocations.fetch_add(1, std::memory_order_relaxed);
    return pool;
}

StagingSlot* free_slot(StagingPool* pool)
{
    const int n = static_cast<int>(pool->slots.size());
    for (int k = 0; k < n; ++k) {
        StagingSlot& slot = pool->slots[static_cast<size_t>((pool->next + k) % n)];
        if (slot.in_flight && slot.released()) slot.in_flight = false;
        if (!slot.in_flight) {
            pool->next = (pool->next + k + 1) % n;
            return &slot;
        }
    }
    return nullptr;
}

// Returns a free slot of at least `bytes`, or nullptr with the status to return.  Never waits.
// Caller holds g_staging_mutex.
StagingSlot* acquire_slot(size_t bytes, ctc_status_t* status_out)
{
    int dev = 0;
    if (!record(hipGetDevice(&dev))) {
        *status_out = CTC_STATUS_HIP_ERROR;
        return nullptr;
    }
    DeviceStaging* d = staging_of(dev);
    const size_t want = std::max(kMinSlotBytes, (2 * bytes + 65535) / 65536 * 65536 - kFlagBytes);
    StagingPool* pool = d->pools.empty() ? nullptr : d->pools.back();
    if (pool && bytes <= pool->slot_bytes) {
        for (auto it = d->pools.rbegin(); it != d->pools.rend(); ++it) {
            if (bytes > (*it)->slot_bytes) continue;
            if (StagingSlot* slot = free_slot(*it)) return slot;
        }
        // every slot is in flight: the caller runs that far ahead of the GPU
        pool = add_pool(d, 2 * static_cast<int>(pool->slots.size()), pool->slot_bytes, kMaxStagingBytes - kSpareStagingBytes,
                        status_out);
    } else if (pool) {
        pool = add_pool(d, static_cast<int>(pool->slots.size()), want, kMaxStagingBytes, status_out);     // a larger image than any before
    } else {
        pool = add_pool(d, kInitialSlots, want, kMaxStagingBytes, status_out);
    }
    if (!pool) return nullptr;
    pool->next = 1;
    return &pool->slots[0];
}

struct Call {
    Mode mode;
    const void* x;
    const int32_t* flat_labels;
    const int32_t* label_lengths;
    const int32_t* input_lengths;
    int T, B, A, blank;
    ctc_dtype_t dtype;
    float* costs;
    void* grads;             // kGrad only
    int32_t* alignment;      // kBest only
    void* ws;
    size_t ws_bytes;
    void* stream;
};

// Validates everything that can be validated on the host, builds the upload image
// (Utt records, run order, labels) and the launch parameters.
ctc_status_t prepare(const Call& c, const Layout& lay, Launch* out, char* image)
{
    if (lay.sumL > 0 && !c.flat_labels) return CTC_STATUS_INVALID_VALUE;
    if (reinterpret_cast<uintptr_t>(c.ws) % kAlign != 0) return CTC_STATUS_INVALID_VALUE;

    const size_t elem = (c.dtype == CTC_DTYPE_F32) ? 4 : 2;
    const size_t tensor_bytes = static_cast<size_t>(c.T) * c.B * c.A * elem;
    if (c.mode == Mode::kGrad) {
        const char* xa = static_cast<const char*>(c.x);
        const char* ga = static_cast<const char*>(c.grads);
        if (xa < ga + tensor_bytes && ga < xa + tensor_bytes) return CTC_STATUS_INVALID_VALUE;
        if (reinterpret_cast<uintptr_t>(c.grads) % elem) return CTC_STATUS_INVALID_VALUE;
    }
    if (reinterpret_cast<uintptr_t>(c.x) % elem) return CTC_STATUS_INVALID_VALUE;
    if (c.mode == Mode::kBest && reinterpret_cast<uintptr_t>(c.alignment) % sizeof(int32_t))
        return CTC_STATUS_INVALID_VALUE;

    Utt* meta = reinterpret_cast<Utt*>(image + lay.meta);
    int32_t* order = reinterpret_cast<int32_t*>(image + lay.order);
    int32_t* labels = reinterpret_cast<int32_t*>(image + lay.labels);
    uint8_t* labels8 = reinterpret_cast<uint8_t*>(image + lay.labels8);

    const Plans& all_plans = plans();
    // Would the launch, planned for latency, put more than two wavefronts on every SIMD?
    int64_t latency_waves = 0;
    for (int b = 0; b < c.B; ++b) latency_waves += all_plans.latency_waves[c.label_lengths[b]];
    const bool crowded = latency_waves * 2 > kCrowdedWaves;
    const PlanTable& plan_of = all_plans.table[crowded];

    // The labels travel as bytes where a symbol fits one and as words otherwise (launch_setup, NarrowImage).
    const bool byte_labels = c.A <= kByteLabelsMaxA;
    const int poll_budget = g_poll_budget.load(std::memory_order_relaxed);
    int64_t lab_off = 0, e_off = 0, ab_off = 0, f_off = 0;
    int n_run = 0, max_waves = 1, max_frames = 0, max_label = 0;
    bool needs_barrier = false;
    for (int b = 0; b < c.B; ++b) {
        const int L = c.label_lengths[b], Tb = c.input_lengths[b];
        const int32_t* const lab = c.flat_labels + lab_off;
        max_label = std::max(max_label, L);
        // (branch-free, so that the compiler makes vector code of it)
        unsigned bad = 0;
        int repeats = 0;
        const unsigned A = static_cast<unsigned>(c.A);
        const int32_t blank = c.blank;
        for (int i = 0; i < L; ++i) bad |= (static_cast<unsigned>(lab[i]) >= A) | (lab[i] == blank);
        for (int i = 1; i < L; ++i) repeats += lab[i] == lab[i - 1];
        if (bad) return CTC_STATUS_INVALID_VALUE;
        if (byte_labels)
            for (int i = 0; i < L; ++i) labels8[lab_off + i] = static_cast<uint8_t>(lab[i]);
        else if (L > 0)
            std::memcpy(labels + lab_off, lab, static_cast<size_t>(L) * sizeof(int32_t));
        // An alignment exists iff every symbol gets a frame and equal neighbours a blank between them.
        const bool runs = Tb > 0 && Tb >= L + repeats;
        Utt m;
        m.Tb = Tb;
        m.L = L;
        m.lab_off = static_cast<int32_t>(lab_off);
        m.flags = (runs ? kUttRuns : 0) | (plan_of.two_pairs(L) ? kUttTwoPairs : 0) |
                  ((Tb > kLinearMaxFrames || tight_fit(Tb, L, repeats)) ? kUttLogDomain : 0);
        m.f_off = static_cast<uint32_t>(f_off);
        m.waves = plan_of.waves1(L);
        m.halo = plan_of.halo1(L);
        m.waves2 = plan_of.waves2(L);
        m.halo2 = plan_of.halo2(L);
        m.poll_budget = poll_budget;
        m.e_off = e_off;
        m.ab_off = ab_off;
        m.e_direct = emission_layout(c.A);
        m.rough = 0;
        m.steep = 0;
        m.e_cols = m.e_direct == kEmitSymbols ? c.A : L;
        meta[b] = m;
        const int64_t padded = padded_frames(Tb);
        lab_off += L;
        e_off += c.A <= kDirectMaxA ? padded * c.A : gathered_emissions(Tb, L);
        f_off += padded;
        ab_off += lattice_words(Tb, L);
        if (runs) {
            order[n_run++] = b;
            max_waves = std::max({max_waves, m.waves, m.waves2});
            needs_barrier = needs_barrier || all_plans.barrier[L];
            max_frames = std::max(max_frames, Tb);
        }
    }
    // The one-barrier-per-step kernel only has the log-domain recursion.
    if (needs_barrier)
        for (int b = 0; b < c.B; ++b) meta[b].flags |= kUttLogDomain;
    // Heaviest chains first, so the longest recursion does not start last; launches of more
    // chains than compute units are ordered for the SIMDs' loads (order_chains).
    auto chain_waves = [&](int b) {
        const bool two = (meta[b].flags & (kUttTwoPairs | kUttLogDomain)) == kUttTwoPairs && c.mode != Mode::kBest;
        return two ? meta[b].waves2 : meta[b].waves;
    };
    // (sorted as numbers: the weight, then the smaller utterance number first)
    thread_local std::vector<uint64_t> by_weight;
    by_weight.resize(static_cast<size_t>(n_run));
    for (int i = 0; i < n_run; ++i) {
        const int b = order[i];
        by_weight[i] = (~static_cast<uint64_t>(chain_weight(meta[b], c.mode == Mode::kBest, crowded)) << 16) | static_cast<uint64_t>(b);
    }
    std::sort(by_weight.begin(), by_weight.end());
    thread_local std::vector<int32_t> running, run_frames, run_waves;
    running.resize(static_cast<size_t>(n_run));
    run_frames.resize(static_cast<size_t>(n_run));
    run_waves.resize(static_cast<size_t>(n_run));
    for (int i = 0; i < n_run; ++i) {
        running[i] = static_cast<int32_t>(by_weight[i] & 0xFFFF);
        run_frames[i] = meta[running[i]].Tb;
        run_waves[i] = chain_waves(running[i]);
    }
    constexpr int dirs = 2;
    order_chains(running.data(), run_frames.data(), run_waves.data(), n_run, dirs, compute_units(), order);
    for (int i = n_run * dirs; i < 2 * c.B; ++i) order[i] = -1;
    // all utterances for the gradient: those without an alignment, then the lightest first
    int32_t* by_end = order + 2 * c.B;
    if (n_run < c.B)
        for (int b = 0; b < c.B; ++b)
            if (!(meta[b].flags & kUttRuns)) *by_end++ = b;
    for (int i = n_run - 1; i >= 0; --i) *by_end++ = running[i];
    const bool narrow_gradient = c.mode == Mode::kGrad && c.A <= kDirectMaxA;
    thread_local std::vector<int32_t> frames_by_end;
    if (narrow_gradient) {
        frames_by_end.assign(static_cast<size_t>(c.B), 0);
        for (int i = 0; i < n_run; ++i) frames_by_end[c.B - 1 - i] = run_frames[i];
    }

    const bool sequential_chains = c.mode == Mode::kGrad && g_sequential_chains.load(std::memory_order_relaxed) != 0;

    if (c.ws_bytes < lay.total) return CTC_STATUS_WORKSPACE_TOO_SMALL;

    out->mode = c.mode;
    out->frames_by_end = narrow_gradient ? frames_by_end.data() : nullptr;
    out->T = c.T; out->B = c.B; out->A = c.A; out->blank = c.blank;
    out->dtype = c.dtype;
    out->n_run = n_run;
    out->n_chains = n_run * dirs;
    out->max_waves = max_waves;
    out->max_frames = max_frames;
    out->max_label = max_label;
    out->needs_barrier = needs_barrier;
    out->x = c.x;
    out->grads = (c.mode == Mode::kGrad) ? c.grads : nullptr;
    out->alignment = (c.mode == Mode::kBest) ? c.alignment : nullptr;
    out->costs = c.costs;
    out->ws = static_cast<char*>(c.ws);
    out->labels = reinterpret_cast<const int32_t*>(static_cast<char*>(c.ws) + lay.labels);
    out->host_image = image;
    out->dev_label_lengths = nullptr;
    out->dev_input_lengths = nullptr;
    out->dev_status = nullptr;
    out->poll_budget = poll_budget;
    out->end_polls = g_end_polls.load(std::memory_order_relaxed);
    out->crowded = crowded;
    out->sequential_chains = sequential_chains;
    out->n_cu = compute_units();
    out->defer = 0;
    out->defer_columns = 0;
    if (c.mode == Mode::kGrad && c.A > kDirectMaxA && !needs_barrier && !sequential_chains && n_run > 0) {
        int64_t rows = static_cast<int64_t>(c.T) * c.B;
        for (int i = 0; i < n_run; ++i) rows -= run_frames[i];
        out->defer = deferred_frames(static_cast<double>(rows) * c.A * elem, max_frames, n_run * dirs, out->n_cu);
        out->defer_columns = columns_frames(static_cast<double>(rows) * c.A * elem, c.A, out->defer);
    }
    out->fused = c.mode == Mode::kGrad && !needs_barrier && !sequential_chains && n_run > 0 &&
                 can_fuse_gradient(c.A, max_waves, n_run * dirs, out->n_cu, c.T, c.B);
    const int overlap = g_overlap.load(std::memory_order_relaxed);
    out->late_percent = overlap <= 100 ? std::max(overlap, 0) : 0;
    if (out->fused && overlap < 0) {
        double last = 0, early = 0, late = 0;
        auto end_of = [&](int i) { return run_frames[i] * chain_us_per_frame(run_waves[i]); };
        const int counted = beside_by_work(max_waves, n_run * dirs, out->n_cu) ? n_run : 0;
        for (int i = 0; i < counted; ++i) last = std::max(last, end_of(i));
        for (int i = 0; i < counted; ++i)
            (end_of(i) < 0.85 * last ? early : late) += static_cast<double>(frame_blocks(run_frames[i])) * std::max(1, label_pieces(meta[running[i]].L));
        out->fused = gradient_in_lattice_launch(early, late, last, max_frames, max_waves, n_run * dirs, out->n_cu);
    }
    out->fused = out->fused && overlap != 0;
    // Blocks times pieces of the utterances whose chains end in the last 15 % of the time (a question of up to a chain per compute unit: blocks_to_share).
    int64_t late_blocks = 0;
    auto weight = [&](int i) { return ~by_weight[i] >> 16; };
    for (int i = 0; i < n_run && narrow_gradient && n_run * dirs <= out->n_cu && 100 * weight(i) >= 85 * weight(0); ++i)
        late_blocks += static_cast<int64_t>(frame_blocks(run_frames[i])) * std::max(1, label_pieces(meta[running[i]].L));
    out->share_last = blocks_to_share(late_blocks, c.A, n_run * dirs, out->n_cu);
    out->folded = c.A <= kDirectMaxA && c.B <= kNarrowMaxB && c.T < (1 << 29);
    out->lay = lay;
    return CTC_STATUS_SUCCESS;
}

// Cheap checks that need neither the layout nor a staging slot.
ctc_status_t precheck(const Call& c)
{
    if (!c.x || !c.label_lengths || !c.input_lengths || !c.costs || !c.ws) return CTC_STATUS_INVALID_VALUE;
    if (c.mode == Mode::kGrad && !c.grads) return CTC_STATUS_INVALID_VALUE;
    if (c.mode == Mode::kBest && !c.alignment) return CTC_STATUS_INVALID_VALUE;
    if (c.T < 1 || c.B < 1 || c.A < 1 || c.blank < 0 || c.blank >= c.A) return CTC_STATUS_INVALID_VALUE;
    return CTC_STATUS_SUCCESS;
}

// HIP events of a profiled call, destroyed however the call ends.
struct Events {
    hipEvent_t ev[CTC_NUM_KERNELS + 3] = {};
    bool create()
    {
        for (auto& e : ev)
            if (!record(hipEventCreate(&e))) return false;
        return true;
    }
    ~Events()
    {
        for (auto& e : ev)
            if (e) (void)hipEventDestroy(e);
    }
};

ctc_status_t run(const Call& c, float* kernel_ms)
{
    ctc_status_t st = precheck(c);
    if (st != CTC_STATUS_SUCCESS) return st;
    Layout lay;
    st = make_layout(c.T, c.B, c.A, c.label_lengths, c.input_lengths, c.dtype, &lay);
    if (st != CTC_STATUS_SUCCESS) return st;

    hipStream_t s = static_cast<hipStream_t>(c.stream);
    // Events 0..CTC_NUM_KERNELS bracket the launches; the last two are recorded back to back
    // and give what an interval with nothing in it reads, which is taken off every interval.
    Events events;
    hipEvent_t* const ev = events.ev;
    Launch p;
    {
        // The image is validated while it is written; on an error nothing has been enqueued and
        // the slot simply stays free.
        std::lock_guard<std::mutex> lock(g_staging_mutex);
        thread_local std::vector<char> scratch;          // validation without a device: see below
        static const bool have_device = [] {
            int ndev = 0;
            const bool ok = hipGetDeviceCount(&ndev) == hipSuccess && ndev > 0;
            if (!ok) (void)hipGetLastError();
            return ok;
        }();
        if (!have_device) {
            // No GPU (host-only checks of the argument validation): build the image in ordinary
            // memory so that every validation error is still reported, then stop.
            scratch.resize(lay.upload_bytes);
            st = prepare(c, lay, &p, scratch.data());
            return st != CTC_STATUS_SUCCESS ? st : CTC_STATUS_HIP_ERROR;
        }
        StagingSlot* const slot = acquire_slot(lay.upload_bytes, &st);
        if (!slot) return st;
        st = prepare(c, lay, &p, slot->image());
        if (st != CTC_STATUS_SUCCESS) return st;
        if (kernel_ms && !events.create()) return CTC_STATUS_HIP_ERROR;
        slot->generation += 1;
        p.host_flag = slot->flag();
        p.host_flag_value = slot->generation;
        // The upload launch's own time is not reported separately: it is a few microseconds and
        // overlaps the tail of whatever ran before on the stream.  (Narrow alphabets have none: their
        // softmax launch reads the image itself, and the lattice launch releases it.)
        if (!p.folded && !record(launch_setup(p, c.stream))) return CTC_STATUS_HIP_ERROR;
        // The image is released by the softmax launch, or by the lattice launch after it (narrow
        // alphabets).  Should the releasing launch fail to go out, nothing would ever release the slot
        // while a kernel may still be reading it: wait for the stream (an error path) and leave the
        // slot free.
        bool out = (!kernel_ms || record(hipEventRecord(ev[0], s))) && record(launch_softmax(p, c.stream)) &&
                   (!kernel_ms || record(hipEventRecord(ev[1], s)));
        if (out && p.folded)
            out = record(launch_lattice(p, c.stream)) && (!kernel_ms || record(hipEventRecord(ev[2], s)));
        if (!out) {
            (void)hipStreamSynchronize(s);
            return CTC_STATUS_HIP_ERROR;
        }
        slot->in_flight = true;
    }

    // Cost-only calls end with the lattice launch.
    int (*const stages[CTC_NUM_KERNELS])(const Launch&, void*) = {
        launch_softmax, launch_lattice,
        c.mode == Mode::kGrad ? (p.fused ? nullptr : launch_gradient) : (c.mode == Mode::kLoss ? nullptr : launch_backtrace)};
    for (int i = p.folded ? 2 : 1; i < CTC_NUM_KERNELS; ++i) {
        if (stages[i] && !record(stages[i](p, c.stream))) return CTC_STATUS_HIP_ERROR;
        if (kernel_ms && !record(hipEventRecord(ev[i + 1], s))) return CTC_STATUS_HIP_ERROR;
    }
    if (kernel_ms) {
        if (!record(hipEventRecord(ev[CTC_NUM_KERNELS + 1], s))) return CTC_STATUS_HIP_ERROR;
        if (!record(hipEventRecord(ev[CTC_NUM_KERNELS + 2], s))) return CTC_STATUS_HIP_ERROR;
        if (!record(hipStreamSynchronize(s))) return CTC_STATUS_HIP_ERROR;
        float empty = 0.0f;
        if (!record(hipEventElapsedTime(&empty, ev[CTC_NUM_KERNELS + 1], ev[CTC_NUM_KERNELS + 2])))
            return CTC_STATUS_HIP_ERROR;
        for (int i = 0; i < CTC_NUM_KERNELS; ++i) {
            if (!record(hipEventElapsedTime(&kernel_ms[i], ev[i], ev[i + 1]))) return CTC_STATUS_HIP_ERROR;
            kernel_ms[i] = stages[i] ? std::max(kernel_ms[i] - empty, 0.0f) : 0.0f;
        }
    }
    return CTC_STATUS_SUCCESS;
}

// Device-metadata call: nothing about the batch is known on the host beyond its bounds, so
// the launch shapes come from the bounds and a planning kernel fills in the rest.  Only kernel
// launches are enqueued (no copies, no host memory, no waiting), so the call may be recorded
// into a HIP graph.
ctc_status_t run_device(const void* x, const int32_t* labels, const int32_t* label_lengths,
                        const int32_t* input_lengths, int max_label, int T, int B, int A, int blank,
                        ctc_dtype_t dtype, float* costs, void* grads, int32_t* status, void* ws,
                        size_t ws_bytes, void* stream, float* kernel_ms = nullptr)
{
    if (!x || !label_lengths || !input_lengths || !costs || !status || !ws) return CTC_STATUS_INVALID_VALUE;
    if (max_label > 0 && !labels) return CTC_STATUS_INVALID_VALUE;
    if (T < 1 || B < 1 || A < 1 || blank < 0 || blank >= A) return CTC_STATUS_INVALID_VALUE;
    Layout lay;
    ctc_status_t st = make_layout_bounds(T, B, A, max_label, dtype, &lay);
    if (st != CTC_STATUS_SUCCESS) return st;
    if (reinterpret_cast<uintptr_t>(ws) % kAlign != 0) return CTC_STATUS_INVALID_VALUE;
    const size_t elem = (dtype == CTC_DTYPE_F32) ? 4 : 2;
    if (reinterpret_cast<uintptr_t>(x) % elem || reinterpret_cast<uintptr_t>(grads) % elem)
        return CTC_STATUS_INVALID_VALUE;
    if (grads) {
        const size_t tensor_bytes = static_cast<size_t>(T) * B * A * elem;
        const char* xa = static_cast<const char*>(x);
        const char* ga = static_cast<const char*>(grads);
        if (xa < ga + tensor_bytes && ga < xa + tensor_bytes) return CTC_STATUS_INVALID_VALUE;
    }
    if (ws_bytes < lay.total) return CTC_STATUS_WORKSPACE_TOO_SMALL;

    Launch p;
    p.mode = grads ? Mode::kGrad : Mode::kLoss;
    p.T = T; p.B = B; p.A = A; p.blank = blank;
    p.dtype = dtype;
    p.n_run = B;                       // a lattice workgroup per utterance and direction; those that do not run leave at once
    p.n_chains = B * 2;
    // Would the launch, planned for latency, put more than two wavefronts on every SIMD (prepare's question)?  The
    // labels' lengths are on the GPU; the answer here is for lengths spread evenly up to the bound.
    const Plans& all_plans = plans();
    p.crowded = static_cast<int64_t>(B) * 2 * all_plans.latency_waves_up_to[max_label] >
                static_cast<int64_t>(kCrowdedWaves) * (max_label + 1);
    p.max_waves = all_plans.most_waves[p.crowded][max_label];
    p.max_frames = T;
    p.max_label = max_label;
    p.needs_barrier = all_plans.barrier[max_label];
    p.x = x;
    p.grads = grads;
    p.alignment = nullptr;
    p.costs = costs;
    p.ws = static_cast<char*>(ws);
    p.labels = labels;
    p.host_image = nullptr;
    p.host_flag = nullptr;
    p.host_flag_value = 0;
    p.dev_label_lengths = label_lengths;
    p.dev_input_lengths = input_lengths;
    p.dev_status = status;
    p.poll_budget = g_poll_budget.load(std::memory_order_relaxed);
    p.end_polls = g_end_polls.load(std::memory_order_relaxed);
    p.n_cu = compute_units();
    p.share_last = blocks_to_share(-1, A, p.n_chains, p.n_cu);
    // (how much padding there is only the GPU knows: taken for a third of the tensor)
    p.defer = grads && A > kDirectMaxA && !p.needs_barrier
                  ? deferred_frames(static_cast<double>(T) * B * A * elem / 3, T / 2, p.n_chains, p.n_cu) : 0;
    p.defer_columns = grads && A > kDirectMaxA && !p.needs_barrier ? columns_frames(static_cast<double>(T) * B * A * elem / 3, A, p.defer) : 0;
    const int overlap = g_overlap.load(std::memory_order_relaxed);
    p.late_percent = overlap <= 100 ? std::max(overlap, 0) : 0;
    p.fused = grads && !p.needs_barrier && overlap != 0 && can_fuse_gradient(A, p.max_waves, p.n_chains, p.n_cu, T, B);
    if (p.fused && overlap < 0) {
        // (lengths spread evenly up to the bounds, as above: one utterance in seven ends late, half the frames are frames)
        const double blocks = static_cast<double>(B) * frame_blocks(T);
        const double late = 0.14 * blocks * std::max(1, label_pieces(max_label * 3 / 4)), all = 0.5 * blocks * std::max(1, label_pieces(max_label / 2));
        p.fused = gradient_in_lattice_launch(std::max(all - late, 0.0), late, T * chain_us_per_frame(all_plans.latency_waves[max_label]),
                                             T, p.max_waves, p.n_chains, p.n_cu);
    }
    // Narrow alphabets: the softmax launch builds the records itself (no planning launch before it); every
    // utterance's setup workgroup weighs all B utterances for the run order, which is worth it up to here.
    p.folded = A <= kDirectMaxA && B <= kDeviceFoldMaxB && max_label > 0;
    p.lay = lay;
    // Per-launch device times for measurements (ctc_profile_kernels_device): events around the launches as in run().
    Events events;
    hipEvent_t* const ev = events.ev;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (kernel_ms && !events.create()) return CTC_STATUS_HIP_ERROR;
    if (!p.folded && !record(launch_plan(p, stream))) return CTC_STATUS_HIP_ERROR;
    int (*const stages[CTC_NUM_KERNELS])(const Launch&, void*) = {launch_softmax, launch_lattice,
                                                                   grads && !p.fused ? launch_gradient : nullptr};
    if (kernel_ms && !record(hipEventRecord(ev[0], s))) return CTC_STATUS_HIP_ERROR;
    for (int i = 0; i < CTC_NUM_KERNELS; ++i) {
        if (stages[i] && !record(stages[i](p, stream))) return CTC_STATUS_HIP_ERROR;
        if (kernel_ms && !record(hipEventRecord(ev[i + 1], s))) return CTC_STATUS_HIP_ERROR;
    }
    if (kernel_ms) {
        if (!record(hipEventRecord(ev[CTC_NUM_KERNELS + 1], s))) return CTC_STATUS_HIP_ERROR;
        if (!record(hipEventRecord(ev[CTC_NUM_KERNELS + 2], s))) return CTC_STATUS_HIP_ERROR;
        if (!record(hipStreamSynchronize(s))) return CTC_STATUS_HIP_ERROR;
        float empty = 0.0f;
        if (!record(hipEventElapsedTime(&empty, ev[CTC_NUM_KERNELS + 1], ev[CTC_NUM_KERNELS + 2])))
            return CTC_STATUS_HIP_ERROR;
        for (int i = 0; i < CTC_NUM_KERNELS; ++i) {
            if (!record(hipEventElapsedTime(&kernel_ms[i], ev[i], ev[i + 1]))) return CTC_STATUS_HIP_ERROR;
            kernel_ms[i] = stages[i] ? std::max(kernel_ms[i] - empty, 0.0f) : 0.0f;
        }
    }
    return CTC_STATUS_SUCCESS;
}

// Address of `scratch` on the current device (each GPU holds its own copy at its own address):
// asked once per device, with that device current, and kept.
void* static_workspace()
{
    constexpr int kMaxDevices = 64;
    static std::mutex mutex;
    static void* address[kMaxDevices] = {};
    int dev = 0;
    if (!record(hipGetDevice(&dev))) return nullptr;
    if (dev < 0 || dev >= kMaxDevices) {
        g_last_hip_error = static_cast<int>(hipErrorInvalidDevice);
        return nullptr;
    }
    std::lock_guard<std::mutex> lock(mutex);
    if (!address[dev]) {
        void* ptr = nullptr;
        if (!record(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)))) return nullptr;
        address[dev] = ptr;
    }
    return address[dev];
}

}  // namespace
}  // namespace ctc

extern "C" {

ctc_status_t ctc_profile_kernels_device(const void* activations, const int32_t* labels,
                                        const int32_t* label_lengths, const int32_t* input_lengths,
                                        int max_label_length, int T, int B, int A, int blank,
                                        ctc_dtype_t dtype, float* costs, void* grads, int32_t* status_out,
                                        void* workspace, size_t workspace_bytes, hipStream_t stream,
                                        float* kernel_ms)
{
    if (!kernel_ms) return CTC_STATUS_INVALID_VALUE;
    return ctc::run_device(activations, labels, label_lengths, input_lengths, max_label_length, T, B, A,
                           blank, dtype, costs, grads, status_out, workspace, workspace_bytes, stream, kernel_ms);
}

ctc_status_t ctc_loss_and_grad_device_static(const void* activations, const int32_t* labels,
                                             const int32_t* label_lengths, const int32_t* input_lengths,
                                             int max_label_length, int T, int B, int A, int blank,
                                             ctc_dtype_t dtype, float* costs, void* grads,
                                             int32_t* status_out, hipStream_t stream)
{
    // Sizes first: a batch shape beyond the static workspace is refused before anything else happens.
    ctc::Layout lay;
    const ctc_status_t st = ctc::make_layout_bounds(T, B, A, max_label_length, dtype, &lay);
    if (st != CTC_STATUS_SUCCESS) return st;
    if (lay.total > CTC_STATIC_WORKSPACE_BYTES) return CTC_STATUS_WORKSPACE_TOO_SMALL;
    void* const ws = ctc::static_workspace();
    if (!ws) return CTC_STATUS_HIP_ERROR;
    return ctc::run_device(activations, labels, label_lengths, input_lengths, max_label_length, T, B, A,
                           blank, dtype, costs, grads, status_out, ws, CTC_STATIC_WORKSPACE_BYTES, stream);
}

ctc_status_t ctc_workspace_size_device(int T, int B, int A, int max_label_length, ctc_dtype_t dtype,
                                       size_t* bytes_out)
{
    if (!bytes_out) return CTC_STATUS_INVALID_VALUE;
    ctc::Layout lay;
    ctc_status_t st = ctc::make_layout_bounds(T, B, A, max_label_length, dtype, &lay);
    if (st == CTC_STATUS_SUCCESS) *bytes_out = lay.total;
    return st;
}

ctc_status_t ctc_loss_and_grad_device(const void* activations, const int32_t* labels,
                                      const int32_t* label_lengths, const int32_t* input_lengths,
                                      int max_label_length, int T, int B, int A, int blank,
                                      ctc_dtype_t dtype, float* costs, void* grads, int32_t* status_out,
                                      void* workspace, size_t workspace_bytes, hipStream_t stream)
{
    return ctc::run_device(activations, labels, label_lengths, input_lengths, max_label_length, T, B, A,
                           blank, dtype, costs, grads, status_out, workspace, workspace_bytes, stream);
}


ctc_status_t ctc_workspace_size(int T, int B, int A, const int32_t* label_lengths,
                                const int32_t* input_lengths, ctc_dtype_t dtype, size_t* bytes_out)
{
    if (!bytes_out) return CTC_STATUS_INVALID_VALUE;
    ctc::Layout lay;
    ctc_status_t st = ctc::make_layout(T, B, A, label_lengths, input_lengths, dtype, &lay);
    if (st == CTC_STATUS_SUCCESS) *bytes_out = lay.total;
    return st;
}

ctc_status_t ctc_loss_and_grad(const void* activations, const int32_t* flat_labels,
                               const int32_t* label_lengths, const int32_t* input_lengths,
                               int T, int B, int A, int blank, ctc_dtype_t dtype, float* costs,
                               void* grads, void* workspace, size_t workspace_bytes, hipStream_t stream)
{
    ctc::Call c{grads ? ctc::Mode::kGrad : ctc::Mode::kLoss, activations, flat_labels, label_lengths,
                input_lengths, T, B, A, blank, dtype, costs, grads, nullptr, workspace, workspace_bytes, stream};
    return ctc::run(c, nullptr);
}

ctc_status_t ctc_profile_kernels(const void* activations, const int32_t* flat_labels,
                                 const int32_t* label_lengths, const int32_t* input_lengths,
                                 int T, int B, int A, int blank, ctc_dtype_t dtype, float* costs,
                                 void* grads, void* workspace, size_t workspace_bytes, hipStream_t stream,
                                 float* kernel_ms)
{
    if (!kernel_ms) return CTC_STATUS_INVALID_VALUE;
    ctc::Call c{grads ? ctc::Mode::kGrad : ctc::Mode::kLoss, activations, flat_labels, label_lengths,
                input_lengths, T, B, A, blank, dtype, costs, grads, nullptr, workspace, workspace_bytes, stream};
    return ctc::run(c, kernel_ms);
}

ctc_status_t ctc_best_path(const void* activations, const int32_t* flat_labels,
                           const int32_t* label_lengths, const int32_t* input_lengths,
                           int T, int B, int A, int blank, ctc_dtype_t dtype, float* scores,
                           int32_t* alignment, void* workspace, size_t workspace_bytes, hipStream_t stream)
{
    ctc::Call c{ctc::Mode::kBest, activations, flat_labels, label_lengths, input_lengths, T, B, A, blank,
                dtype, scores, nullptr, alignment, workspace, workspace_bytes, stream};
    return ctc::run(c, nullptr);
}

ctc_status_t ctc_profile_best_path(const void* activations, const int32_t* flat_labels,
                                   const int32_t* label_lengths, const int32_t* input_lengths,
                                   int T, int B, int A, int blank, ctc_dtype_t dtype, float* scores,
                                   int32_t* alignment, void* workspace, size_t workspace_bytes,
                                   hipStream_t stream, float* kernel_ms)
{
    if (!kernel_ms) return CTC_STATUS_INVALID_VALUE;
    ctc::Call c{ctc::Mode::kBest, activations, flat_labels, label_lengths, input_lengths, T, B, A, blank,
                dtype, scores, nullptr, alignment, workspace, workspace_bytes, stream};
    return ctc::run(c, kernel_ms);
}

const char* ctc_kernel_name(int index)
{
    switch (index) {
        case CTC_KERNEL_SOFTMAX: return "ctc_softmax";
        case CTC_KERNEL_LATTICE: return "ctc_lattice";
        case CTC_KERNEL_GRADIENT: return "ctc_gradient";
        case CTC_KERNEL_BACKTRACE: return "ctc_backtrace";
        default: return nullptr;
    }
}

const char* ctc_status_string(ctc_status_t status)
{
    switch (status) {
        case CTC_STATUS_SUCCESS: return "success";
        case CTC_STATUS_INVALID_VALUE: return "invalid value";
        case CTC_STATUS_WORKSPACE_TOO_SMALL: return "workspace too small";
        case CTC_STATUS_HIP_ERROR: return "HIP runtime error";
        case CTC_STATUS_UNSUPPORTED: return "unsupported size";
        case CTC_STATUS_NOT_READY: return "too many calls in flight";
        default: return "unknown status";
    }
}

int ctc_last_hip_error(void) { return ctc::g_last_hip_error; }

long ctc_debug_staging_allocations(void)
{
    std::lock_guard<std::mutex> lock(ctc::g_staging_mutex);
    long n = 0;
    for (const ctc::DeviceStaging* d : ctc::g_staging) n += d->allocations.load(std::memory_order_relaxed);
    return n;
}

long ctc_debug_replay_emission_fetches(int T, int B, int A, const int32_t* label_lengths, const int32_t* input_lengths,
                                       int max_label_length, long* margin_floats)
{
    using namespace ctc;
    if (!label_lengths || !input_lengths) return -1;
    const bool bounds = max_label_length >= 0;
    Layout lay;
    const ctc_status_t st = bounds ? make_layout_bounds(T, B, A, max_label_length, CTC_DTYPE_F32, &lay)
                                   : make_layout(T, B, A, label_lengths, input_lengths, CTC_DTYPE_F32, &lay);
    if (st != CTC_STATUS_SUCCESS) return -1;
    const bool symbols = emission_layout(A) == kEmitSymbols;
    // the regions as carved: slack, blocks, slack
    const int64_t label_floats = lay.emit_floats + 2 * static_cast<int64_t>(kLabelSlack);
    const int64_t blank_floats = lay.frames + 2 * static_cast<int64_t>(kBlankSlack);
    long violations = 0;
    int64_t margin = INT64_MAX;
    auto touch = [&](int64_t off, int64_t size) {
        if (off < 0 || off >= size) ++violations;
        margin = std::min(margin, std::min(off, size - 1 - off));
    };
    int64_t e_off = 0, f_off = 0;
    for (int b = 0; b < B; ++b) {
        const int L = label_lengths[b], Tb = input_lengths[b];
        // block offsets as the launcher (prepare) and the device-side planner (ctc_plan_kernel) set them
        Utt m{};
        m.Tb = Tb;
        m.L = L;
        m.e_direct = emission_layout(A);
        m.e_cols = symbols ? A : L;
        if (bounds) {
            m.f_off = static_cast<uint32_t>(b * padded_frames(T));
            m.e_off = b * (symbols ? padded_frames(T) * A : gathered_emissions(T, longest_aligned(T, max_label_length)));
        } else {
            m.f_off = static_cast<uint32_t>(f_off);
            m.e_off = e_off;
            e_off += symbols ? padded_frames(Tb) * A : gathered_emissions(Tb, L);
            f_off += padded_frames(Tb);
        }
        if (Tb < 1 || Tb < L) continue;             // its chains do not run
        const int chunks = 2 * frame_blocks(Tb);
        for (int backward = 0; backward < 2; ++backward) {
            // Lanes at the ends of every range a pointer depends on: first and last label position, first
            // and last symbol; a lane without a label state, for either constant.
            struct LaneKind { bool has_label; int symbol, li, constant; };
            const LaneKind kinds[] = {{L > 0, 0, 0, 0}, {L > 0, A - 1, L - 1, 0}, {L > 0, 0, L - 1, 0}, {L > 0, A - 1, 0, 0},
                                      {false, 0, 0, kZeroEmission}, {false, 0, 0, kLogZeroEmission}};
            auto nothing = [](auto, int) {};
            for (const LaneKind& k : kinds) {
                int64_t p = label_emission_offset(m, k.has_label, k.symbol, k.li, chain_chunk(0, chunks, backward != 0), k.constant);
                const int64_t step = label_emission_step(m, k.has_label, backward != 0);
                auto fetch = [&](auto, int) {
                    touch(p, label_floats);
                    touch(p + kChunk - 1, label_floats);
                    p += step;
                };
                chain_schedule(chunks, fetch, nothing);
            }
            auto fetch = [&](auto, int i) {
                if (i < kBlankAhead) return;
                const int64_t w = blank_emission_offset(m, chain_chunk(i - kBlankAhead, chunks, backward != 0));
                touch(w, blank_floats);                          // (the block of doubles has the same extent)
                touch(w + kChunk - 1, blank_floats);
            };
            chain_schedule(chunks, fetch, nothing);
        }
    }
    if (margin_floats) *margin_floats = margin == INT64_MAX ? -1 : static_cast<long>(margin);
    return violations;
}

void ctc_debug_set_overlap(int percent) { ctc::g_overlap.store(percent < 0 ? -1 : percent, std::memory_order_relaxed); }

void ctc_debug_set_sequential_chains(int on)
{
    ctc::g_sequential_chains.store(on ? 1 : 0, std::memory_order_relaxed);
}

void ctc_debug_set_poll_budget(int polls)
{
    ctc::g_poll_budget.store(polls < 0 ? ctc::kDefaultPollBudget : polls, std::memory_order_relaxed);
}

void ctc_debug_set_end_polls(int polls)
{
    ctc::g_end_polls.store(polls < 0 ? ctc::kDefaultEndPolls : polls, std::memory_order_relaxed);
}

}  // extern "C"
