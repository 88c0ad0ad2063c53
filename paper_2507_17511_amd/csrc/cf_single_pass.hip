// Single-pass kernel for channel scales (arxiv 2507.17511, App. D
// "Quantization": v_j = mean_i |z_ij| needs every token of a channel before
// any code of that channel can be chosen).
//
// A two-kernel design reads x and recon twice from HBM.  Here a workgroup
// keeps its share of the operands in registers across the reduction instead:
//   item  = p_rows x 128 channels of one tensor, owned by one workgroup of 256
//           lanes (16 chunks of 8 channels x 16 row-lanes), 128 VGPRs of raw
//           operands per lane: 256 rows of bf16 x and recon (Sec. 3.2's feedback
//           folded into the residual against the reconstruction), half as many
//           of fp32, half as many again when the error buffer is an operand too
//           (the literal and the no-feedback recursions); for contexts of short
//           tensors half as tall and 256 channels wide (32 chunks x 8 row-lanes),
//           for contexts of tall ones twice as tall and 64 wide (8 x 32);
//           k_short_items, small calls: 128 x 64 (half as tall for fp32);
//   group = the items of one such stripe of one tensor; only they have
//           to agree on that stripe's scales, so there is no grid-wide barrier,
//           and different groups drift apart, which keeps HBM busy while some
//           workgroups wait.
// What bounds it is HBM in large calls (114 x [4096, 3072] bf16 1-bit 14.5 GB in 2.64 ms, 5.5 TB/s), waiting for the slowest of a group in tall
// ones (30 x [17776, 1920], 35 items a group, 8.2 GB in 1.66 to 1.74 ms, 4.7 to 4.9 TB/s), and in small calls the chain of an item: its
// operands, the exchange, and its code, which a CU fetches once per launch.  Those take short items (SHORT): a quarter of the rows a lane.
// Per item: load -> |z| tree over the lane's rows -> LDS tree over row-lanes
// -> publish the item's partial (an aligned power-of-two block of the channel
// tree) -> every workgroup of the group fetches the group's partials as they
// appear and finishes the tree itself -> scales -> codes, error and
// reconstruction straight from the registers.
//
// A partial is its own ready flag: it is no less than zero, and its sign bit, which it does not need, tells in which of two
// alternating calls it was stored.  Every item keeps a byte in the workspace with the sign of its last call and turns it over
// when it is done (a word each, whose lines come from memory one for four workgroups of an XCD, cost 114 x [4096, 3072] 15 us); the items of a group always run in the same calls, so they agree on it, the slots need no clearing between
// calls, and a captured call can be replayed.  One store and one load per hop; no counter, no launch before the kernel.
//
// Forward progress does not depend on how the hardware schedules workgroups.
// Items are numbered group-major and dealt to the workgroups in index order
// (or, for short tensors, XCD-major: see the kernel), so the items of a group
// start at about the same time and a waiter normally sees the partials within
// microseconds.  But no workgroup waits for ever: one that has polled a slot
// `sp_wait_polls` times in vain GIVES ITS ITEM UP for the time being and does the missing
// items' sums itself, one after the other: it loads such an item's operands, publishes its partial, and then starts
// its own item again, whose operands it has dropped.  Up to that point it has
// written nothing but partials (codes, error and reconstruction are all
// written after the wait).  The missing item may start meanwhile, and writes over its operands (error and reconstruction are
// updated in place) once all partials of its group are there, its own among them: so the helper stores with a
// compare-and-swap against the partial of the call before.  If that finds one, the item had written nothing yet and the helper
// read what it should; if not, the item's own partial stands.  Both compute the same bits.  This needs every partial of an item to be
// where other XCDs look before the item writes over an operand: the waves that publish wait for their stores (publish_landed) ahead of
// the barrier that all of the item's other stores lie behind.  A helper's loads of operands have returned before its swap, which needs their sum.  A workgroup helps each item of its
// group once at most, so it always ends, on a device shared with other kernels and with a dispatcher that does not go by
// index too, and the outputs are the same bits either way.
#include <cstddef>
#include <cstring>

#include "cf_device.h"
#include "cf_internal.h"

namespace cf {
namespace {

using namespace dev;

__device__ __forceinline__ void publish(uint32_t *p, uint32_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// The wave's stores, publish() among them, are where every XCD sees them: agent-scope stores go through to memory, and loads and stores count down one counter.
__device__ __forceinline__ void publish_landed() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ __forceinline__ uint32_t fetch(const uint32_t *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// What is the same for the whole workgroup and nobody writes while it is looked at, by way of the scalar cache.
template <class T> __device__ __forceinline__ T scalar_load(uint64_t at)
{
    T out;
    const __attribute__((address_space(4))) uint32_t *const from = (const __attribute__((address_space(4))) uint32_t *)at;
    uint32_t words[sizeof(T) / 4];
#pragma unroll
    for (unsigned k = 0; k < sizeof(T) / 4; ++k) words[k] = from[k];
    __builtin_memcpy(&out, words, sizeof(T));
    return out;
}

constexpr int kPollBatch = 8;       // leaves fetched (and re-fetched) together

// tree_over whose leaves are other workgroups' partials: a leaf that does not have the call's sign yet is
// fetched again until its owner has stored it, at most max_polls times (then `missing` is its number and the
// result is meaningless).  The data word is its own ready flag, so a group needs no counter and no
// second round trip.
template <bool IS_MAX, int LV>
__device__ __forceinline__ float tree_over_published(int n, const uint32_t *mine, int64_t stride, uint32_t sign, uint32_t max_polls, int &missing)
{
    constexpr int NB = kPollBatch;
    float stack[LV];
#pragma unroll
    for (int l = 0; l < LV; ++l) stack[l] = 0.0f;
    const int nbatch = (n + NB - 1) / NB;
    int bpad = 1;
    while (bpad < nbatch) bpad <<= 1;
    for (int b = 0; b < bpad; ++b) {
        uint32_t words[NB];         // nothing is done with them before all are asked for
#pragma unroll
        for (int u = 0; u < NB; ++u) words[u] = (b * NB + u < n) ? fetch(mine + (int64_t)(b * NB + u) * stride) : sign;
        uint32_t polls = 0;
        for (;;) {
            uint32_t pending = 0;
#pragma unroll
            for (int u = 0; u < NB; ++u) pending |= ((words[u] ^ sign) >> 31) << u;
            if (pending == 0) break;
            if (polls >= max_polls) {
                const int q = b * NB + __builtin_ctz(pending);
                missing = q < missing ? q : missing;
                break;
            }
            __builtin_amdgcn_s_sleep(1);
#pragma unroll
            for (int u = 0; u < NB; ++u)
                if ((pending >> u) & 1u) words[u] = fetch(mine + (int64_t)(b * NB + u) * stride);
            ++polls;
        }
        float vals[NB];
#pragma unroll
        for (int u = 0; u < NB; ++u) vals[u] = __uint_as_float(words[u] ^ sign);
        // balanced tree over the batch: neighbours, then neighbours of neighbours, ...
#pragma unroll
        for (int w = 1; w < NB; w <<= 1)
#pragma unroll
            for (int u = 0; u < NB; u += 2 * w) vals[u] = comb<IS_MAX>(vals[u], vals[u + w]);
        tree_push<LV, IS_MAX>(stack, vals[0], b);
    }
    return tree_top<LV, IS_MAX>(stack);
}

// SCH: channels per stripe (kStripeChannels, kStripeChannelsWide or kStripeChannelsSlim); the 256 lanes are SCH / 8 chunks across
// by 2048 / SCH row-lanes down.
template <int SCH> struct alignas(16) Shared {
    float red[kPersistThreads / (SCH / kChunk)][SCH];       // 8 KB: level 2 of the tree; afterwards the waves' patches for whole-line stores
    float part[kPersistThreads];    // level 3: the tree over a share of the group's partials
    float scale[SCH];
    int missing;                // the first item whose partial did not come in time, or kNoneMissing
    uint32_t sign;              // of the call's partials: kept here for the end, where a load would wait for the stores before it
};
constexpr int kNoneMissing = 0x7fffffff;
constexpr uint32_t kMaxHelps = 4096u;

// BLOCKS: rows that are no whole blocks of 64 bytes, whose parts at a stripe's ends are left to the L2 to merge (make_layout says for which, kBlocksBytes from which size on).
// help: do no more than store the partial of item rb, which is another workgroup's.  max_polls: of a missing partial.
// Returns kNoneMissing when the item is done, else the item whose partial was missing; nothing but a partial has been written then.
template <int DT, int BITS, int EF, int ET, bool FUSED, int SCH, bool SHORT, bool BLOCKS>
__device__ __forceinline__ int persist_item(const BatchView &v, const TensorDev &d, const TensorPtrs &p, int stripe,
                                            int rb, uint32_t sign, uint32_t max_polls, bool help, Shared<SCH> &sh)
{
    constexpr int kStripeChannels = SCH, kStripeChunks = SCH / kChunk, kRowLanes = kPersistThreads / kStripeChunks;
    constexpr int RPT = single_pass_rows_per_lane(DT, EF) / (SHORT ? kShortFraction : 1);       // rows per lane
    constexpr bool IS_MAX = BITS == 4;
    constexpr bool HAS_B = EF != EF_NAIVE;                      // recon is an operand
    constexpr bool HAS_E = EF == EF_LITERAL || EF == EF_OFF;    // the error buffer is an operand
    const int tid = (int)threadIdx.x, cl = tid & (kStripeChunks - 1), rl = tid / kStripeChunks;
    const int chunk = stripe * kStripeChunks + cl;
    const bool cvalid = chunk < d.n_chunks;
    const int64_t row0 = (int64_t)rb * d.p_rows + rl * RPT;
    const int64_t C = d.n_channels;

    // ---- load the lane's rows (raw), all in flight at once
    Raw8<DT> xr[RPT], br[HAS_B ? RPT : 1];
    Raw8<ET> er[HAS_E ? RPT : 1];
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
        const int64_t row = row0 + k;
        if (cvalid && row < d.n_tokens) {
            const int64_t e = row * C + (int64_t)chunk * kChunk;
            xr[k].load_stream(p.x, e);       // read once: keep the caches for the partials and the outputs
            if (HAS_B) br[HAS_B ? k : 0].load_stream(p.recon, e);
            if (HAS_E) er[HAS_E ? k : 0].load_stream(p.err, e);
        } else {                                    // zero padding of the tree / masked lanes
            xr[k].zero();
            if (HAS_B) br[HAS_B ? k : 0].zero();
            if (HAS_E) er[HAS_E ? k : 0].zero();
        }
    }
    const F8 none = {};

    // ---- a3, level 1: balanced tree over the lane's RPT consecutive rows
    // (a binary-counter stack: after row k the slots hold the partial trees of the rows seen so far;
    // k is a compile-time constant after unrolling, so every branch below folds away)
    constexpr int LVR = (RPT == 32) ? 6 : (RPT == 16) ? 5 : (RPT == 8) ? 4 : (RPT == 4) ? 3 : 2;
    F8 st[LVR];
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
        F8 z = residual8<EF>(xr[k].widen(), HAS_B ? br[HAS_B ? k : 0].widen() : none, HAS_E ? er[HAS_E ? k : 0].widen() : none);
        F8 a;
#pragma unroll
        for (int j = 0; j < 8; ++j) a.v[j] = fabsf(z.v[j]);
        bool carry = true;
#pragma unroll
        for (int l = 0; l < LVR; ++l) {
            if (carry) {
                if ((k >> l) & 1) {
#pragma unroll
                    for (int j = 0; j < 8; ++j) a.v[j] = comb<IS_MAX>(st[l].v[j], a.v[j]);
                } else {
                    st[l] = a;
                    carry = false;
                }
            }
        }
    }
    {
        const F8 &top = st[LVR - 1];
        f32x4 *dst = reinterpret_cast<f32x4 *>(&sh.red[rl][cl * kChunk]);
        f32x4 lo, hi;
        lo.x = top.v[0]; lo.y = top.v[1]; lo.z = top.v[2]; lo.w = top.v[3];
        hi.x = top.v[4]; hi.y = top.v[5]; hi.z = top.v[6]; hi.w = top.v[7];
        dst[0] = lo;
        dst[1] = hi;
    }
    if (tid == 0) {
        sh.missing = kNoneMissing;
        sh.sign = sign;
    }
    __syncthreads();

    // ---- level 2: tree over the row-lanes (consecutive RPT-row blocks); one lane per channel
    const bool owner = tid < kStripeChannels;
    const int64_t col = owner ? (int64_t)stripe * kStripeChannels + tid : C;
    uint32_t *partial = reinterpret_cast<uint32_t *>(v.workspace + d.p_partial_off);
    float res = 0.0f;
    if (owner) {
        float lanes[kRowLanes];
#pragma unroll
        for (int q = 0; q < kRowLanes; ++q) lanes[q] = sh.red[q][tid];
#pragma unroll
        for (int w = 1; w < kRowLanes; w <<= 1)
#pragma unroll
            for (int q = 0; q < kRowLanes; q += 2 * w) lanes[q] = comb<IS_MAX>(lanes[q], lanes[q + w]);
        res = lanes[0];
        if (col < C && d.p_n_rb > 1) {
            uint32_t *const slot = partial + (int64_t)rb * C + col;
            const uint32_t word = (__float_as_uint(res) & ~kPartialSign) | sign;
            if (!help) {
                publish(slot, word);
            } else {        // unless its owner, or another helper, has been faster
                uint32_t old = fetch(slot);
                if ((old & kPartialSign) != sign)
                    (void)__hip_atomic_compare_exchange_strong(slot, &old, word, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
    if (help) return kNoneMissing;
    // The partials are agent-scope atomic stores (written through to where the other XCDs read them)
    // and every partial is its own ready flag: nothing to drain here, no arrival to count.

    // ---- level 3: the same tree continued over the group's item partials as they appear, then the scale.  All 256 lanes fetch: of a
    // 64-channel stripe's lanes each takes a quarter of the tree, of a 128-channel one's half, so that there are as few round
    // trips one after the other as can be.  An item that is alone in its group has nothing to exchange.
    constexpr int kShares = kPersistThreads / SCH;
    if (d.p_n_rb > 1) {
        const int column = stripe * kStripeChannels + (tid & (SCH - 1)), share = tid / SCH;
        int per = kPollBatch;                       // leaves of a share, a power of two: no fewer than one round trip brings
        while (per * kShares < d.p_n_rb) per <<= 1;
        const int lo = share * per, count = d.p_n_rb - lo < per ? d.p_n_rb - lo : per;
        float sum = 0.0f;
        if (column < C && count > 0) {
            int missing = kNoneMissing;
            sum = tree_over_published<IS_MAX, 10>(count, partial + (int64_t)lo * C + column, C, sign, max_polls, missing);
            if (missing != kNoneMissing) atomicMin(&sh.missing, lo + missing);          // a partial did not come in time
        }
        if (kShares > 1 && d.p_n_rb > per) {
            sh.part[tid] = sum;
            __syncthreads();
            if (owner) {
                float shares[kShares];
#pragma unroll
                for (int q = 0; q < kShares; ++q) shares[q] = sh.part[q * SCH + tid];
#pragma unroll
                for (int w = 1; w < kShares; w <<= 1)
#pragma unroll
                    for (int q = 0; q < kShares; q += 2 * w) shares[q] = comb<IS_MAX>(shares[q], shares[q + w]);
                sum = shares[0];
            }
        }
        res = sum;
    }
    if (col < C) {
        const float s = IS_MAX ? res / 7.0f : res / (float)d.n_tokens;
        sh.scale[tid] = s;
    }
    publish_landed();       // costs nothing: the loads of the partials came after
    __syncthreads();
    const int missing_item = __builtin_amdgcn_readfirstlane(sh.missing);
    if (missing_item != kNoneMissing) return missing_item;
    if (rb == 0 && col < C) gmut<float>(p.scales)[col] = sh.scale[tid];

    // ---- a4-a8 from the registers.  z is formed again from the raw operands: keeping the first
    // phase's fp32 residuals alive across the wait would double the register footprint.
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
        xr[k].opaque();
        if (HAS_B) br[HAS_B ? k : 0].opaque();
        if (HAS_E) er[HAS_E ? k : 0].opaque();
    }
    F8 s;
    {
        const f32x4 *src = reinterpret_cast<const f32x4 *>(&sh.scale[cl * kChunk]);
        f32x4 a = src[0], b = src[1];
        s.v[0] = a.x; s.v[1] = a.y; s.v[2] = a.z; s.v[3] = a.w;
        s.v[4] = b.x; s.v[5] = b.y; s.v[6] = b.z; s.v[7] = b.w;
    }
    const int64_t row_bytes = C * BITS / 8;
    const bool wide = (d.n_channels & 31) == 0;
    // fp32 error rows go out as whole lines (see lines_exchange): a run is the kStripeChunks lanes of one row
    // segment; the wave's patch is its 2 KB of `red`, which nobody reads any more
    float *patch = &sh.red[0][0] + (tid >> 6) * 512;
    const int run_valid = d.n_chunks - stripe * kStripeChunks, run_chunks = run_valid < kStripeChunks ? run_valid : kStripeChunks;
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
        const int64_t row = row0 + k;
        const bool rvalid = row < d.n_tokens;
        __builtin_amdgcn_sched_barrier(0);      // one row at a time: keeps the live set inside the register budget
        const int64_t e = row * C + (int64_t)chunk * kChunk;
        const F8 b = HAS_B ? br[HAS_B ? k : 0].widen() : none;
        const F8 eold = HAS_E ? er[HAS_E ? k : 0].widen() : none;
        const F8 z = residual8<EF>(xr[k].widen(), b, eold);         // masked lanes and rows hold zeros
        F8 dq;
        uint32_t packed = quant8<BITS>(z, s, dq);
        if (rvalid && cvalid) store_codes_wide<BITS>(p.codes + row * row_bytes, chunk, packed, wide);
        F8 enew;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            float lost = z.v[j] - dq.v[j];
            if (EF == EF_OFF) lost = eold.v[j] + lost;
            enew.v[j] = lost;
        }
        if (ET == F32) {
            f32x4 pieces[2];
            lines_exchange<kStripeChunks>(patch, tid & 63, enew, pieces);
            if (rvalid) {
                float *const run = static_cast<float *>(p.err) + row * C + (int64_t)stripe * kStripeChannels;
                if (BLOCKS) lines_store_blocks<kStripeChunks>(run, cl, run_valid, pieces);
                else lines_store_stream<kStripeChunks>(run, cl, run_valid, pieces);
            }
        } else if (rvalid && cvalid) {
            Raw8<ET> eo;
            eo.narrow(enew);
            if (!BLOCKS || WholeBlocks(static_cast<uint16_t *>(p.err) + (e - cl * kChunk), run_chunks).has(cl)) {
                eo.store_stream(p.err, e);
                asm volatile("");
            } else {
                eo.store(p.err, e);
            }
        }
        if (FUSED && rvalid && cvalid) {
            F8 nb;
#pragma unroll
            for (int j = 0; j < 8; ++j) nb.v[j] = (EF == EF_NAIVE) ? dq.v[j] : b.v[j] + dq.v[j];
            Raw8<DT> out;
            out.narrow(nb);
            if (DT == BF16 && (!BLOCKS || WholeBlocks(static_cast<uint16_t *>(p.recon) + (e - cl * kChunk), run_chunks).has(cl))) {
                out.store_stream(p.recon, e);
                asm volatile("");
            } else {
                out.store(p.recon, e);
            }
        }
    }
    return kNoneMissing;
}

template <int EF, int ET, bool FUSED, int SCH, bool BLOCKS>
__global__ __launch_bounds__(kPersistThreads, 2) void k_single_pass(SinglePassArgs args)
{
    const BatchView &v = args.v;
    const LaunchRange &r = args.r;
    __shared__ Shared<SCH> sh;
    // Workgroups are handed to the 8 XCDs in turn (blockIdx.x % 8).  Taking item b in workgroup b runs the
    // consecutive items of a reduction group on different XCDs at the same time.  Short tensors
    // (few items per group) do better XCD-major, a run of consecutive items per XCD; the host chooses.
    const uint32_t n_items = r.item_hi - r.item_lo;
    // of direct calls; asked for along with the range, which says whether it is one
    uint32_t begins[kDirectTensors];
#pragma unroll
    for (int q = 1; q < kDirectTensors; ++q) begins[q] = args.direct.descs[q].p_item_begin;
    asm volatile("" : "+s"(begins[1]), "+s"(begins[2]), "+s"(begins[3]), "+s"(begins[4]), "+s"(begins[5]), "+s"(begins[6]), "+s"(begins[7]));
    static_assert(kDirectTensors == 8, "all of them");
    uint32_t vb = blockIdx.x;
    if (r.sp_xcd_major) {
        const uint32_t q = gridDim.x >> 3, rem = gridDim.x & 7u, xcd = blockIdx.x & 7u;
        vb = xcd * q + (xcd < rem ? xcd : rem) + (blockIdx.x >> 3);
    }
    uint32_t gave_up = 0u;          // how often, at this item
    int at = -1;                    // the item of the group that this workgroup helps; -1: it does its own
    for (uint32_t k = vb; k < n_items;) {
        uint32_t item = __builtin_amdgcn_readfirstlane(r.item_lo + k);
        asm volatile("" : "+s"(item));      // a second turn, which hardly ever comes, finds everything anew: kept for it, it would cost registers
        uint64_t desc, set;
        if (r.direct && r.count <= kDirectTensors) {        // both are among the arguments
            uint32_t t = 0;
#pragma unroll
            for (int q = 1; q < kDirectTensors; ++q) t += item >= begins[q] ? 1u : 0u;
            desc = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(SinglePassArgs, direct.descs) + t * sizeof(TensorDev);
            set = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(SinglePassArgs, direct.sets) + t * sizeof(TensorPtrs);
        } else {
            const uint32_t t = scalar_load<uint32_t>((uint64_t)(v.item_tensor + item));
            desc = (uint64_t)(v.descs + t);
            set = r.direct ? (uint64_t)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(SinglePassArgs, direct.sets) + (t - (uint32_t)r.first) * sizeof(TensorPtrs)
                           : (uint64_t)(v.ptrs + t);
        }
        TensorDev d = scalar_load<TensorDev>(desc);         // by value: scalar registers, never re-read
        TensorPtrs p = scalar_load<TensorPtrs>(set);
        uint32_t state = scalar_load<uint32_t>((uint64_t)v.item_state + (item & ~3u));       // four items' bytes
        asm volatile("" : "+s"(d.n_tokens), "+s"(d.n_channels), "+s"(d.n_chunks), "+s"(d.dtype), "+s"(d.bits), "+s"(d.p_partial_off), "+s"(d.p_rows),
                          "+s"(d.p_n_rb), "+s"(d.p_item_begin), "+s"(p.x), "+s"(p.recon), "+s"(p.err), "+s"(p.codes), "+s"(p.scales), "+s"(state));  // one wait for all of them
        const uint32_t local = item - d.p_item_begin;               // group-major: stripe, then row block
        const int stripe = (int)(local / (uint32_t)d.p_n_rb);
        // The groups of a tensor begin on different XCDs unless its row blocks number a multiple of 8: each is turned, so that a row block, all but for a group's
        // last few, is on the XCD of its number in every stripe, whose L2 then sees the stripes' pieces of a line and of a code row.  In order / turned, us, [3300, 3080]
        // (13 row blocks) 487 / 449, [5000, 3080] (20) 506 / 460, 30 x [17776, 1920] (35) 1716 / 1662, [3268, 1504] in short items (26) 15.4 / 14.4.
        int rb = (int)(local % (uint32_t)d.p_n_rb);
        const int turned = rb + (int)((k - (uint32_t)rb) & 7u);
        if (!r.sp_xcd_major && d.p_n_rb >= 8) rb = turned >= d.p_n_rb ? turned - d.p_n_rb : turned;
        if (at >= 0) rb = at;
        const uint32_t sign = ~(state << (24u - 8u * (item & 3u))) & kPartialSign;     // nobody else writes the byte, and this workgroup at the very end
        const uint32_t polls = gave_up ? 0u : r.sp_wait_polls;
        int missing;
        if (d.dtype == BF16) {
            if (d.bits == 1) missing = persist_item<BF16, 1, EF, ET, FUSED, SCH, false, BLOCKS>(v, d, p, stripe, rb, sign, polls, at >= 0, sh);
            else if (d.bits == 2) missing = persist_item<BF16, 2, EF, ET, FUSED, SCH, false, BLOCKS>(v, d, p, stripe, rb, sign, polls, at >= 0, sh);
            else missing = persist_item<BF16, 4, EF, ET, FUSED, SCH, false, BLOCKS>(v, d, p, stripe, rb, sign, polls, at >= 0, sh);
        } else {
            if (d.bits == 1) missing = persist_item<F32, 1, EF, ET, FUSED, SCH, false, BLOCKS>(v, d, p, stripe, rb, sign, polls, at >= 0, sh);
            else if (d.bits == 2) missing = persist_item<F32, 2, EF, ET, FUSED, SCH, false, BLOCKS>(v, d, p, stripe, rb, sign, polls, at >= 0, sh);
            else missing = persist_item<F32, 4, EF, ET, FUSED, SCH, false, BLOCKS>(v, d, p, stripe, rb, sign, polls, at >= 0, sh);
        }
        // The same for all, which the compiler does not see: the loop it then makes, of lanes that leave one by one, took up to 9 % longer in one
        // pass of twenty (114 x [4096, 3072], 2640 us and now and then 2700 to 2900).
        missing = __builtin_amdgcn_readfirstlane(missing);
        __syncthreads();            // the shared arrays are used again
        if (at >= 0) {              // helped; now its own item again
            at = -1;
            continue;
        }
        if (missing != kNoneMissing) {
            at = missing;
            if (++gave_up <= kMaxHelps) continue;       // always: each turn brings a partial that was missing, and no group has that many
            if (threadIdx.x == 0) __hip_atomic_store(v.error_flag, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (threadIdx.x == 0) {
            *gmut<uint8_t>(v.item_state + r.item_lo + k) = (uint8_t)(sh.sign >> 24 | (gave_up ? 1u : 0u));
            if (k == 0) {               // which items the call had, for cf_given_up_items
                *gmut<uint32_t>(v.error_flag + kLastItemsWord) = r.item_lo;
                *gmut<uint32_t>(v.error_flag + kLastItemsWord + 1) = r.item_hi;
                *gmut<uint32_t>(v.error_flag + kLastItemsWord + 2) = 0u;
            }
        }
        at = -1;
        gave_up = 0u;
        k += gridDim.x;
    }
}

// Short items.  A call of them is over before a large one's first operands arrive, so what it waits for is the chain of an item, and of that its descriptor was the
// longest link: range, then which tensor, then descriptor and state, each a load from memory that waits for the one before (3 of the 8 us that one tensor of
// [256, 64] took).  Here the grid says which item a workgroup has: x the row block, y the stripe, z the tensor, as many as the largest tensor of the call has, and
// the descriptor and pointers come with the range, in one round; the state comes while the operands do.  Tensors of unlike shapes would leave most of such a grid
// empty (32,768 workgroups for the 512 items of 7 x [8192, 64] with [64, 4096], 25.3 us): those calls have a workgroup per item, which finds its tensor among the
// arguments and asks again (11.1).
template <int ET, bool FUSED, bool BLOCKS>
__global__ __launch_bounds__(kPersistThreads, 4) void k_short_items(ShortArgs args)
{
    constexpr int EF = EF_RECON, SCH = kShortStripeChannels;
    const BatchView &v = args.v;
    const LaunchRange &r = args.r;
    __shared__ Shared<SCH> sh;
    const uint64_t given = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
    TensorDev d;
    TensorPtrs p;
    const auto load = [&](uint32_t t) {
        d = scalar_load<TensorDev>(given + offsetof(ShortArgs, descs) + t * sizeof(TensorDev));
        p = scalar_load<TensorPtrs>(given + offsetof(ShortArgs, sets) + t * sizeof(TensorPtrs));
    };
    load(blockIdx.z);
    uint8_t *states = v.item_state;
    uint32_t kind = r.sp_short;
    asm volatile("" : "+s"(d.n_tokens), "+s"(d.n_channels), "+s"(d.n_chunks), "+s"(d.dtype), "+s"(d.bits), "+s"(d.p_partial_off), "+s"(d.p_rows), "+s"(d.p_n_rb),
                      "+s"(d.p_n_stripes), "+s"(d.p_item_begin), "+s"(p.x), "+s"(p.recon), "+s"(p.err), "+s"(p.codes), "+s"(p.scales), "+s"(states), "+s"(kind));      // one wait for all of them
    int stripe = (int)blockIdx.y, in_order = (int)blockIdx.x;
    uint32_t group_begin = (blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x;           // the group's first workgroup
    if (__builtin_expect(kind == 2u, 0)) {          // out of the way: the code of the others comes from memory too
        const uint32_t first_item = args.descs[0].p_item_begin, item = first_item + blockIdx.x;
        uint32_t t = 0;
#pragma unroll
        for (int q = 1; q < kDirectTensors; ++q) t += item >= args.descs[q].p_item_begin ? 1u : 0u;
        load(t);
        const uint32_t local = item - d.p_item_begin;               // group-major: stripe, then row block
        stripe = (int)(local / (uint32_t)d.p_n_rb);
        in_order = (int)(local % (uint32_t)d.p_n_rb);
        group_begin = blockIdx.x - (uint32_t)in_order;
    } else if (in_order >= d.p_n_rb || stripe >= d.p_n_stripes) {
        return;                     // uniform over the workgroup: a larger tensor's
    }
    const uint32_t item = d.p_item_begin + (uint32_t)stripe * (uint32_t)d.p_n_rb + (uint32_t)in_order;
    const uint32_t state = scalar_load<uint32_t>((uint64_t)states + (item & ~3u));      // four items' bytes
    // turned as in k_single_pass
    const int turned = in_order + (int)(group_begin & 7u);
    const int mine = d.p_n_rb < 8 ? in_order : turned >= d.p_n_rb ? turned - d.p_n_rb : turned;
    const uint32_t sign = ~(state << (24u - 8u * (item & 3u))) & kPartialSign;     // nobody else writes the byte, and this workgroup at the very end
    uint32_t gave_up = 0u;          // how often
    int at = -1;                    // the item of the group that this workgroup helps; -1: it does its own
    for (;;) {
        const int rb = at >= 0 ? at : mine;
        const uint32_t polls = gave_up ? 0u : r.sp_wait_polls;
        int missing;
        if (d.dtype == BF16) {
            if (d.bits == 1) missing = persist_item<BF16, 1, EF, ET, FUSED, SCH, true, BLOCKS>(v, d, p, stripe, rb, sign, polls, at >= 0, sh);
            else if (d.bits == 2) missing = persist_item<BF16, 2, EF, ET, FUSED, SCH, true, BLOCKS>(v, d, p, stripe, rb, sign, polls, at >= 0, sh);
            else missing = persist_item<BF16, 4, EF, ET, FUSED, SCH, true, BLOCKS>(v, d, p, stripe, rb, sign, polls, at >= 0, sh);
        } else {
            if (d.bits == 1) missing = persist_item<F32, 1, EF, ET, FUSED, SCH, true, BLOCKS>(v, d, p, stripe, rb, sign, polls, at >= 0, sh);
            else if (d.bits == 2) missing = persist_item<F32, 2, EF, ET, FUSED, SCH, true, BLOCKS>(v, d, p, stripe, rb, sign, polls, at >= 0, sh);
            else missing = persist_item<F32, 4, EF, ET, FUSED, SCH, true, BLOCKS>(v, d, p, stripe, rb, sign, polls, at >= 0, sh);
        }
        missing = __builtin_amdgcn_readfirstlane(missing);      // see k_single_pass
        if (at < 0 && missing == kNoneMissing) break;
        __syncthreads();            // the shared arrays are used again
        if (at >= 0) {              // helped; now its own item again
            at = -1;
            continue;
        }
        at = missing;
        if (++gave_up <= kMaxHelps) continue;       // always: each turn brings a partial that was missing, and no group has that many
        if (threadIdx.x == 0) __hip_atomic_store(v.error_flag, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        break;
    }
    if (threadIdx.x == 0) {
        *gmut<uint8_t>(v.item_state + item) = (uint8_t)(sh.sign >> 24 | (gave_up ? 1u : 0u));
        if (item == r.item_lo) {        // which items the call had, for cf_given_up_items
            *gmut<uint32_t>(v.error_flag + kLastItemsWord) = r.item_lo;
            *gmut<uint32_t>(v.error_flag + kLastItemsWord + 1) = r.item_hi;
            *gmut<uint32_t>(v.error_flag + kLastItemsWord + 2) = 1u;
        }
    }
}

// States and partials as before a first call; the states byte by byte: other tensors' lie next to them.
__global__ void k_fresh_partials(u32x4 *partials, uint64_t n_vec, uint8_t *states, uint32_t n_states)
{
    const uint64_t at = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x, step = (uint64_t)gridDim.x * blockDim.x;
    const u32x4 fill = (u32x4)(kFreshPartials);
    for (uint64_t i = at; i < n_vec; i += step) *gmut<u32x4>(partials + i) = fill;
    for (uint64_t i = at; i < n_states; i += step) *gmut<uint8_t>(states + i) = (uint8_t)kFreshPartials;
}

template <int EF, int ET, bool FUSED, int SCH> const void *persistent_fn(bool blocks)
{
    if constexpr (EF == EF_RECON)
        if (blocks) return reinterpret_cast<const void *>(&k_single_pass<EF_RECON, ET, FUSED, SCH, true>);
    return reinterpret_cast<const void *>(&k_single_pass<EF, ET, FUSED, SCH, false>);
}

template <int EF, int SCH> const void *pick_width(int err_dtype, bool fused, bool blocks)
{
    if (err_dtype == BF16) return fused ? persistent_fn<EF, BF16, true, SCH>(blocks) : persistent_fn<EF, BF16, false, SCH>(blocks);
    return fused ? persistent_fn<EF, F32, true, SCH>(blocks) : persistent_fn<EF, F32, false, SCH>(blocks);
}

template <int EF> const void *pick_ef(int err_dtype, bool fused, bool wide, bool slim, bool blocks)
{
    if (slim) return pick_width<EF, kStripeChannelsSlim>(err_dtype, fused, blocks);
    return wide ? pick_width<EF, kStripeChannelsWide>(err_dtype, fused, blocks) : pick_width<EF, kStripeChannels>(err_dtype, fused, blocks);
}

const void *pick(int ef, int err_dtype, bool fused, bool wide, bool slim, bool blocks)
{
    if (ef == EF_LITERAL) return pick_ef<EF_LITERAL>(err_dtype, fused, wide, slim, false);
    if (ef == EF_OFF) return pick_ef<EF_OFF>(err_dtype, fused, wide, slim, false);
    if (ef == EF_NAIVE) return pick_ef<EF_NAIVE>(err_dtype, fused, wide, slim, false);
    return pick_ef<EF_RECON>(err_dtype, fused, wide, slim, blocks);
}

// One stripe width, and the default feedback mode alone: with a third operand a quarter of the rows would be one or two a lane (naive compression
// would have as many as the default; no kernels for it here).
template <int ET, bool FUSED> const void *short_fn(bool blocks)
{
    if constexpr (ET == F32 || FUSED)       // the others write less than kShortBlocksBytes
        if (blocks) return reinterpret_cast<const void *>(&k_short_items<ET, FUSED, true>);
    return reinterpret_cast<const void *>(&k_short_items<ET, FUSED, false>);
}

const void *pick_short(int err_dtype, bool fused, bool blocks)
{
    if (err_dtype == BF16) return fused ? short_fn<BF16, true>(blocks) : short_fn<BF16, false>(blocks);
    return fused ? short_fn<F32, true>(blocks) : short_fn<F32, false>(blocks);
}

hipError_t launch_short_items(const BatchView &v, const LaunchRange &r, int err_dtype, bool fused, hipStream_t s)
{
    ShortArgs a;
    a.v = v;
    a.r = r;
    std::memset(static_cast<void *>(a.sets), 0, sizeof a.sets);
    std::memset(static_cast<void *>(a.descs), 0, sizeof a.descs);
    for (int k = 0; k < kDirectTensors; ++k) {
        if (k < r.count) {
            a.sets[k] = r.direct[k];
            a.descs[k] = r.direct_descs[k];
        } else {
            a.descs[k].p_item_begin = ~0u;      // behind every item
        }
    }
    const ShortGrid grid = short_grid(r.direct_descs, r.count);
    a.r.sp_short = grid.flat ? 2u : 1u;
    void *args[] = {&a};
    return hipLaunchKernel(pick_short(err_dtype, fused, r.sp_blocks != 0), dim3(grid.x, grid.y, grid.z), dim3(kPersistThreads), args, 0, s);
}

}  // namespace

int persistent_max_blocks_per_cu(int ef, int err_dtype, bool fused, bool wide, bool slim)
{
    int n = 0;
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, pick(ef, err_dtype, fused, wide, slim, false), kPersistThreads, 0);
    if (e != hipSuccess) { (void)hipGetLastError(); return 0; }
    return n;
}

hipError_t launch_fresh_partials(uint8_t *partials, size_t bytes, uint8_t *states, uint32_t n_states, hipStream_t s)
{
    const uint64_t n_vec = bytes / 16, want = ((n_vec > n_states ? n_vec : n_states) + 255) / 256;
    if (want == 0) return hipSuccess;
    hipLaunchKernelGGL(k_fresh_partials, dim3((unsigned)(want < 2048 ? want : 2048)), dim3(256), 0, s, reinterpret_cast<u32x4 *>(partials), n_vec, states, n_states);
    return hipGetLastError();
}

// one_shot: one workgroup per item instead of a smaller grid whose workgroups loop over the items.
// A workgroup that loops has to drain its stores before its next loads count as returned (the loads and
// stores of a wave share one in-order counter); one that exits leaves the draining to the memory system
// while the next workgroup already loads: measured faster by 15 % (114 x [4096, 3072] bf16: 2.65 against 3.04 ms).  Neither form needs co-residency to
// finish (see the top of the file); the looping grid is for callers who share the device with other work
// and want the codec to hold a fixed number of workgroup slots.
hipError_t launch_single_pass(const BatchView &v, const LaunchRange &r, int ef, int err_dtype, bool fused, bool wide, int grid,
                             bool one_shot, hipStream_t s)
{
    if (r.item_hi == r.item_lo) return hipSuccess;
    if (r.sp_short) return launch_short_items(v, r, err_dtype, fused, s);
    uint32_t items = r.item_hi - r.item_lo;
    if ((uint32_t)grid > items) grid = (int)items;
    if (grid < 1) grid = 1;
    const uint32_t n_wg = one_shot ? items : (uint32_t)grid;
    SinglePassArgs a;
    a.v = v;
    a.r = r;
    std::memset(static_cast<void *>(&a.direct), 0, sizeof a.direct);
    if (r.direct) std::memcpy(a.direct.sets, r.direct, sizeof(TensorPtrs) * (size_t)(r.count < kSinglePassSets ? r.count : kSinglePassSets));
    for (int k = 0; r.direct && r.count <= kDirectTensors && k < kDirectTensors; ++k) {
        if (k < r.count) a.direct.descs[k] = r.direct_descs[k];
        else a.direct.descs[k].p_item_begin = ~0u;      // behind every item
    }
    void *args[] = {&a};
    return hipLaunchKernel(pick(ef, err_dtype, fused, wide, r.sp_slim != 0, r.sp_blocks != 0), dim3(n_wg), dim3(kPersistThreads), args, 0, s);
}

}  // namespace cf
