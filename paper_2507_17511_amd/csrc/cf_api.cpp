// C-ABI layer of the residual codec: argument validation, workspace layout,
// per-call pointer tables and kernel sequencing.  No arithmetic of the method
// happens here; see cf_kernels.hip, cf_single_pass.hip and cf_lowrank.hip.  Declarations and their citations of
// arxiv 2507.17511 are in include/compactfusion.h.
#include "compactfusion.h"

#include <algorithm>
#include <cstdint>
#include <cstring>
#include <new>
#include <vector>

#include "cf_internal.h"

using namespace cf;

namespace {

constexpr size_t kAlign = 256;
inline size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

// A bf16 tensor whose rows are no whole blocks of 64 bytes, in the default feedback mode (see make_layout); the parts of its blocks may go out without the streaming hint; fused steps
// of more than kUnevenRounds rounds of workgroups over it take two kernels by default.
enum : uint8_t { kUnevenRow = 1, kUnevenBlocks = 2, kUnevenTwo = 4 };

struct Layout {
    size_t off_descs = 0, off_ptrs = 0, off_tile_prefix = 0, off_fin_prefix = 0, off_partials = 0;
    size_t off_item_prefix = 0, off_item_tensor = 0, off_item_state = 0, off_error = 0, off_p_partials = 0;
    std::vector<uint32_t> item_prefix;
    size_t n_items = 0;
    int32_t max_group_items = 0;   // largest reduction group of the single-pass path
    bool sp_wide = false;          // single-pass items are kStripeChannelsWide channels wide (short tensors)
    bool sp_slim = false;          // ... kStripeChannelsSlim channels wide (tall tensors)
    bool sp_uneven = false;        // most of the context is bf16 rows that are no whole blocks of 64 bytes, see make_layout
    std::vector<uint8_t> uneven;   // per tensor, kUnevenRow and what else holds of it
    bool sp_too_tall = false;      // some group is larger than its tensor's limit: two kernels by default, but for small calls
    bool single_pass = false;      // every channel-scale tensor has single-pass geometry
    // Short items: calls whose items leave the device half empty take ones a quarter as tall, kernels of their own with a
    // quarter of the code, which the first workgroup of a CU has to wait for.  Those tensors have a second geometry, with partials and item
    // states of its own.  Sent layer by layer, us, items as tall as in large calls / half / a quarter: 2 x [1024, 3072] bf16 (192 items) 18.1 / 16.2 / 14.6,
    // [2048, 3072] (192) 20.5 / 16.7 / 16.6, [512, 512] (8) 17.1 / 11.3 / 9.6; 2 x [2048, 3072] (384) 28.3 / 25.5 / 31.0, [4096, 3072] (384)
    // 28.6 / 26.9 / 31.9: the line is what the device holds at once.
    std::vector<TensorDev> short_dev;           // p_rows = 0: none
    size_t off_short_state = 0, n_short_items = 0;
    size_t off_lr_slices = 0, lr_slice_bytes = 0;       // slices of the low-rank back-projection, shared by the tensors of a call
    size_t total = 0;
    std::vector<TensorDev> dev;
    std::vector<uint32_t> tile_prefix, fin_prefix, ew_prefix, dec_prefix;
    size_t off_ew_prefix = 0, off_dec_prefix = 0;
    bool any_channel = false, any_rank1 = false, any_lowrank = false;
};

cf_status check_opts(const cf_options *o, cf_options &out)
{
    out.ef = CF_EF_RECON;
    out.err_dtype = CF_F32;
    out.flags = 0;
    out.tile_rows = 0;
    out.encode_rows = 0;
    if (!o) return CF_OK;
    if (o->ef != CF_EF_RECON && o->ef != CF_EF_LITERAL && o->ef != CF_EF_OFF && o->ef != CF_EF_NAIVE) return CF_ERR_UNSUPPORTED;
    if (o->err_dtype != CF_F32 && o->err_dtype != CF_BF16) return CF_ERR_UNSUPPORTED;
    if (o->flags & ~(CF_FLAG_SINGLE_PASS | CF_FLAG_TWO_KERNEL | CF_FLAG_LOWRANK_INT4 | CF_FLAG_FIXED_GRID | CF_FLAG_TEST_NO_WAIT))
        return CF_ERR_UNSUPPORTED;
    if (o->tile_rows != 0 && o->tile_rows != 8 && o->tile_rows != 16 && o->tile_rows != 32 && o->tile_rows != 64)
        return CF_ERR_UNSUPPORTED;
    if (o->encode_rows < 0 || o->encode_rows > 64) return CF_ERR_UNSUPPORTED;
    out = *o;
    return CF_OK;
}

cf_status check_desc(const cf_tensor_desc &d)
{
    if (d.n_tokens < 1 || d.n_channels < 8 || d.n_channels % 8 != 0) return CF_ERR_SHAPE;
    if (d.n_channels > (int64_t)1 << 30 || d.n_tokens > (int64_t)1 << 24) return CF_ERR_SHAPE;
    if (d.n_tokens > ((int64_t)1 << 46) / d.n_channels) return CF_ERR_SHAPE;
    if (d.dtype != CF_F32 && d.dtype != CF_BF16) return CF_ERR_UNSUPPORTED;
    if (d.bits != 1 && d.bits != 2 && d.bits != 4) return CF_ERR_UNSUPPORTED;
    if (d.scale == CF_SCALE_CHANNEL) return CF_OK;
    if (d.scale == CF_SCALE_GROUP) {
        if (d.bits != 4) return CF_ERR_UNSUPPORTED;
        if (d.group != 128 || d.n_channels % 128 != 0) return CF_ERR_SHAPE;
        return CF_OK;
    }
    if (d.scale == CF_LOWRANK) {        // bits = subspace iterations T, group = rank
        if (d.group != kLowRankRank) return CF_ERR_UNSUPPORTED;
        if (d.n_channels % 32 != 0 || d.n_channels > kLowRankMaxChannels) return CF_ERR_SHAPE;
        return CF_OK;
    }
    if (d.scale == CF_SPARSE_NM) {      // bits = N values kept of every group = M channels
        if (d.group != 8 && d.group != 16) return CF_ERR_UNSUPPORTED;
        if (d.n_channels % d.group != 0) return CF_ERR_SHAPE;
        return CF_OK;                   // bits in {1, 2, 4} was checked above
    }
    if (d.scale == CF_SCALE_RANK1) {
        if (d.bits == 4) return CF_ERR_UNSUPPORTED;                  // the paper's u v^T goes with its 1-/2-bit code books
        if (d.n_channels > (int64_t)kMaxRank1Colblocks * kTileChannels) return CF_ERR_SHAPE;
        return CF_OK;
    }
    return CF_ERR_UNSUPPORTED;
}

size_t dtype_size(int32_t dt) { return dt == CF_BF16 ? 2 : 4; }

struct BufferBytes {
    size_t codes, scales, recon, err;      // recon is also the size of x
};

// Byte sizes of one (valid) tensor's buffers.
BufferBytes buffer_bytes(const cf_tensor_desc &d, const cf_options &o)
{
    BufferBytes b;
    const size_t n = (size_t)d.n_tokens, c = (size_t)d.n_channels;
    if (d.scale == CF_LOWRANK) {        // U [N, 32] then V [C, 32] in the storage dtype; the scales entry is the input Q0 [C, 32] fp32
        // 4-bit factors: 16 nibble bytes and one fp32 scale per factor row
        b.codes = (o.flags & CF_FLAG_LOWRANK_INT4) ? (n + c) * 20 : (n + c) * kLowRankRank * dtype_size(d.dtype);
        b.scales = c * kLowRankRank * sizeof(float);
    } else if (d.scale == CF_SPARSE_NM) {      // one mask byte per block of 8, then (16-byte aligned) bits values per block
        b.codes = (n * (c / 8) + 15) / 16 * 16 + n * (c / (size_t)d.group) * (size_t)d.bits * dtype_size(d.dtype);
        b.scales = 0;
    } else {
        b.codes = n * (c * (size_t)d.bits / 8);
        b.scales = sizeof(float) * (d.scale == CF_SCALE_GROUP ? n * (c / 128) : d.scale == CF_SCALE_RANK1 ? c + n : c);
    }
    b.recon = n * c * dtype_size(d.dtype);
    b.err = n * c * dtype_size(o.err_dtype);
    return b;
}

inline bool overlap(const void *a, size_t na, const void *b, size_t nb)
{
    if (!a || !b || na == 0 || nb == 0) return false;
    const uintptr_t pa = reinterpret_cast<uintptr_t>(a), pb = reinterpret_cast<uintptr_t>(b);
    return pa < pb + nb && pb < pa + na;
}

// Rows per tile: as large as still leaves the batched grid a few thousand
// workgroups (256 CUs, several resident workgroups each).
int pick_rb_rows(const cf_tensor_desc *descs, int32_t n, const cf_options &o)
{
    if (o.tile_rows) return o.tile_rows;
    const int cands[] = {64, 32, 16, 8};
    for (int rb : cands) {
        uint64_t tiles = 0;
        for (int32_t t = 0; t < n; ++t) {
            uint64_t rbn = (uint64_t)((descs[t].n_tokens + rb - 1) / rb);
            uint64_t cbn = (uint64_t)((descs[t].n_channels / kChunk + kTileThreads - 1) / kTileThreads);
            tiles += rbn * cbn;
        }
        if (tiles >= 4096) return rb;
    }
    return 8;
}

int64_t lowrank_stripes(int64_t n_channels) { return (n_channels + kLowRankBackChannels - 1) / kLowRankBackChannels; }

// Workgroups that share a channel stripe of the low-rank back-projection in a call of that many stripes (the largest
// low-rank tensor's channels and tokens given): more where the stripes alone would leave the device idle.
// Whole steps with 1 / 2 / 4 sharing, us: [4096, 3072] 1 tensor 339 / 234 / 190, 8 (96 stripes) 633 / 529 / 514, 16 966 / 907 / 889,
// 40 2053 / 2038 / 2066, 57 (684) 2910 / 2881 / 2882; 60 x [8000, 96] 456 / 353 / 311, 100 x [4096, 256] 636 / 531 / 515.  Beyond, the
// shares' memory is not worth it.
int64_t lowrank_split(int64_t max_channels, int64_t max_tokens, int64_t stripes)
{
    return std::min<int64_t>(lowrank_runs(max_tokens, max_channels), stripes <= 128 ? kLowRankMaxRuns : stripes <= 768 ? 2 : 1);
}

size_t lowrank_slice_bytes_of(int64_t max_channels, int64_t split, int64_t count)
{
    return (size_t)((split - 1) * count) * (size_t)max_channels * kLowRankRank * sizeof(float);
}

// What the shares after the first need in calls over any number of these tensors, were they all of the largest size; calls over
// narrower ones that would need more share less.
size_t lowrank_slice_bytes(const cf_tensor_desc *descs, int32_t n)
{
    int64_t c = 0, tok = 0, lowrank = 0;
    for (int32_t t = 0; t < n; ++t)
        if (descs[t].scale == CF_LOWRANK) {
            c = std::max<int64_t>(c, descs[t].n_channels);
            tok = std::max<int64_t>(tok, descs[t].n_tokens);
            ++lowrank;
        }
    size_t most = 0;
    for (int64_t count = 1; count <= lowrank; ++count)
        most = std::max(most, lowrank_slice_bytes_of(c, lowrank_split(c, tok, lowrank_stripes(c) * count), count));
    return align_up(most);
}

// Largest group of 64-channel stripes in a call of any size.  The taller the tensors the longer workgroups wait for the slowest of their group, and a
// stripe of a row is one line of 128 bytes of bf16: where rows are no whole lines it is pieces of two, and where they are multiples of 1024 channels the
// stripe's rows share their memory channels.  Single pass against two kernels in us, 2.6e8 elements of bf16 (1.5e8 of fp32 and with the error as operand):
//   whole lines        [22358, 1920] 44 items 542 / 616, [32598, 3328] 64 497 / 578; naive [19286, 1536] 38 404 / 417, [32598, 3328] 64 365 / 409;
//                      fp32 [16299, 1920] 64 491 / 593, naive 376 / 420; no feedback [16299, 3072] 64 887 / 993, of fp32 [8150, 3072] 724 / 801
//   multiples of 1024  [20310, 3072] 40 items 606 / 610, [26454, 2048] 52 543 / 520, [32598, 4096] 64 404 / 334; naive [12118, 3072] 24 388 / 402, [15190,
//                      3072] 30 434 / 418, [32598, 2048] 64 458 / 353; fp32 [16314, 2048] 64 570 / 610, naive [12203, 3072] 48 706 / 737, 64 871 / 818
//   others             [19286, 1096] 38 1200 / 662, [32598, 1096] 64 1126 / 651; naive [11094, 1096] 22 1004 / 487, [15190, 2056] 30 1440 / 460; fp32 [12218, 3080]
//                      48 596 / 563, [16314, 200] 64 741 / 671; no feedback [12218, 1096] 48 749 / 655, of fp32 50 x [7000,
//                      200] 55 489 / 436, 4 x [7000, 2056] 413 / 371, but 3 x [7000, 3080] 370 / 433
// The lines for the last two kinds are those of a fetch by one lane a channel, which all kinds had once; for rows of no whole lines two kernels are the
// faster choice below them too.
int32_t slim_group_limit(const cf_tensor_desc &d, const cf_options &o)
{
    const bool wide = d.dtype == CF_F32, naive = o.ef == CF_EF_NAIVE, three_operands = o.ef == CF_EF_LITERAL || o.ef == CF_EF_OFF;
    const bool whole_lines = d.n_channels * (wide ? 4 : 2) % 128 == 0;
    if (!whole_lines) return naive ? kSlimGroupLimitNaive : kSlimGroupLimitUneven;
    if (three_operands || (wide && !naive) || d.n_channels % 1024 != 0) return kSlimGroupLimit;
    return !naive ? kSlimGroupLimitUneven : wide ? kNarrowGroupLimit : kSlimGroupLimitNaive;
}

// uneven_stripes: contexts of mostly uneven rows take stripes of their own, which have up to twice the partials
cf_status make_layout(const cf_tensor_desc *descs, int32_t n, const cf_options &o, Layout &L, bool uneven_stripes = true)
{
    if (!descs || n < 1) return CF_ERR_INVALID_ARG;
    for (int32_t t = 0; t < n; ++t) {
        cf_status st = check_desc(descs[t]);
        if (st != CF_OK) return st;
    }
    const int rb = pick_rb_rows(descs, n, o);
    int64_t columns = 0;            // that k_finalize has to finish
    for (int32_t t = 0; t < n; ++t)
        if (descs[t].scale == CF_SCALE_CHANNEL || descs[t].scale == CF_SCALE_RANK1) columns += descs[t].n_channels;
    L.dev.resize(n);
    L.tile_prefix.assign(n + 1, 0);
    L.ew_prefix.assign(n + 1, 0);
    L.dec_prefix.assign(n + 1, 0);
    uint64_t ew_tiles = 0, dec_tiles = 0;
    L.fin_prefix.assign(n + 1, 0);
    uint64_t tiles = 0, fins = 0, items = 0;
    size_t partial_bytes = 0, p_partial_bytes = 0;
    uint32_t lr_tensors = 0;
    L.item_prefix.assign(n + 1, 0);
    L.single_pass = (o.flags & CF_FLAG_TWO_KERNEL) == 0;
    for (int32_t t = 0; t < n; ++t)
        if (descs[t].scale == CF_SCALE_RANK1) L.single_pass = false;   // the single-pass kernel knows channel scales only
    // Single-pass item shape: 256 lanes, each with single_pass_rows_per_lane rows, cover kStripeChannels channels by
    // default; when even the tallest channel-scale tensor would make at most 12 items per group that way (bf16:
    // N <= 3072), items half as tall and twice as wide measure equal or faster.  [N, 3072] bf16 batches of equal
    // size, 128 -> 256 channels, 1- / 2- / 4-bit codes: N = 1024 1.57 / 1.61 / 1.65 -> 1.47 / 1.55 / 1.52 ms,
    // N = 2048 1.49 / 1.51 / 1.60 -> 1.52 / 1.48 / 1.55, N = 3072 1.47 / 1.52 / 1.61 -> 1.46 / 1.50 / 1.58,
    // N = 4096 1.50 / 1.55 / 1.62 -> 1.53 / 1.56 / 1.65, N = 6144 1.56 / 1.59 / 1.68 -> 1.62 / 1.66 / 1.77.
    auto narrow_item_rows = [&](int32_t dtype) { return (kPersistThreads / (kStripeChannels / kChunk)) * single_pass_rows_per_lane(dtype, o.ef); };
    int64_t narrow_max_group = 0, elements = 0, tall_elements = 0, sliver_elements = 0, uneven_elements = 0, uneven_wide = 0, uneven_short = 0, uneven_middle = 0;
    L.uneven.assign(n, 0);
    for (int32_t t = 0; t < n; ++t)
        if (descs[t].scale == CF_SCALE_CHANNEL) {
            const int64_t rows = narrow_item_rows(descs[t].dtype), c = descs[t].n_channels, last = c % kStripeChannelsSlim;
            const int64_t g = (descs[t].n_tokens + rows - 1) / rows;
            if (g > narrow_max_group) narrow_max_group = g;
            elements += descs[t].n_tokens * c;
            if (o.ef == CF_EF_RECON && descs[t].dtype == CF_BF16 && c % 32 != 0) {
                const bool odd = c % 16 != 0;
                const int limit = !odd ? kUnevenGroupLimitEven : o.err_dtype == CF_BF16 ? kUnevenGroupLimitBf16Error : kUnevenWideGroup;
                L.uneven[t] = (uint8_t)(kUnevenRow | (odd ? kUnevenBlocks : 0) | (g > limit ? kUnevenTwo : 0));
                uneven_elements += descs[t].n_tokens * c;
                if (g <= kUnevenWideGroup) uneven_wide += descs[t].n_tokens * c;
                if (g <= kWideGroup) uneven_short += descs[t].n_tokens * c;
                if (g >= 4 && g <= kWideGroup) uneven_middle += descs[t].n_tokens * c;
            }
            if (g > kTallGroupItems) tall_elements += descs[t].n_tokens * c;
            // the last 64-channel stripe of a row is a few short pieces of memory and much of what there is
            if (g > kTallGroupItems && c < kStripeChannels && last > 0 && last < kStripeChannelsSlim / 2) sliver_elements += descs[t].n_tokens * c;
        }
    const bool slivers = sliver_elements > 0 && sliver_elements >= elements - sliver_elements;
    // Uneven rows, bf16 ones that are no whole blocks of 64 bytes: a stripe's piece of a row shares its first and last block with the stripes beside
    // it, and a block that reaches memory in parts costs as much as five whole ones.  Wide stripes have half as many; the parts go out without the
    // streaming hint, so that an L2 that has both makes them whole (`blocks`, in calls that write enough: kBlocksBytes); past both, two kernels, whose rows are written in one run.  In
    // calls of few rounds the caches make more of them whole: 2 x [8000, 1512] (768 items) 76.5 / 60.1 in 128-channel stripes without and with blocks, 76.4 with two kernels.  Steps of 1.6e8
    // elements, us, 128 / 128 blocks / 256 / 256 blocks / two kernels (channels that are an odd multiple of 8: error rows are uneven too):
    //   odd   [1024, 1096] 205 / 161 / 165 / 145 / 181, [4096, 1096] 429 / 409 / 385 / 386 / 409, [4096, 3080] 430 / 405 / 378 / 377 / 389, [4096, 200] 296 / 255 / 247 / 220 / 224,
    //         [5000, 1096] 451 / 447 / 425 / 423 / 417, [8000, 3080] 447 / 417 / 413 / 408 / 385, bf16 error [6100, 1096] 469 / 445 / 460 / 470 / 460, [8000, 1096] 636 / 613 / 617 /
    //         653 / 603; not fused [6100, 1096] 395 / 373 / 411 / 415 / 450, [8000, 1096] 528 / 501 / 558 / 562 / 590
    //   even  [1024, 1104] 333 / 298 / 276 / 265 / 345, [4096, 1104] 371 / 367 / 355 / 369 / 407, [8000, 1104] 391 / 391 / 409 / 425 / 410, [11000, 1104] 407 / 408 / 484 / 488 / 406 (64
    //         channels 479), [17000, 3088] 451 / 449 / 631 / 643 / 411; not fused [8000, 1104] 318 / 327 / 359 / 371 / 390
    // Of 49 to 64 items, as it runs in 128 channels / in 64 / two kernels: 10 x [14000, 1096] 449 / 556 / 404, not fused 309 / 352 / 346, two of them 75 / 88 / 99 and 66 / 74 / 89,
    // 3 x [16000, 3080] not fused 326 / 352 / 319; 10 x [14000, 1104] 405 / 477 / 400, not fused 290 / 322 / 345, two of them 87 / 99 / 99 and 61 / 66 / 88.  Beyond, 64 channels
    // without and with blocks / two kernels: 8 x [17000, 1096] 632 / 550 / 390, not fused 412 / 349 / 337, two of them 161 / 109 / 113 and 109 / 93 / 100.
    // Stripes are the context's.  Wide ones cost whole rows of 13 items and more what uneven ones of so many gain, and what those gain in steps they lose when sent: so three quarters
    // of the context have to be such.  128 / 256 channels: 36 x [4096, 1096] 417 / 395, sent 292 / 303, x [4096, 1104] 380 / 364, sent 275 / 287; 27 x [4096, 1096] with 9 x [4096,
    // 1088] 396 / 382, sent 281 / 297, 20 with 16 379 / 374, sent 272 / 291.  Uneven rows of up to 12 items gain more: half of the context is enough (26 x [1027, 1976] with 15 x
    // [1675, 1024] fp32 223 / 204), and four fifths, if of 4 items at least, next to tensors of up to 24: 110 x [1024, 1096] with one [5000, 3072] 425 / 317, the 110 alone 370 / 276, the
    // one alone 31 / 35, but 10 x [385, 2872], of two items, with one [4629, 64] 38 / 51.
    // Stores and the second kernel are the call's, by most of its elements: 30 x [4800, 1088] of a context with 40 x [4800, 1096] take 305 in the single pass, 324 with blocks, 397 with
    // two kernels.  Calls over both, single pass / two kernels: [4609, 1096] with [4609, 1088] 51 % 751 / 782, 67 % 774 / 775, 80 % 805 / 781, [8000, 3080] with [8000, 3072]
    // 57 % 879 / 860, [14000, 1096] with [14000, 1088] 55 % 890 / 861.
    L.sp_uneven = L.single_pass && uneven_elements > elements - uneven_elements;
    if (narrow_max_group <= 4)          // even ones too: [1024, 1104] above
        for (uint8_t &u : L.uneven) u |= u ? kUnevenBlocks : 0;
    const bool wide_uneven = uneven_stripes && ((narrow_max_group <= kUnevenWideGroup && (uneven_wide >= 3 * (elements - uneven_wide) || uneven_short > elements - uneven_short)) ||
                                                (narrow_max_group <= kNarrowGroupLimit / 2 && uneven_middle >= 4 * (elements - uneven_middle)));
    L.sp_wide = L.single_pass && narrow_max_group > 0 && (narrow_max_group <= kWideGroup || wide_uneven);
    // Tall tensors the other way round: all workgroups of a group wait for its slowest, and the more they are the longer.
    // 128 -> 64 channels on batches of equal size, us: [6144, 3072] bf16 793 -> 790, [8192, 3072] 840 -> 812 (4-bit 858 ->
    // 856), [12288, 3072] 895 -> 854, [16384, 3072] 1030 -> 902, [17776, 1920] with bf16 error 2227 -> 1976.  Tensors that
    // are not tall lose by it, so tall ones that the 128-channel form still serves (up to kNarrowGroupLimit items) must
    // hold half of the context: 40 x [1024, 3072] with one [12288, 3072] 332 -> 357, 40 x [4096, 3072] with one 1027 -> 1042,
    // 20 x [4096, 3072] with seven 1080 -> 1068; beyond that two kernels are the other choice: 40 x [2048, 3072] with four
    // [16384, 3072] 970 against 1078.  Not for slivers: 114 x [11653, 80] 360 -> 434 (x [11653, 64] 272 -> 199, 60 x
    // [17000, 96] 310 -> 298).
    L.sp_slim = L.single_pass && !slivers && !(L.sp_uneven && uneven_stripes && narrow_max_group <= kUnevenNarrowGroup) && narrow_max_group > kTallGroupItems &&
                (narrow_max_group > kNarrowGroupLimit || tall_elements >= elements - tall_elements);
    // Largest group of a call of any size in 128-channel stripes, single pass against two kernels in us: 4 x [10000, 3072], 40, 290 / 307; one [12288,
    // 3072] among 40 x [4096, 3072], 48, 1027 / 1311; slivers, whose second kernel runs across the row ends: 114 x [11653, 80], 46, 351 / 312, x [10500,
    // 72], 42, 344 / 265.  In 64-channel stripes: slim_group_limit.
    const int stripe_channels = L.sp_wide ? kStripeChannelsWide : L.sp_slim ? kStripeChannelsSlim : kStripeChannels;
    for (int32_t t = 0; t < n; ++t) {
        const cf_tensor_desc &d = descs[t];
        TensorDev &v = L.dev[t];
        std::memset(&v, 0, sizeof v);
        v.n_tokens = d.n_tokens;
        v.n_channels = (int32_t)d.n_channels;
        v.n_chunks = (int32_t)(d.n_channels / kChunk);
        v.dtype = d.dtype;
        v.bits = d.bits;
        v.scale = d.scale;
        v.nm_block = d.scale == CF_SPARSE_NM ? (uint32_t)d.group : (d.scale == CF_LOWRANK && (o.flags & CF_FLAG_LOWRANK_INT4)) ? 4u : 0u;
        v.rb_rows = rb;
        v.n_rowblocks = (int32_t)((d.n_tokens + rb - 1) / rb);
        v.n_colblocks = (v.n_chunks + kTileThreads - 1) / kTileThreads;
        v.tile_begin = (uint32_t)tiles;
        v.fin_begin = (uint32_t)fins;
        L.tile_prefix[t] = (uint32_t)tiles;
        L.fin_prefix[t] = (uint32_t)fins;
        tiles += (uint64_t)v.n_rowblocks * (uint64_t)v.n_colblocks;
        // Tiles across the row ends (see cf_kernels.hip) where the last 1024-channel tile of a row would be a part of one;
        // their chunk numbers are 32-bit.  The receiver's kernel, which reads a lane's channel scales once for both rows
        // of a tile, takes them only where whole rows would leave more than an eighth of the lanes idle.  Row tiles / flat, us,
        // 1.5e8 bf16 elements of [2039, C]: warm-up C = 3064 218 / 194, 2600 218 / 192, 1096 277 / 197, 112 216 / 69; sparsifier's
        // encoder 3064 278 / 255, 2600 281 / 255, 1096 384 / 257; receiver, 2-bit channel scales, 2600 117 / 110, 1784 118 / 110,
        // 1096 176 / 111, 520 188 / 115, 112 204 / 37 (1800, just under an eighth, stays with rows at 116).
        const uint64_t chunks = (uint64_t)d.n_tokens * (uint64_t)v.n_chunks;
        const bool ragged = v.n_chunks % kTileThreads != 0 && chunks < (1u << 31) - (1u << 16);
        // element-wise kernels do best with short-lived workgroups: a lane never has to wait for
        // its own stores before it can use its next loads
        v.ew_flat = ragged;
        v.ew_tile_begin = (uint32_t)ew_tiles;
        L.ew_prefix[t] = (uint32_t)ew_tiles;
        ew_tiles += v.ew_flat ? (chunks + kTileThreads - 1) / kTileThreads : (uint64_t)d.n_tokens * (uint64_t)v.n_colblocks;
        if (ew_tiles > 0x7fffffffull) return CF_ERR_SHAPE;
        // the receiver's kernel moves 4 bytes per element, not 10: two rows per workgroup (loaded together, then
        // stored together) keep the workgroup count down; measured 1.43 -> 1.08 ms on 114 x [4096, 3072]
        v.dec_rows = o.encode_rows ? o.encode_rows : 2;
        v.dec_flat = ragged && v.n_chunks * 8 < v.n_colblocks * kTileThreads * 7;
        v.dec_tile_begin = (uint32_t)dec_tiles;
        L.dec_prefix[t] = (uint32_t)dec_tiles;
        const uint64_t dec_run = (uint64_t)v.dec_rows * kTileThreads;
        dec_tiles += v.dec_flat ? (chunks + dec_run - 1) / dec_run
                                : (uint64_t)((d.n_tokens + v.dec_rows - 1) / v.dec_rows) * (uint64_t)v.n_colblocks;
        // a column with a lane of its own takes 2.5 us and 0.058 per partial, however many there are; sixteen lanes a column
        // make a workgroup of 16 columns, 2.8 ns each once the device is full: k_finalize of 57 x [4096, 3072] (64 partials)
        // 10.6 / 30.1 us, 114 x [8192, 1024] (128) 14.3 / 24.0, 16 x [4096, 3072] (128) 11.6 / 12.2, 30 x [17776, 1920] (278)
        // 28.5 / 22.2, 8 x [4096, 3072] (256) 18.4 / 11.0, 1 x [16384, 512] (2048) 121 / 13
        v.fin_columns = v.n_rowblocks > 32 && (int64_t)v.n_rowblocks * 320 > columns ? kFinalizeColumns : kFinalizeThreads;
        fins += (uint64_t)((d.n_channels + v.fin_columns - 1) / v.fin_columns);
        if (tiles > 0x7fffffffull || fins > 0x7fffffffull) return CF_ERR_SHAPE;
        if (d.scale == CF_SCALE_CHANNEL || d.scale == CF_SCALE_RANK1) {
            L.any_channel = true;
            v.partial_off = partial_bytes;   // relative; rebased below
            partial_bytes += align_up((size_t)v.n_rowblocks * (size_t)d.n_channels * sizeof(float));
        }
        if (d.scale == CF_LOWRANK) {
            if (o.ef != CF_EF_RECON) return CF_ERR_UNSUPPORTED;
            L.any_lowrank = true;
            v.lr_slot = lr_tensors++;
            v.lr_p_off = partial_bytes;
            partial_bytes += align_up((size_t)d.n_tokens * kLowRankRank * sizeof(float));
            v.lr_z_off = partial_bytes;
            partial_bytes += align_up((size_t)d.n_channels * kLowRankRank * sizeof(float));
            v.lr_g_off = partial_bytes;
            partial_bytes += align_up(lowrank_g_bytes(d.n_channels));
        }
        if (d.scale == CF_SCALE_RANK1) {
            L.any_rank1 = true;
            v.rowpart_off = partial_bytes;
            partial_bytes += align_up((size_t)d.n_tokens * (size_t)v.n_colblocks * sizeof(float));
        }
        L.item_prefix[t] = (uint32_t)items;
        if (d.scale == CF_SCALE_CHANNEL && L.single_pass) {
            v.p_rows = narrow_item_rows(d.dtype) * kStripeChannels / stripe_channels;
            v.p_n_rb = (int32_t)((d.n_tokens + v.p_rows - 1) / v.p_rows);
            v.p_n_stripes = (int32_t)((d.n_channels + stripe_channels - 1) / stripe_channels);
            v.p_item_begin = (uint32_t)items;
            v.p_partial_off = p_partial_bytes;               // relative; rebased below
            p_partial_bytes += align_up((size_t)v.p_n_rb * (size_t)d.n_channels * sizeof(float));
            items += (uint64_t)v.p_n_rb * (uint64_t)v.p_n_stripes;
            if (v.p_n_rb > L.max_group_items) L.max_group_items = v.p_n_rb;
            if (v.p_n_rb > (L.sp_slim ? slim_group_limit(d, o) : slivers ? kTallGroupItems : L.sp_uneven && uneven_stripes ? kUnevenNarrowGroup : kNarrowGroupLimit)) L.sp_too_tall = true;
            if (items > 0x7fffffffull) return CF_ERR_SHAPE;
        }
    }
    // What else takes two kernels where others of the context decide on the stripes: uneven rows of any length in 64-channel ones; in 128-channel ones those of few row blocks, which
    // do not keep their XCD from stripe to stripe, and with fp32 errors odd ones of more than 12 items and 2048 channels.  Fused, single pass / two kernels: 12 x [2924, 3736] with one
    // [19336, 352] 574 / 365, 8 x [6614, 3280] with one [18008, 112] 548 / 446; 46 x [1508, 3576] with two [12327, 1472] 817 / 649, 59 x [302, 3160] with three [10872, 544]
    // 230 / 190, 40 x [1000, 3080] 427 / 388, 110 x [1024, 1096] with one [5000, 3072] 425 / 389, but 60 x [1000, 1096] 207 / 220 (and of eight row blocks, [2000, 1096], 367 / 403);
    // 30 x [3077, 2696] with one [6457, 192] 776 / 652, but 31 x [4096, 1096] with 20 x [6000, 1088] 624 / 697.
    for (int32_t t = 0; t < n; ++t) {
        if (!L.uneven[t]) continue;
        const int32_t g = L.dev[t].p_n_rb;
        const bool few = g < 8 && L.max_group_items > 4, long_odd = g > kWideGroup && narrow_max_group > kUnevenWideGroup && descs[t].n_channels % 16 != 0 && descs[t].n_channels > 2048 && o.err_dtype == CF_F32;
        if (L.sp_slim || (!L.sp_wide && (few || long_odd))) L.uneven[t] |= kUnevenTwo;
    }
    L.tile_prefix[n] = (uint32_t)tiles;
    L.ew_prefix[n] = (uint32_t)ew_tiles;
    L.dec_prefix[n] = (uint32_t)dec_tiles;
    L.fin_prefix[n] = (uint32_t)fins;
    L.item_prefix[n] = (uint32_t)items;

    size_t off = 0;
    L.off_descs = off;        off = align_up(off + sizeof(TensorDev) * (size_t)n);
    L.off_ptrs = off;         off = align_up(off + sizeof(TensorPtrs) * (size_t)n);
    L.off_tile_prefix = off;  off = align_up(off + sizeof(uint32_t) * (size_t)(n + 1));
    L.off_fin_prefix = off;   off = align_up(off + sizeof(uint32_t) * (size_t)(n + 1));
    L.off_ew_prefix = off;    off = align_up(off + sizeof(uint32_t) * (size_t)(n + 1));
    L.off_dec_prefix = off;   off = align_up(off + sizeof(uint32_t) * (size_t)(n + 1));
    L.off_partials = off;     off = align_up(off + partial_bytes);
    L.off_item_prefix = off;  off = align_up(off + sizeof(uint32_t) * (size_t)(n + 1));
    L.off_item_tensor = off;  off = align_up(off + sizeof(uint32_t) * (size_t)items);
    L.n_items = (size_t)items;
    L.off_error = off;        off = align_up(off + sizeof(uint32_t) * 64);      // error word, and the last single pass's items 128 bytes on
    L.off_item_state = off;   off = align_up(off + (size_t)items);     // one fill with the partials behind them
    L.lr_slice_bytes = lowrank_slice_bytes(descs, n);
    size_t short_bytes = 0, short_items = 0;
    L.short_dev = L.dev;
    for (TensorDev &v : L.short_dev) {
        const int64_t rows = kPersistThreads / (kShortStripeChannels / kChunk) * single_pass_rows_per_lane(v.dtype, o.ef) / kShortFraction;
        const int64_t rb = (v.n_tokens + rows - 1) / rows, stripes = (v.n_channels + kShortStripeChannels - 1) / kShortStripeChannels;
        const bool fits = v.p_rows > 0 && o.ef == CF_EF_RECON && rb <= kShortGroupLimit && rb * stripes <= kShortItems;
        v.p_rows = fits ? (int32_t)rows : 0;
        if (!fits) continue;
        v.p_n_rb = (int32_t)rb;
        v.p_n_stripes = (int32_t)stripes;
        v.p_item_begin = (uint32_t)short_items;
        v.p_partial_off = short_bytes;                      // relative; rebased below
        short_bytes += align_up((size_t)rb * (size_t)v.n_channels * sizeof(float));
        short_items += (size_t)(rb * stripes);
    }
    {   // nor do tensors outgrow the static scratch because of them
        const size_t without = align_up(off + p_partial_bytes), with = align_up(align_up(off + short_items) + p_partial_bytes) + short_bytes;
        if (without <= kStaticScratchBytes && with + L.lr_slice_bytes > kStaticScratchBytes) {
            short_items = 0;
            for (TensorDev &v : L.short_dev) v.p_rows = 0;
        }
    }
    L.n_short_items = short_items;
    L.off_short_state = off;  off = align_up(off + short_items);
    L.off_p_partials = off;   off = align_up(off + p_partial_bytes);
    if (short_items > 0) {
        for (TensorDev &v : L.short_dev) v.p_partial_off += off;
        off += short_bytes;
    }
    L.off_lr_slices = off;
    // no tensors outgrow the static scratch because of the slices: there are fewer then, and the sums are the same
    if (off <= kStaticScratchBytes) L.lr_slice_bytes = std::min(L.lr_slice_bytes, (kStaticScratchBytes - off) / kAlign * kAlign);
    off += L.lr_slice_bytes;
    L.total = off;
    for (int32_t t = 0; t < n; ++t) {
        if (descs[t].scale == CF_SCALE_CHANNEL || descs[t].scale == CF_SCALE_RANK1) {
            L.dev[t].partial_off += L.off_partials;
            L.dev[t].p_partial_off += L.off_p_partials;
        }
        if (descs[t].scale == CF_SCALE_RANK1) L.dev[t].rowpart_off += L.off_partials;
        if (descs[t].scale == CF_LOWRANK) {
            L.dev[t].lr_p_off += L.off_partials;
            L.dev[t].lr_z_off += L.off_partials;
            L.dev[t].lr_g_off += L.off_partials;
        }
    }
    return CF_OK;
}

inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

}  // namespace

struct cf_ctx {
    std::vector<cf_tensor_desc> descs;
    Layout L;
    cf_options opts;
    uint8_t *ws = nullptr;
    size_t ws_bytes = 0;
    std::vector<TensorPtrs> ptrs;      // what the workspace table currently holds (once the uploads on ptrs_stream have run)
    hipStream_t ptrs_stream = nullptr; // stream the pointer uploads were enqueued on
    bool ptrs_synced = false;          // the table matches `ptrs` for work enqueued on ptrs_stream from now on
    hipStream_t sp_stream = nullptr;   // stream of the single passes so far
    bool sp_called = false;
    bool sp_unordered = false;         // single passes were enqueued on several streams or captured: no stream keeps them apart for certain
    bool sp_always_fresh = false;      // every single pass sets its signs anew
    std::vector<uint8_t> warm;
    int32_t last_hip = 0;
    int device = 0;
    int persist_grid[2][2] = {{0, 0}, {0, 0}};   // co-resident workgroups of k_single_pass<err dtype, fused>

    // benchmark instrumentation (cf_profile_next_call)
    std::vector<hipEvent_t> prof_events;
    bool prof_armed = false;
    int32_t prof_count = 0;
    const char *prof_names[16] = {};

    BatchView view() const
    {
        BatchView v;
        v.descs = reinterpret_cast<const TensorDev *>(ws + L.off_descs);
        v.ptrs = reinterpret_cast<const TensorPtrs *>(ws + L.off_ptrs);
        v.tile_prefix = reinterpret_cast<const uint32_t *>(ws + L.off_tile_prefix);
        v.fin_prefix = reinterpret_cast<const uint32_t *>(ws + L.off_fin_prefix);
        v.ew_prefix = reinterpret_cast<const uint32_t *>(ws + L.off_ew_prefix);
        v.dec_prefix = reinterpret_cast<const uint32_t *>(ws + L.off_dec_prefix);
        v.item_prefix = reinterpret_cast<const uint32_t *>(ws + L.off_item_prefix);
        v.item_tensor = reinterpret_cast<const uint32_t *>(ws + L.off_item_tensor);
        v.error_flag = reinterpret_cast<uint32_t *>(ws + L.off_error);
        v.item_state = ws + L.off_item_state;
        v.workspace = ws;
        v.n_tensors = (int32_t)descs.size();
        return v;
    }

    // The single pass's item states and partials as before a first call: every sign the same (see cf_single_pass.hip).
    hipError_t fresh_partials(hipStream_t s) const
    {
        if (L.n_items == 0) return hipSuccess;
        return launch_fill_words(ws + L.off_item_state, kFreshPartials, (L.off_lr_slices - L.off_item_state) / sizeof(uint32_t), s);
    }

    // A single pass takes over the signs that the call before left, which calls that overlapped (against the rules) may leave in disorder.  On one stream
    // no two can; once single passes came on another stream than the ones before, or were recorded into a graph, which may be replayed on any, warm-ups, which
    // the tensors need then, set their signs anew.  hipStreamPerThread is a stream of its own in every thread.
    void note_single_pass(hipStream_t s)
    {
        if (sp_unordered) return;
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(s, &cap) != hipSuccess) {
            (void)hipGetLastError();
            cap = hipStreamCaptureStatusNone;
        }
        sp_unordered = cap != hipStreamCaptureStatusNone || s == hipStreamPerThread || (sp_called && sp_stream != s);
        sp_called = true;
        sp_stream = s;
    }

    // Item states and partials of the range as before a first call, of the items of `devs`: L.dev or L.short_dev.
    hipError_t fresh_partials_of(int32_t first, int32_t count, const std::vector<TensorDev> &devs, size_t off_state, hipStream_t s) const
    {
        uint64_t lo = ~(uint64_t)0, hi = 0;
        uint32_t item_lo = 0, item_hi = 0;
        for (int32_t t = first; t < first + count; ++t) {
            const TensorDev &d = devs[t];
            if (d.p_rows == 0) continue;
            if (hi == 0) {
                lo = d.p_partial_off;
                item_lo = d.p_item_begin;
            }
            hi = d.p_partial_off + align_up((size_t)d.p_n_rb * (size_t)d.n_channels * sizeof(float));
            item_hi = d.p_item_begin + (uint32_t)(d.p_n_rb * d.p_n_stripes);
        }
        if (hi == 0) return hipSuccess;
        return launch_fresh_partials(ws + lo, hi - lo, ws + off_state + item_lo, item_hi - item_lo, s);
    }

    LaunchRange range(int32_t first, int32_t count) const
    {
        LaunchRange r;
        r.first = first;
        r.count = count;
        r.direct = nullptr;
        r.direct_descs = L.dev.data() + first;
        r.tile_lo = L.tile_prefix[first];
        r.tile_hi = L.tile_prefix[first + count];
        r.ew_lo = L.ew_prefix[first];
        r.ew_hi = L.ew_prefix[first + count];
        r.dec_lo = L.dec_prefix[first];
        r.dec_hi = L.dec_prefix[first + count];
        r.fin_lo = L.fin_prefix[first];
        r.fin_hi = L.fin_prefix[first + count];
        r.sp_xcd_major = 0;
        r.sp_wait_polls = kWaitPolls;
        r.sp_slim = L.sp_slim;
        r.sp_short = 0;
        r.item_lo = L.item_prefix[first];
        r.item_hi = L.item_prefix[first + count];
        r.sp_blocks = 0;
        r.only_group_scale = 0;
        r.naive = opts.ef == CF_EF_NAIVE;
        r.dts = descs[first].dtype;
        r.dec_kinds = 0;
        r.lr_max_channels = 0;
        r.lr_max_tokens = 0;
        r.lr_wires = 0;
        r.lr_project_blocks = 0;
        r.lr_project_many = 0;
        r.lr_split = 1;
        r.lr_first_slot = 0;
        r.lr_slices_off = L.off_lr_slices;
        int64_t lr_tensors = 0, lr_stripes = 0, lr_bf16_blocks = 0;
        for (int32_t t = first; t < first + count; ++t) {
            if (descs[t].dtype != descs[first].dtype) r.dts = 2;
            if (descs[t].scale != CF_LOWRANK) r.dec_kinds |= L.dev[t].dec_flat ? 2 : 1;
            if (descs[t].scale == CF_LOWRANK) {
                if (lr_tensors++ == 0) r.lr_first_slot = L.dev[t].lr_slot;
                if (descs[t].n_channels > r.lr_max_channels) r.lr_max_channels = (int32_t)descs[t].n_channels;
                if (descs[t].n_tokens > r.lr_max_tokens) r.lr_max_tokens = descs[t].n_tokens;
                r.lr_wires |= descs[t].dtype == CF_BF16 && !(opts.flags & CF_FLAG_LOWRANK_INT4) ? 1 : 2;
                const int64_t tokens = lowrank_project_tokens(descs[t].n_channels), blocks = (descs[t].n_tokens + tokens - 1) / tokens;
                r.lr_project_blocks = std::max<int32_t>(r.lr_project_blocks, (int32_t)blocks);
                if (descs[t].dtype == CF_BF16) lr_bf16_blocks += blocks;
                lr_stripes += lowrank_stripes(descs[t].n_channels);
            }
        }
        if (r.lr_max_channels > 0) {    // as many shares as the rule says and the workspace holds; the sums are the same either way
            r.lr_project_many = lr_bf16_blocks >= kLowRankProjectMany;
            r.lr_split = (int32_t)lowrank_split(r.lr_max_channels, r.lr_max_tokens, lr_stripes);
            while (lowrank_slice_bytes_of(r.lr_max_channels, r.lr_split, lr_tensors) > L.lr_slice_bytes) r.lr_split /= 2;
        }
        return r;
    }

    // Whether most of the call's elements with channel scales are tensors of that kind, in a context of mostly uneven rows.
    bool mostly(int32_t first, int32_t count, uint8_t kind) const
    {
        if (!L.sp_uneven) return false;
        int64_t of_kind = 0, others = 0;
        for (int32_t t = first; t < first + count; ++t)
            if (descs[t].scale == CF_SCALE_CHANNEL) (L.uneven[t] & kind ? of_kind : others) += descs[t].n_tokens * descs[t].n_channels;
        return of_kind > others;
    }

    // Bytes of errors and, fused, reconstructions that the call writes for tensors with channel scales.
    int64_t written_bytes(int32_t first, int32_t count, bool fused) const
    {
        int64_t bytes = 0;
        for (int32_t t = first; t < first + count; ++t)
            if (descs[t].scale == CF_SCALE_CHANNEL) bytes += descs[t].n_tokens * descs[t].n_channels * (int64_t)(dtype_size(opts.err_dtype) + (fused ? dtype_size(descs[t].dtype) : 0));
        return bytes;
    }

    // Whether short items serve the call: `r` and `v` are theirs then.  resident: how many the device holds at once.
    bool take_short(int32_t first, int32_t count, uint32_t resident, bool fused, LaunchRange &r, BatchView &v) const
    {
        uint32_t items = 0;
        for (int32_t t = first; t < first + count; ++t) {
            if (L.n_short_items == 0 || L.short_dev[t].p_rows == 0) return false;
            items += (uint32_t)(L.short_dev[t].p_n_rb * L.short_dev[t].p_n_stripes);
        }
        if (items > (uint32_t)kShortItems || items > resident) return false;
        r.sp_short = 1;
        r.sp_blocks = items > (uint32_t)kShortBlocksItems && mostly(first, count, kUnevenRow) && written_bytes(first, count, fused) >= kShortBlocksBytes;
        r.item_lo = L.short_dev[first].p_item_begin;
        r.item_hi = r.item_lo + items;
        r.direct_descs = L.short_dev.data() + first;
        v.item_state = ws + L.off_short_state;
        return true;
    }

    // anything for k_encode (with_channel: channel-scale tensors too; not when the single-pass kernel took them)
    bool range_has_quantised(int32_t first, int32_t count, bool with_channel) const
    {
        for (int32_t t = first; t < first + count; ++t) {
            const int sc = descs[t].scale;
            if (sc == CF_SCALE_GROUP || sc == CF_SCALE_RANK1 || (with_channel && sc == CF_SCALE_CHANNEL)) return true;
        }
        return false;
    }

    bool range_has_sparse(int32_t first, int32_t count, int block) const   // anything for k_encode_nm of that block length
    {
        for (int32_t t = first; t < first + count; ++t)
            if (descs[t].scale == CF_SPARSE_NM && descs[t].group == block) return true;
        return false;
    }

    bool range_has_channel(int32_t first, int32_t count) const      // anything that needs the reduction kernels
    {
        for (int32_t t = first; t < first + count; ++t)
            if (descs[t].scale == CF_SCALE_CHANNEL || descs[t].scale == CF_SCALE_RANK1) return true;
        return false;
    }

    bool range_all_channel(int32_t first, int32_t count) const
    {
        for (int32_t t = first; t < first + count; ++t)
            if (descs[t].scale != CF_SCALE_CHANNEL) return false;
        return true;
    }

    int range_lowrank_iters(int32_t first, int32_t count) const       // most subspace iterations any tensor asks for; -1 = no such tensor
    {
        int iters = -1;
        for (int32_t t = first; t < first + count; ++t)
            if (descs[t].scale == CF_LOWRANK && descs[t].bits > iters) iters = descs[t].bits;
        return iters;
    }

    bool range_has_elementwise(int32_t first, int32_t count) const    // anything k_encode / k_decode handle
    {
        for (int32_t t = first; t < first + count; ++t)
            if (descs[t].scale != CF_LOWRANK) return true;
        return false;
    }

    bool range_has_rank1(int32_t first, int32_t count) const
    {
        for (int32_t t = first; t < first + count; ++t)
            if (descs[t].scale == CF_SCALE_RANK1) return true;
        return false;
    }
};

namespace {

cf_status check_range(const cf_ctx *ctx, int32_t first, int32_t count)
{
    if (!ctx) return CF_ERR_INVALID_ARG;
    if (first < 0 || count < 0 || (int64_t)first + count > (int64_t)ctx->descs.size()) return CF_ERR_INVALID_ARG;
    return CF_OK;
}

cf_status check_warm(const cf_ctx *ctx, int32_t first, int32_t count)
{
    for (int32_t t = first; t < first + count; ++t)
        if (!ctx->warm[t]) return CF_ERR_STATE;
    return CF_OK;
}

// Validates one pointer array (host array of `count` device pointers).
cf_status check_ptrs(const void *const *arr, int32_t count)
{
    if (!arr) return CF_ERR_INVALID_ARG;
    for (int32_t k = 0; k < count; ++k)
        if (!arr[k] || !aligned16(arr[k])) return CF_ERR_INVALID_ARG;
    return CF_OK;
}

// Scale buffers: the N:M sparsifier has none, its entries are ignored and may be null.
cf_status check_scale_ptrs(const cf_ctx *ctx, int32_t first, int32_t count, const void *const *arr)
{
    if (!arr) return CF_ERR_INVALID_ARG;
    for (int32_t k = 0; k < count; ++k) {
        if (ctx->descs[first + k].scale == CF_SPARSE_NM) {
            if (arr[k] && !aligned16(arr[k])) return CF_ERR_INVALID_ARG;
        } else if (!arr[k] || !aligned16(arr[k])) {
            return CF_ERR_INVALID_ARG;
        }
    }
    return CF_OK;
}

cf_status device_fail(cf_ctx *ctx, hipError_t e)
{
    ctx->last_hip = (int32_t)e;
    return CF_ERR_DEVICE;
}

// Builds a context over `workspace` and brings its tables there.  Everything travels inside kernel arguments
// (no host-to-device copy, no memset), so this works wherever a kernel launch does.
cf_status make_ctx(cf_ctx **out, const cf_tensor_desc *descs, int32_t n_tensors, const cf_options &o, void *workspace,
                   size_t workspace_bytes, hipStream_t s, bool uneven_stripes = true)
{
    cf_ctx *ctx = new (std::nothrow) cf_ctx;
    if (!ctx) return CF_ERR_INVALID_ARG;
    cf_status st = make_layout(descs, n_tensors, o, ctx->L, uneven_stripes);
    if (st != CF_OK) { delete ctx; return st; }
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) % kAlign) != 0 || workspace_bytes < ctx->L.total) {
        delete ctx;
        return CF_ERR_WORKSPACE;
    }
    ctx->descs.assign(descs, descs + n_tensors);
    ctx->opts = o;
    ctx->ws = static_cast<uint8_t *>(workspace);
    ctx->ws_bytes = workspace_bytes;
    ctx->ptrs.resize(n_tensors);
    std::memset(ctx->ptrs.data(), 0, sizeof(TensorPtrs) * (size_t)n_tensors);
    ctx->warm.assign(n_tensors, 0);

    const Layout &L = ctx->L;
    const size_t prefix_bytes = sizeof(uint32_t) * (size_t)(n_tensors + 1);
    hipError_t e = hipGetDevice(&ctx->device);
    if (e == hipSuccess) e = launch_upload_bytes(L.dev.data(), ctx->ws + L.off_descs, sizeof(TensorDev) * (size_t)n_tensors, s);
    if (e == hipSuccess) e = launch_upload_bytes(L.tile_prefix.data(), ctx->ws + L.off_tile_prefix, prefix_bytes, s);
    if (e == hipSuccess) e = launch_upload_bytes(L.fin_prefix.data(), ctx->ws + L.off_fin_prefix, prefix_bytes, s);
    if (e == hipSuccess) e = launch_upload_bytes(L.ew_prefix.data(), ctx->ws + L.off_ew_prefix, prefix_bytes, s);
    if (e == hipSuccess) e = launch_upload_bytes(L.dec_prefix.data(), ctx->ws + L.off_dec_prefix, prefix_bytes, s);
    if (e == hipSuccess) e = launch_upload_bytes(L.item_prefix.data(), ctx->ws + L.off_item_prefix, prefix_bytes, s);
    if (e == hipSuccess && L.n_items > 0)
        e = launch_fill_item_tensor(reinterpret_cast<const uint32_t *>(ctx->ws + L.off_item_prefix),
                                    reinterpret_cast<uint32_t *>(ctx->ws + L.off_item_tensor), n_tensors, s);
    if (e == hipSuccess) e = launch_fill_words(ctx->ws + L.off_ptrs, 0u, sizeof(TensorPtrs) * (size_t)n_tensors / 4, s);
    if (e == hipSuccess) e = launch_fill_words(ctx->ws + L.off_error, 0u, 64, s);
    if (e == hipSuccess) e = ctx->fresh_partials(s);
    if (e == hipSuccess && L.single_pass && L.max_group_items > 0) {
        int n_cu = 0;
        e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, ctx->device);
        if (e == hipSuccess)
            for (int et = 0; et < 2; ++et)
                for (int fu = 0; fu < 2; ++fu)
                    ctx->persist_grid[et][fu] = persistent_max_blocks_per_cu(o.ef, et, fu != 0, L.sp_wide, L.sp_slim) * n_cu;
    }
    if (e != hipSuccess) {
        (void)hipGetLastError();
        delete ctx;
        return CF_ERR_DEVICE;
    }
    *out = ctx;
    return CF_OK;
}

// Runs one launch; when the call is being profiled, brackets it with the caller's events.
template <class F>
hipError_t launch(cf_ctx *ctx, hipStream_t s, const char *name, F &&f)
{
    const int32_t k = ctx->prof_count;
    const bool rec = ctx->prof_armed && (size_t)(2 * k + 1) < ctx->prof_events.size();
    if (ctx->prof_armed && k < 16) ctx->prof_names[k] = name;
    if (ctx->prof_armed) ctx->prof_count = k + 1;
    hipError_t e = hipSuccess;
    if (rec) e = hipEventRecord(ctx->prof_events[2 * k], s);
    if (e == hipSuccess) e = f();
    if (e == hipSuccess && rec) e = hipEventRecord(ctx->prof_events[2 * k + 1], s);
    return e;
}

struct ProfileScope {      // a profiled call is exactly one entry-point call
    cf_ctx *ctx;
    explicit ProfileScope(cf_ctx *c) : ctx(c) { if (ctx->prof_armed) ctx->prof_count = 0; }
    ~ProfileScope() { ctx->prof_armed = false; }
};

// Brings the workspace pointer table up to date for [first, first+count).
// Arrays that an entry point does not take are passed as nullptr and keep
// their last value.  Nothing is launched when no pointer changed.
cf_status sync_ptrs(cf_ctx *ctx, int32_t first, int32_t count, const void *const *x, void *const *recon,
                    void *const *err, void *const *codes, void *const *scales, hipStream_t s)
{
    bool changed = false;
    for (int32_t k = 0; k < count; ++k) {
        TensorPtrs &p = ctx->ptrs[first + k];
        TensorPtrs q = p;
        if (x) q.x = x[k];
        if (recon) q.recon = recon[k];
        if (err) q.err = err[k];
        if (codes) q.codes = static_cast<uint8_t *>(codes[k]);
        if (scales) q.scales = static_cast<float *>(scales[k]);
        if (std::memcmp(&p, &q, sizeof p) != 0) {
            p = q;
            changed = true;
        }
    }
    // The mirror describes the table as work enqueued on ptrs_stream after the last upload sees it.  On another
    // stream nothing orders that upload before this call, and while a stream is being captured into a graph the
    // upload is recorded, not run (nobody knows whether or when the graph will): in both cases the whole table
    // is uploaded, and after a captured call it counts as unknown again.
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &cap) != hipSuccess) {
        (void)hipGetLastError();
        cap = hipStreamCaptureStatusNone;
    }
    const bool capturing = cap != hipStreamCaptureStatusNone;
    const bool whole = capturing || !ctx->ptrs_synced || ctx->ptrs_stream != s;
    if (!changed && !whole) return CF_OK;
    const int32_t lo = whole ? 0 : first, n = whole ? (int32_t)ctx->ptrs.size() : count;
    TensorPtrs *table = reinterpret_cast<TensorPtrs *>(ctx->ws + ctx->L.off_ptrs);
    ctx->ptrs_synced = false;
    for (int32_t k0 = 0; k0 < n; k0 += kMaxUploadTensors) {
        int m = n - k0 < kMaxUploadTensors ? n - k0 : kMaxUploadTensors;
        PtrChunk chunk;
        std::memset(&chunk, 0, sizeof chunk);
        for (int k = 0; k < m; ++k) chunk.p[k] = ctx->ptrs[lo + k0 + k];
        hipError_t e = launch(ctx, s, "k_upload_ptrs", [&] { return launch_upload_ptrs(chunk, table + lo + k0, m, s); });
        if (e != hipSuccess) return device_fail(ctx, e);       // the table counts as unknown: the next call uploads all of it
    }
    ctx->ptrs_synced = !capturing;
    ctx->ptrs_stream = s;
    return CF_OK;
}

// Calls over few tensors whose kernels read no table: the pointers go into the kernels' arguments.  Table and mirror stay as
// they are, so this holds on any stream and under capture.  False, and nothing done, for calls over more tensors.
struct DirectPtrs {
    TensorPtrs sets[kSinglePassSets];
    bool take(LaunchRange &r, const void *const *x, const void *const *recon, const void *const *err, const void *const *codes, const void *const *scales,
              int32_t most = kDirectTensors)
    {
        if (r.count > most) return false;
        std::memset(sets, 0, sizeof(TensorPtrs) * (size_t)r.count);
        for (int32_t k = 0; k < r.count; ++k) {
            if (x) sets[k].x = x[k];
            if (recon) sets[k].recon = const_cast<void *>(recon[k]);
            if (err) sets[k].err = const_cast<void *>(err[k]);
            if (codes) sets[k].codes = static_cast<uint8_t *>(const_cast<void *>(codes[k]));
            if (scales) sets[k].scales = static_cast<float *>(const_cast<void *>(scales[k]));
        }
        r.direct = sets;
        return true;
    }
};

// Alg. 3 on the low-rank tensors of the range: Q <- orth(Q0); T x { P <- A Q; Z <- A^T P; Q <- orth(Z) };
// U <- A Q; then D = U V^T, error and reconstruction.
cf_status run_lowrank_sender(cf_ctx *ctx, int32_t first, int32_t count, const BatchView &v, const LaunchRange &r,
                             bool fused, hipStream_t s)
{
    const int iters = ctx->range_lowrank_iters(first, count);
    if (iters < 0) return CF_OK;
    if (count > 65535) return CF_ERR_SHAPE;     // the low-rank kernels index the tensors of a call with blockIdx.y
    hipError_t e = launch(ctx, s, "k_lr_orth", [&] { return launch_lr_orth(v, r, true, 0, s); });
    if (e != hipSuccess) return device_fail(ctx, e);
    for (int it = 1; it <= iters; ++it) {       // tensors that asked for fewer iterations sit the later ones out
        e = launch(ctx, s, "k_lr_project", [&] { return launch_lr_project(v, r, false, it, s); });
        if (e != hipSuccess) return device_fail(ctx, e);
        e = launch(ctx, s, "k_lr_backproject", [&] { return launch_lr_backproject(v, r, it, s); });
        if (e != hipSuccess) return device_fail(ctx, e);
        e = launch(ctx, s, "k_lr_orth", [&] { return launch_lr_orth(v, r, false, it, s); });
        if (e != hipSuccess) return device_fail(ctx, e);
    }
    e = launch(ctx, s, "k_lr_project", [&] { return launch_lr_project(v, r, true, 0, s); });
    if (e != hipSuccess) return device_fail(ctx, e);
    if (ctx->opts.flags & CF_FLAG_LOWRANK_INT4) {
        e = launch(ctx, s, "k_lr_quant_u", [&] { return launch_lr_quant_u(v, r, s); });
        if (e != hipSuccess) return device_fail(ctx, e);
    }
    e = launch(ctx, s, "k_lr_apply", [&] { return launch_lr_encode(v, r, ctx->opts.err_dtype, fused, s); });
    if (e != hipSuccess) return device_fail(ctx, e);
    return CF_OK;
}

// The row-local encoders over the element-wise tiles of the range: k_encode for the quantisers (channel-scale
// tensors only when with_channel: not when the single-pass kernel already took them, r.only_group_scale),
// k_encode_nm for the sparsifier (once per block length); each only if the range holds such a tensor.
hipError_t run_row_local(cf_ctx *ctx, int32_t first, int32_t count, const BatchView &v, const LaunchRange &r, bool fused,
                         bool with_channel, hipStream_t s)
{
    const int ef = ctx->opts.ef, et = ctx->opts.err_dtype;
    hipError_t e = hipSuccess;
    if (ctx->range_has_quantised(first, count, with_channel)) {
        e = launch(ctx, s, "k_encode", [&] { return launch_encode(v, r, ef, et, fused, s); });
        if (e != hipSuccess) return e;
    }
    for (int pair = 0; pair < 2 && e == hipSuccess; ++pair)
        if (ctx->range_has_sparse(first, count, pair ? 16 : 8))
            e = launch(ctx, s, "k_encode_nm", [&] { return launch_encode_nm(v, r, ef, et, fused, pair != 0, s); });
    return e;
}

cf_status run_sender(cf_ctx *ctx, int32_t first, int32_t count, const void *const *x, void *const *recon,
                     void *const *err, void *const *codes, void *const *scales, void *stream, bool fused)
{
    cf_status st = check_range(ctx, first, count);
    if (st != CF_OK) return st;
    if (count == 0) return CF_OK;
    if ((st = check_ptrs(x, count)) != CF_OK) return st;
    if ((st = check_ptrs(recon, count)) != CF_OK) return st;
    if ((st = check_ptrs(err, count)) != CF_OK) return st;
    if ((st = check_ptrs(codes, count)) != CF_OK) return st;
    if ((st = check_scale_ptrs(ctx, first, count, reinterpret_cast<const void *const *>(scales))) != CF_OK) return st;
    for (int32_t k = 0; k < count; ++k) {       // the buffers of one tensor must not overlap one another
        const BufferBytes b = buffer_bytes(ctx->descs[first + k], ctx->opts);
        const void *px = x[k], *pr = recon[k], *pe = err[k], *pc = codes[k], *ps = scales[k];
        if (overlap(px, b.recon, pr, b.recon) || overlap(px, b.recon, pe, b.err) || overlap(pr, b.recon, pe, b.err)) return CF_ERR_INVALID_ARG;
        if (overlap(pc, b.codes, px, b.recon) || overlap(pc, b.codes, pr, b.recon) || overlap(pc, b.codes, pe, b.err)) return CF_ERR_INVALID_ARG;
        if (overlap(ps, b.scales, px, b.recon) || overlap(ps, b.scales, pr, b.recon) || overlap(ps, b.scales, pe, b.err) ||
            overlap(ps, b.scales, pc, b.codes))
            return CF_ERR_INVALID_ARG;
    }
    if ((st = check_warm(ctx, first, count)) != CF_OK) return st;

    hipStream_t s = static_cast<hipStream_t>(stream);
    ProfileScope prof(ctx);
    BatchView v = ctx->view();
    LaunchRange r = ctx->range(first, count);
    const int ef = ctx->opts.ef, et = ctx->opts.err_dtype;
    hipError_t e;
    const int grid = ctx->persist_grid[et == CF_BF16 ? 1 : 0][fused ? 1 : 0];
    const bool forced = (ctx->opts.flags & CF_FLAG_SINGLE_PASS) != 0;
    // unless asked for, not for very tall tensors (see sp_too_tall) in calls of more than a round of workgroups, 512 on the whole MI355X (us, single pass / two kernels:
    // one tensor of [32768, 3072], 3072 items, 303 / 259, of [65536, 1024], 2048 items, 249 / 177; 4 x [20000, 128], 320
    // items, 34 / 48; one [65536, 128], 256 items in groups of 128, 35 / 52, [131072, 64], 256 in one group, 46 / 60, [40000,
    // 384], 474 in groups of 79, 48 / 81, [30000, 256] fp32 39 / 59)
    const uint32_t items = r.item_hi - r.item_lo;
    const bool small_call = grid > 0 && items <= (uint32_t)grid;
    // nor, in calls of more than a round, for tensors of fewer than 256 tokens that leave too much of their items empty.  Single pass / two kernels, us, 114 and 57
    // tensors of 3072 channels:
    //   groups of one item of 128 rows (bf16)   30 % full 53.6 / 50.9 and 30.5 / 30.7, 34 % 57.3 / 54.5 and 31.2 / 33.5, 40 % 60.0 / 60.3 and 32.2 / 36.0, 100 % 104 / 124 and 54 / 66;
    //                                           of [50, 1096], whose last stripe is 28 % of one, 39 % 35.3 / 35.3
    //                      64 rows              fp32 20 % 34.7 / 37.8 and 19.9 / 24.7, bf16 without feedback 20 % 34.7 / 34.6 and 20.4 / 23.0, literal 20 % 37.5 / 34.4, 25 % 38.2 / 37.6
    //                      32 rows              fp32 without feedback 9 % 21.9 / 23.9 and 12.3 / 19.7
    //     (an empty row costs the less the fewer of them a lane has)
    //   groups of two, which wait for another   bf16 51 % 141 / 126 and 73.6 / 68.0, 60 % 147 / 145 and 76.7 / 77.5, 70 % 155 / 161 and 81.5 / 87.4; fp32 51 % 128 / 111 and
    //                                           63.6 / 59.4, 60 % 135 / 132 and 67.6 / 68.0, 70 % 142 / 154; without feedback 59 % 91.2 / 82.1 and 46.7 / 48.5, 70 % 94.4 / 93.4
    //   of three and more                       two thirds full at least: 187 / 218 (68 %) and better
    // Several shapes count by their items: 57 x [256, 3072] with 57 x [20, 3072] 123 / 137, 20 with 80 79 / 66; 30 x [1024, 64] with 90 x [16, 3072] 52 / 44.  Two kernels
    // take a tall tensor through one latency after another, whatever else the call has: 40 x [16, 3072] with 10 x [3072, 64] (720 items) 34 / 51, 110 with one
    // (1344) 50 / 55, 100 with 10 (1440) 54 / 63, 114 with 20 (1848) 71 / 63, 60 x [20, 3072] with 3 x [2048, 512] 33 / 46, 80 x [16, 3072] with 10 x [1536, 64] 46 / 42.
    // Calls of a round, whatever their shape: 114 x [8, 1024] bf16 (456 items) 20.8 / 25.2, 30 x [128, 512] (60) 20.2 / 20.2, 9 x [64, 256] (9) 18.3 / 19.5; with their
    // pointers along 8 x [64, 256] 9.6 / 19.3, [1, 8] 9.9 / 19.2, [4096, 256] 14.1 / 17.0, [16384, 64] 20.0 / 23.1 (what Python adds to a call, some 9 us, hides what
    // the kernel takes below that).  Replayed from a graph, where launches cost less, tiny bf16 calls of more than eight tensors are the slower ones: 9 x [64, 256]
    // 15.5 / 13.1, 60 x [16, 256] 15.5 / 14.0, but 20 x [250, 1024] 19.0 / 27.6.
    const double rounds = grid > 0 ? (double)items / grid : 0.0;
    const int stripe = ctx->L.sp_wide ? kStripeChannelsWide : ctx->L.sp_slim ? kStripeChannelsSlim : kStripeChannels;
    double gain = 0.0;              // over the items, how far each is filled less how far it has to be
    bool tall = false;
    for (int32_t t = first; t < first + count; ++t) {
        const TensorDev &d = ctx->L.dev[t];
        if (d.p_rows == 0) continue;
        const int rows_per_lane = single_pass_rows_per_lane(d.dtype, ef);
        const double rows = (double)d.n_tokens / d.p_rows, width = (double)d.n_channels / stripe;         // in items
        tall |= d.n_tokens >= 2048;
        if (d.n_tokens >= 256 || d.p_n_rb > 2) gain += d.p_n_stripes * d.p_n_rb * (rounds <= 3.0 ? 0.4 : 0.3);      // as full as can be
        else if (d.p_n_rb == 2) gain += d.p_n_stripes * (rows - (rounds <= 3.0 ? 1.2 : 1.4));
        else gain += rows * width - d.p_n_stripes * (rows_per_lane < 8 ? 0.1 : rows_per_lane < 16 ? 0.25 : rounds <= 2.0 ? 1.0 / 3.0 : 0.4);
    }
    const bool worth_it = forced || small_call || (!ctx->L.sp_too_tall && !(fused && rounds > kUnevenRounds && ctx->mostly(first, count, kUnevenTwo)) && (gain >= 0.0 || (tall && rounds <= 3.0)));
    // (a group larger than what the device holds at once would have its first workgroups wait for ones that cannot
    // start before they leave: correct, they give up and compute the missing sums, but slow: such tensors take two kernels)
    const bool single_pass = ctx->L.single_pass && grid >= ctx->L.max_group_items && grid >= 1 && r.item_hi > r.item_lo && worth_it;
    r.sp_blocks = ctx->mostly(first, count, kUnevenBlocks) &&
                  ctx->written_bytes(first, count, fused) >= (ctx->L.sp_wide ? kBlocksBytesWide : ctx->L.sp_slim ? kBlocksBytesSlim : kBlocksBytes);
    DirectPtrs direct;
    // kernels that take their pointers as arguments: the row-local ones, and the single pass
    const bool one_pass = single_pass && ctx->range_all_channel(first, count);
    const bool is_direct = (one_pass || !ctx->range_has_channel(first, count)) && ctx->range_lowrank_iters(first, count) < 0 &&
                           direct.take(r, x, recon, err, codes, reinterpret_cast<const void *const *>(scales), one_pass ? kSinglePassSets : kDirectTensors);
    if (is_direct && !one_pass) {
        e = run_row_local(ctx, first, count, v, r, fused, true, s);
        return e == hipSuccess ? CF_OK : device_fail(ctx, e);
    }
    if (is_direct && count <= kDirectTensors && !(ctx->opts.flags & CF_FLAG_FIXED_GRID)) ctx->take_short(first, count, 2u * (uint32_t)grid, fused, r, v);       // they need half the registers
    if (!is_direct && (st = sync_ptrs(ctx, first, count, x, recon, err, codes, scales, s)) != CF_OK) return st;
    if (single_pass) {
        // channel-scale tensors: one pass, the operands stay in registers across the scale reduction
        // measured on [N, 3072] bf16 batches: up to 4 row blocks per tensor a run of consecutive items per XCD is
        // 4-20 % faster (the stripes of a code row meet in one L2), from 6 on dealing them round the XCDs is 8-15 % faster
        r.sp_xcd_major = !r.sp_short && ctx->L.max_group_items <= 4;
        r.sp_wait_polls = (ctx->opts.flags & CF_FLAG_TEST_NO_WAIT) ? 0u : kWaitPolls;
        const bool one_shot = (ctx->opts.flags & CF_FLAG_FIXED_GRID) == 0;
        if (ctx->sp_always_fresh) {
            e = launch(ctx, s, "k_fresh_partials", [&] {
                return r.sp_short ? ctx->fresh_partials_of(first, count, ctx->L.short_dev, ctx->L.off_short_state, s)
                                  : ctx->fresh_partials_of(first, count, ctx->L.dev, ctx->L.off_item_state, s);
            });
            if (e != hipSuccess) return device_fail(ctx, e);
        }
        ctx->note_single_pass(s);
        e = launch(ctx, s, r.sp_short ? "k_short_items" : "k_single_pass", [&] { return launch_single_pass(v, r, ef, et, fused, ctx->L.sp_wide, grid, one_shot, s); });
        if (e != hipSuccess) return device_fail(ctx, e);
        r.only_group_scale = 1;
        if ((e = run_row_local(ctx, first, count, v, r, fused, false, s)) != hipSuccess) return device_fail(ctx, e);
        return run_lowrank_sender(ctx, first, count, v, r, fused, s);
    }
    if (ctx->range_has_channel(first, count)) {
        e = launch(ctx, s, "k_colreduce", [&] { return launch_colreduce(v, r, ef, et, s); });
        if (e != hipSuccess) return device_fail(ctx, e);
        // the rank-1 form does k_finalize's work too
        if (ctx->range_has_rank1(first, count)) e = launch(ctx, s, "k_finalize_rank1", [&] { return launch_finalize_rank1(v, r, s); });
        else e = launch(ctx, s, "k_finalize", [&] { return launch_finalize(v, r, s); });
        if (e != hipSuccess) return device_fail(ctx, e);
    }
    if ((e = run_row_local(ctx, first, count, v, r, fused, true, s)) != hipSuccess) return device_fail(ctx, e);
    return run_lowrank_sender(ctx, first, count, v, r, fused, s);
}

}  // namespace

extern "C" {

const char *cf_status_string(cf_status s)
{
    switch (s) {
    case CF_OK: return "ok";
    case CF_ERR_INVALID_ARG: return "invalid argument";
    case CF_ERR_SHAPE: return "unsupported shape";
    case CF_ERR_UNSUPPORTED: return "unsupported configuration";
    case CF_ERR_STATE: return "tensor not warmed up";
    case CF_ERR_WORKSPACE: return "workspace too small or misaligned";
    case CF_ERR_DEVICE: return "HIP call failed";
    }
    return "unknown status";
}

cf_status cf_sizes(const cf_tensor_desc *desc, const cf_options *opts, size_t *codes_bytes, size_t *scales_bytes,
                   size_t *recon_bytes, size_t *err_bytes)
{
    if (!desc) return CF_ERR_INVALID_ARG;
    cf_options o;
    cf_status st = check_opts(opts, o);
    if (st != CF_OK) return st;
    if ((st = check_desc(*desc)) != CF_OK) return st;
    BufferBytes b = buffer_bytes(*desc, o);
    if (codes_bytes) *codes_bytes = b.codes;
    if (scales_bytes) *scales_bytes = b.scales;
    if (recon_bytes) *recon_bytes = b.recon;
    if (err_bytes) *err_bytes = b.err;
    return CF_OK;
}

size_t cf_workspace_bytes(const cf_tensor_desc *descs, int32_t n_tensors, const cf_options *opts)
{
    cf_options o;
    if (check_opts(opts, o) != CF_OK) return 0;
    Layout L;
    if (make_layout(descs, n_tensors, o, L) != CF_OK) return 0;
    return L.total;
}

cf_status cf_init(cf_ctx **out, const cf_tensor_desc *descs, int32_t n_tensors, const cf_options *opts,
                  void *workspace, size_t workspace_bytes, void *stream)
{
    if (!out) return CF_ERR_INVALID_ARG;
    *out = nullptr;
    cf_options o;
    cf_status st = check_opts(opts, o);
    if (st != CF_OK) return st;
    return make_ctx(out, descs, n_tensors, o, workspace, workspace_bytes, static_cast<hipStream_t>(stream));
}

void cf_destroy(cf_ctx *ctx) { delete ctx; }

int32_t cf_last_hip_error(const cf_ctx *ctx) { return ctx ? ctx->last_hip : 0; }

cf_status cf_profile_next_call(cf_ctx *ctx, void *const *events, int32_t n_pairs)
{
    if (!ctx || n_pairs < 0 || (n_pairs > 0 && !events)) return CF_ERR_INVALID_ARG;
    ctx->prof_events.clear();
    for (int32_t k = 0; k < 2 * n_pairs; ++k) {
        if (!events[k]) { ctx->prof_events.clear(); return CF_ERR_INVALID_ARG; }
        ctx->prof_events.push_back(static_cast<hipEvent_t>(events[k]));
    }
    ctx->prof_armed = n_pairs > 0;
    ctx->prof_count = 0;
    return CF_OK;
}

cf_status cf_check_device(cf_ctx *ctx, void *stream)
{
    if (!ctx) return CF_ERR_INVALID_ARG;
    hipError_t e = hipStreamSynchronize(static_cast<hipStream_t>(stream));
    uint32_t flag = 0;
    if (e == hipSuccess) e = hipMemcpy(&flag, ctx->ws + ctx->L.off_error, sizeof flag, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return device_fail(ctx, e);
    if (flag) {
        ctx->last_hip = 0;
        return CF_ERR_DEVICE;
    }
    return CF_OK;
}

cf_status cf_given_up_items(cf_ctx *ctx, void *stream, uint32_t *count)
{
    if (!ctx || !count) return CF_ERR_INVALID_ARG;
    hipError_t e = hipStreamSynchronize(static_cast<hipStream_t>(stream));
    uint32_t items[3] = {0, 0, 0};          // of the last single pass, and whether they were short ones
    if (e == hipSuccess) e = hipMemcpy(items, ctx->ws + ctx->L.off_error + sizeof(uint32_t) * kLastItemsWord, sizeof items, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return device_fail(ctx, e);
    uint32_t n = 0;
    const size_t off_state = items[2] ? ctx->L.off_short_state : ctx->L.off_item_state;
    for (uint32_t at = items[0]; at < items[1] && items[1] <= (items[2] ? ctx->L.n_short_items : ctx->L.n_items);) {
        uint8_t state[4096];
        const uint32_t m = std::min<uint32_t>(items[1] - at, sizeof state);
        e = hipMemcpy(state, ctx->ws + off_state + at, m, hipMemcpyDeviceToHost);
        if (e != hipSuccess) return device_fail(ctx, e);
        for (uint32_t k = 0; k < m; ++k) n += state[k] & 1u;
        at += m;
    }
    *count = n;
    return CF_OK;
}

int32_t cf_profile_launch_count(const cf_ctx *ctx) { return ctx ? ctx->prof_count : 0; }

const char *cf_profile_kernel_name(const cf_ctx *ctx, int32_t k)
{
    if (!ctx || k < 0 || k >= ctx->prof_count || k >= 16) return nullptr;
    return ctx->prof_names[k];
}

cf_status cf_set_warm(cf_ctx *ctx, int32_t first, int32_t count, int32_t warm)
{
    cf_status st = check_range(ctx, first, count);
    if (st != CF_OK) return st;
    for (int32_t t = first; t < first + count; ++t) ctx->warm[t] = warm ? 1 : 0;
    return CF_OK;
}

cf_status cf_warmup(cf_ctx *ctx, int32_t first, int32_t count, const void *const *x0, void *const *recon,
                    void *const *err, void *stream)
{
    cf_status st = check_range(ctx, first, count);
    if (st != CF_OK) return st;
    if (count == 0) return CF_OK;
    if ((st = check_ptrs(x0, count)) != CF_OK) return st;
    if ((st = check_ptrs(recon, count)) != CF_OK) return st;
    if ((st = check_ptrs(err, count)) != CF_OK) return st;
    for (int32_t k = 0; k < count; ++k) {
        const BufferBytes b = buffer_bytes(ctx->descs[first + k], ctx->opts);
        if (overlap(x0[k], b.recon, recon[k], b.recon) || overlap(x0[k], b.recon, err[k], b.err) || overlap(recon[k], b.recon, err[k], b.err))
            return CF_ERR_INVALID_ARG;
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    LaunchRange r = ctx->range(first, count);
    DirectPtrs direct;
    if (!direct.take(r, x0, recon, err, nullptr, nullptr) &&
        (st = sync_ptrs(ctx, first, count, x0, recon, err, nullptr, nullptr, s)) != CF_OK)
        return st;
    hipError_t e = launch_warmup(ctx->view(), r, ctx->opts.err_dtype, s);
    if (e == hipSuccess && ctx->sp_unordered) {
        e = ctx->fresh_partials_of(first, count, ctx->L.dev, ctx->L.off_item_state, s);
        if (e == hipSuccess) e = ctx->fresh_partials_of(first, count, ctx->L.short_dev, ctx->L.off_short_state, s);
    }
    if (e != hipSuccess) return device_fail(ctx, e);
    for (int32_t t = first; t < first + count; ++t) ctx->warm[t] = 1;
    return CF_OK;
}

cf_status cf_compress(cf_ctx *ctx, int32_t first, int32_t count, const void *const *x, const void *const *recon,
                      void *const *err, void *const *codes, void *const *scales, void *stream)
{
    return run_sender(ctx, first, count, x, const_cast<void *const *>(reinterpret_cast<const void *const *>(recon)), err,
                      codes, scales, stream, false);
}

cf_status cf_step_fused(cf_ctx *ctx, int32_t first, int32_t count, const void *const *x, void *const *recon,
                        void *const *err, void *const *codes, void *const *scales, void *stream)
{
    return run_sender(ctx, first, count, x, recon, err, codes, scales, stream, true);
}

cf_status cf_decompress(cf_ctx *ctx, int32_t first, int32_t count, const void *const *codes,
                        const void *const *scales, void *const *recon, void *stream)
{
    cf_status st = check_range(ctx, first, count);
    if (st != CF_OK) return st;
    if (count == 0) return CF_OK;
    if ((st = check_ptrs(codes, count)) != CF_OK) return st;
    if ((st = check_scale_ptrs(ctx, first, count, scales)) != CF_OK) return st;
    if ((st = check_ptrs(recon, count)) != CF_OK) return st;
    for (int32_t k = 0; k < count; ++k) {
        const BufferBytes b = buffer_bytes(ctx->descs[first + k], ctx->opts);
        if (overlap(codes[k], b.codes, recon[k], b.recon)) return CF_ERR_INVALID_ARG;
        if (overlap(scales[k], b.scales, codes[k], b.codes) || overlap(scales[k], b.scales, recon[k], b.recon)) return CF_ERR_INVALID_ARG;
    }
    if ((st = check_warm(ctx, first, count)) != CF_OK) return st;
    hipStream_t s = static_cast<hipStream_t>(stream);
    ProfileScope prof(ctx);
    LaunchRange r = ctx->range(first, count);
    DirectPtrs direct;
    if (!direct.take(r, nullptr, recon, nullptr, codes, scales) &&
        (st = sync_ptrs(ctx, first, count, nullptr, recon, nullptr, const_cast<void *const *>(codes),
                        const_cast<void *const *>(scales), s)) != CF_OK)
        return st;
    hipError_t e = hipSuccess;
    if (ctx->range_has_elementwise(first, count)) {
        e = launch(ctx, s, "k_decode", [&] { return launch_decode(ctx->view(), r, s); });
        if (e != hipSuccess) return device_fail(ctx, e);
    }
    if (ctx->range_lowrank_iters(first, count) >= 0) {
        e = launch(ctx, s, "k_lr_apply", [&] { return launch_lr_decode(ctx->view(), r, s); });
        if (e != hipSuccess) return device_fail(ctx, e);
    }
    return CF_OK;
}

namespace {
constexpr int kMaxStaticDevices = 64;
cf_ctx *g_static_ctx[kMaxStaticDevices];       // the context over each device's static scratch, kept while the tensors stay the same
}  // namespace

cf_status cf_step_fused_static(const cf_tensor_desc *descs, int32_t n_tensors, const cf_options *opts, const void *const *x,
                               void *const *recon, void *const *err, void *const *codes, void *const *scales, void *stream)
{
    cf_options o;
    cf_status st = check_opts(opts, o);
    if (st != CF_OK) return st;
    if (!descs || n_tensors < 1) return CF_ERR_INVALID_ARG;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxStaticDevices) {
        (void)hipGetLastError();
        return CF_ERR_DEVICE;
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    cf_ctx *&ctx = g_static_ctx[dev];
    const bool same = ctx && ctx->descs.size() == (size_t)n_tensors &&
                      std::memcmp(ctx->descs.data(), descs, sizeof(cf_tensor_desc) * (size_t)n_tensors) == 0 &&
                      std::memcmp(&ctx->opts, &o, sizeof o) == 0;
    if (!same) {
        delete ctx;
        ctx = nullptr;
        void *ws = nullptr;
        if (static_scratch(&ws) != hipSuccess) {
            (void)hipGetLastError();
            return CF_ERR_DEVICE;
        }
        // lays the tables out in the scratch array afresh (CF_ERR_WORKSPACE if these tensors need more than it holds)
        st = make_ctx(&ctx, descs, n_tensors, o, ws, kStaticScratchBytes, s);
        // no tensors outgrow the scratch because of the stripes of uneven rows
        if (st == CF_ERR_WORKSPACE) st = make_ctx(&ctx, descs, n_tensors, o, ws, kStaticScratchBytes, s, false);
        if (st != CF_OK) return st;
        for (auto &w : ctx->warm) w = 1;        // the caller vouches for recon and err
        ctx->sp_unordered = ctx->sp_always_fresh = true;        // every caller on the GPU shares the scratch, and nobody warms up
    }
    return run_sender(ctx, 0, n_tensors, x, recon, err, codes, scales, stream, true);
}

}  // extern "C"
