// Internal interface between the C-ABI layer (cf_api.cpp) and the gfx950
// kernels (cf_kernels.hip).  Not installed; not part of the ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace cf {

// Every tile of the tiled kernels is TILE_ROWS(rb) x TILE_CHANNELS: 128 lanes
// each own 8 consecutive channels (one 128-bit load of bf16).
constexpr int kTileThreads = 128;
constexpr int kChunk = 8;                                   // channels per lane
constexpr int kTileChannels = kTileThreads * kChunk;        // 1024
constexpr int kFinalizeThreads = 256;
constexpr int kFinalizeColumns = 16;                        // columns per finalise block, kFinalizeThreads where columns are many or have few partials
constexpr int kRank1Threads = 1024;                         // one block per tensor finishes the token scales u
constexpr int kMaxRank1Colblocks = 128;                     // rank-1 scales: C <= 128 * 1024
constexpr int kMaxUploadTensors = 64;                       // pointer sets per upload launch
// Calls of one kernel over at most so many tensors (one layer's K and V of four peers) carry their pointers in the kernel's
// arguments and skip the upload to the table, a launch and a gap, where pointers change from call to call: receivers of n x [1024, 3072], bf16, 2-bit,
// table / arguments, us: n = 1 8.6 / 4.8, 4 13.5 / 11.3, 6 17.4 / 15.4, 8 22.1 / 19.4; with room for 16 tensors 12 29.5 / 27.3, 16 37.5 / 35.2, the
// small calls the same.  (With room for 16 the arguments are 340 bytes longer; the lead is open.)  n x [64, 256]: 8.6 / 4.4 for any n.
constexpr int kDirectTensors = 8;
// k_single_pass takes the pointers of up to so many tensors along, and finds the descriptors of more than kDirectTensors in the table.
constexpr int kSinglePassSets = 64;
// Single-pass path: one workgroup of 256 lanes keeps an item of p_rows x 128
// channels (x and recon, raw) in registers between the scale reduction and the
// encode; lanes are 16 chunks x 16 row-lanes, so a row segment is 256 bytes of
// bf16 and a row's 1-bit codes of one item are 16 bytes.  Measured on 114 x
// [4096, 3072] bf16: 64- / 128- / 256-channel stripes (8 / 16 / 32 items per
// reduction group) 2.94 / 2.86 / 2.92 ms; 32-channel ones (64-byte segments)
// were 50 % slower.  Short tensors do better with the wide stripe (items half
// as tall, twice as many per group): 57 x [1024, 3072] 0.417 -> 0.382 ms; a
// context whose tallest channel-scale tensor makes at most 12 items per group
// with the narrow stripe (bf16: N <= 3072) takes the wide one, and one of mostly
// tensors of more than 40 (N > 10240) the slim one, whose items are twice as tall;
// contexts of mostly bf16 rows that are no whole blocks of 64 bytes have lines of
// their own (kUnevenWideGroup, kUnevenNarrowGroup).
constexpr int kPersistThreads = 256;
constexpr int kStripeChannels = 128;
constexpr int kStripeChannelsWide = 2 * kStripeChannels;    // 256
constexpr int kStripeChannelsSlim = kStripeChannels / 2;    // 64
// Rows a lane of the single-pass kernel keeps in registers: 128 VGPRs of raw operands, i.e. 16 rows of bf16 x and
// recon, half as many of fp32, half as many again when the error buffer is an operand too (CF_EF_LITERAL = 1,
// CF_EF_OFF = 2).  Measured on 114 x [4096, 3072] bf16 (two waves per SIMD): 16 rows 2.65 ms; 8 rows at three
// waves per SIMD 2.97 ms, at four (spills) 4.8 ms.  dtype: cf_dtype (CF_F32 = 0).
// Short items, of calls that leave most of the device idle otherwise, have a quarter of them and are 64 channels wide (128 channels, 32 rows to
// 64 of bf16 and groups of twice the items: [4096, 512] 14.9 us against 12.3, 2 x [1024, 3072] 15.3 / 14.7, 8 x [512, 1024] 11.8 / 12.3); see Layout::short_dev.
constexpr int kShortFraction = 4;
constexpr int kShortStripeChannels = 64;
constexpr int kShortItems = 1024;                           // the most of a call: four workgroups a CU of the whole MI355X; a part of one takes as many as it holds
constexpr int kShortGroupLimit = 64;                        // the most of a group
// Workgroups without an item that a call of short items may have.  Steps, us, with / by looking up: 2 x [1024, 3072] (none) 12.9 / 13.3, [2048, 512] + [1024, 512] (64) 8.4 / 8.6,
// [1024, 3072] + [768, 3072] (96) 12.2 / 12.1, + [512, 3072] (192) 12.1 / 11.6, [1024, 2048] + 2 x [512, 2048] (256) 11.6 / 10.1, [8192, 64] + [8, 61440] (121,856) 151 / 8.8.
constexpr uint64_t kShortEmpty = 64;
constexpr int single_pass_rows_per_lane(int dtype, int ef) { return 16 / (dtype == 0 ? 2 : 1) / ((ef == 1 || ef == 2) ? 2 : 1); }
// A workgroup polls a missing partial this many times (a microsecond or two each) before it gives its item up.
constexpr uint32_t kWaitPolls = 4096;
// A tensor of more 128-channel items per group than kTallGroupItems is tall: contexts of mostly such take 64-channel
// stripes.  Groups of more items than the limit of the stripe in use take two kernels by default, unless the device holds
// the whole call at once: nothing has to wait for a second round of workgroups then.
constexpr int kWideGroup = 12;
constexpr int kTallGroupItems = 40;
constexpr int kNarrowGroupLimit = 48;
constexpr int kSlimGroupLimit = 64;                         // see slim_group_limit
constexpr int kSlimGroupLimitUneven = 38;
constexpr int kSlimGroupLimitNaive = 24;
// Contexts of mostly uneven rows, in 128-channel items a group: 256-channel stripes up to the first (of those that are three quarters of the context), no 64-channel ones
// up to kUnevenNarrowGroup, nor two kernels because of kNarrowGroupLimit; fused calls of more than kUnevenRounds rounds by two kernels where most are past the first, or past these where the error is bf16 or the channels a
// multiple of 16.  make_layout has the figures.
constexpr int kUnevenWideGroup = 18;
constexpr int kUnevenNarrowGroup = 64;
constexpr int kUnevenGroupLimitBf16Error = 28;
constexpr int kUnevenGroupLimitEven = 32;
constexpr double kUnevenRounds = 2.5;
// Calls over uneven rows leave parts of blocks to the L2 from so many bytes of errors and reconstructions on, more than its 32 MB hold: what it holds at a kernel's end has to be
// written then, and smaller calls wait for that.  All streamed / parts left, us: steps of 12 x [300, 1096] (24 MB) 18.2 / 20.5, 24 (47) 23.8 / 25.6, 36 (71) 41.5 / 41.8, 9 x [1000,
// 1096] (59) 28.0 / 27.2, 12 (79) 34.6 / 29.4, [12000, 328] (24) 21.5 / 24.0, [8400, 1096] (55) 34.4 / 31.2, three (166) 91 / 70, with bf16 errors (37) 27.3 / 29.2, two (74) 53.7 / 50.1;
// sent, 9 x [2000, 520] (37) 21.9 / 23.8, 15 (62) 39.1 / 39.3, [8400, 1096] two (74) 50.9 / 49.6, with bf16 errors (37) 41.1 / 43.3, three (55) 50.6 / 52.2.
// Narrower stripes have more parts: 128 channels, 2 x [10078, 440] (53) 34.5 / 29.8, sent (35) 25.8 / 25.9; 64 channels, [17320, 376] (39) 28 / 25, three [18773, 152] (51) 40 / 33.
constexpr int64_t kBlocksBytesWide = 54000000, kBlocksBytes = 45000000, kBlocksBytesSlim = 36000000;
// Short items, steps: 6 x [512, 1096] (432 items, 20 MB) 15.1 / 15.4, 2 x [2048, 1096] (576, 27) 16.0 / 13.5, 6 x [1024, 1096] (864, 40) 22.5 / 16.7, [1024, 3080] (392, 19) 11.4 / 11.1, two
// (784, 38) 18.5 / 20.8; sent, 4 x [1024, 1096] (576, 18) 12.4 / 11.7, 6 (864, 27) 16.8 / 14.8, with bf16 errors (13) 13.1 / 14.2.
constexpr int kShortBlocksItems = 448;
constexpr int64_t kShortBlocksBytes = 17000000;
constexpr int kLastItemsWord = 32;                          // 128 bytes behind the error word: the first item of the last single pass, and the one past its last

// The single pass's partials carry the sign of their call in this bit; item states and partials are filled with the other word before a first call.
constexpr uint32_t kPartialSign = 0x80000000u;
constexpr uint32_t kFreshPartials = 0x80808080u;

// Static description of one tensor; built at cf_init, lives in the workspace.
struct alignas(16) TensorDev {
    int64_t n_tokens;
    int32_t n_channels;
    int32_t n_chunks;       // C / 8
    int32_t dtype;          // cf_dtype
    int32_t bits;           // 1 | 2 | 4
    int32_t scale;          // cf_scale_kind
    int32_t rb_rows;        // rows per tile (power of two, multiple of 8)
    int32_t n_rowblocks;    // ceil(N / rb_rows)
    int32_t n_colblocks;    // ceil(n_chunks / 128)
    uint32_t tile_begin;    // id of this tensor's first tile in the batched grids
    uint32_t fin_begin;     // id of its first finalise block
    uint64_t partial_off;   // byte offset in the workspace of partial[n_rowblocks][C] (channel scales)
    // single-pass path (channel scales): items of p_rows x kStripeChannels (or kStripeChannelsWide)
    uint64_t p_partial_off; // byte offset of partial[p_n_rb][C]
    int32_t p_rows;         // rows per item (row-lanes x single_pass_rows_per_lane); 0 = tensor not on this path
    int32_t p_n_rb;         // ceil(N / p_rows): items per reduction group
    int32_t p_n_stripes;    // ceil(C / stripe width of the context): reduction groups of this tensor
    uint32_t p_item_begin;  // id of this tensor's first item
    int32_t fin_columns;    // columns per finalise block
    // element-wise kernels (warm-up, encode): tiles of one row x 1024 channels, or flat ones of 128 chunks across row ends
    int32_t ew_flat;
    uint32_t ew_tile_begin;
    // the receiver's kernel does less per row and likes taller tiles: dec_rows x 1024 channels, or dec_rows x 128 chunks
    int32_t dec_rows;
    int32_t dec_flat;
    uint32_t dec_tile_begin;
    // rank-1 scales: per-row sums of |z| over each 1024-channel tile, rowpart[N][n_colblocks]
    uint32_t nm_block;      // N:M sparsifier: M, channels per block (8 or 16)
                            // low-rank compressor: 4 when the factors travel as 4-bit integers, else 0
    uint32_t lr_slot;       // low-rank tensors before this one in the context
    uint64_t rowpart_off;
    // low-rank compressor: P = A Q [N][32] fp32; Z = A^T P [C][32] fp32, which the high and mid pieces of Q take the place of in
    // the order k_lr_project reads them; partial sums of Z^T Z, one [32][32] fp64 matrix per 256 channels (C > 256 only), behind them
    // the low pieces of Q, and a word of k_lr_orth's at the end of their area
    uint64_t lr_p_off, lr_z_off, lr_g_off;
};

static_assert(sizeof(TensorDev) % 4 == 0, "tables travel as 4-byte words");

// Per-call device pointers of one tensor; uploaded into the workspace.
struct TensorPtrs {
    const void *x;
    void *recon;
    void *err;
    uint8_t *codes;
    float *scales;
};

struct PtrChunk {
    TensorPtrs p[kMaxUploadTensors];
};

// A piece of one of the context's tables on its way to the workspace inside a kernel's arguments.
constexpr int kUploadWords = 896;
struct WordChunk {
    uint32_t w[kUploadWords];
};

// Device view of a context's workspace.
struct BatchView {
    const TensorDev *descs;     // [n_tensors]
    const TensorPtrs *ptrs;     // [n_tensors]
    const uint32_t *tile_prefix;    // [n_tensors + 1] reduction tiles
    const uint32_t *ew_prefix;      // [n_tensors + 1] element-wise tiles
    const uint32_t *dec_prefix;     // [n_tensors + 1] decode tiles
    const uint32_t *fin_prefix;     // [n_tensors + 1]
    const uint32_t *item_prefix;    // [n_tensors + 1] items of the single-pass path
    const uint32_t *item_tensor;    // [n_items] tensor of every item: one load where a search over the prefix would be seven
    uint32_t *error_flag;           // set if a partial is missing that a workgroup has stored itself (cannot happen); kLastItemsWord words on: the last call's items
    uint8_t *item_state;            // [n_items] single-pass path: the sign (bit 7) of the item's partial in its last call, and in bit 0 whether it gave up waiting in it
    uint8_t *workspace;
    int32_t n_tensors;
};

struct LaunchRange {
    int32_t first, count;       // tensors
    uint32_t tile_lo, tile_hi;  // reduction tiles of [first, first+count)
    uint32_t ew_lo, ew_hi;      // element-wise tiles
    uint32_t dec_lo, dec_hi;    // decode tiles
    uint32_t fin_lo, fin_hi;    // finalise blocks
    uint32_t item_lo, item_hi;  // single-pass items
    uint32_t sp_xcd_major;      // single-pass kernel: deal the items XCD-major (a run of consecutive items per XCD)
    uint32_t sp_wait_polls;     // single-pass kernel: polls of a missing partial before the workgroup computes it itself
    uint32_t sp_slim;           // single-pass kernel: items of kStripeChannelsSlim channels (tall tensors)
    uint32_t sp_blocks;         // single-pass kernel: parts of 64-byte blocks go out without the streaming hint
    uint32_t sp_short;          // single-pass kernel: short items (2: workgroups look their tensors up, see short_grid); item_lo, item_hi, direct_descs and the view's item_state are theirs
    int32_t dts;                // storage dtype of every tensor in the range (cf_dtype), or 2 if mixed
    int32_t only_group_scale;   // tiled encode: skip tensors the single-pass kernel covers
    int32_t naive;              // decode: recon_t = D instead of recon_{t-1} + D (CF_EF_NAIVE)
    int32_t dec_kinds;          // decode: bit 0, tensors with row tiles in the range; bit 1, with flat ones
    int32_t lr_max_channels;    // low-rank tensors of the range: largest C and N (0 = none)
    int64_t lr_max_tokens;
    int32_t lr_wires;           // bit 0: factors that travel as bf16 in the range; bit 1: others
    int32_t lr_project_blocks;  // workgroups of k_lr_project for the tensor that needs most, one block of tokens per wave
    int32_t lr_project_many;    // whether the bf16 tensors of the range together have enough of them for several blocks a wave
    int32_t lr_split;           // low-rank back-projection: at most so many workgroups share a channel stripe's runs of tokens (1, 2 or 4)
    uint32_t lr_first_slot;     // lr_slot of the range's first low-rank tensor
    uint64_t lr_slices_off;     // workspace offset of the shares after the first, [low-rank tensors][lr_split - 1][lr_max_channels][32] fp32
    const TensorPtrs *direct;   // host memory: the call's pointers, kDirectTensors sets at most (k_single_pass kSinglePassSets), for kernels to take as arguments; null: they are in the table
    const TensorDev *direct_descs;      // host memory: the descriptors of the call's tensors
};

// The same with the call's pointers along: what kernels of direct calls take in the range's place, in instances of their own
// (a choice between the sets and the table within one instance cost the large kernels 3-5 %).
// The sets begin 256 bytes into the arguments, behind the BatchView: 16 bytes earlier, receivers of 6 x [1024, 3072] took 17.87 instead of 17.55 us.
struct DirectRange : LaunchRange {
    char unused[256 - sizeof(BatchView) - sizeof(LaunchRange)] = {};
    TensorPtrs sets[kDirectTensors];
    explicit DirectRange(const LaunchRange &r) : LaunchRange(r), sets()
    {
        for (int k = 0; k < r.count && k < kDirectTensors; ++k) sets[k] = r.direct[k];
    }
};

// The arguments of k_single_pass: direct calls bring their tensors' pointers along, and descriptors.
struct SinglePassArgs {
    BatchView v;
    LaunchRange r;
    struct {
        TensorPtrs sets[kSinglePassSets];
        TensorDev descs[kDirectTensors];
    } direct;
};

static_assert(sizeof(BatchView) + sizeof(DirectRange) == 256 + sizeof(TensorPtrs) * kDirectTensors, "where the sets begin");

static_assert(sizeof(SinglePassArgs) <= 4096, "a kernel's arguments");

// The grid of k_short_items: row blocks x stripes x tensors, as many as the largest of the call's tensors have, where no more than kShortEmpty workgroups of it are
// without an item; else one workgroup per item, which looks its tensor up first.
struct ShortGrid {
    uint32_t x, y, z;
    bool flat;
};
inline ShortGrid short_grid(const TensorDev *descs, int count)
{
    uint64_t rb = 0, stripes = 0, items = 0;
    for (int k = 0; k < count; ++k) {
        rb = (uint64_t)descs[k].p_n_rb > rb ? (uint64_t)descs[k].p_n_rb : rb;
        stripes = (uint64_t)descs[k].p_n_stripes > stripes ? (uint64_t)descs[k].p_n_stripes : stripes;
        items += (uint64_t)descs[k].p_n_rb * (uint64_t)descs[k].p_n_stripes;
    }
    if (rb * stripes * (uint64_t)count > items + kShortEmpty) return {(uint32_t)items, 1u, 1u, true};
    return {(uint32_t)rb, (uint32_t)stripes, (uint32_t)count, false};
}

// The arguments of k_short_items: nothing of a call is elsewhere.
struct ShortArgs {
    BatchView v;
    LaunchRange r;
    TensorPtrs sets[kDirectTensors];
    TensorDev descs[kDirectTensors];
};

// f(range) with the kind of range the call's kernels take
template <class F> auto with_range(const LaunchRange &r, F &&f) { return r.direct ? f(DirectRange(r)) : f(r); }

enum class Op { Compress, StepFused };

hipError_t launch_upload_ptrs(const PtrChunk &chunk, TensorPtrs *dst, int n, hipStream_t s);
// Host tables (multiples of 4 bytes) to the workspace through kernel arguments; fills; the item -> tensor table
hipError_t launch_upload_bytes(const void *src, void *dst, size_t bytes, hipStream_t s);
hipError_t launch_fill_words(void *dst, uint32_t value, size_t n_words, hipStream_t s);
hipError_t launch_fill_item_tensor(const uint32_t *item_prefix, uint32_t *item_tensor, int n_tensors, hipStream_t s);

// The library's own scratch for callers that cannot allocate (cf_static.hip): one array per device, resolved on
// first use with that device current.
constexpr size_t kStaticScratchBytes = (size_t)16 << 20;
hipError_t static_scratch(void **ptr);
hipError_t launch_warmup(const BatchView &v, const LaunchRange &r, int err_dtype, hipStream_t s);
hipError_t launch_colreduce(const BatchView &v, const LaunchRange &r, int ef, int err_dtype, hipStream_t s);
hipError_t launch_finalize(const BatchView &v, const LaunchRange &r, hipStream_t s);
hipError_t launch_finalize_rank1(const BatchView &v, const LaunchRange &r, hipStream_t s);
hipError_t launch_encode(const BatchView &v, const LaunchRange &r, int ef, int err_dtype, bool fused, hipStream_t s);
hipError_t launch_encode_nm(const BatchView &v, const LaunchRange &r, int ef, int err_dtype, bool fused, bool pair, hipStream_t s);
hipError_t launch_decode(const BatchView &v, const LaunchRange &r, hipStream_t s);

// Low-rank compressor (cf_lowrank.hip): rank 32, C a multiple of 32 and at most kLowRankMaxChannels.
constexpr int kLowRankRank = 32;
constexpr int kLowRankMaxChannels = 3072;
// The back-projection's workgroups own kLowRankBackChannels channels each.  A tensor's tokens are summed in lowrank_runs
// runs, a property of the tensor alone: the sum has one order in every call.  Runs cost a workgroup that takes them all a
// drained pipeline and a sum over its waves each, so short tensors have fewer, wide ones above all: steps with 2 / 4
// runs, us: 114 x [1100, 2048] T = 2 1740 / 1818, 100 x [2000, 3072] 2595 / 2660, 6 x [2000, 3072] 262 / 261; 20 x [2000, 1024]
// 257 / 262, one [2048, 64] 91 / 85, one [2900, 1024] T = 2 266 / 213.
constexpr int kLowRankBackChannels = 256;
constexpr int kLowRankMaxRuns = 4;
constexpr int lowrank_runs(int64_t n_tokens, int64_t n_channels)
{
    return n_tokens <= 384 ? 1 : n_tokens <= (n_channels <= 1024 ? 1024 : 2048) ? 2 : kLowRankMaxRuns;
}
// The area of the Gram matrices: partial sums, 8 KB per 256 channels (none up to 256 channels), Q's low pieces behind them, and in the last
// word whether k_lr_orth left the tensor over.
constexpr size_t lowrank_g_bytes(int64_t n_channels) { return (size_t)n_channels * kLowRankRank * sizeof(float); }
constexpr size_t lowrank_q_low_off(int64_t n_channels) { return n_channels > 256 ? (size_t)n_channels * 32 + 8192 : 0; }
constexpr bool lowrank_g_area_fits()
{
    for (int64_t c = 32; c <= kLowRankMaxChannels; c += 32) {
        const size_t sums = c > 256 ? (size_t)((c + 255) / 256) * 8192 : 0;
        if (sums > lowrank_q_low_off(c) || lowrank_q_low_off(c) + (size_t)c * kLowRankRank * 2 + sizeof(uint32_t) > lowrank_g_bytes(c)) return false;
    }
    return true;
}
static_assert(lowrank_g_area_fits(), "partial sums, low pieces and the word have places of their own");
// Shares of the channels that P = A Q is the sum of, 64-channel stages dealt in turn: none has fewer than one stage's but where the stages
// are no multiple of the shares (96 channels 64 / 32, 160 channels 64 / 64 / 32 and an empty one).
constexpr int lowrank_project_parts(int64_t n_channels) { return n_channels > 128 ? 4 : n_channels > 64 ? 2 : 1; }
constexpr int lowrank_project_tokens(int64_t n_channels) { return 128 / lowrank_project_parts(n_channels); }        // of a workgroup, a block of 32 per wave
// Blocks of 32 tokens that a wave of k_lr_project<bf16> takes in calls whose bf16 tensors have kLowRankProjectMany workgroups' blocks (seven a
// CU) and more, one block after the other against the same pieces of Q, which otherwise take as much of a CU's 64 bytes per clock as the
// operands.  Steps of bf16, one block / three, us: [4096, 3072] 1 tensor 190 / 242, 8 (1024 blocks) 523 / 529, 12 812 / 846, 14 (1792) 842 / 844, 16
// 935 / 907, 24 1402 / 1361, 57 3089 / 2875; 57 x [1024, 3072] (1824) 927 / 906, 114 x [4096, 256] 571 / 567, 60 x [8000, 96] 303 / 311.
// fp32 tensors take one: 28 of them 2778 / 2860.
constexpr int kLowRankProjectBlocks = 3;
constexpr int64_t kLowRankProjectMany = 1792;
// k_lr_apply: a wave owns 32 tokens and one or two tiles of 64 channels, two where widening the factors costs more than the products.  The
// waves are counted through the rows of a tensor and on into the next 32 tokens, whatever workgroup they fall into, so that no width
// leaves waves without tiles; of eight tiles in a row, wave k of four has tiles k and k + 4, so that the four lie side by side.
constexpr int kLowRankApplyChannels = 64;
constexpr int kLowRankApplyTokens = 32;
struct ApplyTiles {
    int first, step, end;       // tiles first, first + step ... below end; no more than the wave's one or two
};
constexpr int lowrank_apply_waves(int n_channels, int tiles_per_wave)       // of 32 tokens
{
    const int tiles = (n_channels + kLowRankApplyChannels - 1) / kLowRankApplyChannels;
    return tiles_per_wave == 1 ? tiles : tiles / 8 * 4 + (tiles % 8 + 1) / 2;
}
constexpr ApplyTiles lowrank_apply_tiles(int n_channels, int tiles_per_wave, int wave)
{
    const int tiles = (n_channels + kLowRankApplyChannels - 1) / kLowRankApplyChannels;
    if (tiles_per_wave == 1) return {wave, 1, wave + 1};
    const int whole = tiles / 8 * 4, half = (tiles % 8 + 1) / 2;
    if (wave < whole) return {wave / 4 * 8 + wave % 4, 4, wave / 4 * 8 + 8};
    return {2 * whole + wave - whole, half, tiles};
}
// min_iters: only tensors whose descriptor asks for at least that many subspace iterations take part
hipError_t launch_lr_orth(const BatchView &v, const LaunchRange &r, bool from_q0, int min_iters, hipStream_t s);
hipError_t launch_lr_project(const BatchView &v, const LaunchRange &r, bool wire, int min_iters, hipStream_t s);
hipError_t launch_lr_backproject(const BatchView &v, const LaunchRange &r, int min_iters, hipStream_t s);
// 4-bit factors: U from P (fp32, in the workspace) onto the wire, after the last projection
hipError_t launch_lr_quant_u(const BatchView &v, const LaunchRange &r, hipStream_t s);
hipError_t launch_lr_encode(const BatchView &v, const LaunchRange &r, int err_dtype, bool fused, hipStream_t s);
hipError_t launch_lr_decode(const BatchView &v, const LaunchRange &r, hipStream_t s);

// Single-pass kernel (channel scales, every error-feedback mode).
int persistent_max_blocks_per_cu(int ef, int err_dtype, bool fused, bool wide, bool slim);
// wide: items of kStripeChannelsWide channels (the layout's choice, fixed at cf_init); one_shot: a workgroup per
// item, else `grid` workgroups that loop over the items
hipError_t launch_single_pass(const BatchView &v, const LaunchRange &r, int ef, int err_dtype, bool fused, bool wide, int grid,
                             bool one_shot, hipStream_t s);
// a range's partials (offset and size multiples of 256 bytes) and item states as cf_init leaves them
hipError_t launch_fresh_partials(uint8_t *partials, size_t bytes, uint8_t *states, uint32_t n_states, hipStream_t s);

}  // namespace cf
