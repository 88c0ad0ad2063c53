// Low-rank compressor (arxiv 2507.17511, Alg. 3 and App. D "Low-Rank Compression") under the
// residual recursion of Sec. 3.1: A = x_t - recon_{t-1} [tokens, channels] is sent as rank-32 factors
// U = A Q [tokens, 32], V = Q [channels, 32] found by T steps of subspace iteration
//     Q <- orth(Q0);  T x { Z <- A^T (A Q);  Q <- orth(Z) };  U <- A Q,
// and both ends add D = U V^T to the reconstruction; e_t = A - D stays at the sender.
//
// This is the one dense contraction of the codec, so it runs on the matrix cores: project and backproject in bf16 pieces of
// fp32 operands (see split2 below), apply on the bf16 factors as they travel or, for other wires, in fp32.  A is never
// materialised: each pass re-forms it from x and recon (4 bytes per element in bf16 storage, the same as reading an fp32 A
// would cost) and is bound by that stream.  Bytes written between the reads of a stream cost far more than they are: P, 1 % of what
// a projection reads, took 12 % of its time, so nothing is written that the next kernel does not need.
//
// Operand layouts: an instruction computes D[m][n] += sum_k A[m][k] B[k][n]; any relabelling of k that both operands
// share, and any relabelling of m or n that the epilogue undoes, is free.
//   project      P = A Q     m = token, k = channel: by way of a wave's LDS patch.
//   backproject  Z = A^T P   m = channel, k = token: a lane loads 8 consecutive channels of 4 tokens and
//                            spends them on 8 channel tiles (tile j holds channels = j mod 8).
//   apply        D = U V^T   m = token, n = channel, k = rank; D comes back row-major by way of a wave's LDS patch.
#include "cf_device.h"
#include "cf_internal.h"

namespace cf {
namespace {

using namespace dev;

typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kRank = 32;
constexpr float kDrop2 = 1e-8f;     // (1e-4)^2: a column left with less than 1e-4 of its length is dropped

__device__ __forceinline__ f32x16 mfma32(float a, float b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }

// Operands a pass reads once.  Streaming hint for bf16 only, whose lanes take their 16 bytes in one load: fp32 lanes take
// 32 bytes in two, and the hint lets go of the line in between.  Steps of [4096, 3072], plain and with the hint, us: 57 of bf16
// 2888 / 2870, 28 of fp32 2756 / 3027.
// `base` uniform over the wave, `off` the lane's byte offset.
__device__ __forceinline__ void load_once(Raw8<BF16> &r, const void *base, uint32_t off) { r.load_stream_at(base, off); }
__device__ __forceinline__ void load_once(Raw8<F32> &r, const void *base, uint32_t off) { r.load_at(base, off); }

template <int DT> __device__ __forceinline__ void load16(const void *base, int64_t elem, float (&out)[16])
{
    Raw8<DT> lo, hi;
    lo.load(base, elem);
    hi.load(base, elem + 8);
    const F8 a = lo.widen(), b = hi.widen();
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        out[k] = a.v[k];
        out[8 + k] = b.v[k];
    }
}

__device__ __forceinline__ uint8_t *wire_u(const TensorPtrs &p) { return p.codes; }
__device__ __forceinline__ uint8_t *wire_v(const TensorDev &d, const TensorPtrs &p)
{
    return p.codes + d.n_tokens * kRank * (d.dtype == BF16 ? 2 : 4);
}

// Factors as 4-bit integers (Sec. 3.4 and App. D name INT4 factors; the format is this library's): every
// factor row of 32 entries has one fp32 scale s = absmax / 7 and travels as 32 nibbles q = clamp(rint(f / s),
// -7, 7), two's complement, entry k in byte k / 2, even k in the low nibble -- the 4-bit group quantiser of
// the activations with the rank index in place of the channel.  On the wire: U nibbles [N, 16 bytes],
// V nibbles [C, 16 bytes], U scales [N] fp32, V scales [C] fp32.
__device__ __forceinline__ bool factors_int4(const TensorDev &d) { return d.nm_block == 4u; }
__device__ __forceinline__ uint8_t *wire4_u(const TensorPtrs &p) { return p.codes; }
__device__ __forceinline__ uint8_t *wire4_v(const TensorDev &d, const TensorPtrs &p) { return p.codes + d.n_tokens * 16; }
__device__ __forceinline__ float *wire4_u_scales(const TensorDev &d, const TensorPtrs &p)
{
    return reinterpret_cast<float *>(p.codes + (d.n_tokens + (int64_t)d.n_channels) * 16);
}
__device__ __forceinline__ float *wire4_v_scales(const TensorDev &d, const TensorPtrs &p) { return wire4_u_scales(d, p) + d.n_tokens; }

// One factor row (32 fp32 values) onto the wire.
__device__ __forceinline__ void quantise_factor_row(const float (&f)[kRank], uint8_t *nibbles16, float *scale)
{
    float amax = 0.0f;
#pragma unroll
    for (int k = 0; k < kRank; ++k) amax = fmaxf(amax, fabsf(f[k]));
    const float s = amax / 7.0f;
    u32x4 w;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        F8 z, sv, dq;
#pragma unroll
        for (int k = 0; k < 8; ++k) { z.v[k] = f[8 * g + k]; sv.v[k] = s; }
        const uint32_t packed = quant8<4>(z, sv, dq);
        if (g == 0) w.x = packed; else if (g == 1) w.y = packed; else if (g == 2) w.z = packed; else w.w = packed;
    }
    *gmut<u32x4>(nibbles16) = w;
    *gmut<float>(scale) = s;
}

// ---------------------------------------------------------------- fp32 operands on the bf16 matrix cores

// An fp32 value is exactly the sum of three bf16 ones: high, its upper 16 bits, mid, those of what that leaves, and low, the
// rest (8 significant bits each).  A product of two values is then nine products of pieces, that of the two low ones below 2^-30 of it
// and left out (of values below 2^-110 the low piece is cut at 2^-133).  The matrix cores form products of bf16 exactly and add 16 or 32 of them up where the fp32 instructions round every 2
// or 4, in 8/16 or 10/16 of their time.
// Errors against fp64, fp32 storage, rms (largest) x 2^-24, fp32 instructions / pieces.  U = A V, C = 64, 512, 3072:
//   random operands, of the sum of the terms' sizes   0.50 (4.2), 0.75 (4.7), 1.40 (12.4) / 0.18 (1.4), 0.11 (0.7), 0.09 (0.6)
//   positive products, of the sum                      1.9 (5.3), 5.9 (15), 14.4 (45) / 0.5 (1.0), 0.6 (1.7), 0.6 (1.5)
//   one product a sum, of the product                  0.43 (0.98), 0.42 (0.98), 0.42 (0.99) / the same (with six of nine 1.02 (5.9), 1.08 (5.0), 1.08 (5.7))
//   one product of size 1, others of 1e-4              2.5 (14), 6.2 (31), 16 (87) / 1.3 (5.4), 1.4 (6.0), 1.7 (7.3)
//   one product of size 1, others of 1e-8              1.3 (9.3), 2.2 (17), 2.6 (20) / 1.0 (5.5), 1.1 (5.3), 1.2 (5.6)
// First column of V, which is that of Z to length one, C = 2048, N = 64, 4096, 20000:
//   random operands, of the entries' rms               2.8 (11), 3.3 (23), 4.1 (40) / 1.5 (8.5), 1.6 (15), 1.8 (21)
//   positive products, of the entry                    0.88 (3.6), 1.2 (5.3), 2.4 (9.0) / 0.77 (2.7), 0.91 (3.4), 1.4 (5.3) (six of nine in the sum's own accumulator 0.92, 1.3, 2.7)
//   one product an entry, of the entry                 0.68 (2.4), 0.61 (1.6), 0.60 (1.5) / 0.69 (2.8), 0.61 (1.6), 0.60 (1.5) (six of nine 1.03 (5.3), 1.12 (4.7), 1.19 (5.3))
//   one product of size 1, others of 1e-3              2.7 (13), 5.5 (20), 11 (45) / 1.5 (7.2), 2.5 (12), 4.1 (13)
// The one kind found where fp32 was closer: [20000, 128], others of 1e-6, P of four products a row, 0.86 (2.7) / 0.95 (3.4).
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ f32x16 mfma32_bf16(u32x4 a, u32x4 b, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

__device__ __forceinline__ f32x4 mfma16_bf16(u32x4 a, u32x4 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

struct Split4 {
    u32x2 high, mid, low;       // 4 values each, in order
};

// The upper halves of two values in one word, the first value's in its lower half.
__device__ __forceinline__ uint32_t upper_halves(float lo, float hi) { return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u); }
__device__ __forceinline__ float upper_half(float f) { return __uint_as_float(__float_as_uint(f) & 0xffff0000u); }

__device__ __forceinline__ void split2(float a, float b, uint32_t &high, uint32_t &mid, uint32_t &low)
{
    high = upper_halves(a, b);
    const float ra = a - upper_half(a), rb = b - upper_half(b);
    mid = upper_halves(ra, rb);
    low = upper_halves(ra - upper_half(ra), rb - upper_half(rb));
}

__device__ __forceinline__ Split4 split4(const float (&v)[4])
{
    uint32_t w[2][3];
#pragma unroll
    for (int k = 0; k < 2; ++k) split2(v[2 * k], v[2 * k + 1], w[k][0], w[k][1], w[k][2]);
    return {{w[0][0], w[1][0]}, {w[0][1], w[1][1]}, {w[0][2], w[1][2]}};
}

__device__ __forceinline__ u32x4 join(u32x2 a, u32x2 b) { return __builtin_shufflevector(a, b, 0, 1, 2, 3); }

__device__ __forceinline__ float element(const Raw8<BF16> &r, int j) { return (j & 1) ? bf16_hi(r.w[j / 2]) : bf16_lo(r.w[j / 2]); }
__device__ __forceinline__ float element(const Raw8<F32> &r, int j) { return j < 4 ? r.a[j] : r.b[j - 4]; }

struct Split8 {
    u32x4 high, mid, low;       // 8 values each, in order
};

__device__ __forceinline__ Split8 split8(const float (&v)[8])
{
    uint32_t w[4][3];
#pragma unroll
    for (int k = 0; k < 4; ++k) split2(v[2 * k], v[2 * k + 1], w[k][0], w[k][1], w[k][2]);
    return {{w[0][0], w[1][0], w[2][0], w[3][0]}, {w[0][1], w[1][1], w[2][1], w[3][1]}, {w[0][2], w[1][2], w[2][2], w[3][2]}};
}

// Q as k_lr_project reads it: per 32 channels and piece 2 KB, the 8 channels of octet o and rank column n at (32 o + n) * 16
// bytes, so that a lane of either bf16 instruction takes its 8 channels of one column in one load and a wave whole lines.  High and
// mid take the place of Z (the same 4 KB per 32 channels), low lies in the Gram matrices' area behind their partial sums.
__device__ __forceinline__ uint8_t *lr_q(const BatchView &v, const TensorDev &d, int step, int piece)
{
    if (piece < 2) return v.workspace + d.lr_z_off + (int64_t)step * 4096 + piece * 2048;
    return v.workspace + d.lr_g_off + lowrank_q_low_off(d.n_channels) + (int64_t)step * 2048;
}

// ---------------------------------------------------------------- P = A Q  (and U on the wire)

// The MFMA wants a lane to hold one token's channels, memory wants neighbouring lanes on neighbouring channels: a wave
// reads [32 tokens][64 channels] of x and recon row-major (8 lanes = 128 bytes of a bf16 row), leaves the residual in its
// own LDS patch and picks it up again with lane (m, h) on token m, channels 8 h ... of each 16-channel step.
//
// The channels are cut into lowrank_project_parts = 4, 2 or 1 shares, 64-channel stages dealt in turn, and P is the sum of the
// shares' chains.  A wave takes a share of TB blocks of 32 tokens, one block after the other within a stage, and the waves of
// the same tokens add up in LDS; the bits do not depend on TB.
// What rounds in a stage of 64 channels: the products of the leading pieces, exact each, in one accumulator that starts from
// zero, the small ones in another; then one addition of the two and one to the wave's sum, as the vector units round it.
// The matrix cores cut off what lies below the last bits of the largest product of eight and round once per instruction, so small
// products in the sum's own accumulator would cost it a rounding each (sums of 3072 positive products: 6.1e-6).
constexpr int kProjThreads = 256;
constexpr int kProjChannels = 64;
constexpr int kProjPitch = kProjChannels + 4;               // floats per token row of the patch
constexpr int kProjSumPitch = kRank + 4;
// The kernel at 57 x [4096, 3072] bf16 (six products of pieces): one block of tokens a wave 636 us, two 566, three 535, four 605 (11 registers
// spilled); fp32 MFMA 587.  408 of that is the stream alone, 50 or 25 the stores of P or U.  With eight products 543.
constexpr int kProjBlocks = kLowRankProjectBlocks;
typedef float ProjPatches[kProjThreads / 64][32 * kProjPitch];

// What a wave reads of a stage: 8 tokens x 128 bytes an instruction.  Loads without branches: tokens and channels outside the
// tensor read its last ones; those tokens are not stored and those channels not used.
template <int DT> struct ProjStage {
    Raw8<DT> x[4], b[4];
    __device__ __forceinline__ void fetch(const TensorDev &d, const TensorPtrs &p, int64_t row_base, int stage)
    {
        constexpr uint32_t kBytes = DT == BF16 ? 2 : 4;
        const int lane = (int)threadIdx.x & 63;
        const int ch = stage * kProjChannels + (lane & 7) * 8;
        const int64_t last = d.n_tokens - 1, base = row_base < last ? row_base : last;
        const int room = last - base < 31 ? (int)(last - base) : 31;        // tokens after the first that exist
        const char *px = static_cast<const char *>(p.x) + base * d.n_channels * kBytes;
        const char *pb = static_cast<const char *>(p.recon) + base * d.n_channels * kBytes;
        const uint32_t at = (uint32_t)(ch < d.n_channels ? ch : d.n_channels - 8) * kBytes;
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int tok = (lane >> 3) + 8 * it;
            const uint32_t off = (uint32_t)(tok < room ? tok : room) * ((uint32_t)d.n_channels * kBytes) + at;
            load_once(x[it], px, off);
            load_once(b[it], pb, off);
        }
    }
    __device__ __forceinline__ void leave(float *patch) const
    {
        const int lane = (int)threadIdx.x & 63;
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const F8 xv = x[it].widen(), bv = b[it].widen();
            f32x4 lo, hi;
            lo.x = xv.v[0] - bv.v[0]; lo.y = xv.v[1] - bv.v[1]; lo.z = xv.v[2] - bv.v[2]; lo.w = xv.v[3] - bv.v[3];
            hi.x = xv.v[4] - bv.v[4]; hi.y = xv.v[5] - bv.v[5]; hi.z = xv.v[6] - bv.v[6]; hi.w = xv.v[7] - bv.v[7];
            f32x4 *dst = reinterpret_cast<f32x4 *>(patch + ((lane >> 3) + 8 * it) * kProjPitch + (lane & 7) * 8);
            dst[0] = lo;
            dst[1] = hi;
        }
    }
};

// lead + small += (16 channels of the wave's 32 tokens) * Q, u: which 16 of the patch's 64; q: the lane's pieces of Q
__device__ __forceinline__ void project16(const float *patch, int u, const u32x4 (&q)[3], f32x16 &lead, f32x16 &small)
{
    const int lane = (int)threadIdx.x & 63;
    const f32x4 *src = reinterpret_cast<const f32x4 *>(patch + (lane & 31) * kProjPitch + 16 * u + 8 * (lane >> 5));
    const f32x4 w0 = src[0], w1 = src[1];
    const float z[8] = {w0.x, w0.y, w0.z, w0.w, w1.x, w1.y, w1.z, w1.w};
    const Split8 a = split8(z);
    lead = mfma32_bf16(a.high, q[0], lead);
    small = mfma32_bf16(a.low, q[1], small);
    small = mfma32_bf16(a.mid, q[2], small);
    small = mfma32_bf16(a.low, q[0], small);
    small = mfma32_bf16(a.high, q[2], small);
    small = mfma32_bf16(a.mid, q[1], small);
    small = mfma32_bf16(a.mid, q[0], small);
    small = mfma32_bf16(a.high, q[1], small);
}

// acc += the products of a stage's first U * 16 channels
template <int U> __device__ __forceinline__ void project_stage(const float *patch, const u32x4 (&q)[4][3], f32x16 &acc)
{
    f32x16 lead = {}, small = {};
#pragma unroll
    for (int u = 0; u < U; ++u) project16(patch, u, q[u], lead, small);
    acc += lead + small;
}

// 4 columns of a finished row.  Written bytes cost a stream of reads dearly, 1.7 us per MB: the last projection leaves U
// only, but for 4-bit factors, which k_lr_quant_u makes of P.
template <int DT> __device__ __forceinline__ void project_store(const BatchView &v, const TensorDev &d, const TensorPtrs &p, bool wire,
                                                                int64_t row, int col, f32x4 sum)
{
    if (row >= d.n_tokens) return;
    if (!wire || factors_int4(d)) {
        __builtin_nontemporal_store(sum, gmut<f32x4>(v.workspace + d.lr_p_off) + row * (kRank / 4) + col / 4);
    } else if (DT == BF16) {
        u32x2 w;
        w.x = bf16_rne(sum.x) | (bf16_rne(sum.y) << 16);
        w.y = bf16_rne(sum.z) | (bf16_rne(sum.w) << 16);
        *gmut<u32x2>(wire_u(p) + (row * kRank + col) * 2) = w;
    } else {
        *gmut<f32x4>(wire_u(p) + (row * kRank + col) * 4) = sum;
    }
}

// Accumulator register i of lane (m, h): row 8 * (i / 4) + 4 * h + i % 4 of the tile, column m.
__device__ __forceinline__ void project_leave_sum(float *patch, const f32x16 &acc)
{
    const int lane = (int)threadIdx.x & 63, m = lane & 31, h = lane >> 5;
#pragma unroll
    for (int i = 0; i < 16; ++i) patch[(8 * (i >> 2) + 4 * h + (i & 3)) * kProjSumPitch + m] = acc[i];
}

template <int DT, int TB>
__device__ __forceinline__ void lr_project_body(const BatchView &v, const TensorDev &d, const TensorPtrs &p, bool wire, ProjPatches &patches)
{
    const int lane = (int)threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int m = lane & 31, h = lane >> 5;
    const int parts = lowrank_project_parts(d.n_channels), part = wave & (parts - 1);
    const int64_t wg_row = (int64_t)blockIdx.x * (32 * TB * (4 / parts)), row_base = wg_row + 32 * TB * (wave / parts);
    const int steps = d.n_channels / 32, stages = (steps + 1) / 2;
    float *patch = patches[wave];
    f32x16 acc[TB];
#pragma unroll
    for (int b = 0; b < TB; ++b) acc[b] = (f32x16)(0.0f);
    ProjStage<DT> raw;
    if (row_base < d.n_tokens && part < stages) {           // uniform over the wave
        raw.fetch(d, p, row_base, part);
        for (int stage = part; stage < stages; stage += parts) {
            u32x4 q[4][3];
#pragma unroll
            for (int b = 0; b < TB; ++b) {
                raw.leave(patch);
                // Q first, then the prefetch: loads return in issue order, so the MFMAs below wait for Q only
                if (b == 0) {
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int step = 2 * stage + (u >> 1) < steps ? 2 * stage + (u >> 1) : steps - 1;
#pragma unroll
                        for (int k = 0; k < 3; ++k) q[u][k] = gconst<u32x4>(lr_q(v, d, step, k))[(2 * (u & 1) + h) * 32 + m];
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
                if (b + 1 < TB) raw.fetch(d, p, row_base + 32 * (b + 1), stage);
                else if (stage + parts < stages) raw.fetch(d, p, row_base, stage + parts);
                __builtin_amdgcn_sched_barrier(0);
                wave_lds_fence();
                if (2 * stage + 1 < steps) project_stage<4>(patch, q, acc[b]);         // uniform over the wave
                else project_stage<2>(patch, q, acc[b]);
                __builtin_amdgcn_sched_barrier(0);
                wave_lds_fence();
            }
        }
    }
    const int row = (int)threadIdx.x >> 3, col = 4 * ((int)threadIdx.x & 7);
#pragma unroll
    for (int b = 0; b < TB; ++b) {
        project_leave_sum(patch, acc[b]);
        __syncthreads();
        for (int g = 0; g < 4 / parts; ++g) {               // uniform: the workgroup's sets of waves that share tokens
            auto of = [&](int k) { return *reinterpret_cast<const f32x4 *>(patches[g * parts + k] + row * kProjSumPitch + col); };
            f32x4 sum = of(0);
            if (parts > 1) sum += of(1);
            if (parts > 2) sum += of(2) + of(3);
            project_store<DT>(v, d, p, wire, wg_row + 32 * (TB * g + b) + row, col, sum);
        }
        if (b + 1 < TB) __syncthreads();
    }
}

// min_iters: tensors that asked for fewer subspace iterations than this sit the launch out.
// A kernel per storage type: fp32 operands take twice the registers, and bf16 tensors would pay for them in occupancy.
template <int DT, int TB>
__global__ __launch_bounds__(kProjThreads, TB == 1 && DT == BF16 ? 3 : 2) void k_lr_project(BatchView v, LaunchRange r, int wire, int min_iters)
{
    __shared__ __attribute__((aligned(16))) ProjPatches patches;
    const int t = r.first + (int)blockIdx.y;
    const TensorDev d = v.descs[t];
    if (d.scale != LOWRANK || d.dtype != DT || d.bits < min_iters) return;
    if ((int64_t)blockIdx.x * (TB * lowrank_project_tokens(d.n_channels)) >= d.n_tokens) return;        // uniform over the workgroup
    const TensorPtrs p = v.ptrs[t];
    lr_project_body<DT, TB>(v, d, p, wire != 0, patches);
}

// ---------------------------------------------------------------- Z = A^T P

// Workgroups that share the runs of one stripe of a tensor.
__device__ __forceinline__ int lr_shares(const LaunchRange &r, const TensorDev &d)
{
    const int runs = lowrank_runs(d.n_tokens, d.n_channels);
    return r.lr_split < runs ? r.lr_split : runs;
}

// Where share `share` of a tensor leaves its part of Z: the first in Z itself.
__device__ __forceinline__ uint8_t *lr_slice(const BatchView &v, const LaunchRange &r, const TensorDev &d, int share)
{
    if (share == 0) return v.workspace + d.lr_z_off;
    return v.workspace + r.lr_slices_off + ((uint64_t)(d.lr_slot - r.lr_first_slot) * (uint64_t)(r.lr_split - 1) + (uint64_t)(share - 1)) * (uint64_t)r.lr_max_channels * (kRank * sizeof(float));
}

// The tokens are cut into lowrank_runs = 1, 2 or 4 runs.  Z is the sum (run 0 + run 1) + (run 2 + run 3), each run the
// sum over the waves that share its batches of 16 tokens, so the bits depend on the tensor's shape alone, whoever adds: a workgroup
// owns a stripe of 256 channels and either takes all runs one after the other, or, in calls of few tensors, one or two
// of them, and the orthogonalisation adds the shares.
// v_mfma_f32_16x16x32_bf16 takes 8 entries of row l % 16 of A and of column l % 16 of B from lane l, for k = 8 (l / 16) ...:
// lane (q, g) holds channels 8q..8q+7 of its wave's 128 of 4 tokens, straight from 128-bit loads, and makes of channel j of these
// tokens the row of channel tile j (tile j holds channels = j mod 8): two pieces of 4 values each, against two pieces of 4 rows
// of P, or one piece and zeros: (mid, low) (low, mid) + (mid, low) (0, high) + (high, mid) (low, mid) + (high, mid) (mid, high) are the
// small products, (high, mid) (high, 0) the leading one.  Per batch of 16 tokens each of the two starts from zero, and the vector units
// add them up and to the sum, as in project.  Not with the form of half the length for the lone pieces: an accumulator that went
// from v_mfma_f32_16x16x16_bf16 to v_mfma_f32_16x16x32_bf16 within two instructions came back wrong.
// What bounds it, 57 x [4096, 3072] bf16, in a trace about 600 us on average (550-700): the stream of x and recon, alone 550 in 128-channel
// stripes and 400-430 in wider ones.  A wave has one batch in registers; the next is asked for once the residual is formed, so that it is
// in flight while the products are: one tensor 79 -> 56 us, 28 of fp32 570 -> 536, the 57 681 -> 608 (asked for after the products).
constexpr int kBackThreads = 256;
constexpr int kBackChannels = kLowRankBackChannels;
constexpr int kBackEntries = kBackChannels * kRank;
constexpr int kBackWaveChannels = kBackChannels / 2;

template <int DT>
__device__ __forceinline__ void lr_backproject_body(const BatchView &v, const LaunchRange &r, const TensorDev &d, const TensorPtrs &p,
                                                    int stripe, int share, float *sums, float *total)
{
    const int lane = (int)threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int q = lane & 15, g = lane >> 4;
    const int64_t last = d.n_tokens - 1, n_quads = (d.n_tokens + 3) / 4;
    const int n_runs = lowrank_runs(d.n_tokens, d.n_channels), n_mine = n_runs / lr_shares(r, d), first_run = share * n_mine;
    const int64_t per_run = (n_quads + n_runs - 1) / n_runs;
    // Loads without branches: rows and channels outside the tensor read its last ones, P counts as zero there and the
    // channels are not stored.
    constexpr uint32_t kBytes = DT == BF16 ? 2 : 4;
    const uint32_t row_bytes = (uint32_t)d.n_channels * kBytes;
    // two waves side by side and every second batch each, or, where a stripe is no wider than one, every fourth
    const int turns = d.n_channels - stripe * kBackChannels > kBackWaveChannels ? 2 : 4;
    const int half = turns == 2 ? wave & 1 : 0, turn = turns == 2 ? wave >> 1 : wave;
    const int ch0 = stripe * kBackChannels + half * kBackWaveChannels + 8 * q;
    const uint32_t ch = (uint32_t)(ch0 < d.n_channels ? ch0 : d.n_channels - 8) * kBytes;
    struct Batch {                                          // 16 tokens: a lane has rows 4 g .. 4 g + 3
        Raw8<DT> x[4], b[4];
        float p[2][4];
    } batch;
    auto fetch = [&](Batch &w, int64_t quad0) {
        const int64_t row0 = 4 * quad0 < last ? 4 * quad0 : last;
        const int room = last - row0 < 15 ? (int)(last - row0) : 15;        // rows after the first that exist
        const char *px = static_cast<const char *>(p.x) + row0 * row_bytes, *pb = static_cast<const char *>(p.recon) + row0 * row_bytes;
        const char *P = reinterpret_cast<const char *>(v.workspace + d.lr_p_off) + row0 * (kRank * 4);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const uint32_t row = (uint32_t)(4 * g + t < room ? 4 * g + t : room);
            load_once(w.x[t], px, row * row_bytes + ch);
            load_once(w.b[t], pb, row * row_bytes + ch);
            w.p[0][t] = *gconst<float>(P + (row * (kRank * 4) + 4 * q));
            w.p[1][t] = *gconst<float>(P + (row * (kRank * 4) + 64 + 4 * q));
        }
    };
    CF_GLOBAL float *Z = gmut<float>(lr_slice(v, r, d, share)) + (int64_t)stripe * kBackEntries;
    const int n_out = (d.n_channels - stripe * kBackChannels) * kRank;      // entries of the stripe that exist
    for (int run = first_run; run < first_run + n_mine; ++run) {            // uniform over the workgroup
        const int64_t lo = run * per_run + 4 * turn;        // may lie beyond the last quad: such a wave adds zeros
        const int64_t hi = (run + 1) * per_run < n_quads ? (run + 1) * per_run : n_quads;
        f32x4 acc[8][2];
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j][0] = acc[j][1] = (f32x4)(0.0f);
        if (lo < hi) {
            if (run == first_run) fetch(batch, lo);
            for (int64_t quad0 = lo; quad0 < hi; quad0 += 4 * turns) {
                Batch &w = batch;
                const int64_t quad = quad0 + g;
                u32x4 pp[2][4];                             // (low, mid), (0, high), (mid, high), (high, 0)
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    float pv[4];
#pragma unroll
                    for (int t = 0; t < 4; ++t) pv[t] = quad < hi && 4 * quad + t <= last ? w.p[c][t] : 0.0f;
                    const Split4 s = split4(pv);
                    pp[c][0] = join(s.low, s.mid);
                    pp[c][1] = join((u32x2)(0u), s.high);
                    pp[c][2] = join(s.mid, s.high);
                    pp[c][3] = join(s.high, (u32x2)(0u));
                }
                float z[8][4];
#pragma unroll
                for (int j = 0; j < 8; ++j)
#pragma unroll
                    for (int t = 0; t < 4; ++t) z[j][t] = element(w.x[t], j) - element(w.b[t], j);
                __builtin_amdgcn_sched_barrier(0);
                // the next batch, or the first of the next run: in flight while this one's products are formed and the waves' sums meet
                fetch(w, quad0 + 4 * turns < hi ? quad0 + 4 * turns : (run + 1) * per_run + 4 * turn);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const Split4 s = split4(z[j]);
                    const u32x4 a0 = join(s.high, s.mid), a1 = join(s.mid, s.low);
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        f32x4 small = mfma16_bf16(a1, pp[c][0], (f32x4)(0.0f));
                        small = mfma16_bf16(a1, pp[c][1], small);
                        small = mfma16_bf16(a0, pp[c][0], small);
                        small = mfma16_bf16(a0, pp[c][2], small);
                        acc[j][c] += mfma16_bf16(a0, pp[c][3], (f32x4)(0.0f)) + small;
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        // tile j, register i of lane (q, g): channel 8 * (4 * g + i) + j of the stripe, column q (and 16 + q)
        for (int w = 0; w < turns; ++w) {
            if (turn == w) {
                float *mine = sums + half * (kBackWaveChannels * kRank);
#pragma unroll
                for (int j = 0; j < 8; ++j)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            const int idx = (8 * (4 * g + i) + j) * kRank + 16 * h + q;
                            mine[idx] = (w == 0) ? acc[j][h][i] : mine[idx] + acc[j][h][i];
                        }
            }
            __syncthreads();
        }
        // a lane keeps to its own entries of `total` and of Z
        const bool opens = run == first_run || (run & 1) == 0, closes = run + 1 == first_run + n_mine || (run & 1) == 1;
        for (int k = (int)threadIdx.x; k < kBackEntries; k += kBackThreads) {
            float pair = sums[k];
            if (!opens) pair = total[k] + pair;
            if (!closes) total[k] = pair;
            else if (k < n_out) Z[k] = run < first_run + 2 ? pair : Z[k] + pair;
        }
        __syncthreads();                                    // before the next run's first waves write their sums
    }
}

template <int DT>
__global__ __launch_bounds__(kBackThreads, 2) void k_lr_backproject(BatchView v, LaunchRange r, int min_iters)
{
    __shared__ float sums[kBackEntries], total[kBackEntries];
    const int t = r.first + (int)blockIdx.y;
    const TensorDev d = v.descs[t];
    if (d.scale != LOWRANK || d.dtype != DT || d.bits < min_iters) return;
    const int n_stripes = (d.n_channels + kBackChannels - 1) / kBackChannels;
    const int stripe = (int)blockIdx.x % n_stripes, share = (int)blockIdx.x / n_stripes;
    if (share >= lr_shares(r, d)) return;                   // uniform over the workgroup: narrower or shorter than the largest tensor
    const TensorPtrs p = v.ptrs[t];
    lr_backproject_body<DT>(v, r, d, p, stripe, share, sums, total);
}

// ---------------------------------------------------------------- Q = orth(Z)

// Gram-Schmidt over the 32 columns, left to right; a column left with less than 1e-4 of its length is dropped
// (zero): a residual of rank < 32 then gives zero columns rather than amplified rounding noise.
//
// Done on the Gram matrix: with G = Z^T Z and R its (upper) Cholesky factor, Q = Z R^-1 is what Gram-Schmidt
// gives, and the squared length a column is left with is the pivot of its elimination step.  G, R and the
// substitution are fp64: the products of two fp32 entries are exact.  What bounds it: nothing but latency.
// Projecting column by column is 96 rounds of workgroup-wide sums, one after the other, on one workgroup per tensor
// (279 us for 57 x [3072, 32] on 57 of 256 CUs); here every workgroup takes 256 channel rows, k_lr_gram sums their
// products on the fp64 matrix cores, and every workgroup of k_lr_orth adds those partial sums up and eliminates the
// 32 x 32 matrix for itself, most of it the 31 dependent steps of the elimination.
//
// The 1e-4 rule does not bound the conditioning of Z: columns that each lean on the one before compound, and what is
// left of a column is then rounding noise of G.  What is left of column i is sum_j u_ij z_j with u_ii = 1 and the
// row of L^-1 (R^T = L D^1/2) before it, so an error of eta |z_j| |z_k| in the entries of G moves its pivot by eta
// sum_j (|u_ij| |z_j|)^2.  The elimination carries u along in the unused triangle, and a tensor is left to k_lr_orth_twice,
// the column by column form, unless every term of a kept column's sum is at most kLeanMost pivots and a dropped column
// stays under the 1e-4 line with kLeanNoise times its terms added.  eta comes out at 4e-16 to 1.5e-15 over cosines, bumps,
// powers, chains and steep spectra as columns, and a sum at 9 times its largest term at most: inner products of kept
// columns stay below 9 * kLeanMost * 1.5e-15 = 4.5e-7 (1.0e-7 is the worst seen), what projecting twice in fp32 reaches.
// Drifts as they are met have terms up to 1e4 pivots and stay at the rounding of V.  NaN and infinities fail the
// comparisons too.
constexpr double kLeanMost = 33554432.0;                    // 2^25
constexpr double kLeanNoise = 32.0 * 3.6e-15;               // 32 terms, 2^-48 each
constexpr int kOrthThreads = 256;                           // one channel row per lane
constexpr int kGramEntries = kRank * kRank;                 // of which the upper triangle is used

// Whether k_lr_orth left the tensor to k_lr_orth_twice: the last word of the Gram matrices' area, of whose 128 C bytes the partial
// sums and Q's low pieces fill at most 96 C + 8192 (64 C where C <= 256 and there are no partial sums).
__device__ __forceinline__ CF_GLOBAL uint32_t *lr_left_over(const BatchView &v, const TensorDev &d)
{
    return gmut<uint32_t>(v.workspace + d.lr_g_off) + (int64_t)d.n_channels * kRank - 1;
}

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

// Sums of products of the 256 channel rows from `first` on: the three 16 x 16 tiles on or above the diagonal, one
// partial per wave (to be added up in wave order).  v_mfma_f64_16x16x4_f64 takes column l % 16 of row l / 16 from
// lane l on both sides, so a lane's two loads of a step (columns c and 16 + c) feed all three.  Register i of lane l
// holds row 4 * i + l / 16, column l % 16 of a tile.
typedef double GramParts[kOrthThreads / 64][3][256];
// The rows are Q0's, or Z's; where several workgroups shared Z the sum of the shares is formed here and left in Z.
__device__ __forceinline__ void gram_block(const BatchView &v, const LaunchRange &r, const TensorDev &d, int t, bool from_q0, int first, GramParts &part)
{
    const int n_channels = d.n_channels;
    const int n_shares = from_q0 ? 1 : lr_shares(r, d);
    const CF_GLOBAL float *src = from_q0 ? gconst<float>(v.ptrs[t].scales) : gconst<float>(v.workspace + d.lr_z_off);
    const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
    const int col = lane & 15;
    const int row0 = first + wave * 64 + (lane >> 4);
    float lo[16], hi[16];
#pragma unroll
    for (int s = 0; s < 16; ++s) {
        const int row = row0 + 4 * s;
        const bool valid = row < n_channels;
        lo[s] = valid ? src[(int64_t)row * kRank + col] : 0.0f;
        hi[s] = valid ? src[(int64_t)row * kRank + 16 + col] : 0.0f;
    }
    if (n_shares > 1) {         // uniform over the workgroup; 2 or 4
        const CF_GLOBAL float *s1 = gconst<float>(lr_slice(v, r, d, 1));
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            const int row = row0 + 4 * s;
            const bool valid = row < n_channels;
            lo[s] += valid ? s1[(int64_t)row * kRank + col] : 0.0f;
            hi[s] += valid ? s1[(int64_t)row * kRank + 16 + col] : 0.0f;
        }
        if (n_shares > 2) {
            const CF_GLOBAL float *s2 = gconst<float>(lr_slice(v, r, d, 2)), *s3 = gconst<float>(lr_slice(v, r, d, 3));
#pragma unroll
            for (int s = 0; s < 16; ++s) {
                const int row = row0 + 4 * s;
                const bool valid = row < n_channels;
                lo[s] += valid ? s2[(int64_t)row * kRank + col] + s3[(int64_t)row * kRank + col] : 0.0f;
                hi[s] += valid ? s2[(int64_t)row * kRank + 16 + col] + s3[(int64_t)row * kRank + 16 + col] : 0.0f;
            }
        }
        CF_GLOBAL float *Z = gmut<float>(v.workspace + d.lr_z_off);
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            const int row = row0 + 4 * s;
            if (row < n_channels) {
                Z[(int64_t)row * kRank + col] = lo[s];
                Z[(int64_t)row * kRank + 16 + col] = hi[s];
            }
        }
    }
    f64x4 g00 = {}, g01 = {}, g11 = {};
#pragma unroll
    for (int s = 0; s < 16; ++s) {
        const double a = (double)lo[s], b = (double)hi[s];
        g00 = __builtin_amdgcn_mfma_f64_16x16x4f64(a, a, g00, 0, 0, 0);
        g01 = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, g01, 0, 0, 0);
        g11 = __builtin_amdgcn_mfma_f64_16x16x4f64(b, b, g11, 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int e = (4 * i + (lane >> 4)) * 16 + col;
        part[wave][0][e] = g00[i];
        part[wave][1][e] = g01[i];
        part[wave][2][e] = g11[i];
    }
    __syncthreads();
}

__device__ __forceinline__ double gram_sum(const GramParts &part, int tile, int e)
{
    return (part[0][tile][e] + part[1][tile][e]) + (part[2][tile][e] + part[3][tile][e]);
}

// Partial G of 256 channel rows, for tensors of more than 256 channels.
__global__ __launch_bounds__(kOrthThreads) void k_lr_gram(BatchView v, LaunchRange r, int from_q0, int min_iters)
{
    __shared__ GramParts part;
    const int t = r.first + (int)blockIdx.y;
    const TensorDev d = v.descs[t];
    if (d.scale != LOWRANK || d.bits < min_iters) return;
    if (d.n_channels <= kOrthThreads || (int)blockIdx.x * kOrthThreads >= d.n_channels) return;     // uniform over the workgroup
    gram_block(v, r, d, t, from_q0 != 0, (int)blockIdx.x * kOrthThreads, part);
    CF_GLOBAL double *out = gmut<double>(v.workspace + d.lr_g_off) + (int64_t)blockIdx.x * kGramEntries;
    const int row = (int)threadIdx.x >> 4, c = (int)threadIdx.x & 15;
#pragma unroll
    for (int tile = 0; tile < 3; ++tile)
        out[(row + (tile == 2 ? 16 : 0)) * kRank + c + (tile >= 1 ? 16 : 0)] = gram_sum(part, tile, (int)threadIdx.x);
}

// 1 / p by two Newton steps on the hardware's estimate: the elimination's steps depend on each other, and a full
// divide is most of a step.  p is a squared length, far from the ends of the fp64 range.
__device__ __forceinline__ double reciprocal(double p)
{
    double x = __builtin_amdgcn_rcp(p);
    x = __builtin_fma(__builtin_fma(-p, x, 1.0), x, x);
    return __builtin_fma(__builtin_fma(-p, x, 1.0), x, x);
}

// Q rows of 256 channels, in the order k_lr_project reads them, and V = Q on the wire.  Q goes where Z was (a
// workgroup has its rows in registers before it writes them, and both orders keep 32 channels in the same 4 KB).
__global__ __launch_bounds__(kOrthThreads) void k_lr_orth(BatchView v, LaunchRange r, int from_q0, int min_iters)
{
    constexpr int kPitch = kRank + 2;                       // doubles; even, so that pairs of a row stay 16-byte aligned
    __shared__ __attribute__((aligned(16))) double G[kRank][kPitch];
    __shared__ double start2[kRank], inv_len[kRank];
    __shared__ GramParts parts;
    const int t = r.first + (int)blockIdx.y;
    const TensorDev d = v.descs[t];
    if (d.scale != LOWRANK || d.bits < min_iters) return;
    if ((int)blockIdx.x * kOrthThreads >= d.n_channels) return;     // uniform over the workgroup
    const TensorPtrs p = v.ptrs[t];
    const int tid = (int)threadIdx.x;
    const int ch = (int)blockIdx.x * kOrthThreads + tid;
    const bool valid = ch < d.n_channels;
    const CF_GLOBAL f32x4 *src = (from_q0 ? gconst<f32x4>(p.scales) : gconst<f32x4>(v.workspace + d.lr_z_off)) + (int64_t)ch * (kRank / 4);
    f32x4 raw[kRank / 4];

    // G: this lane's entries are rows row0 + 8 * q of column col, on or above the diagonal
    const int n_blocks = (d.n_channels + kOrthThreads - 1) / kOrthThreads;
    const int col = tid & (kRank - 1), row0 = tid / kRank;
    double g[4] = {0.0, 0.0, 0.0, 0.0};
    if (n_blocks == 1) {        // uniform: the rows of this workgroup are all there are
        gram_block(v, r, d, t, from_q0 != 0, 0, parts);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int row = row0 + 8 * q;
            if (row <= col) g[q] = gram_sum(parts, (row >> 4) + (col >> 4), (row & 15) * 16 + (col & 15));
        }
    } else {                    // the partial sums of k_lr_gram, in channel order
        const CF_GLOBAL double *part = gconst<double>(v.workspace + d.lr_g_off);
        constexpr int kAtOnce = 6;                          // blocks whose partial sums are in flight together
        for (int b0 = 0; b0 < n_blocks; b0 += kAtOnce) {
            double w[kAtOnce][4];
#pragma unroll
            for (int u = 0; u < kAtOnce; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    w[u][q] = (b0 + u < n_blocks && row0 + 8 * q <= col) ? part[(int64_t)(b0 + u) * kGramEntries + tid + 256 * q] : 0.0;
#pragma unroll
            for (int u = 0; u < kAtOnce; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q) g[q] += w[u][q];
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        G[row0 + 8 * q][col] = g[q];
        if (row0 + 8 * q == col) start2[col] = g[q];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kRank / 4; ++k) raw[k] = valid ? src[k] : (f32x4)(0.0f);    // after gram_block, which may only now have formed Z
    // elimination: after step k the rows below it hold what is left of G on and above the diagonal, and below it the
    // coefficients of L^-1; a dropped column eliminates nothing
    for (int k = 0; k + 1 < kRank; ++k) {
        const double pivot = G[k][k], start = start2[k];
        const bool keep = start > 0.0 && pivot > (double)kDrop2 * start;
        const double f = keep ? (col == k ? 1.0 : G[k][col]) * reciprocal(pivot) : 0.0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = row0 + 8 * q;
            if (i > k && (i <= col || col <= k)) {
                g[q] = __builtin_fma(-G[k][i], f, g[q]);
                G[i][col] = g[q];
            }
        }
        __syncthreads();
    }
    if (tid < kRank) {
        const double pivot = G[tid][tid], start = start2[tid];
        inv_len[tid] = start > 0.0 && pivot > (double)kDrop2 * start ? 1.0 / __builtin_sqrt(pivot) : 0.0;
    }
    __syncthreads();
    bool clear = true;          // of this lane's entries below the diagonal; the comparisons fail on NaN
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int i = row0 + 8 * q;
        const double term = g[q] * g[q] * start2[col], inv = inv_len[i];
        if (col < i) clear = clear && (inv > 0.0 ? term * inv * inv <= kLeanMost : G[i][i] + kLeanNoise * term <= (double)kDrop2 * start2[i]);
        if (col == i) clear = clear && start2[i] <= 1.7e308;
    }
    const bool left_over = __syncthreads_or(!clear) != 0;   // the same in every workgroup of the tensor: same sums, same steps
    if (blockIdx.x == 0 && tid == 0) *lr_left_over(v, d) = left_over ? 1u : 0u;
    if (left_over) return;                                  // Z stays as it is
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if (row0 + 8 * q < col) G[row0 + 8 * q][col] = g[q] * inv_len[row0 + 8 * q];        // R above the diagonal
#pragma unroll
    for (int k = 0; k < kRank / 4; ++k) asm volatile("" : "+v"(raw[k]));       // the row has arrived before any lane writes Q over it
    __syncthreads();

    // this lane's row: q_j = (z_j - sum_{i < j} q_i R_ij) / R_jj
    double z[kRank];
#pragma unroll
    for (int k = 0; k < kRank / 4; ++k) {
        z[4 * k] = (double)raw[k].x; z[4 * k + 1] = (double)raw[k].y; z[4 * k + 2] = (double)raw[k].z; z[4 * k + 3] = (double)raw[k].w;
    }
    float a[kRank];
#pragma unroll
    for (int i = 0; i < kRank; ++i) {
        const double q = z[i] * inv_len[i];
        a[i] = (float)q;
        if ((i & 1) == 0) z[i + 1] = __builtin_fma(-q, G[i][i + 1], z[i + 1]);
#pragma unroll
        for (int j = (i / 2 + 1) * 2; j < kRank; j += 2) {
            const f64x2 rr = *reinterpret_cast<const f64x2 *>(&G[i][j]);
            z[j] = __builtin_fma(-q, rr.x, z[j]);
            z[j + 1] = __builtin_fma(-q, rr.y, z[j + 1]);
        }
    }
    // Q in the order and the pieces k_lr_project reads: the wave's rows turn in its part of LDS, 32 channels at a time
    float *turn = reinterpret_cast<float *>(parts[tid >> 6]);
    constexpr int kTurnPitch = kRank + 1;
    static_assert(32 * kTurnPitch * sizeof(float) <= sizeof(parts[0]), "32 rows fit a wave's part");
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        const int step = (ch - (tid & 63)) / 32 + half;
        if (32 * step >= d.n_channels) break;               // uniform over the wave
        wave_lds_fence();
        if (((tid >> 5) & 1) == half)
#pragma unroll
            for (int n = 0; n < kRank; ++n) turn[(tid & 31) * kTurnPitch + n] = a[n];
        wave_lds_fence();
        const int octet = (tid & 63) >> 4;
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) {
            const int n = 16 * rt + (tid & 15);
            float f[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) f[i] = turn[(8 * octet + i) * kTurnPitch + n];
            const Split8 q = split8(f);
            gmut<u32x4>(lr_q(v, d, step, 0))[octet * 32 + n] = q.high;
            gmut<u32x4>(lr_q(v, d, step, 1))[octet * 32 + n] = q.mid;
            gmut<u32x4>(lr_q(v, d, step, 2))[octet * 32 + n] = q.low;
        }
    }
    if (!valid) return;
    uint8_t *V = wire_v(d, p);
    if (factors_int4(d)) {
        quantise_factor_row(a, wire4_v(d, p) + (int64_t)ch * 16, wire4_v_scales(d, p) + ch);
        return;
    }
#pragma unroll
    for (int k = 0; k < kRank / 8; ++k) {
        F8 f;
#pragma unroll
        for (int n = 0; n < 8; ++n) f.v[n] = a[8 * k + n];
        if (d.dtype == BF16) {
            Raw8<BF16> o;
            o.narrow(f);
            o.store(V, (int64_t)ch * kRank + 8 * k);
        } else {
            Raw8<F32> o;
            o.narrow(f);
            o.store(V, (int64_t)ch * kRank + 8 * k);
        }
    }
}

// 4-bit factors: U = P (fp32, in the workspace) onto the wire, one lane per token.
__global__ __launch_bounds__(256) void k_lr_quant_u(BatchView v, LaunchRange r)
{
    const int t = r.first + (int)blockIdx.y;
    const TensorDev d = v.descs[t];
    if (d.scale != LOWRANK || !factors_int4(d)) return;
    const TensorPtrs p = v.ptrs[t];
    const int64_t row = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (row >= d.n_tokens) return;
    const CF_GLOBAL f32x4 *src = gconst<f32x4>(v.workspace + d.lr_p_off) + row * (kRank / 4);
    float f[kRank];
#pragma unroll
    for (int k = 0; k < kRank / 4; ++k) {
        const f32x4 w = src[k];
        f[4 * k] = w.x; f[4 * k + 1] = w.y; f[4 * k + 2] = w.z; f[4 * k + 3] = w.w;
    }
    quantise_factor_row(f, wire4_u(p) + row * 16, wire4_u_scales(d, p) + row);
}

// Q = orth(Z) column by column, every column projected twice, for the tensors k_lr_orth left over (normally none: the
// launch is empty).  One workgroup of 1024 lanes per tensor holds the matrix in registers (3 channel rows per lane: C <=
// 3072).  Bound by its 96 rounds of workgroup-wide sums, about 280 us a tensor of 3072 channels.
constexpr int kTwiceThreads = 1024;
constexpr int kTwiceRows = 3;

struct TwiceShared {
    float part[kTwiceThreads / 64][kRank + 1];
    float total[kRank + 1];
};

// Sums `val` over the workgroup into sh.total[slot]; the caller places the barriers.
__device__ __forceinline__ void twice_partial(TwiceShared &sh, int slot, float val)
{
    const float w = wave_tree_sum(val);
    if (((int)threadIdx.x & 63) == 0) sh.part[(int)threadIdx.x >> 6][slot] = w;
}

__device__ __forceinline__ void twice_finish(TwiceShared &sh, int n_slots)
{
    __syncthreads();
    if ((int)threadIdx.x < n_slots) {
        float s = 0.0f;
#pragma unroll
        for (int w = 0; w < kTwiceThreads / 64; ++w) s += sh.part[w][threadIdx.x];
        sh.total[threadIdx.x] = s;
    }
    __syncthreads();
}

// Column K: project it on the finished columns 0..K-1 (twice), then normalise or drop it.  K is a
// template parameter so that every register of the matrix is addressed statically.
template <int K>
__device__ __forceinline__ void twice_column(float (&a)[kTwiceRows][kRank], TwiceShared &sh)
{
    float start2 = 0.0f;
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
        // <q_j, a_K> for every finished column j < K, and (first pass) the column's own length
#pragma unroll
        for (int j = 0; j < K; ++j) {
            float dot = 0.0f;
#pragma unroll
            for (int rr = 0; rr < kTwiceRows; ++rr) dot += a[rr][j] * a[rr][K];
            twice_partial(sh, j, dot);
        }
        if (pass == 0) {
            float own = 0.0f;
#pragma unroll
            for (int rr = 0; rr < kTwiceRows; ++rr) own += a[rr][K] * a[rr][K];
            twice_partial(sh, K, own);
        }
        twice_finish(sh, pass == 0 ? K + 1 : K);
        if (pass == 0) start2 = sh.total[K];
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const float c = sh.total[j];
#pragma unroll
            for (int rr = 0; rr < kTwiceRows; ++rr) a[rr][K] -= c * a[rr][j];
        }
    }
    float own = 0.0f;
#pragma unroll
    for (int rr = 0; rr < kTwiceRows; ++rr) own += a[rr][K] * a[rr][K];
    twice_partial(sh, 0, own);
    twice_finish(sh, 1);
    const float left2 = sh.total[0];
    const bool keep = start2 > 0.0f && left2 > kDrop2 * start2;
    const float len = sqrtf(left2);
#pragma unroll
    for (int rr = 0; rr < kTwiceRows; ++rr) a[rr][K] = keep ? a[rr][K] / len : 0.0f;
    __syncthreads();                                        // sh.total is rewritten by the next column
}

template <int K>
__device__ __forceinline__ void twice_columns_from(float (&a)[kTwiceRows][kRank], TwiceShared &sh)
{
    twice_column<K>(a, sh);
    if constexpr (K + 1 < kRank) twice_columns_from<K + 1>(a, sh);
}

__global__ __launch_bounds__(kTwiceThreads) void k_lr_orth_twice(BatchView v, LaunchRange r, int from_q0, int min_iters)
{
    __shared__ TwiceShared sh;
    const int t = r.first + (int)blockIdx.x;
    const TensorDev d = v.descs[t];
    if (d.scale != LOWRANK || d.bits < min_iters || *lr_left_over(v, d) == 0u) return;      // uniform over the workgroup
    const TensorPtrs p = v.ptrs[t];
    const CF_GLOBAL f32x4 *src = from_q0 ? gconst<f32x4>(p.scales) : gconst<f32x4>(v.workspace + d.lr_z_off);
    float a[kTwiceRows][kRank];
#pragma unroll
    for (int rr = 0; rr < kTwiceRows; ++rr) {
        const int ch = (int)threadIdx.x + kTwiceThreads * rr;
#pragma unroll
        for (int k = 0; k < kRank / 4; ++k) {
            f32x4 w = {};
            if (ch < d.n_channels) w = src[(int64_t)ch * (kRank / 4) + k];
            a[rr][4 * k] = w.x; a[rr][4 * k + 1] = w.y; a[rr][4 * k + 2] = w.z; a[rr][4 * k + 3] = w.w;
        }
    }
    twice_columns_from<0>(a, sh);
    uint8_t *V = wire_v(d, p);
#pragma unroll
    for (int rr = 0; rr < kTwiceRows; ++rr) {
        const int ch = (int)threadIdx.x + kTwiceThreads * rr;
        if (ch >= d.n_channels) continue;
#pragma unroll
        for (int n = 0; n < kRank; ++n) {
            const int64_t at = (((ch & 31) >> 3) * 32 + n) * 8 + (ch & 7);
            const float high = (float)(__bf16)a[rr][n], mid = (float)(__bf16)(a[rr][n] - high);
            gmut<__bf16>(lr_q(v, d, ch >> 5, 0))[at] = (__bf16)high;
            gmut<__bf16>(lr_q(v, d, ch >> 5, 1))[at] = (__bf16)mid;
            gmut<__bf16>(lr_q(v, d, ch >> 5, 2))[at] = (__bf16)(a[rr][n] - high - mid);
            if (factors_int4(d)) continue;
            if (d.dtype == BF16) gmut<uint16_t>(V)[(int64_t)ch * kRank + n] = (uint16_t)bf16_rne(a[rr][n]);
            else gmut<float>(V)[(int64_t)ch * kRank + n] = a[rr][n];
        }
        if (factors_int4(d)) quantise_factor_row(a[rr], wire4_v(d, p) + (int64_t)ch * 16, wire4_v_scales(d, p) + ch);
    }
}

// ---------------------------------------------------------------- D = U V^T, error and reconstruction

// 16 consecutive rank entries (16 * h ...) of one row of a factor on the wire, widened.
// int4: `base` holds rows of 16 nibble bytes and `scales` one fp32 per row.
template <int DT> __device__ __forceinline__ void factor16(const uint8_t *base, const float *scales, bool int4, int64_t row, int h,
                                                           bool valid, float (&out)[16])
{
    const int64_t r0 = valid ? row : 0;                             // row 0 always exists; its values are discarded
    if (int4) {                                                     // uniform over the launch's tensor
        const u32x2 w = *gconst<u32x2>(base + r0 * 16 + 8 * h);
        const float s = *gconst<float>(scales + r0);
        F8 sv, lo, hi;
#pragma unroll
        for (int k = 0; k < 8; ++k) sv.v[k] = s;
        dequant8<4>(w.x, sv, lo);
        dequant8<4>(w.y, sv, hi);
#pragma unroll
        for (int k = 0; k < 8; ++k) { out[k] = lo.v[k]; out[8 + k] = hi.v[k]; }
    } else {
        load16<DT>(base, r0 * kRank + 16 * h, out);
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) out[k] = valid ? out[k] : 0.0f;
}

// One row of a factor on the wire as the MFMAs of D take it, this lane's half of its 32 entries; times() is a 32 x 32 tile of
// rows against rows.  BFW: bf16 factors, whose products the bf16 matrix cores form exactly and add up in fp32, two instructions
// where the fp32 ones take sixteen.
template <int DT, bool BFW> struct Factors {
    float f[16];                // entries 16 h ...
    __device__ __forceinline__ void load(const uint8_t *base, const float *scales, bool int4, int64_t row, int h, bool valid)
    {
        factor16<DT>(base, scales, int4, row, h, valid, f);
    }
    __device__ __forceinline__ f32x16 times(const Factors &other) const
    {
        f32x16 acc = {};
#pragma unroll
        for (int j = 0; j < 16; ++j) acc = mfma32(f[j], other.f[j], acc);
        return acc;
    }
};
template <> struct Factors<BF16, true> {
    u32x4 w[2];                 // entries 8 h ... and 16 + 8 h ...
    __device__ __forceinline__ void load(const uint8_t *base, const float *, bool, int64_t row, int h, bool valid)
    {
        const CF_GLOBAL u32x4 *src = gconst<u32x4>(base + (valid ? row : 0) * (kRank * 2)) + h;     // row 0 always exists
        w[0] = valid ? src[0] : (u32x4)(0u);
        w[1] = valid ? src[2] : (u32x4)(0u);
    }
    __device__ __forceinline__ f32x16 times(const Factors &other) const
    {
        return mfma32_bf16(w[1], other.w[1], mfma32_bf16(w[0], other.w[0], (f32x16)(0.0f)));
    }
};

// A wave owns 32 tokens x 64 channels, or two such tiles; the waves of a workgroup lie side by side.  The MFMA leaves lane (n, h) with
// channel n of 16 tokens, which is the wrong way round for row-major memory, so the tile of D goes
// through the wave's own LDS patch [32 tokens][64 channels] and comes back as 8 consecutive channels
// of one token per lane: 8 lanes then cover 128 bytes of a bf16 row (256 of the fp32 error row).
// SENDER: also forms A again and writes e = A - D.  UPDATE: writes recon + D.
// What bounds it is HBM, and how well depends on how much of a row a workgroup has open and how many do: 57 x [4096, 3072],
// waves below one another, 128 channels wide, fp32 MFMA, two workgroups per CU 1322 us; bf16 MFMA, four of them per CU 1410, two 1358;
// waves side by side, 256 channels, three per CU 1245, two 1196 (512 channels 1254 / 1199).
// Waves that lie side by side in workgroups of their own per 32 tokens idle where a row's tiles are no multiple of theirs.  Receivers, us,
// waves below one another, 128 channels wide / side by side, 256 or 512 channels / counted through: 60 x [8000, 32] bf16 28 / 41 / 19, 4-bit 27 / 54 / 24,
// [8000, 64] fp32 56 / 69 / 56, 30 x [4000, 544] fp32 137 / 193 / 133, bf16 79 / 60 / 57, 4-bit 76 / 110 / 72; 57 x [4096, 3072] bf16 731 / 504 / 504.
constexpr int kApplyChannels = kLowRankApplyChannels;
constexpr int kApplyTokens = kLowRankApplyTokens;
// 4-bit factors cost a wave more to widen than the products: it makes two tiles of its rows of U.
constexpr int apply_tiles_per_wave(bool bf16_wire) { return bf16_wire ? 1 : 2; }
constexpr int kApplyPitch = kApplyChannels + 4;             // floats per token row of the patch
constexpr unsigned kApplyCapLds = 40000;                    // dynamic LDS that nobody touches: two workgroups per CU of senders (the receiver 512 us, 573 capped)

template <int DT, int ET, bool SENDER, bool UPDATE, bool BFW>
__device__ __forceinline__ void lr_apply_body(const TensorDev &d, const TensorPtrs &p, float *patch)
{
    const int lane = (int)threadIdx.x & 63;
    const int n = lane & 31, h = lane >> 5;
    const uint32_t item = blockIdx.x * 4u + (uint32_t)__builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const uint32_t row_waves = (uint32_t)lowrank_apply_waves(d.n_channels, apply_tiles_per_wave(BFW));
    const int64_t tok_base = (int64_t)(item / row_waves) * kApplyTokens;
    if (tok_base >= d.n_tokens) return;                     // uniform over the wave
    const ApplyTiles tiles = lowrank_apply_tiles(d.n_channels, apply_tiles_per_wave(BFW), (int)(item % row_waves));
    const int64_t C = d.n_channels;
    const bool int4 = factors_int4(d);
    Factors<DT, BFW> u;
    u.load(int4 ? wire4_u(p) : wire_u(p), wire4_u_scales(d, p), int4, tok_base + n, h, tok_base + n < d.n_tokens);
    const uint8_t *V = int4 ? wire4_v(d, p) : wire_v(d, p);
    const float *Vs = wire4_v_scales(d, p);
    const int chunk = lane & 7, trow = lane >> 3;           // row-major side: 8 chunks of 8 channels, 8 tokens per sweep
    const int n_sub = d.n_channels / 32;
#pragma unroll 1
    for (int tile = tiles.first; tile < tiles.end; tile += tiles.step) {
        const int sub0 = 2 * tile;
        const int cnt = n_sub - sub0 < 2 ? 1 : 2;
        // Issue order matters because loads return in order: first the V rows the MFMAs need, then the
        // tile's x and recon, which are only needed once D has come back through the patch.
        Factors<DT, BFW> vv[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) vv[c].load(V, Vs, int4, (int64_t)(sub0 + (c < cnt ? c : 0)) * 32 + n, h, true);
        Raw8<DT> xr[4], br[4];
        bool live[4];
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int64_t tok = tok_base + trow + 8 * it;
            live[it] = tok < d.n_tokens && chunk * 8 < cnt * 32;
            const int64_t e0 = tok * C + (int64_t)sub0 * 32 + chunk * 8;
            if (live[it]) {
                if (UPDATE) br[it].load_stream(p.recon, e0);        // written back below: the streaming hint pays
                else br[it].load(p.recon, e0);
                if (SENDER) xr[it].load(p.x, e0); else xr[it].zero();
            } else {
                br[it].zero();
                xr[it].zero();
            }
        }
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            if (c < cnt) {                                  // uniform over the wave
                const f32x16 acc = u.times(vv[c]);
#pragma unroll
                for (int i = 0; i < 16; ++i) patch[(8 * (i >> 2) + 4 * h + (i & 3)) * kApplyPitch + c * 32 + n] = acc[i];
            }
        }
        wave_lds_fence();
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int tl = trow + 8 * it;
            const int64_t tok = tok_base + tl;
            float *row = patch + tl * kApplyPitch;
            f32x4 *mine = reinterpret_cast<f32x4 *>(row + chunk * 8);
            const f32x4 d0 = mine[0], d1 = mine[1];
            F8 D;
            D.v[0] = d0.x; D.v[1] = d0.y; D.v[2] = d0.z; D.v[3] = d0.w;
            D.v[4] = d1.x; D.v[5] = d1.y; D.v[6] = d1.z; D.v[7] = d1.w;
            const int64_t e0 = tok * C + (int64_t)sub0 * 32 + chunk * 8;
            const F8 b = br[it].widen();
            if (SENDER) {
                const F8 x = xr[it].widen();
                F8 lost;
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const float z = x.v[k] - b.v[k];
                    lost.v[k] = z - D.v[k];
                }
                if (ET == F32) {        // the 8 lanes of a token row take its error back from D's place as two whole lines (dead lanes go along)
                    Raw8<F32> eo;
                    eo.narrow(lost);
                    mine[0] = eo.a;
                    mine[1] = eo.b;
                    wave_lds_fence();
                    const f32x4 pieces[2] = {*reinterpret_cast<const f32x4 *>(row + 4 * chunk), *reinterpret_cast<const f32x4 *>(row + 32 + 4 * chunk)};
                    if (tok < d.n_tokens)
                        lines_store_stream<8>(static_cast<float *>(p.err) + tok * C + (int64_t)sub0 * 32, chunk, cnt * 4, pieces);
                } else if (live[it]) {
                    Raw8<ET> eo;
                    eo.narrow(lost);
                    eo.store_stream(p.err, e0);
                }
            }
            if (UPDATE && live[it]) {
                F8 nb;
#pragma unroll
                for (int k = 0; k < 8; ++k) nb.v[k] = b.v[k] + D.v[k];
                Raw8<DT> out;
                out.narrow(nb);
                if (DT == BF16) out.store_stream(p.recon, e0); else out.store(p.recon, e0);
            }
        }
        wave_lds_fence();
    }
}

// BFW: tensors whose factors travel as bf16, else the others (fp32 and 4-bit factors).
template <int ET, bool SENDER, bool UPDATE, bool BFW, class R>
__global__ __launch_bounds__(256, BFW ? 3 : 2) void k_lr_apply(BatchView v, R r)
{
    __shared__ __attribute__((aligned(16))) float patches[4][32 * kApplyPitch];
    const int t = r.first + (int)blockIdx.y;
    const TensorDev d = v.descs[t];
    if (d.scale != LOWRANK || (d.dtype == BF16 && !factors_int4(d)) != BFW) return;
    const TensorPtrs p = call_ptrs(v, r, t);
    float *patch = patches[(int)threadIdx.x >> 6];
    if constexpr (BFW) lr_apply_body<BF16, ET, SENDER, UPDATE, true>(d, p, patch);
    else if (d.dtype == BF16) lr_apply_body<BF16, ET, SENDER, UPDATE, false>(d, p, patch);
    else lr_apply_body<F32, ET, SENDER, UPDATE, false>(d, p, patch);
}

}  // namespace

hipError_t launch_lr_orth(const BatchView &v, const LaunchRange &r, bool from_q0, int min_iters, hipStream_t s)
{
    if (r.count == 0 || r.lr_max_channels == 0) return hipSuccess;
    dim3 grid((unsigned)((r.lr_max_channels + kOrthThreads - 1) / kOrthThreads), (unsigned)r.count);
    if (r.lr_max_channels > kOrthThreads) {
        hipLaunchKernelGGL(k_lr_gram, grid, dim3(kOrthThreads), 0, s, v, r, from_q0 ? 1 : 0, min_iters);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_lr_orth, grid, dim3(kOrthThreads), 0, s, v, r, from_q0 ? 1 : 0, min_iters);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_lr_orth_twice, dim3((unsigned)r.count), dim3(kTwiceThreads), 0, s, v, r, from_q0 ? 1 : 0, min_iters);
    return hipGetLastError();
}

hipError_t launch_lr_project(const BatchView &v, const LaunchRange &r, bool wire, int min_iters, hipStream_t s)
{
    if (r.count == 0 || r.lr_max_tokens == 0) return hipSuccess;
    const dim3 grid((unsigned)r.lr_project_blocks, (unsigned)r.count), block(kProjThreads);
    if (r.dts != F32) {
        if (r.lr_project_many)
            hipLaunchKernelGGL((k_lr_project<BF16, kProjBlocks>), dim3((grid.x + kProjBlocks - 1) / kProjBlocks, grid.y), block, 0, s, v, r, wire ? 1 : 0, min_iters);
        else
            hipLaunchKernelGGL((k_lr_project<BF16, 1>), grid, block, 0, s, v, r, wire ? 1 : 0, min_iters);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (r.dts != BF16) hipLaunchKernelGGL((k_lr_project<F32, 1>), grid, block, 0, s, v, r, wire ? 1 : 0, min_iters);
    return hipGetLastError();
}

hipError_t launch_lr_backproject(const BatchView &v, const LaunchRange &r, int min_iters, hipStream_t s)
{
    if (r.count == 0 || r.lr_max_channels == 0) return hipSuccess;
    dim3 grid((unsigned)((r.lr_max_channels + kBackChannels - 1) / kBackChannels * r.lr_split), (unsigned)r.count);
    if (r.dts != F32) hipLaunchKernelGGL(k_lr_backproject<BF16>, grid, dim3(kBackThreads), 0, s, v, r, min_iters);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (r.dts != BF16) hipLaunchKernelGGL(k_lr_backproject<F32>, grid, dim3(kBackThreads), 0, s, v, r, min_iters);
    return hipGetLastError();
}

// Workgroups of four waves for the largest low-rank tensor of the range; waves beyond a smaller one's last tokens return at once.
static dim3 apply_grid(const LaunchRange &r, bool bf16_wire)
{
    const int64_t waves = (r.lr_max_tokens + kApplyTokens - 1) / kApplyTokens * lowrank_apply_waves(r.lr_max_channels, apply_tiles_per_wave(bf16_wire));
    return dim3((unsigned)((waves + 3) / 4), (unsigned)r.count);
}

hipError_t launch_lr_quant_u(const BatchView &v, const LaunchRange &r, hipStream_t s)
{
    if (r.count == 0 || r.lr_max_tokens == 0) return hipSuccess;
    dim3 grid((unsigned)((r.lr_max_tokens + 255) / 256), (unsigned)r.count);
    hipLaunchKernelGGL(k_lr_quant_u, grid, dim3(256), 0, s, v, r);
    return hipGetLastError();
}

// one launch per kind of factors in the range
template <int ET, bool SENDER, bool UPDATE, class R>
static hipError_t launch_apply(const BatchView &v, const R &r, hipStream_t s)
{
    if (r.lr_wires & 1) {
        hipLaunchKernelGGL((k_lr_apply<ET, SENDER, UPDATE, true, R>), apply_grid(r, true), dim3(256), SENDER ? kApplyCapLds : 0u, s, v, r);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (r.lr_wires & 2) hipLaunchKernelGGL((k_lr_apply<ET, SENDER, UPDATE, false, R>), apply_grid(r, false), dim3(256), 0, s, v, r);
    return hipGetLastError();
}

hipError_t launch_lr_encode(const BatchView &v, const LaunchRange &r, int err_dtype, bool fused, hipStream_t s)
{
    if (r.count == 0 || r.lr_max_tokens == 0) return hipSuccess;
    if (err_dtype == BF16) return fused ? launch_apply<BF16, true, true>(v, r, s) : launch_apply<BF16, true, false>(v, r, s);
    return fused ? launch_apply<F32, true, true>(v, r, s) : launch_apply<F32, true, false>(v, r, s);
}

hipError_t launch_lr_decode(const BatchView &v, const LaunchRange &range, hipStream_t s)
{
    if (range.count == 0 || range.lr_max_tokens == 0) return hipSuccess;
    return with_range(range, [&](const auto &r) { return launch_apply<F32, false, true>(v, r, s); });
}

}  // namespace cf
