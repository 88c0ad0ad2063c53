// Low-rank compressor (arxiv 2507.17511, Alg. 3 and App. D "Low-Rank Compression") under the
// residual recursion of Sec. 3.1: A = x_t - recon_{t-1} [tokens, channels] is sent as rank-32 factors
// U = A Q [tokens, 32], V = Q [channels, 32] found by T steps of subspace iteration
//     Q <- orth(Q0);  T x { Z <- A^T (A Q);  Q <- orth(Z) };  U <- A Q,
// and both ends add D = U V^T to the reconstruction; e_t = A - D stays at the sender.
//
// This is the one dense contraction of the codec, so it runs on the matrix cores: every product is a
// chain of v_mfma_f32_32x32x2_f32 (fp32 in, fp32 accumulate; 32 = the rank fills the N side of the
// tile exactly).  A is never materialised: each pass re-forms it from x and recon (4 bytes per element
// in bf16 storage, the same as reading an fp32 A would cost) and is bound by that stream.
//
// Operand layouts are chosen so that every lane feeds the MFMA straight from a 128-bit row-major
// load, with no staging through LDS.  The instruction computes D[m][n] += sum_k A[m][k] B[k][n] with
// lane l holding A[l % 32][l / 32] and B[l / 32][l % 32]: any relabelling of k that both operands share,
// and any relabelling of m or n that the epilogue undoes, is free.
//   project      P = A Q     m = token, k = channel: a lane loads 16 consecutive channels of its token
//                            and spends them on 16 instructions; Q is kept in that per-lane order.
//   backproject  Z = A^T P   m = channel, k = token: a lane loads 8 consecutive channels of its token and
//                            spends them on 8 channel tiles (tile j holds channels = j mod 8); 16x16x4 tiles.
//   encode       D^T = V U^T m = channel (relabelled so that a lane ends up with 16 consecutive channels
//                            of its token), n = token, k = rank.
#include "cf_device.h"
#include "cf_internal.h"

namespace cf {
namespace {

using namespace dev;

typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kRank = 32;
constexpr float kDrop2 = 1e-8f;     // (1e-4)^2: a column left with less than 1e-4 of its length is dropped

__device__ __forceinline__ f32x16 mfma32(float a, float b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }

__device__ __forceinline__ f32x4 mfma16(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// Operands a pass reads once.  Streaming hint for bf16 only, whose lanes take their 16 bytes in one load: fp32 lanes take
// 32 bytes in two, and the hint lets go of the line in between.  57 x [4096, 3072], plain and with the hint: bf16 project
// 600 / 585 us, back-projection 616 / 593; fp32 project 1094 / 1263, back-projection 1348 / 1779 (at four waves per SIMD).
template <int DT> __device__ __forceinline__ void load_once(Raw8<DT> &r, const void *base, int64_t elem)
{
    if (DT == BF16) r.load_stream(base, elem); else r.load(base, elem);
}

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

// 16 consecutive elements of the residual x - recon of one token, or zeros.
template <int DT> __device__ __forceinline__ void residual16(const TensorPtrs &p, int64_t elem, bool valid, float (&z)[16])
{
    if (valid) {
        float x[16], b[16];
        load16<DT>(p.x, elem, x);
        load16<DT>(p.recon, elem, b);
#pragma unroll
        for (int k = 0; k < 16; ++k) z[k] = x[k] - b[k];
    } else {
#pragma unroll
        for (int k = 0; k < 16; ++k) z[k] = 0.0f;
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

// ---------------------------------------------------------------- P = A Q  (and U on the wire)

// A wave owns 64 tokens (two accumulator tiles that share the Q operand), a workgroup of two waves 128, and walks
// the channels 64 at a time.  The MFMA wants a lane to hold one token's channels, memory wants
// neighbouring lanes on neighbouring channels: the wave reads its [64 tokens][64 channels] of x and
// recon row-major (8 lanes = 128 bytes of a bf16 row), leaves the residual in its own LDS patch and
// picks it up again with lane (m, h) on token m (and m + 32), channels 16 * h ... of each 32-channel step.
// Q is read in its per-lane order: step s (32 channels), lane l, 16 floats at ((s * 64 + l) * 16).
constexpr int kProjThreads = 128;                           // two waves: their LDS patches stay under 64 KB at four workgroups per CU
constexpr int kProjTokens = 128;
constexpr int kProjChannels = 64;
constexpr int kProjPitch = kProjChannels + 4;               // floats per token row of the patch

template <int DT>
__device__ __forceinline__ void lr_project_body(const BatchView &v, const TensorDev &d, const TensorPtrs &p, bool wire, float *patch)
{
    const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
    const int m = lane & 31, h = lane >> 5;
    const int64_t row_base = (int64_t)blockIdx.x * kProjTokens + wave * 64;
    if (row_base >= d.n_tokens) return;                     // uniform over the wave
    const int64_t C = d.n_channels;
    const CF_GLOBAL f32x4 *qs = gconst<f32x4>(v.workspace + d.lr_z_off);
    f32x16 acc0 = {}, acc1 = {};
    const int steps = d.n_channels / 32;
    const int chunk = lane & 7, trow = lane >> 3;           // row-major side: 8 chunks of 8 channels, 8 tokens per sweep
    // The loads of the next 64 channels are issued as soon as the current ones have gone to the patch,
    // so that they are in flight while the 64 MFMAs of the current ones run.
    Raw8<DT> xr[8], br[8];
    auto fetch = [&](int s0) {
        const int ch = s0 * 32 + chunk * 8;
#pragma unroll
        for (int it = 0; it < 8; ++it) {
            const int64_t tok = row_base + trow + 8 * it;
            if (s0 < steps && tok < d.n_tokens && ch < d.n_channels) {
                load_once<DT>(xr[it], p.x, tok * C + ch);
                load_once<DT>(br[it], p.recon, tok * C + ch);
            } else {
                xr[it].zero();
                br[it].zero();
            }
        }
    };
    fetch(0);
    for (int s0 = 0; s0 < steps; s0 += 2) {
#pragma unroll
        for (int it = 0; it < 8; ++it) {
            const F8 x = xr[it].widen(), b = br[it].widen();
            f32x4 lo, hi;
            lo.x = x.v[0] - b.v[0]; lo.y = x.v[1] - b.v[1]; lo.z = x.v[2] - b.v[2]; lo.w = x.v[3] - b.v[3];
            hi.x = x.v[4] - b.v[4]; hi.y = x.v[5] - b.v[5]; hi.z = x.v[6] - b.v[6]; hi.w = x.v[7] - b.v[7];
            f32x4 *dst = reinterpret_cast<f32x4 *>(patch + (trow + 8 * it) * kProjPitch + chunk * 8);
            dst[0] = lo;
            dst[1] = hi;
        }
        // Q first, then the prefetch: loads return in issue order, so the MFMAs below wait for Q only
        float q[2][16];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const CF_GLOBAL f32x4 *qp = qs + ((int64_t)(s0 + u < steps ? s0 + u : s0) * 64 + lane) * 4;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const f32x4 wq = qp[k];
                q[u][4 * k] = wq.x; q[u][4 * k + 1] = wq.y; q[u][4 * k + 2] = wq.z; q[u][4 * k + 3] = wq.w;
            }
        }
        fetch(s0 + 2);
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (s0 + u < steps) {                           // uniform over the wave
                float z0[16], z1[16];
                const f32x4 *a0 = reinterpret_cast<const f32x4 *>(patch + m * kProjPitch + 32 * u + 16 * h);
                const f32x4 *a1 = reinterpret_cast<const f32x4 *>(patch + (m + 32) * kProjPitch + 32 * u + 16 * h);
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const f32x4 w0 = a0[k], w1 = a1[k];
                    z0[4 * k] = w0.x; z0[4 * k + 1] = w0.y; z0[4 * k + 2] = w0.z; z0[4 * k + 3] = w0.w;
                    z1[4 * k] = w1.x; z1[4 * k + 1] = w1.y; z1[4 * k + 2] = w1.z; z1[4 * k + 3] = w1.w;
                }
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    acc0 = mfma32(z0[j], q[u][j], acc0);
                    acc1 = mfma32(z1[j], q[u][j], acc1);
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
    // accumulator register i of lane (m, h): row 8 * (i / 4) + 4 * h + i % 4 of the tile, column m
    CF_GLOBAL float *P = gmut<float>(v.workspace + d.lr_p_off);
    uint8_t *U = wire_u(p);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int row = 8 * (i >> 2) + 4 * h + (i & 3);
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int64_t rr = row_base + 32 * half + row;
            const float val = half ? acc1[i] : acc0[i];
            if (rr < d.n_tokens) {
                P[rr * kRank + m] = val;
                if (wire && !factors_int4(d)) {     // 4-bit factors are quantised from P by k_lr_quant_u
                    if (DT == BF16) gmut<uint16_t>(U)[rr * kRank + m] = (uint16_t)bf16_rne(val);
                    else gmut<float>(U)[rr * kRank + m] = val;
                }
            }
        }
    }
}

// min_iters: tensors that asked for fewer subspace iterations than this sit the launch out.
__global__ __launch_bounds__(kProjThreads, 2) void k_lr_project(BatchView v, LaunchRange r, int wire, int min_iters)
{
    __shared__ __attribute__((aligned(16))) float patches[kProjThreads / 64][64 * kProjPitch];
    const int t = r.first + (int)blockIdx.y;
    const TensorDev d = v.descs[t];
    if (d.scale != LOWRANK || d.bits < min_iters) return;
    const TensorPtrs p = v.ptrs[t];
    float *patch = patches[(int)threadIdx.x >> 6];
    if (d.dtype == BF16) lr_project_body<BF16>(v, d, p, wire != 0, patch);
    else lr_project_body<F32>(v, d, p, wire != 0, patch);
}

// ---------------------------------------------------------------- Z = A^T P

// Workgroups that share the runs of one stripe of a tensor.
__device__ __forceinline__ int lr_shares(const LaunchRange &r, const TensorDev &d)
{
    const int runs = lowrank_runs(d.n_tokens, d.n_channels);
    return r.lr_split < runs ? r.lr_split : runs;
}

// Where share `share` of tensor t leaves its part of Z: the first in Z itself.
__device__ __forceinline__ uint8_t *lr_slice(const BatchView &v, const LaunchRange &r, const TensorDev &d, int t, int share)
{
    if (share == 0) return v.workspace + d.lr_z_off;
    return v.workspace + r.lr_slices_off + (uint64_t)((t - r.first) * (r.lr_split - 1) + share - 1) * (uint64_t)r.lr_max_channels * (kRank * sizeof(float));
}

// The tokens are cut into lowrank_runs = 1, 2 or 4 runs.  Z is the sum (run 0 + run 1) + (run 2 + run 3), each run the
// sum (w0 + w1) + (w2 + w3) over its 4 waves, so the bits depend on the tensor's shape alone, whoever adds: a workgroup
// owns a stripe of 128 channels and either takes all runs one after the other, or, in calls of few tensors, one or two
// of them, and the orthogonalisation adds the shares.
// v_mfma_f32_16x16x4_f32 takes A[l % 16][l / 16] and B[l / 16][l % 16] from lane l: lane (q, g) holds channels
// 8q..8q+7 of the stripe of token 4 * quad + g, straight from a 128-bit load, and spends them on 8 channel tiles
// (tile j holds channels = j mod 8) times 2 rank tiles.  What bounds it is how much a CU has in flight:
// three waves per SIMD (142 registers, 64 of them accumulators), each with the loads of one quad, about 2 KB; the loop asks
// for R quads ahead, the compiler moves their loads down to the quad before their use.  57 x [4096, 3072], us: bf16 621
// (713 with 256 channels and two waves per SIMD; 635 at four waves with one run), fp32 1185 (1187; 1769 at four waves and with the hint).
// The sums cost a drained pipeline and two barriers a run: four turns of one wave each instead of two of two took 1 %
// longer at 57 x [1000, 3072].
constexpr int kBackThreads = 256;
constexpr int kBackChannels = kLowRankBackChannels;
constexpr int kBackEntries = kBackChannels * kRank;
typedef float BackSums[2][kBackEntries];                    // of waves 0 + 1 and 2 + 3

template <int DT>
__device__ __forceinline__ void lr_backproject_body(const BatchView &v, const LaunchRange &r, const TensorDev &d, const TensorPtrs &p, int t,
                                                    int stripe, int share, BackSums &sums, float *total)
{
    const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
    const int q = lane & 15, g = lane >> 4;
    const int64_t C = d.n_channels, last = d.n_tokens - 1;
    const int64_t n_quads = (d.n_tokens + 3) / 4;
    const int n_runs = lowrank_runs(d.n_tokens, d.n_channels), n_mine = n_runs / lr_shares(r, d), first_run = share * n_mine;
    const int64_t per_wave = (n_quads + 4 * n_runs - 1) / (4 * n_runs);
    // Loads without branches: rows and channels outside the tensor read its last ones, P counts as zero there and the
    // channels are not stored.
    const int ch0 = stripe * kBackChannels + 8 * q;
    const int ch = ch0 < d.n_channels ? ch0 : d.n_channels - 8;
    const CF_GLOBAL float *P = gconst<float>(v.workspace + d.lr_p_off) + q;
    constexpr int R = (DT == F32) ? 4 : 8;                  // quads asked for ahead (fp32 rows take twice the registers)
    Raw8<DT> xr[R], br[R];
    float pv[R][2];
    auto fetch = [&](int slot, int64_t quad) {
        const int64_t row = 4 * quad + g;
        const int64_t at = row < last ? row : last;
        load_once<DT>(xr[slot], p.x, at * C + ch);
        load_once<DT>(br[slot], p.recon, at * C + ch);
        pv[slot][0] = P[at * kRank];
        pv[slot][1] = P[at * kRank + 16];
    };
    CF_GLOBAL float *Z = gmut<float>(lr_slice(v, r, d, t, share)) + (int64_t)stripe * kBackEntries;
    const int n_out = (d.n_channels - stripe * kBackChannels) * kRank;      // entries of the stripe that exist
    for (int run = first_run; run < first_run + n_mine; ++run) {            // uniform over the workgroup
        const int64_t lo = (run * 4 + wave) * per_wave;     // may lie beyond the last quad: such a wave adds zeros
        const int64_t hi = lo + per_wave < n_quads ? lo + per_wave : n_quads;
        f32x4 acc[8][2];
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j][0] = acc[j][1] = (f32x4)(0.0f);
        if (lo < hi) {
#pragma unroll
            for (int u = 0; u < R; ++u) fetch(u, lo + u);
            for (int64_t quad0 = lo; quad0 < hi; quad0 += R) {
#pragma unroll
                for (int u = 0; u < R; ++u) {
                    const F8 x = xr[u].widen(), b = br[u].widen();
                    F8 z;
#pragma unroll
                    for (int j = 0; j < 8; ++j) z.v[j] = x.v[j] - b.v[j];
                    const bool valid = quad0 + u < hi && 4 * (quad0 + u) + g <= last;
                    const float p0 = valid ? pv[u][0] : 0.0f, p1 = valid ? pv[u][1] : 0.0f;
                    fetch(u, quad0 + R + u);
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        acc[j][0] = mfma16(z.v[j], p0, acc[j][0]);
                        acc[j][1] = mfma16(z.v[j], p1, acc[j][1]);
                    }
                }
            }
        }
        // tile j, register i of lane (q, g): channel 8 * (4 * g + i) + j of the stripe, column q (and 16 + q)
        for (int w = 0; w < 2; ++w) {
            if ((wave & 1) == w) {
                float *mine = sums[wave >> 1];
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
            float pair = sums[0][k] + sums[1][k];
            if (!opens) pair = total[k] + pair;
            if (!closes) total[k] = pair;
            else if (k < n_out) Z[k] = run < first_run + 2 ? pair : Z[k] + pair;
        }
        __syncthreads();                                    // before the next run's first waves write their sums
    }
}

__global__ __launch_bounds__(kBackThreads, 3) void k_lr_backproject(BatchView v, LaunchRange r, int min_iters)
{
    __shared__ BackSums sums;
    __shared__ float total[kBackEntries];
    const int t = r.first + (int)blockIdx.y;
    const TensorDev d = v.descs[t];
    if (d.scale != LOWRANK || d.bits < min_iters) return;
    const int n_stripes = (d.n_channels + kBackChannels - 1) / kBackChannels;
    const int stripe = (int)blockIdx.x % n_stripes, share = (int)blockIdx.x / n_stripes;
    if (share >= lr_shares(r, d)) return;                   // uniform over the workgroup: narrower or shorter than the largest tensor
    const TensorPtrs p = v.ptrs[t];
    if (d.dtype == BF16) lr_backproject_body<BF16>(v, r, d, p, t, stripe, share, sums, total);
    else lr_backproject_body<F32>(v, r, d, p, t, stripe, share, sums, total);
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

// Whether k_lr_orth left the tensor to k_lr_orth_twice: the last word of the Gram matrices' area, whose partial sums
// fill at most 32 C + 8160 of its 128 C bytes (and which k_lr_orth alone uses where C <= 256).
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
        const CF_GLOBAL float *s1 = gconst<float>(lr_slice(v, r, d, t, 1));
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            const int row = row0 + 4 * s;
            const bool valid = row < n_channels;
            lo[s] += valid ? s1[(int64_t)row * kRank + col] : 0.0f;
            hi[s] += valid ? s1[(int64_t)row * kRank + 16 + col] : 0.0f;
        }
        if (n_shares > 2) {
            const CF_GLOBAL float *s2 = gconst<float>(lr_slice(v, r, d, t, 2)), *s3 = gconst<float>(lr_slice(v, r, d, t, 3));
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
    if (!valid) return;
    CF_GLOBAL float *qs = gmut<float>(v.workspace + d.lr_z_off);
    uint8_t *V = wire_v(d, p);
    const int s = ch >> 5, c = ch & 31, hh = c >> 4, j = c & 15;
#pragma unroll
    for (int n = 0; n < kRank; ++n) qs[((int64_t)s * 64 + hh * 32 + n) * 16 + j] = a[n];
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
    CF_GLOBAL float *qs = gmut<float>(v.workspace + d.lr_z_off);
    uint8_t *V = wire_v(d, p);
#pragma unroll
    for (int rr = 0; rr < kTwiceRows; ++rr) {
        const int ch = (int)threadIdx.x + kTwiceThreads * rr;
        if (ch >= d.n_channels) continue;
        const int s = ch >> 5, c = ch & 31, hh = c >> 4, j = c & 15;
#pragma unroll
        for (int n = 0; n < kRank; ++n) {
            qs[((int64_t)s * 64 + hh * 32 + n) * 16 + j] = a[rr][n];
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

// A wave owns 32 tokens and kApplySpan channels, which it walks in tiles of 64 (a workgroup that
// looped over all channels would have to drain its stores before each tile's loads count as returned).  The MFMA leaves lane (n, h) with
// channel n of 16 tokens, which is the wrong way round for row-major memory, so the tile of D goes
// through the wave's own LDS patch [32 tokens][64 channels] and comes back as 8 consecutive channels
// of one token per lane: 8 lanes then cover 128 bytes of a bf16 row (256 of the fp32 error row).
// SENDER: also forms A again and writes e = A - D.  UPDATE: writes recon + D.
constexpr int kApplyChannels = 64;
#ifndef CF_APPLY_SPAN
#define CF_APPLY_SPAN 128
#endif
constexpr int kApplySpan = CF_APPLY_SPAN;                   // channels per workgroup
constexpr int kApplyPitch = kApplyChannels + 4;             // floats per token row of the patch

template <int DT, int ET, bool SENDER, bool UPDATE>
__device__ __forceinline__ void lr_apply_body(const TensorDev &d, const TensorPtrs &p, float *patch, float *epatch)
{
    const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
    const int n = lane & 31, h = lane >> 5;
    const int n_spans = (d.n_channels + kApplySpan - 1) / kApplySpan;
    const int span = (int)(blockIdx.x % (unsigned)n_spans);
    const int64_t tok_base = (int64_t)(blockIdx.x / (unsigned)n_spans) * 128 + wave * 32;
    if (tok_base >= d.n_tokens) return;                     // uniform over the wave
    const int64_t C = d.n_channels;
    float u[16];
    const bool int4 = factors_int4(d);
    factor16<DT>(int4 ? wire4_u(p) : wire_u(p), wire4_u_scales(d, p), int4, tok_base + n, h, tok_base + n < d.n_tokens, u);
    const uint8_t *V = int4 ? wire4_v(d, p) : wire_v(d, p);
    const float *Vs = wire4_v_scales(d, p);
    const int sub_lo = span * (kApplySpan / 32);
    const int n_sub = d.n_channels / 32 < sub_lo + kApplySpan / 32 ? d.n_channels / 32 : sub_lo + kApplySpan / 32;
    const int chunk = lane & 7, trow = lane >> 3;           // row-major side: 8 chunks of 8 channels, 8 tokens per sweep
    for (int sub0 = sub_lo; sub0 < n_sub; sub0 += 2) {
        const int cnt = n_sub - sub0 < 2 ? 1 : 2;
        // Issue order matters because loads return in order: first the V rows the MFMAs need, then the
        // tile's x and recon, which are only needed once D has come back through the patch.
        float vv[2][16];
#pragma unroll
        for (int c = 0; c < 2; ++c) factor16<DT>(V, Vs, int4, (int64_t)(sub0 + (c < cnt ? c : 0)) * 32 + n, h, true, vv[c]);
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
                f32x16 acc = {};
#pragma unroll
                for (int j = 0; j < 16; ++j) acc = mfma32(u[j], vv[c][j], acc);
#pragma unroll
                for (int i = 0; i < 16; ++i) patch[(8 * (i >> 2) + 4 * h + (i & 3)) * kApplyPitch + c * 32 + n] = acc[i];
            }
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int tl = trow + 8 * it;
            const int64_t tok = tok_base + tl;
            // every lane goes through the exchange of the error row (dead lanes carry values nobody stores)
            const f32x4 *src = reinterpret_cast<const f32x4 *>(patch + tl * kApplyPitch + chunk * 8);
            const f32x4 d0 = src[0], d1 = src[1];
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
                if (ET == F32) {        // the 8 lanes of a token row send its 256 bytes as two whole lines
                    f32x4 pieces[2];
                    lines_exchange<8>(epatch, lane, lost, pieces);
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
        __builtin_amdgcn_wave_barrier();
    }
}

template <int ET, bool SENDER, bool UPDATE>
__global__ __launch_bounds__(256) void k_lr_apply(BatchView v, LaunchRange r)
{
    __shared__ __attribute__((aligned(16))) float patches[4][32 * kApplyPitch];
    const int t = r.first + (int)blockIdx.y;
    const TensorDev d = v.descs[t];
    if (d.scale != LOWRANK) return;
    const TensorPtrs p = v.ptrs[t];
    __shared__ __attribute__((aligned(16))) float epatches[4][512];       // the error rows' way to whole lines (2 KB per wave)
    float *patch = patches[(int)threadIdx.x >> 6];
    float *epatch = epatches[(int)threadIdx.x >> 6];
    if (d.dtype == BF16) lr_apply_body<BF16, ET, SENDER, UPDATE>(d, p, patch, epatch);
    else lr_apply_body<F32, ET, SENDER, UPDATE>(d, p, patch, epatch);
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
    dim3 grid((unsigned)((r.lr_max_tokens + kProjTokens - 1) / kProjTokens), (unsigned)r.count);
    hipLaunchKernelGGL(k_lr_project, grid, dim3(kProjThreads), 0, s, v, r, wire ? 1 : 0, min_iters);
    return hipGetLastError();
}

hipError_t launch_lr_backproject(const BatchView &v, const LaunchRange &r, int min_iters, hipStream_t s)
{
    if (r.count == 0 || r.lr_max_channels == 0) return hipSuccess;
    dim3 grid((unsigned)((r.lr_max_channels + kBackChannels - 1) / kBackChannels * r.lr_split), (unsigned)r.count);
    hipLaunchKernelGGL(k_lr_backproject, grid, dim3(kBackThreads), 0, s, v, r, min_iters);
    return hipGetLastError();
}

// Blocks of 128 tokens x kApplySpan channels, for the largest low-rank tensor of the range; a tensor with
// fewer channel spans sees block indices beyond its own and returns at once (tok_base >= n_tokens).
static unsigned apply_blocks(const LaunchRange &r)
{
    return (unsigned)((r.lr_max_tokens + 127) / 128) * (unsigned)((r.lr_max_channels + kApplySpan - 1) / kApplySpan);
}

hipError_t launch_lr_quant_u(const BatchView &v, const LaunchRange &r, hipStream_t s)
{
    if (r.count == 0 || r.lr_max_tokens == 0) return hipSuccess;
    dim3 grid((unsigned)((r.lr_max_tokens + 255) / 256), (unsigned)r.count);
    hipLaunchKernelGGL(k_lr_quant_u, grid, dim3(256), 0, s, v, r);
    return hipGetLastError();
}

hipError_t launch_lr_encode(const BatchView &v, const LaunchRange &r, int err_dtype, bool fused, hipStream_t s)
{
    if (r.count == 0 || r.lr_max_tokens == 0) return hipSuccess;
    dim3 grid(apply_blocks(r), (unsigned)r.count), block(256);
    if (err_dtype == BF16) {
        if (fused) hipLaunchKernelGGL((k_lr_apply<BF16, true, true>), grid, block, 0, s, v, r);
        else hipLaunchKernelGGL((k_lr_apply<BF16, true, false>), grid, block, 0, s, v, r);
    } else {
        if (fused) hipLaunchKernelGGL((k_lr_apply<F32, true, true>), grid, block, 0, s, v, r);
        else hipLaunchKernelGGL((k_lr_apply<F32, true, false>), grid, block, 0, s, v, r);
    }
    return hipGetLastError();
}

hipError_t launch_lr_decode(const BatchView &v, const LaunchRange &r, hipStream_t s)
{
    if (r.count == 0 || r.lr_max_tokens == 0) return hipSuccess;
    dim3 grid(apply_blocks(r), (unsigned)r.count);
    hipLaunchKernelGGL((k_lr_apply<F32, false, true>), grid, dim3(256), 0, s, v, r);
    return hipGetLastError();
}

}  // namespace cf
