// milo_compress_w3lr: the MiLo compression loop (Algorithm 1) on the device.
//
// One outer iteration is  R = W - U V;  a few half-quadratic updates of the zero-points z for the
// target R with the scales fixed (Section 3.2, Eq. update_We / update_z);  E = W - W_dq;  a truncated
// SVD of E split as U = U^ S^(1/2), V = S^(1/2) V^ (Eq. UV);  the error eps_t (Eq. epsilon).  The host
// reads eps_t after every iteration and applies the stop rule (Eq. stop_condition).
//
// The SVD is the only step that is not a plain transcription: an exact SVD of a 14336 x 4096 matrix
// per iteration is what makes the method slow on the paper's own hardware, and the loop only needs the
// leading r (<= 128) triplets.  They come from a block subspace iteration with l = r + 8 vectors:
//     Y = E Vb^T,  Y^T Y = L L^T,  B = L^-1 Y^T E  (= Q^T E for the orthonormal Q = Y L^-T),
//     next basis: the rows of B, orthonormalized by a Cholesky factorization of B B^T
// and after the last round B B^T = Ub S^2 Ub^T (Jacobi), U = Q Ub_r S_r^(1/2), V = S_r^(-1/2) Ub_r^T B.
// Only the space that a basis spans matters to the next round, so the eigenvectors are formed once per
// outer iteration and not once per round.  The first outer iteration starts from a random basis with a
// few extra rounds, later ones from the previous right singular vectors (E changes little between outer
// iterations, so the outer loop itself is the power iteration).
//
// Each round reads E twice; both products are tall-skinny (l <= 136), so they are bound by HBM as long as
// the fp32 matrix cores do the arithmetic: 16 x 16 x 4 tiles, no operand converted, fp32 throughout.
// 14336 x 4096, r = 32: 67 us for Y, 71 us for Y^T E (E is 235 MB:
// 3.5 TB/s), against about 330 us each on the vector units.
//
// Compiled with -ffp-contract=off like the quantizer: the half-quadratic update follows its
// formulas one rounding per operation.
#include <math.h>

#include <type_traits>

#include "milo_device.h"
#include "milo_host.h"
#include "pack_device.h"

namespace milo {

constexpr int kSketchExtra = 8;                                   // l = r + 8 basis vectors
constexpr int kSketchMax = MILO_COMPRESS_MAX_RANK + kSketchExtra;
constexpr int kSmallThreads = 512;            // the one-workgroup factorizations and the pass that one runs beside

// ------------------------------------------------------------------ half-quadratic zero-point updates
// The whole quantization step of one outer iteration for the target R: FIRST: R = W, the scales
// s = fp16((max - min) / 7) (1 for a degenerate group) and the start z = -min / s come from W's group and
// s is stored; otherwise R is in RE and s, z are read.  RE receives E = W - s (W_q - z) with the codes and z
// of the last update, z the zero-points.
//
// One lane owns a group: the 64 targets, divided by the scale, stay in its registers over all updates and the
// group's mean needs no cross-lane step.  An update is, per weight,
//     q = clamp(rint(r / s + z));  e = r - s (q - z);  m = shrink(e);  z' = mean(q - (r - m) / s)
// and shrink(e), which takes |e|^(p-1) / beta off |e|, is exactly zero as long as |e| <= beta^(-1/(2-p)), 0.17 for
// the defaults: residuals of that size do not occur in a weight of usual magnitude.  A wave bounds the |e| of its
// groups by half a step, or by what the ends of the group lose to the clamp, and evaluates the shrinkage (a logarithm and
// an exponential per weight, three quarters of the work) only when that is above the limit (less a margin for the
// rounding of the power).  The sums keep one order (four in turn, then pairs), with or without the shrinkage: a zero-point
// that is off by one rounding moves a code at a boundary now and then, and from there on everything that follows.
// Without the shrinkage an update that returns every zero-point of the wave is a fixed point: the rest of the updates would
// repeat it (a normal weight takes 7 to 17 of them until the last of a wave's 64 groups is there, 11 in the mean).
// Bound: the vector units, five operations per weight and update, and HBM (W in, E out: 90 us).  14336 x 4096, 20
// updates: 143 us (167 when all were carried out); with 16 lanes per group and the shrinkage always evaluated 772 us + 48 us
// for the scales + 71 us for a copy of W.
// Sum of 64 values: four in turn, then pairs.  four(k, a) gives values 4 k .. 4 k + 3; the barriers keep the scheduler from
// forming all of them before the first addition (128 registers hold the group already).
template <typename F>
__device__ __forceinline__ float group_sum(F&& four) {
    float a[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        float v[4];
        four(k, v);
        a[k] = ((v[0] + v[1]) + v[2]) + v[3];
        if (k % 2 == 1) __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int d = 1; d < 16; d <<= 1)
#pragma unroll
        for (int k = 0; k < 16; k += 2 * d) a[k] += a[k + d];
    return a[0];
}

template <bool FIRST>
__global__ __launch_bounds__(kRowBlockThreads, 2) void hqq_kernel(const float* __restrict__ W, float* __restrict__ RE,
                                                               float* __restrict__ s, float* __restrict__ z, int64_t N, int64_t K,
                                                               int iters, float pm1, float beta, float kappa, float edge, float edge_step) {
    __shared__ __attribute__((aligned(16))) unsigned char lds[kRowBlockWaves * kRowBlockBytes];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t G = K / kGroup;
    int64_t n0, g0;
    if (!row_block_item(N, G, wave, &n0, &g0)) return;
    unsigned char* const area = lds + wave * kRowBlockBytes;
    const int row = lane & 15, gl = lane >> 4;
    const bool live = g0 + gl < G;
    const int64_t gu = (n0 + row) * G + g0 + gl;
    stage_row_block(FIRST ? W : RE, K, n0, N, g0, K, area, lane);
    wait_vmem();
    float t[64];
    read_unit64(area, lane, t);
    float sf, zf, mn = t[0], mx = t[0];
#pragma unroll
    for (int i = 1; i < 64; ++i) {
        mn = fminf(mn, t[i]);
        mx = fmaxf(mx, t[i]);
    }
    if (FIRST) {
        sf = (float)(f16)((mx - mn) / 7.0f);
        if (!(sf > 0.0f && sf <= 65504.0f)) sf = 1.0f;
        zf = (-mn) / sf;
        if (live) s[gu] = sf;
    } else {
        sf = live ? s[gu] : 1.0f;
        zf = live ? z[gu] : 0.0f;
    }
    const float inv_s = 1.0f / sf;
    mn = div_by(mn, sf, inv_s);
    mx = div_by(mx, sf, inv_s);
    float p[64];                    // r / s as the mean takes it: by the reciprocal
#pragma unroll
    for (int i = 0; i < 64; ++i) {
        p[i] = t[i] * inv_s;
        t[i] = div_by(t[i], sf, inv_s);
    }
    int it = 0;
    bool settled = false;
    for (; it < iters; ++it) {
        // largest residual of the group: a rounding, or a clamp at one of its ends
        const float most = fmaxf(0.5f, fmaxf((mx + zf) - 7.0f, -(mn + zf))) * sf;
        if (__builtin_amdgcn_ballot_w64(live && !(most <= edge)) != 0ull) break;
        if (!settled) {
            const float zn = group_sum([&](int k, float (&v)[4]) {
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = fminf(fmaxf(__builtin_rintf(t[4 * k + i] + zf), 0.0f), 7.0f) - p[4 * k + i];
            }) * (1.0f / 64.0f);
            // an update that gives every group of the wave its zero-point back, bit for bit, is the last one that does anything
            settled = __builtin_amdgcn_ballot_w64(__builtin_bit_cast(uint32_t, zn) != __builtin_bit_cast(uint32_t, zf)) == 0ull;
            zf = zn;
        }
        beta *= kappa;
        edge *= edge_step;
    }
    // From the first update on that needs it, with the shrinkage: |e|^(p-1) through the hardware's exp2 and log2
    // (about 1 ulp each; the threshold is a smooth function, no decision hangs on its last bits).  The targets
    // come from LDS again, so that the loop above has the registers to itself.
    for (; it < iters; ++it) {
        const float inv_beta = 1.0f / beta;
        int unit_at = row * 1024 + gl * 256;
        asm volatile("" : "+v"(unit_at));           // (read in every update, not kept)
        zf = group_sum([&](int k, float (&v)[4]) {
            const float4 r4 = *reinterpret_cast<const float4*>(area + unit_at + ((k ^ row) << 4));
            const float r[4] = {r4.x, r4.y, r4.z, r4.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float q = fminf(fmaxf(__builtin_rintf(div_by(r[i], sf, inv_s) + zf), 0.0f), 7.0f);
                const float e = r[i] - sf * (q - zf), ae = fabsf(e);
                const float thr = ae > 0.0f ? __builtin_amdgcn_exp2f(pm1 * __builtin_amdgcn_logf(ae)) * inv_beta : 0.0f;
                const float m = copysignf(fmaxf(ae - thr, 0.0f), e);
                v[i] = q - (r[i] - m) * inv_s;
            }
        }) * (1.0f / 64.0f);
        beta *= kappa;
    }
    read_unit64(area, lane, t);
#pragma unroll
    for (int i = 0; i < 64; ++i) t[i] = fminf(fmaxf(__builtin_rintf(div_by(t[i], sf, inv_s) + zf), 0.0f), 7.0f);
    if (!FIRST) {                                   // the area holds R
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        stage_row_block(W, K, n0, N, g0, K, area, lane);
        wait_vmem();
    }
#pragma unroll
    for (int c = 0; c < 16; ++c) {
        float4* const at = reinterpret_cast<float4*>(area + row * 1024 + gl * 256 + ((c ^ row) << 4));
        const float4 w = *at;
        *at = float4{w.x - sf * (t[4 * c] - zf), w.y - sf * (t[4 * c + 1] - zf), w.z - sf * (t[4 * c + 2] - zf),
                     w.w - sf * (t[4 * c + 3] - zf)};
    }
    if (live) z[gu] = zf;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    // out again as whole rows: lane l carries segment l % 16 of group l / 16
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const float4 v = *reinterpret_cast<const float4*>(area + i * 1024 + gl * 256 + ((row ^ i) << 4));
        if (live) *reinterpret_cast<float4*>(RE + (n0 + i) * K + (g0 + gl) * kGroup + 4 * row) = v;
    }
}

// The same for few groups (kHqqFewUnits): 16 lanes per group, four targets each, the shrinkage always evaluated.  Bit for
// bit the same: the mean is summed in the same order, and where the kernel above leaves the shrinkage out it is zero.
constexpr int kHqqFewThreads = 256, kHqqFewPerBlock = kHqqFewThreads / 16;
template <bool FIRST>
__global__ __launch_bounds__(kHqqFewThreads) void hqq_few_kernel(const float* __restrict__ W, float* __restrict__ RE, float* __restrict__ s,
                                                                 float* __restrict__ z, int64_t units, int iters, float pm1, float beta,
                                                                 float kappa) {
    const int64_t gu = (int64_t)blockIdx.x * kHqqFewPerBlock + (threadIdx.x >> 4);
    const int l16 = threadIdx.x & 15;
    if (gu >= units) return;                        // whole 16-lane groups leave together
    const int64_t at = gu * kGroup + 4 * l16;
    const float4 w4 = *reinterpret_cast<const float4*>(W + at);
    const float4 r4 = FIRST ? w4 : *reinterpret_cast<const float4*>(RE + at);
    const float w[4] = {w4.x, w4.y, w4.z, w4.w}, r[4] = {r4.x, r4.y, r4.z, r4.w};
    float sf, zf;
    if (FIRST) {
        float mn = fminf(fminf(w[0], w[1]), fminf(w[2], w[3])), mx = fmaxf(fmaxf(w[0], w[1]), fmaxf(w[2], w[3]));
#pragma unroll
        for (int m = 1; m < 16; m <<= 1) {
            mn = fminf(mn, __shfl_xor(mn, m, 16));
            mx = fmaxf(mx, __shfl_xor(mx, m, 16));
        }
        sf = (float)(f16)((mx - mn) / 7.0f);
        if (!(sf > 0.0f && sf <= 65504.0f)) sf = 1.0f;
        zf = (-mn) / sf;
        if (l16 == 0) s[gu] = sf;
    } else {
        sf = s[gu];
        zf = z[gu];
    }
    const float inv_s = 1.0f / sf;
    auto code = [&](int i) { return fminf(fmaxf(__builtin_rintf(r[i] / sf + zf), 0.0f), 7.0f); };
    for (int it = 0; it < iters; ++it) {
        const float inv_beta = 1.0f / beta;
        float v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float q = code(i), e = r[i] - sf * (q - zf), ae = fabsf(e);
            const float thr = ae > 0.0f ? __builtin_amdgcn_exp2f(pm1 * __builtin_amdgcn_logf(ae)) * inv_beta : 0.0f;
            const float m = copysignf(fmaxf(ae - thr, 0.0f), e);
            v[i] = q - (r[i] - m) * inv_s;
        }
        float sum = ((v[0] + v[1]) + v[2]) + v[3];
#pragma unroll
        for (int m = 1; m < 16; m <<= 1) sum += __shfl_xor(sum, m, 16);
        zf = sum * (1.0f / 64.0f);
        beta *= kappa;
    }
    float e[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) e[i] = w[i] - sf * (code(i) - zf);
    *reinterpret_cast<float4*>(RE + at) = float4{e[0], e[1], e[2], e[3]};
    if (l16 == 0) z[gu] = zf;
}
// Up to here the chip has lanes to spare and the longest chain counts.  One outer iteration at rank 0, us, 16 lanes / one:
// 512 x 512 (4096 groups) 39 / 50, 768 x 1024 (12288) 46 / 49, 1024 x 1024 (16384) 49.6 / 49.5, 1024 x 1536 57 / 53.
constexpr int64_t kHqqFewUnits = 16384;

// ------------------------------------------------------------------ In - U V: the new target, its norm, the codes
// A wave computes 16 rows x 64 columns of U V with 16x16x4 fp32 MFMAs at a time.  Column tile c (of four) is
// made of the columns 4 i + c, so that lane (i, k) of the result holds 4 consecutive columns of row 4 k + v and
// In is read and written as whole 256-byte row pieces.  U rows of the wave wait in LDS (row length r + 1: the
// 16 rows of a fragment lie on different banks).
//   RESID_TARGET: Out = In - U V.   RESID_NORM: fp64 sum of squares of In - U V to partial[workgroup].
//   RESID_PACK: codes of In - U V with the given scales and z rounded to fp16, packed (Section 3.3).
// Bound by HBM: In is read once (and written once).  14336 x 4096, r = 32: 66 us for the norm (80 on the
// vector units), 105 us for target and packing in one pass (177 as two kernels).
enum { RESID_TARGET = 0, RESID_NORM = 1, RESID_PACK = 2 };
constexpr int kResidCols = 256;        // columns of a wave's work item
typedef f32x4 Tile4[4];

__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

template <int MODE>
__global__ __launch_bounds__(256, 2) void resid_kernel(const float* __restrict__ In, const float* __restrict__ U,
                                                    const float* __restrict__ V, int r, int64_t N, int64_t K, float* __restrict__ Out,
                                                    double* __restrict__ partial, const float* __restrict__ s, const float* __restrict__ z,
                                                    uint32_t* __restrict__ planeA, uint32_t* __restrict__ planeB) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, i = lane & 15, kq = lane >> 4;
    const int64_t G = K / kGroup;
    // RESID_PACK: the wave's 16 rows x 256 columns of the target, swizzled as stage_row_block does
    unsigned char* const area = lds_raw + wave * kRowBlockBytes;
    float* const Us = reinterpret_cast<float*>(lds_raw + (MODE == RESID_PACK ? 4 * kRowBlockBytes : 0));     // [16][r + 1]
    // blockIdx.x: 16 rows; blockIdx.y: a share of the 256-column items, dealt to the four waves
    const int64_t n0 = (int64_t)blockIdx.x * 16;
    const int ldu = r + 1;
    const int64_t items = (K + kResidCols - 1) / kResidCols;
    double sq = 0.0;
    // a pack wave has few neighbours on its CU (LDS), so it requests its next item while it forms the codes of the last
    constexpr int AHEAD = MODE == RESID_PACK ? 4 : 1;
    float4 all[AHEAD][4];
    auto column = [&](int64_t c0, int sub) { return c0 + 64 * sub < K ? c0 + 64 * sub + 4 * i : c0 + 4 * i; };   // (past K: anywhere)
    auto load_in = [&](int64_t c0, int sub, float4 (&in)[4]) {
#pragma unroll
        for (int v = 0; v < 4; ++v) in[v] = *reinterpret_cast<const float4*>(In + (n0 + 4 * kq + v) * K + column(c0, sub));
    };
    auto load_item = [&](int64_t it) {
        if (AHEAD == 4 && it < items) {
#pragma unroll
            for (int sub = 0; sub < AHEAD; ++sub) load_in(it * kResidCols, sub, all[sub]);
        }
    };
    load_item((int64_t)blockIdx.y * 4 + wave);
    for (int e = tid; e < 16 * r; e += 256) Us[(e / r) * ldu + e % r] = U[n0 * r + e];
    __syncthreads();
    for (int64_t it = (int64_t)blockIdx.y * 4 + wave; it < items; it += (int64_t)gridDim.y * 4) {
        const int64_t c0 = it * kResidCols;
        // SUBS sub-tiles at a time: a pack wave takes all four, so that V costs it one round trip per 16 ranks and item
        constexpr int SUBS = AHEAD;
#pragma unroll
        for (int sub0 = 0; sub0 < 4; sub0 += SUBS) {
            if (c0 + 64 * sub0 >= K) break;
            if (AHEAD == 1) load_in(c0, sub0, all[0]);
            Tile4 acc[SUBS];
#pragma unroll
            for (int u = 0; u < SUBS; ++u)
#pragma unroll
                for (int c = 0; c < 4; ++c) acc[u][c] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            for (int k0 = 0; k0 < r; k0 += 16) {           // sixteen ranks' loads at once
                float a[4];
                float4 b[SUBS][4];
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const int k = k0 + 4 * x + kq, kc = k < r ? k : r - 1;          // (past the rank: a = 0)
#pragma unroll
                    for (int u = 0; u < SUBS; ++u)
                        b[u][x] = *reinterpret_cast<const float4*>(V + (int64_t)kc * K + column(c0, sub0 + u));
                    a[x] = Us[i * ldu + kc];
                    if (k >= r) a[x] = 0.0f;
                }
#pragma unroll
                for (int u = 0; u < SUBS; ++u)
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        acc[u][0] = mfma_f32(a[x], b[u][x].x, acc[u][0]);
                        acc[u][1] = mfma_f32(a[x], b[u][x].y, acc[u][1]);
                        acc[u][2] = mfma_f32(a[x], b[u][x].z, acc[u][2]);
                        acc[u][3] = mfma_f32(a[x], b[u][x].w, acc[u][3]);
                    }
            }
#pragma unroll
            for (int u = 0; u < SUBS; ++u)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float4 in = all[u][v];
                    const float4 o = {in.x - acc[u][0][v], in.y - acc[u][1][v], in.z - acc[u][2][v], in.w - acc[u][3][v]};
                    if (MODE == RESID_TARGET) *reinterpret_cast<float4*>(Out + (n0 + 4 * kq + v) * K + column(c0, sub0 + u)) = o;
                    if (MODE == RESID_NORM) sq += (double)o.x * o.x + (double)o.y * o.y + (double)o.z * o.z + (double)o.w * o.w;
                    if (MODE == RESID_PACK) {
                        const int row = 4 * kq + v;
                        *reinterpret_cast<float4*>(area + row * 1024 + (sub0 + u) * 256 + ((i ^ row) << 4)) = o;
                    }
                }
        }
        if (MODE == RESID_PACK) {
            load_item(it + (int64_t)gridDim.y * 4);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");          // (the area is this wave's own)
            const int64_t g0 = c0 / kGroup;
            if (g0 + kq < G) {
                float q[64];
                read_unit64(area, lane, q);
                const int64_t gu = (n0 + i) * G + g0 + kq;
                const float sf = s[gu], inv_s = 1.0f / sf;
                const f16 z16 = (f16)fminf(fmaxf(z[gu], -65504.0f), 65504.0f);
#pragma unroll
                for (int e = 0; e < 64; ++e)
                    q[e] = fminf(fmaxf(__builtin_rintf(div_by_any(q[e], sf, inv_s) + (float)z16), 0.0f), 7.0f);
                uint32_t d[6];
                unit_words(q, d);
                store_row_block_unit(d, scale_zero_word((f16)sf, z16), ((n0 >> 4) * G + g0) * 16 + lane, planeA, planeB);
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        }
    }
    if (MODE == RESID_NORM) {
        __shared__ double red[4];
#pragma unroll
        for (int m = 1; m < 64; m <<= 1) sq += __shfl_xor(sq, m, 64);
        if (lane == 0) red[wave] = sq;
        __syncthreads();
        if (tid == 0) partial[(int64_t)blockIdx.x * gridDim.y + blockIdx.y] = ((red[0] + red[1]) + (red[2] + red[3]));
    }
}

__global__ __launch_bounds__(kSmallThreads) void sum_partials_kernel(const double* __restrict__ partial, int64_t count,
                                                                     double* __restrict__ out) {
    __shared__ double red[kSmallThreads];
    double a = 0.0;
    for (int64_t i = threadIdx.x; i < count; i += kSmallThreads) a += partial[i];
    red[threadIdx.x] = a;
    __syncthreads();
    for (int h = kSmallThreads / 2; h > 0; h >>= 1) {
        if (threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = red[0];
}

__device__ __forceinline__ float4 add4(float4 a, float4 b) { return float4{a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w}; }
// sum of S parts of four consecutive floats, sixteen loads in flight
__device__ __forceinline__ float4 sum_parts4(const float* __restrict__ at, int S, int64_t stride) {
    float4 a = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int z0 = 0; z0 < S; z0 += 16) {
        float4 v[16];
#pragma unroll
        for (int z = 0; z < 16; ++z) v[z] = *reinterpret_cast<const float4*>(at + (int64_t)(z0 + z < S ? z0 + z : z0) * stride);
#pragma unroll
        for (int z = 0; z < 16; ++z)
            if (z0 + z < S) a = add4(a, v[z]);
    }
    return a;
}

// ------------------------------------------------------------------ the inverse Cholesky factor of a small Gram matrix (one workgroup)
// A chain of l dependent steps; what a step costs is its barrier and LDS round trips, so the update is one sweep
// over the matrix between two barriers.
// Rows and columns below n of the sum of the parts [ld x ld] to LDS, row length w.
template <int THREADS>
__device__ __forceinline__ void load_gram(const float* __restrict__ Gp, int parts, int ld, int n, float* lds, int w) {
    const int quads = ld / 4;
    for (int e = threadIdx.x; e < n * quads; e += THREADS) {
        const int i = e / quads, j = 4 * (e % quads);
        if (j >= n) continue;
        const float4 a = sum_parts4(Gp + (int64_t)i * ld + j, parts, (int64_t)ld * ld);
        lds[i * w + j] = a.x;
        if (j + 1 < n) lds[i * w + j + 1] = a.y;
        if (j + 2 < n) lds[i * w + j + 2] = a.z;
        if (j + 3 < n) lds[i * w + j + 3] = a.w;
    }
}

// Gm = sum of the parts, [l x l] symmetric positive definite (a Gram matrix Y^T Y) = L L^T.  Writes Linv = L^-1
// (lower triangular, dense, row length l), so that Q = Y Linv^T has orthonormal columns.  Elimination on [Gm | 1]: after
// step j the right half of row i > j holds the multipliers of the rows eliminated so far; row i leaves scaled by
// the root of its pivot.  A pivot that is not safely positive (a rank-deficient sketch) is replaced by a small
// multiple of the mean diagonal: the result stays finite and the directions concerned carry no weight in the
// later steps.  l = 40: 19 us, with three barriers per column and a substitution by single threads 62.
__device__ __forceinline__ void cholesky_inverse(const float* __restrict__ Gp, int parts, int ld, int l, float* __restrict__ Linv,
                                                 float* lds) {
    const int w = 2 * l + 1;
    float* const A = lds;                          // [l][2 l + 1]
    const int tid = threadIdx.x;
    const int col = tid % l, row0 = tid / l, rows = kSmallThreads / l;
    const bool on = row0 < rows;
    load_gram<kSmallThreads>(Gp, parts, ld, l, A, w);
    if (on)
        for (int i = row0; i < l; i += rows) A[i * w + l + col] = i == col ? 1.0f : 0.0f;
    __syncthreads();
    float tr = 0.0f;
    for (int i = 0; i < l; ++i) tr += A[i * w + i];
    const float floor_pivot = fmaxf(tr / (float)l * 1e-10f, 1e-37f);
    __syncthreads();
    for (int j = 0; j < l; ++j) {
        const float rd = __builtin_amdgcn_rcpf(fmaxf(A[j * w + j], floor_pivot));
        const int at = col > j ? col : l + col;    // row j is non-zero in the columns above j and l .. l + j
        const float top = A[j * w + at];
        if (on)
            for (int i = j + 1 + row0; i < l; i += rows) A[i * w + at] -= A[i * w + j] * rd * top;
        __syncthreads();
    }
    if (on)
        for (int i = row0; i < l; i += rows) {
            const float d = fmaxf(A[i * w + i], floor_pivot);
            Linv[i * l + col] = col <= i ? A[i * w + l + col] / sqrtf(d) : 0.0f;
        }
}

__global__ __launch_bounds__(kSmallThreads) void cholesky_inverse_kernel(const float* __restrict__ Gp, int parts, int ld, int l,
                                                                         float* __restrict__ Linv) {
    extern __shared__ __attribute__((aligned(16))) float lds[];
    cholesky_inverse(Gp, parts, ld, l, Linv, lds);
}

// ------------------------------------------------------------------ the two passes over E
// Rows and columns of the sketch are padded with zeros to ld = 16 ceil(l / 16).
//
// Y = E Vb^T, [N x ld], as the sum of parts over K.  A workgroup takes 64 rows (16 per wave), the RB rank tiles
// from 16 RB blockIdx.z on and the share blockIdx.y of the 64-column chunks.  Lane (i, k) reads E[row i][16 c + 4 k ..
// + 3], four steps of 16 columns per chunk; the basis chunk goes through LDS ([16 RB rows][64], double
// buffered, segment p of row j at p ^ (j % 16)), read in the same order of k, which is a permutation both
// operands share.
template <int RB>
__global__ __launch_bounds__(256) void sketch_y_kernel(const float* __restrict__ E, const float* __restrict__ Vb, int64_t N, int64_t K,
                                                       int ld, int splits, float* __restrict__ Yp) {
    __shared__ __attribute__((aligned(16))) unsigned char basis[2][RB * 16 * 256];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, i = lane & 15, kq = lane >> 4;
    const int64_t n0 = (int64_t)blockIdx.x * 64 + 16 * wave;
    const int j0 = (int)blockIdx.z * 16 * RB;
    const int chunks = (int)(K / 64), per = (chunks + splits - 1) / splits;
    const int c_lo = (int)blockIdx.y * per, c_hi = c_lo + per < chunks ? c_lo + per : chunks;
    const bool mine = n0 < N;
    const float* const erow = E + (mine ? n0 + i : 0) * K + 4 * kq;
    // copy x of the wave: 4 basis rows, 256 bytes each
    auto stage = [&](int c, int b) {
#pragma unroll
        for (int x = 0; x < RB; ++x) {
            const int r4 = j0 + 4 * (wave * RB + x), rl = 4 * (wave * RB + x) + (lane >> 4);
            const BufRsrc vb = make_rsrc(Vb + (int64_t)r4 * K, r4 < ld ? (uint64_t)K * 16u : 0u);      // (rows past ld read as zero)
            const uint32_t o = ((uint32_t)(lane >> 4) * (uint32_t)K + (uint32_t)c * 64u) * 4u + (uint32_t)(((lane & 15) ^ (rl & 15)) << 4);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(vb, (PackLdsPtr)(&basis[b][(wave * RB + x) * 1024]), 16, o, 0, 0, 0);
        }
    };
    f32x4 acc[RB];
#pragma unroll
    for (int x = 0; x < RB; ++x) acc[x] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    float4 e[4], nx[4];
    if (c_lo < c_hi) {
        stage(c_lo, 0);
#pragma unroll
        for (int x = 0; x < 4; ++x) e[x] = *reinterpret_cast<const float4*>(erow + (int64_t)c_lo * 64 + 16 * x);
    }
    for (int c = c_lo; c < c_hi; ++c) {
        const int b = (c - c_lo) & 1;
        wait_vmem();
        __syncthreads();
        const int cn = c + 1 < c_hi ? c + 1 : c;
        if (c + 1 < c_hi) stage(cn, b ^ 1);
#pragma unroll
        for (int x = 0; x < 4; ++x) nx[x] = *reinterpret_cast<const float4*>(erow + (int64_t)cn * 64 + 16 * x);
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            float4 v[RB];
#pragma unroll
            for (int y = 0; y < RB; ++y)
                v[y] = *reinterpret_cast<const float4*>(&basis[b][(16 * y + i) * 256 + (((4 * x + kq) ^ i) << 4)]);
#pragma unroll
            for (int y = 0; y < RB; ++y) acc[y] = mfma_f32(e[x].x, v[y].x, acc[y]);
#pragma unroll
            for (int y = 0; y < RB; ++y) acc[y] = mfma_f32(e[x].y, v[y].y, acc[y]);
#pragma unroll
            for (int y = 0; y < RB; ++y) acc[y] = mfma_f32(e[x].z, v[y].z, acc[y]);
#pragma unroll
            for (int y = 0; y < RB; ++y) acc[y] = mfma_f32(e[x].w, v[y].w, acc[y]);
        }
#pragma unroll
        for (int x = 0; x < 4; ++x) e[x] = nx[x];
    }
    if (!mine) return;
    float* const out = Yp + (int64_t)blockIdx.y * N * ld;
#pragma unroll
    for (int y = 0; y < RB; ++y)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (j0 + 16 * y < ld) out[(n0 + 4 * kq + v) * ld + j0 + 16 * y + i] = acc[y][v];
}

// Y^T E, [ld x K], as the sum of parts over N.  A workgroup takes 256 columns (a contiguous KB of every row: with 64
// columns per workgroup the rows, 16 KB apart, met on few memory channels and the pass took 112 us), the RB rank
// tiles from 16 RB blockIdx.z on and the share blockIdx.y of the 16-row blocks.  Wave w takes columns
// 64 (w % 4) .. and every second block from w / 4 on; the two sums meet in LDS.  Lane (i, k) reads
// E[row k][4 i .. 4 i + 3]: one 16-byte load carries the B operands of four column tiles (tile c = columns 4 i + c) for a
// step of four rows; the A operand is Y[row k][rank i].
// One more workgroup (blockIdx.x = 0) factors Y^T Y meanwhile: its result is
// needed after this pass, and 20 us of a single workgroup would be idle time of all others.
template <int RB>
__global__ __launch_bounds__(kSmallThreads) void sketch_b_kernel(const float* __restrict__ E, const float* __restrict__ Y, int64_t N,
                                                                 int64_t K, int ld, int splits, float* __restrict__ Bp,
                                                                 const float* __restrict__ Gp, int gram_parts, int l,
                                                                 float* __restrict__ Linv) {
    extern __shared__ __attribute__((aligned(16))) float sketch_lds[];
    if (blockIdx.x == 0) {
        if (blockIdx.y == 0 && blockIdx.z == 0) cholesky_inverse(Gp, gram_parts, ld, l, Linv, sketch_lds);
        return;
    }
    f32x4 (*const red)[RB * 4 * 64] = reinterpret_cast<f32x4 (*)[RB * 4 * 64]>(sketch_lds);
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, i = lane & 15, kq = lane >> 4;
    const int cw = wave & 3, rw = wave >> 2;
    const int64_t c0 = (int64_t)(blockIdx.x - 1) * 256 + 64 * cw;
    const bool mine = c0 < K;
    const int j0 = (int)blockIdx.z * 16 * RB;
    const int blocks = (int)(N / 16), per = (blocks + splits - 1) / splits;
    const int b_lo = (int)blockIdx.y * per, b_hi = b_lo + per < blocks ? b_lo + per : blocks;
    Tile4 acc[RB];
#pragma unroll
    for (int y = 0; y < RB; ++y)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[y][c] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    float4 e[4], ne[4];
    float a[4][RB], na[4][RB];
    const float* const ep = E + (mine ? c0 : 0) + 4 * i + kq * K;
    const float* const yp = Y + j0 + i + kq * ld;
    auto load = [&](int b, float4 (&ev)[4], float (&av)[4][RB]) {
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const int64_t n = (int64_t)b * 16 + 4 * x;
            ev[x] = *reinterpret_cast<const float4*>(ep + n * K);
#pragma unroll
            for (int y = 0; y < RB; ++y) av[x][y] = j0 + 16 * y < ld ? yp[n * ld + 16 * y] : 0.0f;
        }
    };
    const int b0 = b_lo + rw;
    if (b0 < b_hi) load(b0, e, a);
    for (int b = b0; b < b_hi; b += 2) {
        load(b + 2 < b_hi ? b + 2 : b, ne, na);
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
            for (int y = 0; y < RB; ++y) {
                acc[y][0] = mfma_f32(a[x][y], e[x].x, acc[y][0]);
                acc[y][1] = mfma_f32(a[x][y], e[x].y, acc[y][1]);
                acc[y][2] = mfma_f32(a[x][y], e[x].z, acc[y][2]);
                acc[y][3] = mfma_f32(a[x][y], e[x].w, acc[y][3]);
            }
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            e[x] = ne[x];
#pragma unroll
            for (int y = 0; y < RB; ++y) a[x][y] = na[x][y];
        }
    }
    if (rw > 0) {
#pragma unroll
        for (int y = 0; y < RB; ++y)
#pragma unroll
            for (int c = 0; c < 4; ++c) red[cw][(4 * y + c) * 64 + lane] = acc[y][c];
    }
    __syncthreads();
    if (rw > 0 || !mine) return;
    float* const out = Bp + (int64_t)blockIdx.y * ld * K;
#pragma unroll
    for (int y = 0; y < RB; ++y) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const f32x4 p = red[cw][(4 * y + c) * 64 + lane];
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[y][c][v] += p[v];
        }
        if (j0 + 16 * y >= ld) continue;
#pragma unroll
        for (int v = 0; v < 4; ++v)
            *reinterpret_cast<float4*>(out + (int64_t)(j0 + 16 * y + 4 * kq + v) * K + c0 + 4 * i) =
                float4{acc[y][0][v], acc[y][1][v], acc[y][2][v], acc[y][3][v]};
    }
}

// ------------------------------------------------------------------ small products around them
// These move a few megabytes and do little arithmetic: what they cost is memory round trips, so every thread has
// all its loads of a step in flight at once (16 bytes each) and the products run on the matrix cores from LDS.
// Y = sum of its parts, and this workgroup's share (kGramRows rows) of the Gram matrix Y^T Y.
constexpr int kGramRows = 256, kGramStep = 128, kGramThreads = 1024;
static_assert((kSketchMax + 15) / 16 == 9, "81 tiles at most: 6 per wave");

template <int PERW>                                 // tiles of the Gram matrix per wave
__global__ __launch_bounds__(kGramThreads) void gram_rows_kernel(const float* __restrict__ Yp, int splits, int64_t N, int ld,
                                                                 float* __restrict__ Y, float* __restrict__ Gp) {
    extern __shared__ float rows[];                 // [kGramStep][ld + 1]
    const int tid = threadIdx.x, lds_ld = ld + 1, quads = ld / 4;
    const int64_t n_lo = (int64_t)blockIdx.x * kGramRows, n_hi = n_lo + kGramRows < N ? n_lo + kGramRows : N;
    // 16 x 16 tiles of the Gram matrix, dealt to the waves; lane (i, k): D rows 4 k + v, column i
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, i = lane & 15, kq = lane >> 4;
    const int rt = ld / 16, tiles = rt * rt;
    f32x4 acc[PERW];
#pragma unroll
    for (int x = 0; x < PERW; ++x) acc[x] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    for (int64_t n = n_lo; n < n_hi; n += kGramStep) {
        const int cnt = (int)(n_hi - n < kGramStep ? n_hi - n : kGramStep) * quads;
        for (int e = tid; e < kGramStep * quads; e += kGramThreads) {
            float4 a = {0.0f, 0.0f, 0.0f, 0.0f};
            if (e < cnt) {
                a = sum_parts4(Yp + n * ld + 4 * e, splits, N * ld);
                *reinterpret_cast<float4*>(Y + n * ld + 4 * e) = a;
            }
            float* const at = rows + (e / quads) * lds_ld + 4 * (e % quads);
            at[0] = a.x; at[1] = a.y; at[2] = a.z; at[3] = a.w;
        }
        __syncthreads();
#pragma unroll
        for (int x = 0; x < PERW; ++x) {
            const int t = wave + 16 * x;
            if (t < tiles) {
                const int ta = (t / rt) * 16 + i, tb = (t % rt) * 16 + i;
#pragma unroll 8
                for (int k = 0; k < kGramStep; k += 4)
                    acc[x] = mfma_f32(rows[(k + kq) * lds_ld + ta], rows[(k + kq) * lds_ld + tb], acc[x]);
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int x = 0; x < PERW; ++x) {
        const int t = wave + 16 * x;
        if (t < tiles)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                Gp[((int64_t)blockIdx.x * ld + (t / rt) * 16 + 4 * kq + v) * ld + (t % rt) * 16 + i] = acc[x][v];
    }
}

// Out [rows_out x K] = M [rows_out x l] (sum of the S parts of In [ld x K]), 64 columns per workgroup; rows from
// rows_out to the next multiple of 16 are written as zeros if they are below ld_out.  With Gp also this
// workgroup's share of Out Out^T [ld_out x ld_out].
constexpr int kLeftThreads = 512;
__global__ __launch_bounds__(kLeftThreads) void apply_left_kernel(const float* __restrict__ M, int rows_out, int ld_out, int l,
                                                                  const float* __restrict__ In, int S, int64_t part_stride, int64_t K,
                                                                  float* __restrict__ Out, float* __restrict__ Gp) {
    extern __shared__ float sm[];
    const int lk = (l + 3) & ~3, tiles_out = (ld_out + 15) / 16;
    constexpr int LDB = 65;
    float* const Bs = sm;                           // [lk][64 + 1]
    float* const Os = Bs + lk * LDB;                // [16 tiles_out][64 + 1]
    float* const Ms = Os + 16 * tiles_out * LDB;    // [16 tiles_out][lk + 1], zeros past rows_out and l
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, i = lane & 15, kq = lane >> 4;
    constexpr int WAVES = kLeftThreads / 64;
    const int64_t c0 = (int64_t)blockIdx.x * 64;
    for (int e = tid; e < lk * 16; e += kLeftThreads) {
        const int k = e >> 4, j = 4 * (e & 15);
        float4 a = {0.0f, 0.0f, 0.0f, 0.0f};
        if (k < l) a = sum_parts4(In + (int64_t)k * K + c0 + j, S, part_stride);
        float* const at = Bs + k * LDB + j;
        at[0] = a.x; at[1] = a.y; at[2] = a.z; at[3] = a.w;
    }
    for (int e = tid; e < 16 * tiles_out * lk; e += kLeftThreads) {
        const int n = e / lk, k = e % lk;
        Ms[n * (lk + 1) + k] = n < rows_out && k < l ? M[n * l + k] : 0.0f;
    }
    __syncthreads();
    // 16 x 16 tiles (row tile t / 4, column tile t % 4)
    for (int t = wave; t < 4 * tiles_out; t += WAVES) {
        const int row = (t >> 2) * 16 + i, j = (t & 3) * 16 + i;
        f32x4 o = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 4
        for (int k = kq; k < lk; k += 4) o = mfma_f32(Ms[row * (lk + 1) + k], Bs[k * LDB + j], o);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int n = (t >> 2) * 16 + 4 * kq + v;
            if (n < ld_out) Out[(int64_t)n * K + c0 + j] = o[v];
            Os[n * LDB + j] = o[v];
        }
    }
    if (!Gp) return;
    __syncthreads();
    for (int t = wave; t < tiles_out * tiles_out; t += WAVES) {
        const int ta = (t / tiles_out) * 16, tb = (t % tiles_out) * 16;
        f32x4 g = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 8
        for (int k = 0; k < 64; k += 4) g = mfma_f32(Os[(ta + i) * LDB + k + kq], Os[(tb + i) * LDB + k + kq], g);
#pragma unroll
        for (int v = 0; v < 4; ++v) Gp[((int64_t)blockIdx.x * ld_out + ta + 4 * kq + v) * ld_out + tb + i] = g[v];
    }
}

// U [N x r] = Y [N x ld] P [l x r], 64 rows per workgroup.
__global__ __launch_bounds__(256) void apply_right_kernel(const float* __restrict__ Y, int ld, int l, const float* __restrict__ P, int r,
                                                          int64_t N, float* __restrict__ U) {
    extern __shared__ float sm[];
    float* const Ps = sm;                           // [l][r]
    float* const Ys = sm + l * r;                   // [64][l + 1]
    const int tid = threadIdx.x;
    const int64_t n0 = (int64_t)blockIdx.x * 64;
    const int rows = N - n0 < 64 ? (int)(N - n0) : 64;
    for (int e = tid; e < l * r; e += 256) Ps[e] = P[e];
    for (int e = tid; e < rows * l; e += 256) Ys[(e / l) * (l + 1) + e % l] = Y[(n0 + e / l) * ld + e % l];
    __syncthreads();
    for (int e = tid; e < rows * r; e += 256) {
        const int n = e / r, j = e % r;
        float a = 0.0f;
        for (int k = 0; k < l; ++k) a = fmaf(Ys[n * (l + 1) + k], Ps[k * r + j], a);
        U[n0 * r + e] = a;
    }
}

// Uniform numbers in (-1, 1) from a counter hash: the starting basis of the subspace iteration (zeros from
// element `live` on: the padding rows).
__global__ __launch_bounds__(256) void random_basis_kernel(float* __restrict__ out, int64_t count, int64_t live, uint32_t seed) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= count) return;
    uint32_t h = (uint32_t)i * 0x9E3779B1u + seed;
    h ^= (uint32_t)(i >> 32) * 0x85EBCA77u;
    h ^= h >> 16; h *= 0x7FEB352Du;
    h ^= h >> 15; h *= 0x846CA68Bu;
    h ^= h >> 16;
    out[i] = i < live ? ((float)(h >> 8) + 0.5f) * (1.0f / 8388608.0f) - 1.0f : 0.0f;
}

// ------------------------------------------------------------------ eigenvectors of the small Gram matrix
// (p, q) turned by the angle with sine s and half-angle tangent h: cos = 1 - s h is not formed, so a small angle takes
// nothing from the length of (p, q) by the rounding of its cosine.
__device__ __forceinline__ void turn(float& p, float& q, float s, float h) {
    const float p0 = p;
    p = fmaf(-s, fmaf(h, p0, q), p0);
    q = fmaf(s, fmaf(-h, q, p0), q);
}

// Gm = sum of the parts, [l x l] symmetric (B B^T) = Ub diag(lambda) Ub^T by cyclic Jacobi rotations, l / 2 disjoint
// pairs per step in round-robin order, at most `sweeps` sweeps (fewer when they have converged).  With
// sigma = sqrt(lambda) sorted descending it writes Vm [r x l] = sigma_r^(-1/2) Ub_r^T, Wm [l x l] = sigma^-1 Ub^T (rows
// whose sigma is negligible are zero) and P [l x r] = Linv^T Ub_r sigma_r^(1/2), so that U = Y P.
//
// The two players of pair m sit on rows (columns) 2 m and 2 m + 1, and a step moves everyone to the seat of the next
// step as it writes: the blocks J1^T A J2 it works on (pair x pair, rows and columns at once) are read as aligned
// 8-byte pieces without bank conflicts.  After the n - 1 steps of a sweep all sit where they began.  Lane m of
// a wave (of each of its `subs` parts) owns column pair m: it works out that pair's rotation itself, gets the one of
// its row pair from another lane, and so nothing but the matrix itself crosses waves; with two copies of the
// matrix (TWO, as long as they fit) a step costs one barrier.  PASSES: column pairs per lane (more than 64 pairs).
// l = 40: 171 us; with three barriers per step (rotations, columns, rows) and scattered reads 555.
// THREADS: a step is bound by instructions, many of them the same in every wave (the rotations), so up to three
// row-pair rounds of a 40-wide matrix eight waves are faster than sixteen, and slower on larger ones.
template <int THREADS, int PASSES, bool TWO>
__global__ __launch_bounds__(THREADS) void jacobi_factors_kernel(const float* __restrict__ Gp, int parts, int ld, int l, int r,
                                                                        int sweeps, const float* __restrict__ Linv,
                                                                        float* __restrict__ P, float* __restrict__ Vm,
                                                                        float* __restrict__ Wm) {
    extern __shared__ float lds[];
    constexpr int WAVES = THREADS / 64;
    constexpr int ROUNDS = THREADS == 512 ? 2 : PASSES == 1 ? 4 : 5;      // row pairs of a wave: at most 24 / 16, 64 / 16 or 68 / 16
    const int n = (l + 1) & ~1;            // players of the round-robin; for an odd l the last one is a zero row
    const int half = n / 2, w = n + 2;
    float* const Ev = lds;                 // eigenvectors in columns
    float* A = lds + n * w;                // [n][w]
    float* B = TWO ? lds + 2 * n * w : A;  // where a step writes
    __shared__ float lam[kSketchMax];
    __shared__ int place[kSketchMax];
    __shared__ int again[2];
    __shared__ float top;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    for (int e = tid; e < n * n; e += THREADS) {
        const int i = e / n, j = e % n;
        if (i >= l || j >= l) A[i * w + j] = 0.0f;
        Ev[i * w + j] = i == j ? 1.0f : 0.0f;
    }
    load_gram<THREADS>(Gp, parts, ld, l, A, w);
    if (tid < 2) again[tid] = 0;
    __syncthreads();
    const int subs = PASSES == 1 ? 64 / half : 1;
    const int sub = lane / half < subs ? lane / half : subs - 1, m = lane - sub * half;
    const bool on = m < half;
    const int stride = WAVES * subs, first = wave * subs + sub;
    // next seats of the players of pair x: the upper ones move up a pair, the lower ones down, seat 0 stays
    auto next_upper = [&](int x) { return x == 0 ? 0 : (x == half - 1 ? n - 1 : 2 * x + 2); };
    auto next_lower = [&](int x) { return x == 0 ? (half > 1 ? 2 : 1) : 2 * x - 1; };
    int at[PASSES], nu[PASSES], nl[PASSES];         // this lane's columns, now and next (pairs past the last one repeat it)
#pragma unroll
    for (int y = 0; y < PASSES; ++y) {
        const int x = m + 64 * y < half ? m + 64 * y : half - 1;
        at[y] = 2 * x;
        nu[y] = next_upper(x);
        nl[y] = next_lower(x);
    }
    for (int sweep = 0; sweep < sweeps; ++sweep) {
        for (int step = 0; step < n - 1; ++step) {
            float s2[PASSES], h2[PASSES];               // sine, tangent of half the angle
#pragma unroll
            for (int y = 0; y < PASSES; ++y) {
                const float2 upper = *reinterpret_cast<const float2*>(A + at[y] * w + at[y]);
                const float app = upper.x, apq = upper.y, aqq = A[(at[y] + 1) * w + at[y] + 1];
                const float mean = __builtin_amdgcn_sqrtf(fabsf(app * aqq));
                const bool rotate = fabsf(apq) > 1e-30f && fabsf(apq) > 6e-8f * mean;
                const float tau = (aqq - app) * 0.5f * __builtin_amdgcn_rcpf(apq);
                const float t = copysignf(__builtin_amdgcn_rcpf(fabsf(tau) + __builtin_amdgcn_sqrtf(fmaf(tau, tau, 1.0f))), tau);
                const float c = __builtin_amdgcn_rsqf(fmaf(t, t, 1.0f));
                s2[y] = rotate ? t * c : 0.0f;
                h2[y] = rotate ? s2[y] * __builtin_amdgcn_rcpf(1.0f + c) : 0.0f;
                if (rotate && (fabsf(t) > 2e-4f || fabsf(apq) > 2e-4f * mean)) again[sweep & 1] = 1;
            }
            float blk[ROUNDS][PASSES][4];
#pragma unroll
            for (int k = 0; k < ROUNDS; ++k) {
                if (wave * subs + k * stride >= half) break;
                const int x = first + k * stride < half ? first + k * stride : half - 1;
                float s1 = __shfl(s2[0], x & 63, 64), h1 = __shfl(h2[0], x & 63, 64);
                if (PASSES == 2) {
                    const float sh = __shfl(s2[PASSES - 1], x & 63, 64), hh = __shfl(h2[PASSES - 1], x & 63, 64);
                    if (x >= 64) { s1 = sh; h1 = hh; }
                }
#pragma unroll
                for (int y = 0; y < PASSES; ++y) {
                    const float2 u = *reinterpret_cast<const float2*>(A + 2 * x * w + at[y]);
                    const float2 v = *reinterpret_cast<const float2*>(A + (2 * x + 1) * w + at[y]);
                    float up = u.x, uq = u.y, vp = v.x, vq = v.y;
                    turn(up, vp, s1, h1);                       // rows: J1^T
                    turn(uq, vq, s1, h1);
                    turn(up, uq, s2[y], h2[y]);                 // columns: J2
                    turn(vp, vq, s2[y], h2[y]);
                    blk[k][y][0] = up;
                    blk[k][y][1] = uq;
                    blk[k][y][2] = vp;
                    blk[k][y][3] = vq;
                }
            }
            if (!TWO) __syncthreads();                  // everyone has read
#pragma unroll
            for (int k = 0; k < ROUNDS; ++k) {
                if (wave * subs + k * stride >= half) break;
                const int x = first + k * stride;
                float* const ru = B + next_upper(x) * w;
                float* const rl = B + next_lower(x) * w;
#pragma unroll
                for (int y = 0; y < PASSES; ++y)
                    if (x < half && on && m + 64 * y < half) {
                        ru[nu[y]] = blk[k][y][0];
                        ru[nl[y]] = blk[k][y][1];
                        rl[nu[y]] = blk[k][y][2];
                        rl[nl[y]] = blk[k][y][3];
                    }
            }
            // rows of Ev: always the same wave's, no one else looks at them
            for (int i = first; i < l; i += stride) {
                float* const ev = Ev + i * w;
                float2 e[PASSES];
#pragma unroll
                for (int y = 0; y < PASSES; ++y) e[y] = *reinterpret_cast<const float2*>(ev + at[y]);
#pragma unroll
                for (int y = 0; y < PASSES; ++y)
                    if (on && m + 64 * y < half) {
                        turn(e[y].x, e[y].y, s2[y], h2[y]);
                        ev[nu[y]] = e[y].x;
                        ev[nl[y]] = e[y].y;
                    }
            }
            __syncthreads();
            if (TWO) { float* const o = A; A = B; B = o; }
        }
        // A rotation leaves products of an angle and an off-diagonal element behind: after a sweep in which
        // all of both were below 2e-4 what is left is below the working precision.
        const int more = again[sweep & 1];
        if (more == 0) break;
        if (tid == 0) again[(sweep + 1) & 1] = 0;
        __syncthreads();
    }
    // order: place[i] = position of eigenvalue i in descending order
    for (int i = tid; i < l; i += THREADS) lam[i] = A[i * w + i];
    __syncthreads();
    for (int i = tid; i < l; i += THREADS) {
        int pos = 0;
        for (int j = 0; j < l; ++j) pos += (lam[j] > lam[i] || (lam[j] == lam[i] && j < i)) ? 1 : 0;
        place[i] = pos;
    }
    if (tid == 0) {
        float t = 0.0f;
        for (int i = 0; i < l; ++i) t = fmaxf(t, lam[i]);
        top = sqrtf(fmaxf(t, 0.0f));
    }
    __syncthreads();
    // A is free now: Ub_r sigma_r^(1/2) in its columns
    for (int e = tid; e < l * l; e += THREADS) {
        const int i = e / l, c = e % l;          // eigenvector c (unsorted), component i
        const int k = place[c];
        const float sg = sqrtf(fmaxf(lam[c], 0.0f));
        const bool live = sg > 1e-7f * top && sg > 0.0f;
        const float u = Ev[i * w + c];
        Wm[k * l + i] = live ? u / sg : 0.0f;
        if (k < r) {
            const float h = sqrtf(sg);
            A[i * w + k] = u * h;
            Vm[k * l + i] = live ? u / h : 0.0f;
        }
    }
    __syncthreads();
    for (int e = tid; e < l * r; e += THREADS) {
        const int i = e / r, k = e % r;
        float a = 0.0f;
        for (int x = i; x < l; ++x) a = fmaf(Linv[x * l + i], A[x * w + k], a);       // (Linv is lower triangular)
        P[e] = a;
    }
}

// ------------------------------------------------------------------ host side
struct CompressLayout {
    int l, ld;                     // width of the sketch; padded to whole 16-rank tiles
    int rb, groups;                // rank tiles per workgroup of the two passes, and how many such groups
    int split_y, split_b;          // parts of Y and of Y^T E
    int gram_parts;                // room for this many partial Gram matrices
    int64_t norm_x;                // workgroups per 16 rows of the residual kernels
    size_t RE, s, z, Vb, Bm, Y, Yp, Bp, Gp, LinvY, LinvB, P, Vm, Wm, partial, eps2, total;
};

static CompressLayout compress_layout(int64_t N, int64_t K, int r) {
    CompressLayout L{};
    int64_t l = (int64_t)r + kSketchExtra;
    if (l > N) l = N;
    if (l > K) l = K;
    if (r == 0) l = 0;
    L.l = (int)l;
    L.ld = (int)((l + 15) / 16 * 16);
    const int tiles = L.ld / 16;
    L.rb = tiles < 4 ? (tiles > 0 ? tiles : 1) : 4;
    L.groups = tiles > 0 ? (tiles + L.rb - 1) / L.rb : 1;
    // Four workgroups of the first pass fit on a CU, one of the second (whose launch has one more, see there): as
    // many parts as fill the chip that way, while a part keeps a few hundred columns (rows) to walk.
    const int64_t cus = device_cus(), wy = ((N + 63) / 64) * L.groups, wb = ((K + 255) / 256) * L.groups;
    int64_t sy = 4 * cus / wy, sb = (cus - 1) / wb;
    if (sy > K / 256) sy = K / 256;
    if (sb > N / 256) sb = N / 256;
    L.split_y = (int)(sy < 1 ? 1 : sy > 16 ? 16 : sy);
    L.split_b = (int)(sb < 1 ? 1 : sb > 32 ? 32 : sb);
    const int64_t gy = (N + kGramRows - 1) / kGramRows, gb = K / 64;
    L.gram_parts = (int)(gy > gb ? gy : gb);
    const int64_t items = (K + kResidCols - 1) / kResidCols;
    L.norm_x = (items + 3) / 4 < 4 ? (items + 3) / 4 : 4;
    const int64_t G = K / kGroup;
    size_t at = 0;
    auto take = [&](size_t bytes) { size_t o = at; at = align_up(at + bytes, 256); return o; };
    const size_t ld = (size_t)L.ld;
    L.RE = take((size_t)N * K * 4);
    L.s = take((size_t)N * G * 4);
    L.z = take((size_t)N * G * 4);
    L.Vb = take(ld * K * 4);
    L.Bm = take(ld * K * 4);
    L.Y = take((size_t)N * ld * 4);
    L.Yp = take((size_t)L.split_y * N * ld * 4);
    L.Bp = take((size_t)L.split_b * ld * K * 4);
    L.Gp = take((size_t)L.gram_parts * ld * ld * 4);
    L.LinvY = take(ld * ld * 4);
    L.LinvB = take(ld * ld * 4);
    L.P = take(ld * (size_t)(r > 0 ? r : 1) * 4);
    L.Vm = take(ld * (size_t)(r > 0 ? r : 1) * 4);
    L.Wm = take(ld * ld * 4);
    L.partial = take((size_t)(N / 16) * L.norm_x * 8);
    L.eps2 = take(8);
    L.total = at;
    return L;
}

static bool compress_shape_ok(int64_t N, int64_t K) {
    return weight_shape_ok(N, K) && N < (int64_t(1) << 24) && K < (int64_t(1) << 24);
}

template <typename F>
static void by_rank_tiles(int rb, F&& f) {
    if (rb == 1) f(std::integral_constant<int, 1>{});
    else if (rb == 2) f(std::integral_constant<int, 2>{});
    else if (rb == 3) f(std::integral_constant<int, 3>{});
    else f(std::integral_constant<int, 4>{});
}

// Sliding-mean stop rule of Eq. stop_condition on the errors so far (the mean of the last three, or of
// as many as there are, against the same mean one iteration earlier).
static bool stop_rule(const double* eps, int count, double tol) {
    if (count < 2) return false;
    auto mean = [&](int lo, int hi) {      // [lo, hi)
        double a = 0.0;
        for (int i = lo; i < hi; ++i) a += eps[i];
        return a / (double)(hi - lo);
    };
    const double cur = mean(count >= 3 ? count - 3 : 0, count);
    const double prev = count >= 4 ? mean(count - 4, count - 1) : mean(0, count - 1);
    return (prev - cur) / prev < tol;
}

}  // namespace milo

using namespace milo;

extern "C" size_t milo_compress_w3lr_workspace(int64_t N, int64_t K, int r) {
    if (!compress_shape_ok(N, K) || r < 0 || r > MILO_COMPRESS_MAX_RANK || r > N || r > K) return 0;
    return compress_layout(N, K, r).total;
}

extern "C" int milo_compress_w3lr(const float* W, int64_t N, int64_t K, const milo_compress_params* prm, void* q3, float* U,
                                  float* V, double* eps, int* iters_run, void* workspace, size_t workspace_bytes,
                                  void* stream) {
    if (!W || !prm || !q3 || !workspace || !eps || !iters_run) return MILO_ERR_NULL;
    const int r = prm->rank;
    if (r < 0 || r > MILO_COMPRESS_MAX_RANK || r > N || r > K) return MILO_ERR_RANK;
    if (r > 0 && (!U || !V)) return MILO_ERR_NULL;
    if (!compress_shape_ok(N, K)) return MILO_ERR_SHAPE;
    if (prm->iters < 1 || prm->hqq_iters < 0 || prm->power_iters < 0 || prm->refine_iters < 0 || !(prm->p > 0.0f && prm->p < 1.0f) ||
        !(prm->beta > 0.0f) || !(prm->kappa > 0.0f))
        return MILO_ERR_SHAPE;
    if (!aligned16(W) || !aligned16(q3) || !aligned16(workspace) || (r > 0 && (!aligned16(U) || !aligned16(V))))
        return MILO_ERR_ALIGN;
    const CompressLayout L = compress_layout(N, K, r);
    if (workspace_bytes < L.total) return MILO_ERR_WORKSPACE;

    hipStream_t st = (hipStream_t)stream;
    char* ws = reinterpret_cast<char*>(workspace);
    float* RE = reinterpret_cast<float*>(ws + L.RE);
    float* s = reinterpret_cast<float*>(ws + L.s);
    float* z = reinterpret_cast<float*>(ws + L.z);
    float* Vb = reinterpret_cast<float*>(ws + L.Vb);
    float* Bm = reinterpret_cast<float*>(ws + L.Bm);
    float* Y = reinterpret_cast<float*>(ws + L.Y);
    float* Yp = reinterpret_cast<float*>(ws + L.Yp);
    float* Bp = reinterpret_cast<float*>(ws + L.Bp);
    float* Gp = reinterpret_cast<float*>(ws + L.Gp);
    float* LinvY = reinterpret_cast<float*>(ws + L.LinvY);
    float* LinvB = reinterpret_cast<float*>(ws + L.LinvB);
    float* P = reinterpret_cast<float*>(ws + L.P);
    float* Vm = reinterpret_cast<float*>(ws + L.Vm);
    float* Wm = reinterpret_cast<float*>(ws + L.Wm);
    double* partial = reinterpret_cast<double*>(ws + L.partial);
    double* eps2 = reinterpret_cast<double*>(ws + L.eps2);
    uint32_t* planeA = reinterpret_cast<uint32_t*>(q3);
    uint32_t* planeB = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(q3) + (N * K) / 4);

    const int l = L.l, ld = L.ld;
    const int even = (l + 1) & ~1;
    const size_t chol_lds = (size_t)l * (2 * l + 1) * sizeof(float), one = (size_t)even * (even + 2) * sizeof(float);
    const bool two = 3 * one <= 156 * 1024;           // (the kernel has a KB of its own beside it)
    const size_t jac_lds = (two ? 3 : 2) * one;
    const int jac_threads = l <= 48 ? 512 : 1024;
    auto jacobi = l <= 48 ? jacobi_factors_kernel<512, 1, true> : two ? jacobi_factors_kernel<1024, 1, true>
                : l <= 128 ? jacobi_factors_kernel<1024, 1, false> : jacobi_factors_kernel<1024, 2, false>;
    const size_t left_k = (l + 3) & ~3, left_lds = ((left_k + ld) * 65 + ld * (left_k + 1)) * sizeof(float), right_lds = ((size_t)l * r + 64 * (l + 1)) * sizeof(float);
    const size_t gram_lds = (size_t)kGramStep * (ld + 1) * sizeof(float);
    const size_t resid_lds = (size_t)16 * (r + 1) * sizeof(float), pack_lds = 4 * kRowBlockBytes + resid_lds;
    auto raise = [](const void* k, size_t bytes) {
        return bytes <= 65536 || hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) == hipSuccess;
    };
    const void* const sketch_b = L.rb == 1 ? reinterpret_cast<const void*>(&sketch_b_kernel<1>) : L.rb == 2 ? reinterpret_cast<const void*>(&sketch_b_kernel<2>)
                               : L.rb == 3 ? reinterpret_cast<const void*>(&sketch_b_kernel<3>) : reinterpret_cast<const void*>(&sketch_b_kernel<4>);
    if (!raise(reinterpret_cast<const void*>(&cholesky_inverse_kernel), chol_lds) || !raise(sketch_b, chol_lds) ||
        !raise(reinterpret_cast<const void*>(jacobi), jac_lds) ||
        !raise(reinterpret_cast<const void*>(&gram_rows_kernel<6>), gram_lds) ||
        !raise(reinterpret_cast<const void*>(&apply_left_kernel), left_lds) ||
        !raise(reinterpret_cast<const void*>(&apply_right_kernel), right_lds) ||
        !raise(reinterpret_cast<const void*>(&resid_kernel<RESID_PACK>), pack_lds))
        return MILO_ERR_HIP;

    const dim3 cols((unsigned)(K / 64));
    const int64_t units = N * (K / kGroup);
    const unsigned hqq_grid = (unsigned)row_block_grid(N, K);
    const dim3 resid_grid((unsigned)(N / 16), (unsigned)L.norm_x);
    const int64_t part_b = (int64_t)ld * K;
    const int gram_y = (int)((N + kGramRows - 1) / kGramRows), gram_b = (int)(K / 64);
    if (l > 0)
        random_basis_kernel<<<dim3((unsigned)((part_b + 255) / 256)), dim3(256), 0, st>>>(Vb, part_b, (int64_t)l * K, prm->seed);
    // largest residual that the shrinkage certainly maps to zero, and how it moves as beta grows
    const float edge = (float)(0.999 * pow((double)prm->beta, -1.0 / (2.0 - (double)prm->p)));
    const float edge_step = (float)pow((double)prm->kappa, -1.0 / (2.0 - (double)prm->p));
    *iters_run = 0;
    for (int t = 0; t < prm->iters; ++t) {
        if (t > 0)
            resid_kernel<RESID_TARGET><<<resid_grid, dim3(256), resid_lds, st>>>(W, U, V, r, N, K, RE, nullptr, nullptr, nullptr, nullptr, nullptr);
        if (units <= kHqqFewUnits) {
            auto few = t == 0 ? hqq_few_kernel<true> : hqq_few_kernel<false>;       // (the first target is W itself)
            few<<<dim3((unsigned)((units + kHqqFewPerBlock - 1) / kHqqFewPerBlock)), dim3(kHqqFewThreads), 0, st>>>(
                W, RE, s, z, units, prm->hqq_iters, prm->p - 1.0f, prm->beta, prm->kappa);
        } else if (t == 0) {
            hqq_kernel<true><<<dim3(hqq_grid), dim3(kRowBlockThreads), 0, st>>>(W, RE, s, z, N, K, prm->hqq_iters, prm->p - 1.0f, prm->beta,
                                                                                prm->kappa, edge, edge_step);
        } else {
            hqq_kernel<false><<<dim3(hqq_grid), dim3(kRowBlockThreads), 0, st>>>(W, RE, s, z, N, K, prm->hqq_iters, prm->p - 1.0f, prm->beta,
                                                                                 prm->kappa, edge, edge_step);
        }
        if (r > 0) {
            const int rounds = 1 + (t == 0 ? prm->power_iters : prm->refine_iters);
            for (int it = 0; it < rounds; ++it) {
                by_rank_tiles(L.rb, [&](auto rb) {
                    constexpr int RB = decltype(rb)::value;
                    sketch_y_kernel<RB><<<dim3((unsigned)((N + 63) / 64), (unsigned)L.split_y, (unsigned)L.groups), dim3(256), 0, st>>>(
                        RE, Vb, N, K, ld, L.split_y, Yp);
                });
                const int gram_tiles = (ld / 16) * (ld / 16);
                auto gram = gram_tiles <= 16 ? gram_rows_kernel<1> : gram_rows_kernel<6>;
                gram<<<dim3((unsigned)gram_y), dim3(kGramThreads), gram_lds, st>>>(Yp, L.split_y, N, ld, Y, Gp);
                by_rank_tiles(L.rb, [&](auto rb) {
                    constexpr int RB = decltype(rb)::value;
                    const size_t red = (size_t)RB * 16384;
                    sketch_b_kernel<RB><<<dim3((unsigned)((K + 255) / 256) + 1u, (unsigned)L.split_b, (unsigned)L.groups), dim3(kSmallThreads),
                                          red > chol_lds ? red : chol_lds, st>>>(RE, Y, N, K, ld, L.split_b, Bp, Gp, gram_y, l, LinvY);
                });
                apply_left_kernel<<<cols, dim3(kLeftThreads), left_lds, st>>>(LinvY, l, ld, l, Bp, L.split_b, part_b, K, Bm, Gp);      // B, B B^T
                if (it + 1 < rounds) {
                    cholesky_inverse_kernel<<<dim3(1), dim3(kSmallThreads), chol_lds, st>>>(Gp, gram_b, ld, l, LinvB);
                    apply_left_kernel<<<cols, dim3(kLeftThreads), left_lds, st>>>(LinvB, l, ld, l, Bm, 1, part_b, K, Vb, nullptr);      // next basis
                }
            }
            jacobi<<<dim3(1), dim3((unsigned)jac_threads), jac_lds, st>>>(Gp, gram_b, ld, l, r, 12, LinvY, P, Vm, Wm);
            apply_right_kernel<<<dim3((unsigned)((N + 63) / 64)), dim3(256), right_lds, st>>>(Y, ld, l, P, r, N, U);
            apply_left_kernel<<<cols, dim3(kLeftThreads), left_lds, st>>>(Vm, r, r, l, Bm, 1, part_b, K, V, nullptr);
            if (t + 1 < prm->iters)
                apply_left_kernel<<<cols, dim3(kLeftThreads), left_lds, st>>>(Wm, l, ld, l, Bm, 1, part_b, K, Vb, nullptr);
        }
        resid_kernel<RESID_NORM><<<resid_grid, dim3(256), resid_lds, st>>>(RE, U, V, r, N, K, nullptr, partial, nullptr, nullptr, nullptr, nullptr);
        sum_partials_kernel<<<dim3(1), dim3(kSmallThreads), 0, st>>>(partial, (N / 16) * L.norm_x, eps2);
        double e2 = 0.0;
        if (hipMemcpyAsync(&e2, eps2, sizeof(double), hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipStreamSynchronize(st) != hipSuccess)
            return MILO_ERR_HIP;
        eps[t] = sqrt(e2);
        *iters_run = t + 1;
        if (!(eps[t] == eps[t])) break;                                   // not a number: nothing more to gain
        if (prm->tol >= 0.0f && stop_rule(eps, t + 1, (double)prm->tol)) break;
    }
    // the stored format: target W - U V, fixed scales, z rounded to fp16
    const dim3 pack_grid((unsigned)(N / 16), (unsigned)((L.norm_x + 1) / 2));
    resid_kernel<RESID_PACK><<<pack_grid, dim3(256), pack_lds, st>>>(W, U, V, r, N, K, nullptr, nullptr, s, z, planeA, planeB);
    return launch_status();
}
