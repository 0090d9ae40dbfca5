// milo_pack_w3 / milo_unpack_w3 / milo_dequant_w3: group quantizer (Eq. wq, round-to-nearest
// reading), the zero-waste 3-bit packer (Section 3.3) and the two test aids.
//
// This translation unit is compiled with -ffp-contract=off: the quantizer must perform one
// binary32 rounding per operation (no fused multiply-add) so that its codes are reproducible
// bit for bit.
#include "milo_device.h"
#include "milo_host.h"
#include "pack_device.h"

namespace milo {

// One quantization group: scale, zero-point and codes (as whole floats).  SYM = false: asymmetric quantizer
// (Eq. wq).  SYM = true: the symmetric INT3 quantizer (Eq. symm_int3) in the same storage: the scale word
// holds the step 2 * max|w| / 7, the zero word 4.
template <bool SYM>
__device__ __forceinline__ uint32_t quantize_group(float (&v)[64]) {
    float mn = v[0], mx = v[0];
#pragma unroll
    for (int i = 1; i < 64; ++i) {
        mn = fminf(mn, v[i]);
        mx = fmaxf(mx, v[i]);
    }
    const float span = SYM ? fmaxf(mx, -mn) + fmaxf(mx, -mn) : mx - mn;      // (SYM: twice the largest magnitude)
    f16 s16 = (f16)(span / 7.0f), z16;
    float sf = (float)s16;
    float lift;                             // what is added to w / s before rounding
    const bool degenerate = !(sf > 0.0f && sf <= 65504.0f);                  // zero, NaN or overflowed scale
    if (degenerate) s16 = (f16)1.0f;
    if (SYM) {
        z16 = (f16)4.0f;
        lift = 4.0f;
    } else {
        float z = __builtin_rintf((-mn) / sf);
        z = fminf(fmaxf(z, -65504.0f), 65504.0f);
        z16 = degenerate ? (f16)(-mn) : (f16)z;
        lift = (float)z16;
    }
    const float inv = 1.0f / sf;
#pragma unroll
    for (int i = 0; i < 64; ++i) {
        float t = div_by(v[i], sf, inv);
        if (SYM) {                          // rounded before the shift, so that it is exact
            t = __builtin_rintf(t);
            t = t + 4.0f;
        } else {
            t = t + lift;
            t = __builtin_rintf(t);
        }
        t = fminf(fmaxf(t, 0.0f), 7.0f);
        v[i] = degenerate ? (SYM ? 4.0f : 0.0f) : t;
    }
    return scale_zero_word(s16, z16);
}

// Row n of the source is W + n * row_stride for n < n_valid and zeros for the rows from n_valid up to N.
template <bool SYM>
__global__ __launch_bounds__(kRowBlockThreads) void pack_w3_kernel(const float* __restrict__ W, int64_t N, int64_t K,
                                                                   int64_t row_stride, int64_t n_valid,
                                                                   uint32_t* __restrict__ planeA, uint32_t* __restrict__ planeB) {
    __shared__ __attribute__((aligned(16))) unsigned char lds[kRowBlockWaves * kRowBlockBytes];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t G = K / kGroup;
    int64_t n0, g0;
    if (!row_block_item(N, G, wave, &n0, &g0)) return;
    unsigned char* const area = lds + wave * kRowBlockBytes;
    stage_row_block(W, row_stride, n0, n_valid, g0, K, area, lane);
    wait_vmem();
    float v[64];
    read_unit64(area, lane, v);
    if (g0 + (lane >> 4) >= G) return;
    const uint32_t sz = quantize_group<SYM>(v);
    uint32_t d[6];
    unit_words(v, d);
    store_row_block_unit(d, sz, ((n0 >> 4) * G + g0) * 16 + lane, planeA, planeB);
}

// The transposed factor of milo_pack_lr3 (symmetric quantizer): element (n, k) = W[n + k * col_stride] for
// n < n_valid, zero above.  A few rows, small: one lane per unit, straight from memory (neighbouring lanes
// are neighbouring rows, which are adjacent here).
__global__ __launch_bounds__(256) void pack_w3_transposed_kernel(const float* __restrict__ W, int64_t N, int64_t K,
                                                                 int64_t col_stride, int64_t n_valid,
                                                                 uint32_t* __restrict__ planeA, uint32_t* __restrict__ planeB) {
    const int64_t G = K / kGroup;
    const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= N * G) return;
    const int64_t rest = u >> 4, n = (rest / G) * 16 + (u & 15), g = rest % G;
    float v[64];
#pragma unroll
    for (int i = 0; i < 64; ++i) v[i] = n < n_valid ? W[n + (g * kGroup + i) * col_stride] : 0.0f;
    const uint32_t sz = quantize_group<true>(v);
    uint32_t d[6];
    unit_words(v, d);
    store_row_block_unit(d, sz, u, planeA, planeB);
}

// One thread per unit: unpack to bytes / dequantize to fp16.  Test aids, not tuned.
__global__ __launch_bounds__(256) void unpack_w3_kernel(W3View w, int64_t N, int64_t K,
                                                        uint8_t* __restrict__ codes,
                                                        unsigned short* __restrict__ scales,
                                                        unsigned short* __restrict__ zeros) {
    const int64_t G = w.G;
    const int64_t gu = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gu >= N * G) return;
    const int64_t n = gu / G, g = gu - n * G;
    const int64_t u = unit_index(n, g, G);
    const RawUnit ru = load_unit(w, u);
    const uint32_t d[6] = {ru.a.x, ru.a.y, ru.a.z, ru.a.w, ru.b.x, ru.b.y};
    if (scales) scales[gu] = (unsigned short)(ru.sz & 0xffffu);
    if (zeros) zeros[gu] = (unsigned short)(ru.sz >> 16);
    if (!codes) return;
    uint8_t* out = codes + n * K + g * kGroup;
    for (int P = 0; P < 32; ++P) {
        uint32_t lo, hi;
        if (P < 30) {
            const int j = P / 5, c = P % 5;
            lo = (d[j] >> (3 * c)) & 7u;
            hi = (d[j] >> (16 + 3 * c)) & 7u;
        } else {
            const int base = (P == 30) ? 0 : 3;
            lo = hi = 0u;
            for (int i = 0; i < 3; ++i) {
                lo |= ((d[base + i] >> 15) & 1u) << i;
                hi |= ((d[base + i] >> 31) & 1u) << i;
            }
        }
        out[2 * P] = (uint8_t)lo;
        out[2 * P + 1] = (uint8_t)hi;
    }
}

__global__ __launch_bounds__(256) void dequant_w3_kernel(W3View w, int64_t N, int64_t K,
                                                         f16* __restrict__ Wdq) {
    const int64_t G = w.G;
    const int64_t gu = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gu >= N * G) return;
    const int64_t n = gu / G, g = gu - n * G;
    const RawUnit ru = load_unit(w, unit_index(n, g, G));
    uint32_t wv[32];
    dequant_unit(ru, wv);
    u32x4* out = reinterpret_cast<u32x4*>(Wdq + n * K + g * kGroup);
#pragma unroll
    for (int i = 0; i < 8; ++i) out[i] = u32x4{wv[4 * i], wv[4 * i + 1], wv[4 * i + 2], wv[4 * i + 3]};
}

}  // namespace milo

using namespace milo;

extern "C" size_t milo_w3_packed_bytes(int64_t N, int64_t K) {
    if (!weight_shape_ok(N, K)) return 0;
    return (size_t)(N * K / 64 * 28);
}

template <bool SYM>
static int pack_launch(const float* W, int64_t N, int64_t K, int group_size, void* q3, void* stream) {
    if (!W || !q3) return MILO_ERR_NULL;
    if (group_size != kGroup) return MILO_ERR_GROUP;
    if (!weight_shape_ok(N, K)) return MILO_ERR_SHAPE;
    if (!aligned16(W) || !aligned16(q3)) return MILO_ERR_ALIGN;
    const int64_t blocks = row_block_grid(N, K);
    if (blocks > 0x7fffffff) return MILO_ERR_SHAPE;
    uint32_t* planeA = reinterpret_cast<uint32_t*>(q3);
    uint32_t* planeB = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(q3) + (N * K) / 4);
    pack_w3_kernel<SYM><<<dim3((unsigned)blocks), dim3(kRowBlockThreads), 0, (hipStream_t)stream>>>(W, N, K, K, N, planeA,
                                                                                                   planeB);
    return launch_status();
}

static int64_t rank_rows(int r) { return ((int64_t)r + 15) / 16 * 16; }

extern "C" int milo_lr3_packed_bytes(int64_t N, int64_t K, int r, size_t* u_bytes, size_t* v_bytes) {
    if (r <= 0 || r > MILO_LR3_MAX_RANK) return MILO_ERR_RANK;
    if (!weight_shape_ok(N, K) || (N % kGroup) != 0 || !weight_shape_ok(rank_rows(r), N) || !weight_shape_ok(rank_rows(r), K))
        return MILO_ERR_SHAPE;
    if (u_bytes) *u_bytes = (size_t)(rank_rows(r) * N / 64 * 28);
    if (v_bytes) *v_bytes = (size_t)(rank_rows(r) * K / 64 * 28);
    return MILO_OK;
}

extern "C" int milo_pack_lr3(const float* U, const float* V, int64_t N, int64_t K, int r, void* u3, void* v3,
                             void* stream) {
    if (!U || !V || !u3 || !v3) return MILO_ERR_NULL;
    const int st = milo_lr3_packed_bytes(N, K, r, nullptr, nullptr);
    if (st != MILO_OK) return st;
    if (!aligned16(U) || !aligned16(V) || !aligned16(u3) || !aligned16(v3)) return MILO_ERR_ALIGN;
    const int64_t rp = rank_rows(r);
    // U^T: [rp x N], element (j, n) = U[n * r + j], groups of 64 along N
    {
        const int64_t units = rp * (N / kGroup), blocks = (units + 255) / 256;
        uint32_t* planeA = reinterpret_cast<uint32_t*>(u3);
        uint32_t* planeB = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(u3) + (rp * N) / 4);
        pack_w3_transposed_kernel<<<dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream>>>(U, rp, N, r, r, planeA, planeB);
        if (launch_status() != MILO_OK) return MILO_ERR_HIP;
    }
    // V: [rp x K], element (j, k) = V[j * K + k], groups of 64 along K
    {
        const int64_t blocks = row_block_grid(rp, K);
        uint32_t* planeA = reinterpret_cast<uint32_t*>(v3);
        uint32_t* planeB = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(v3) + (rp * K) / 4);
        pack_w3_kernel<true><<<dim3((unsigned)blocks), dim3(kRowBlockThreads), 0, (hipStream_t)stream>>>(V, rp, K, K, r, planeA,
                                                                                                    planeB);
    }
    return launch_status();
}

extern "C" int milo_pack_w3(const float* W, int64_t N, int64_t K, int group_size, void* q3, void* stream) {
    return pack_launch<false>(W, N, K, group_size, q3, stream);
}

extern "C" int milo_pack_w3_sym(const float* W, int64_t N, int64_t K, int group_size, void* q3, void* stream) {
    return pack_launch<true>(W, N, K, group_size, q3, stream);
}

extern "C" int milo_unpack_w3(const void* q3, int64_t N, int64_t K, uint8_t* codes, milo_half* scales,
                              milo_half* zeros, void* stream) {
    if (!q3 || (!codes && !scales && !zeros)) return MILO_ERR_NULL;
    if (!weight_shape_ok(N, K)) return MILO_ERR_SHAPE;
    if (!aligned16(q3)) return MILO_ERR_ALIGN;
    const int64_t units = N * (K / kGroup);
    const int64_t blocks = (units + 255) / 256;
    if (blocks > 0x7fffffff) return MILO_ERR_SHAPE;
    W3View w = make_view(q3, N, K);
    unpack_w3_kernel<<<dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream>>>(w, N, K, codes, scales, zeros);
    return launch_status();
}

extern "C" int milo_dequant_w3(const void* q3, int64_t N, int64_t K, milo_half* W_dq, void* stream) {
    if (!q3 || !W_dq) return MILO_ERR_NULL;
    if (!weight_shape_ok(N, K)) return MILO_ERR_SHAPE;
    if (!aligned16(q3) || !aligned16(W_dq)) return MILO_ERR_ALIGN;
    const int64_t units = N * (K / kGroup);
    const int64_t blocks = (units + 255) / 256;
    if (blocks > 0x7fffffff) return MILO_ERR_SHAPE;
    W3View w = make_view(q3, N, K);
    dequant_w3_kernel<<<dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream>>>(
        w, N, K, reinterpret_cast<f16*>(W_dq));
    return launch_status();
}
