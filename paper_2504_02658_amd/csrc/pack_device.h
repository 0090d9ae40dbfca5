// Shared by the two quantizers (pack.hip, compress.hip): building units of the zero-waste 3-bit layout
// (Section 3.3) from fp32 weights, one lane per unit.
//
// The quantizers are bound by HBM (4 bytes read per weight) only if the vector units keep up.  With 16
// lanes per unit (four weights each) they did not: 32 cross-lane steps and some fifty instructions of bit
// assembly for every four weights, 103 us for a 14336 x 4096 weight (2.5 TB/s).  Here one lane owns a whole
// unit, so the minimum, the maximum and the words are formed in its own registers with compile-time
// positions, about ten instructions per weight.  A row-major weight read that way would touch 64 lines per
// load, so the wave brings its 64 units in through LDS: 16 rows x 4 groups (the units of one row block, whose
// packed form is contiguous), one 1-KB row piece per buffer-to-LDS copy; eight waves with 16 KB on their way
// each keep a CU's share of the HBM busy.  14336 x 4096: 48 us, 5.4 TB/s, the rate of a device copy.
#pragma once
#include "milo_device.h"

namespace milo {

constexpr int kRowBlockWaves = 4;                              // waves of a workgroup, each on its own units
constexpr int kRowBlockThreads = 64 * kRowBlockWaves;
constexpr int kRowBlockBytes = 16 * 1024;                     // 16 rows x 4 groups of fp32, one wave

typedef __attribute__((address_space(3))) void* PackLdsPtr;

// Copies rows n0 .. n0 + 15, columns 64 g0 .. 64 g0 + 255 of W [. x K] into the wave's LDS area.  Rows from
// n_valid on and columns past K read as zero.  The 16-byte segment at position p of (row, group) is
// segment p ^ row, so that the lanes of a quad, which read 16 rows, meet no bank conflict.  The caller
// waits for the copies.
__device__ __forceinline__ void stage_row_block(const float* __restrict__ W, int64_t row_stride, int64_t n0, int64_t n_valid,
                                                int64_t g0, int64_t K, unsigned char* area, int lane) {
    const int64_t left = (K - g0 * kGroup) * 4;
    const uint32_t bytes = left >= 1024 ? 1024u : (uint32_t)left;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const BufRsrc rb = make_rsrc(W + (n0 + i) * row_stride + g0 * kGroup, n0 + i < n_valid ? bytes : 0u);
        const uint32_t off = ((uint32_t)lane & 48u) * 16u + ((((uint32_t)lane & 15u) ^ (uint32_t)i) << 4);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (PackLdsPtr)(area + i * 1024), 16, off, 0, 0, 0);
    }
    asm volatile("" ::: "memory");
}
// Lane l's unit of the staged block: row l % 16, group l / 16.
__device__ __forceinline__ void read_unit64(const unsigned char* area, int lane, float (&v)[64]) {
    const int row = lane & 15, g = lane >> 4;
#pragma unroll
    for (int t = 0; t < 16; ++t) {
        const float4 f = *reinterpret_cast<const float4*>(area + row * 1024 + g * 256 + ((t ^ row) << 4));
        v[4 * t] = f.x; v[4 * t + 1] = f.y; v[4 * t + 2] = f.z; v[4 * t + 3] = f.w;
    }
}

// a / b rounded as the division instruction sequence rounds it, for y = 1 / b correctly rounded and b a
// binary16 value: q = RN(a y) is off by at most one unit in the last place, its remainder a - q b is exact in
// an fma, and one correction gives RN(a / b) (Markstein's theorem; its exception, a significand of all
// ones, cannot occur in 11 bits).  Quotients too small for an exact remainder vanish in the sum with the
// zero-point.  Three instructions instead of the ten of a division.
__device__ __forceinline__ float div_by(float a, float b, float y) {
    const float q = a * y;
    return __builtin_fmaf(__builtin_fmaf(-q, b, a), y, q);
}
// The same for a quotient that may be infinite, which the remainder would turn into not-a-number.
__device__ __forceinline__ float div_by_any(float a, float b, float y) {
    const float q = a * y;
    return fabsf(q) < __builtin_inff() ? __builtin_fmaf(__builtin_fmaf(-q, b, a), y, q) : q;
}

// The words of a unit from its 64 codes (whole numbers 0..7 as floats).
__device__ __forceinline__ void unit_words(const float (&code)[64], uint32_t (&d)[6]) {
#pragma unroll
    for (int j = 0; j < 6; ++j) {
        d[j] = 0u;
#pragma unroll
        for (int c = 0; c < 5; ++c) {
            const int P = 5 * j + c;
            d[j] |= ((uint32_t)code[2 * P] << (3 * c)) | ((uint32_t)code[2 * P + 1] << (16 + 3 * c));
        }
        const int P = j < 3 ? 30 : 31, bit = j % 3;             // the spare bits 15 and 31 carry pairs 30 and 31
        d[j] |= ((((uint32_t)code[2 * P] >> bit) & 1u) << 15) | ((((uint32_t)code[2 * P + 1] >> bit) & 1u) << 31);
    }
}
// Stores lane l's unit u0 + l of the wave's row block (64 consecutive units, 16 and 12 bytes each).
__device__ __forceinline__ void store_row_block_unit(const uint32_t (&d)[6], uint32_t sz, int64_t u, uint32_t* __restrict__ planeA,
                                                     uint32_t* __restrict__ planeB) {
    *reinterpret_cast<u32x4*>(planeA + 4 * u) = u32x4{d[0], d[1], d[2], d[3]};
    struct Tail { uint32_t w[3]; };
    *reinterpret_cast<Tail*>(planeB + 3 * u) = Tail{{d[4], d[5], sz}};
}
__device__ __forceinline__ uint32_t scale_zero_word(f16 s, f16 z) {
    return (uint32_t)__builtin_bit_cast(unsigned short, s) | ((uint32_t)__builtin_bit_cast(unsigned short, z) << 16);
}
// Work item of a wave: row block and first group of 4; false past the end.
__device__ __forceinline__ bool row_block_item(int64_t N, int64_t G, int wave, int64_t* n0, int64_t* g0) {
    const int64_t per_row = (G + 3) >> 2;
    const int64_t item = (int64_t)blockIdx.x * kRowBlockWaves + wave;
    const int64_t rb = item / per_row;
    *n0 = rb * 16;
    *g0 = (item - rb * per_row) * 4;
    return *n0 < N;
}
inline int64_t row_block_grid(int64_t N, int64_t K) {
    return ((N / 16) * ((K / kGroup + 3) / 4) + kRowBlockWaves - 1) / kRowBlockWaves;
}

}  // namespace milo
