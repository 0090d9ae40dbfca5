// Pieces that the two weight-streaming kernels share (gemm_decode.hip: one linear; gemm_few.hip: the experts of an
// MoE layer): both walk K in chunks of 256 columns, a chunk's activations are the B operand of every 16-row block,
// staged in an 8-KB LDS slot that belongs to one wave.
#pragma once

#include <type_traits>

#include "milo_device.h"

namespace milo {

typedef __attribute__((address_space(3))) void* LdsPtr;

// Compile-time loop: f(std::integral_constant<int, I>) for I in [B, E).
template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        static_for<B + 1, E>(f);
    }
}

constexpr int kStreamSlotBytes = 16 * 512;                      // one chunk of X: 16 rows x 256 k

// B fragments of a staged chunk: step t, lane (j16, q) = X[j16][8 (8q + t) .. + 7] of the chunk.
__device__ __forceinline__ void read_bfrags(const unsigned char* slot, int j16, int q, f16x8 (&bfrag)[8]) {
#pragma unroll
    for (int t = 0; t < 8; ++t)
        bfrag[t] = __builtin_bit_cast(
            f16x8, *reinterpret_cast<const u32x4*>(slot + j16 * 512 + (((8 * q + t) ^ j16) << 4)));
}

// Most k-steps of 32 ranks that the low-rank term takes through LDS.
constexpr int kStreamKS = 4;

// Scatters the dequantized unit of one rank (64 consecutive output features, w[P] = features 2P and
// 2P + 1 of the group) into the U fragments of the R row blocks that start O16 blocks into the
// group: feature 16 (O16 + b) + jj of rank j goes to fragment (b, j / 32), lane (jj, (j % 32) / 8),
// element j % 8.  `frag0` points at that element of block 0's fragment for jj = 0.
template <int R, int O16>
__device__ __forceinline__ void scatter_u_rank(const uint32_t (&w)[32], unsigned char* frag0) {
#pragma unroll
    for (int b = 0; b < R; ++b)
#pragma unroll
        for (int jj = 0; jj < 16; ++jj) {
            const int n = 16 * (O16 + b) + jj;
            const uint32_t v = w[n >> 1];
            *reinterpret_cast<unsigned short*>(frag0 + b * (kStreamKS * 1024) + jj * 16) =
                (unsigned short)((n & 1) ? (v >> 16) : v);
        }
}

}  // namespace milo
