// Kernel of the compensated W3A16 linear for batches of 17 rows up to where the tiled kernel's tiles fill the chip: one
// launch, no K splits across workgroups and no second kernel.
//
// Work split.  A workgroup of eight waves owns 32 S output features (a band) and up to 32 MB rows over the whole K; the waves
// take every eighth 128-column chunk of K and add up in LDS at the end, in wave order.  A wave loads the units of its S
// 32-feature streams, converts them in registers (milo_device.h) and feeds them as the A operand of 32x32x16 MFMAs; the
// chunk's activations are the B operand, copied into a slot of the wave's own in LDS, so the loop has no barrier.  The
// fragments of a chunk are read into registers at once (MB = 2, or a single stream; else in two halves), which frees the slot
// for the next chunk's copies while this one is multiplied.
//
// Why.  At such sizes the tiled kernel has a few dozen tiles: it splits K over workgroups, writes fp32 partial sums and adds
// them in a second kernel, and T = X V^T passes through partial sums, a counter and a flag.  us, tiled / this kernel at
// r = 32: 32 rows of 1024 x 1024 11.8 / 5.7, 2048 x 1408 14.2 / 6.6, 4096 x 4096 15.3 / 8.6, 14336 x 4096 18.5 / 13.5;
// 64 rows of 4096 x 14336 27.9 / 21.2; 77 of 14336 x 4096 31 / 20; 128 of 4096 x 4096 21.5 / 11.9.
//
// Bound: latency.  The launch, the first data and the epilogue take about 4 us; in the loop a wave waits for its chunk, converts and
// multiplies in turn, with one workgroup of eight waves per CU (two with 32-row tiles) to fill in.  Counters: 77 rows of 14336 x 4096, INT3
// r = 32 (21 us) matrix cores busy for 17 % and vector units for 20 % of the SIMD-cycles, waves waiting 43 % of their time, no bank conflicts;
// 400 of 4096 x 4096 (30 us) 18, 28 and 32 %; 32 of 4096 x 4096 (8 us) 3, 8 and 53 %.  X comes from L2 once per workgroup, 1 KB per copy
// instruction, as whole 256-byte row pieces (64-byte pieces of four times as many rows per copy: 32 rows of 4096 x 14336 25 us, now 19).
// Tried without gain: sixteen waves per workgroup, weights requested two chunks ahead, chunks rotated per workgroup.
#include <type_traits>

#include "milo_host.h"
#include "milo_kernels.h"
#include "stream_device.h"

namespace milo {

constexpr int kMidWaves = 8;                            // waves of a workgroup, which share K
constexpr int kMidThreads = 64 * kMidWaves;
constexpr uint32_t kMidNoUnit = 1u << 27;               // past the end of every weight the host accepts

__device__ __forceinline__ uint32_t mid_tag(const MidArgs& a, uint32_t wg) {
    const unsigned long long v =
        __hip_atomic_load(a.epoch + (wg % kDecGroups) * kDecGroupStride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return (uint32_t)(v >> 16) + 1u;
}

// Copies a 128-column chunk of 4 NC rows into a slot ([row][256 B], the sixteen 16-byte segments of a row at position s ^
// (row % 16), so that the 32 rows of a fragment are read without bank conflicts).  Copy i moves rows 4 i .. 4 i + 3 with one
// 1-KB buffer-to-LDS load of whole 256-byte pieces.  Rows past the end of the buffer read as zero, and so do the upper 64
// columns of a chunk that has none.
struct ChunkCopy {
    uint32_t seg, row;      // byte of this lane's segment of copy 0 in its row, offset of the row
    __device__ __forceinline__ ChunkCopy(int lane, uint32_t ldb) {
        const uint32_t r = (uint32_t)lane >> 4;
        seg = (((uint32_t)lane & 15u) ^ r) << 4;
        row = r * ldb;
    }
    template <int NC>
    __device__ __forceinline__ void issue(BufRsrc b, unsigned char* slot, uint32_t base, uint32_t ldb, bool lower_only) const {
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            uint32_t flip = 64u * (i & 3), uni = __builtin_amdgcn_readfirstlane(base + (uint32_t)i * 4u * ldb);
            asm volatile("" : "+s"(flip), "+s"(uni));       // (formed here, not kept in registers)
            const uint32_t s = seg ^ flip, off = s + row + uni;
            const uint32_t at = lower_only && s >= 128u ? kOobOffset : off;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(b, (LdsPtr)(slot + i * 1024), 16, at, 0, 0, 0);
        }
        asm volatile("" ::: "memory");
    }
};
// Fragment of step t of a slot: row i32 of block mb (i: the row that is read in its place), segment 8 h + t.
__device__ __forceinline__ f16x8 chunk_frag(const unsigned char* slot, int mb, int t, int i, int h) {
    return __builtin_bit_cast(
        f16x8, *reinterpret_cast<const u32x4*>(slot + (mb * 32 + i) * 256 + (((8 * h + t) ^ (i & 15)) << 4)));
}
template <bool BF>
__device__ __forceinline__ f32x16 mfma32_any(f16x8 x, f16x8 y, f32x16 c) {
    return BF ? mfma32_bf16(__builtin_bit_cast(bf16x8, x), __builtin_bit_cast(bf16x8, y), c) : mfma32(x, y, c);
}
__device__ __forceinline__ f32x16 zero_f32x16() {
    f32x16 v;
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = 0.0f;
    return v;
}

// One T worker: 32 ranks x 32 rows of T over a part of K, fp32.  Each wave takes every eighth chunk of the part; both operands
// are staged through its own 8 KB of LDS.
template <bool BF>
__device__ __forceinline__ void mid_t_worker(const MidArgs& a, unsigned char* smem) {
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, i32 = lane & 31, h = lane >> 5;
    const uint32_t item = blockIdx.x;
    const uint32_t part = item % a.t_parts, x = item / a.t_parts, rb = x % a.rank_blocks, blk = x / a.rank_blocks;
    const uint32_t K = a.K, G = K / kGroup, nchunks = (G + 1u) / 2u, ldb = K * 2u;
    const bool odd = (G & 1u) != 0;
    // tag of the launch, from the counter of a workgroup that does not move it on before it has read what is formed here
    uint32_t tag = 0u;
    if (tid == 0) tag = mid_tag(a, (blk * 32u / a.tile_rows) * a.bands);
    const uint32_t cpp = (nchunks + a.t_parts - 1u) / a.t_parts, c_lo = part * cpp, c_hi = c_lo + cpp < nchunks ? c_lo + cpp : nchunks;
    const BufRsrc xb = make_rsrc(a.X, a.x_bytes);
    const bool q = (a.w.flags & MILO_LR_INT3) != 0;
    const BufRsrc vb = make_rsrc(a.w.V, q ? 0u : (uint64_t)(uint32_t)a.w.r * K * 2u);
    const W3Buf vq = make_w3buf(a.w.V, q ? (int64_t)a.ldt : 0, K);
    unsigned char* const slot = smem + wave * 8192;
    f32x16 acc = zero_f32x16();
    if (q) {
        // V as units: whole chunks, so that the columns of a lane are those of its unit
        const ChunkCopy cc(lane, ldb);
        auto issue = [&](uint32_t c) { cc.issue<8>(xb, slot, blk * 32u * ldb + c * 256u, ldb, odd && c == nchunks - 1u); };
        if (c_lo + wave < c_hi) issue(c_lo + wave);
        for (uint32_t c = c_lo + wave; c < c_hi; c += kMidWaves) {
            const uint32_t rank = rb * 32u + i32;
            const bool none = rank >= a.ldt || (odd && c == nchunks - 1u && h == 1);
            const RawUnit u = load_unit_buf(vq, none ? kMidNoUnit : ((rank >> 4) * G + 2u * c + h) * 16u + (rank & 15u));
            wait_vmem();
            f16x8 x[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) x[t] = chunk_frag(slot, 0, t, i32, h);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // the slot is free again
            if (c + kMidWaves < c_hi) issue(c + kMidWaves);
            dequant_unit_steps<true>(u, [&](int t, f16x8 frag) { acc = mfma32(frag, x[t], acc); });
        }
    } else {
        // 64 columns of both at a time: 32 rows of 128 bytes, segment s at position s ^ (row % 8); copies of 8 rows
        const uint32_t crow = (uint32_t)lane >> 3, own = crow * ldb + ((((uint32_t)lane & 7u) ^ crow) << 4);
        auto issue = [&](uint32_t g) {
#pragma unroll
            for (uint32_t i = 0; i < 4; ++i) {
                const uint32_t xo = own + (blk * 32u + 8u * i) * ldb + g * 128u, vo = own + (rb * 32u + 8u * i) * ldb + g * 128u;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(xb, (LdsPtr)(slot + i * 1024), 16, xo, 0, 0, 0);
                __builtin_amdgcn_raw_ptr_buffer_load_lds(vb, (LdsPtr)(slot + 4096 + i * 1024), 16, vo, 0, 0, 0);
            }
            asm volatile("" ::: "memory");
        };
        const uint32_t g_hi = 2u * c_hi < G ? 2u * c_hi : G;
        uint32_t g = 2u * c_lo + wave;
        if (g < g_hi) issue(g);
        for (; g < g_hi; g += kMidWaves) {
            wait_vmem();
            f16x8 x[4], v[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const unsigned char* const at = slot + i32 * 128 + (((2 * t + h) ^ (i32 & 7)) << 4);
                x[t] = __builtin_bit_cast(f16x8, *reinterpret_cast<const u32x4*>(at));
                v[t] = __builtin_bit_cast(f16x8, *reinterpret_cast<const u32x4*>(at + 4096));
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            if (g + kMidWaves < g_hi) issue(g + kMidWaves);
#pragma unroll
            for (int t = 0; t < 4; ++t) acc = mfma32_any<BF>(v[t], x[t], acc);
        }
    }
    __syncthreads();
    f32x4* const red = reinterpret_cast<f32x4*>(smem);          // [wave][4][64 lanes]
#pragma unroll
    for (int v = 0; v < 4; ++v) red[(wave * 4 + v) * 64 + lane] = f32x4{acc[4 * v], acc[4 * v + 1], acc[4 * v + 2], acc[4 * v + 3]};
    __syncthreads();
    if (wave < 4) {
        f32x4 p[kMidWaves];
#pragma unroll
        for (int w = 0; w < kMidWaves; ++w) p[w] = red[(w * 4 + wave) * 64 + lane];
        f32x4 sum = p[0];
#pragma unroll
        for (int w = 1; w < kMidWaves; ++w)
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[e] += p[w][e];
        // element e of quad v: rank 32 rb + 8 v + 4 h + e, row 32 blk + i32
        const uint32_t rank = rb * 32u + 8u * wave + 4u * h, row = blk * 32u + i32;
        const BufRsrc tb = make_rsrc(a.T, a.t_bytes);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, sum), tb,
                                               rank < a.ldt && row < a.M ? ((part * a.M + row) * a.ldt + rank) * 4u : kOobOffset, 0, 17);
    }
    wait_vmem();
    __syncthreads();
    if (tid == 0) __hip_atomic_store(a.ready + item, (unsigned long long)tag << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // counters without a workgroup of this launch move on here
    if (item == 0 && (uint32_t)tid < kDecGroups && (uint32_t)tid >= a.nmain) atomicAdd(a.epoch + (uint32_t)tid * kDecGroupStride, 65536ull);
}

// MB: 32-row blocks of a tile, ROWS: rows of a tile that are staged; S: 32-feature streams of a wave.
template <int MB, int ROWS, int S, int MODE>
__global__ __launch_bounds__(kMidThreads, MB == 1 ? 4 : 2) void w3lr_mid_kernel(const MidArgs a) {
    constexpr bool SYM = MODE == 1, BF = MODE == 2;
    constexpr int SLOT = ROWS * 256;                // bytes of a wave's slot: one chunk
    constexpr int NC = ROWS / 4;                    // 1-KB copies of a chunk
    constexpr bool WHOLE = MB == 2 || (MB == 1 && S == 1);     // a chunk's fragments fit the registers at once
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    if (blockIdx.x < a.nt) {
        mid_t_worker<BF>(a, smem);
        return;
    }
    const int tid = threadIdx.x, lane = tid & 63, i32 = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t wg = blockIdx.x - a.nt;
    const uint32_t band = wg % a.bands, tile = wg / a.bands;        // (tiles of a band: the same weights)
    const uint32_t K = a.K, N = a.N, G = K / kGroup, nchunks = (G + 1u) / 2u, ldb = K * 2u;
    const bool odd = (G & 1u) != 0;
    const uint32_t row0 = tile * a.tile_rows, rows = a.M - row0 < a.tile_rows ? a.M - row0 : a.tile_rows;
    const uint32_t n0 = band * (32u * S);

    const W3Buf wb = make_w3buf(a.w.q3, N, K);
    uint32_t unit0[S];                              // unit of this lane in chunk 0
#pragma unroll
    for (int s = 0; s < S; ++s) {
        const uint32_t n = n0 + 32u * s + i32;
        unit0[s] = n < N ? (n >> 4) * G * 16u + (n & 15u) + 16u * h : kMidNoUnit;
    }
    const BufRsrc xb = make_rsrc(a.X, a.x_bytes);
    unsigned char* const slot = smem + wave * SLOT;
    const ChunkCopy cc(lane, ldb);
    const uint32_t xbase = row0 * ldb;
    const uint32_t iters = (nchunks + kMidWaves - 1u) / kMidWaves;
    auto chunk_of = [&](uint32_t j) { return wave + kMidWaves * j; };
    auto issue_x = [&](uint32_t c) {
        const bool none = c >= nchunks;        // (requested like any other, out of range)
        cc.issue<NC>(xb, slot, none ? 0x80000000u : xbase + c * 256u, none ? 0u : ldb, odd && c == nchunks - 1u);
    };
    auto issue_w = [&](uint32_t c, RawUnit (&u)[S]) {
        const bool none = c >= nchunks || (odd && c == nchunks - 1u && h == 1);
#pragma unroll
        for (int s = 0; s < S; ++s)
            u[s] = a.once ? load_unit_buf_once(wb, none ? kMidNoUnit : unit0[s] + c * 32u) : load_unit_buf(wb, none ? kMidNoUnit : unit0[s] + c * 32u);
        asm volatile("" ::: "memory");
    };

    f32x16 acc[S][MB];
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[s][mb] = zero_f32x16();

    RawUnit ring[2][S];
    issue_w(chunk_of(0), ring[0]);
    issue_x(chunk_of(0));
    for (uint32_t j0 = 0; j0 < iters; j0 += 2) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const uint32_t j = j0 + u, c = chunk_of(j), next = chunk_of(j + 1);
            if (c >= nchunks) break;
            RawUnit (&cur)[S] = ring[u];
            constexpr int FT = WHOLE ? 8 : 4;
            f16x8 b[MB][FT];
            auto fetch = [&](int t0) {
#pragma unroll
                for (int t = 0; t < FT; ++t)
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb) b[mb][t] = chunk_frag(slot, mb, t0 + t, mb * 32 + 32 > ROWS ? i32 & 15 : i32, h);
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // (the slot is free again after the last of them)
            };
            wait_vmem();
            fetch(0);
            if (WHOLE) issue_x(next);
            issue_w(next, ring[u ^ 1]);
#pragma unroll
            for (int s = 0; s < S; ++s) pin_unit(cur[s]);
            auto step = [&](int t, auto... fr) {
                if (!WHOLE && t == 4) {
                    __builtin_amdgcn_sched_barrier(0);
                    fetch(4);
                    issue_x(next);
                }
                const f16x8 af[S] = {__builtin_bit_cast(f16x8, fr)...};
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                    for (int s = 0; s < S; ++s) acc[s][mb] = mfma32_any<BF>(af[s], b[mb][t % FT], acc[s][mb]);
            };
            if constexpr (S == 2) {
                if constexpr (BF) dequant_units2_steps_bf16(cur[0], cur[1], step);
                else dequant_units2_steps<SYM>(cur[0], cur[1], step);
            } else {
                if constexpr (BF) dequant_unit_steps_bf16(cur[0], step);
                else dequant_unit_steps<SYM>(cur[0], step);
            }
        }
    }

    wait_vmem();
    const int r = a.w.r;
    if (r > 0) {
        const bool uq = (a.w.flags & MILO_LR_INT3) != 0;
        const int ldu = (int)a.ldt + 8;
        f16* const UL = reinterpret_cast<f16*>(smem);
        if (uq) {
            // the band's groups of 64 features of U^T, rank by rank, as columns of UL[feature of the band][rank]
            constexpr int BAND = 32 * S, NG = (BAND + 63) / 64, PER = kMidWaves / NG;
            __syncthreads();
            const uint32_t GN = N >> 6, f0 = band * BAND, g = (f0 >> 6) + wave % NG, j = (wave / NG) * 64u + lane;
            static_assert(PER * 64 >= MILO_LR3_MAX_RANK, "a thread per rank and group");
            if (j < a.ldt) {
                const RawUnit u = load_unit_buf(make_w3buf(a.w.U, a.ldt, N), g < GN ? ((j >> 4) * GN + g) * 16u + (j & 15u) : kMidNoUnit);
                uint32_t wv[32];
                dequant_unit<true>(u, wv);
                if constexpr (BAND >= 64) {
                    f16* col = UL + 64 * (wave % NG) * ldu + j;
#pragma unroll
                    for (int P = 0; P < 32; ++P) {
                        const f16x2 pr = __builtin_bit_cast(f16x2, wv[P]);
                        col[(2 * P) * ldu] = pr[0];
                        col[(2 * P + 1) * ldu] = pr[1];
                    }
                } else {
                    const uint32_t up = (f0 & 32u) != 0 ? 0xffffffffu : 0u;
#pragma unroll
                    for (int P = 0; P < 16; ++P) {
                        const f16x2 pr = __builtin_bit_cast(f16x2, (wv[P + 16] & up) | (wv[P] & ~up));
                        UL[(2 * P) * ldu + j] = pr[0];
                        UL[(2 * P + 1) * ldu + j] = pr[1];
                    }
                }
            }
            __syncthreads();
        }
        // (k-step of 16 ranks, row block) pairs, dealt to the waves that share K
        const uint32_t nks = (uint32_t)(r + 15) / 16u, mbs = (rows + 31u) / 32u;
        const uint32_t tag = mid_tag(a, wg);
        const BufRsrc tb = make_rsrc(a.T, a.t_bytes);
        for (uint32_t f = wave; f < nks * mbs; f += kMidWaves) {
            const uint32_t mb = f % mbs, ks = f / mbs, k0 = 16u * ks + 8u * h;
            f16x8 av[S];
#pragma unroll
            for (int s = 0; s < S; ++s) {
                av[s] = zero_f16x8();
                const uint32_t n = n0 + 32u * s + i32;
                if (uq) {
                    if (k0 < a.ldt) av[s] = load_f16x8(UL + (int64_t)(32 * s + i32) * ldu + k0);
                } else if (n < N && k0 < (uint32_t)r) {
                    av[s] = load_row8(a.w.U + (int64_t)n * r, k0, r, (r & 7) == 0);
                }
            }
            const unsigned long long* const word = a.ready + ((row0 / 32u + mb) * a.rank_blocks + ks / 2u) * a.t_parts;
            for (uint32_t spins = 0;; ++spins) {
                const unsigned long long v = (uint32_t)lane < a.t_parts ? __hip_atomic_load(word + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                                                                        : (unsigned long long)tag << 32;
                if (__builtin_amdgcn_ballot_w64((uint32_t)(v >> 32) != tag) == 0ull) break;
                if (spins > a.spin_limit) {
                    if (lane == 0) atomicOr(a.status, 1u);
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
            asm volatile("" ::: "memory");          // (T is read after the words)
            const uint32_t m = row0 + 32u * mb + i32;
            float sum[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
            for (uint32_t p0 = 0; p0 < a.t_parts; p0 += 4) {           // four parts' loads at once
                u32x4 v[4][2];
#pragma unroll
                for (uint32_t i = 0; i < 4; ++i) {
                    const uint32_t p = p0 + i;
                    const uint32_t at = p < a.t_parts && m < a.M && k0 < a.ldt ? ((p * a.M + m) * a.ldt + k0) * 4u : kOobOffset;
                    v[i][0] = buf_load16_coherent(tb, at);
                    v[i][1] = buf_load16_coherent(tb, at == kOobOffset ? at : at + 16u);
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) {                           // (a part past the last adds zeros)
                    const f32x4 lo = __builtin_bit_cast(f32x4, v[i][0]), hi = __builtin_bit_cast(f32x4, v[i][1]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        sum[e] += lo[e];
                        sum[4 + e] += hi[e];
                    }
                }
            }
            f16x8 bv;
            if (BF) {
                bv = __builtin_bit_cast(f16x8, u32x4{pack_bf16(sum[0], sum[1]), pack_bf16(sum[2], sum[3]),
                                                     pack_bf16(sum[4], sum[5]), pack_bf16(sum[6], sum[7])});
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) bv[e] = (f16)sum[e];
            }
#pragma unroll
            for (int b = 0; b < MB; ++b)
                if (mb == (uint32_t)b)
#pragma unroll
                    for (int s = 0; s < S; ++s) acc[s][b] = mfma32_any<BF>(av[s], bv, acc[s][b]);
        }
    }

    // The waves that share K add up in LDS, in wave order; RS streams at a time.  A wave finishes pairs of quads: sixteen
    // features of the 32 rows of a block.
    constexpr int RS = (MB * S <= 4) ? S : 1, PAIRS = RS * MB * 2;
    f32x4* const red = reinterpret_cast<f32x4*>(smem);              // [wave][RS * MB * 4][64 lanes]
#pragma unroll
    for (int s0 = 0; s0 < S; s0 += RS) {
        __syncthreads();
        if (s0 == 0 && r > 0 && tid == kMidThreads - 1) {        // T has been read: this workgroup's share of its counter
            const uint32_t all = a.bands * a.tiles, members = (all - wg % kDecGroups + kDecGroups - 1u) / kDecGroups;
            atomicAdd(a.epoch + (wg % kDecGroups) * kDecGroupStride, wg < kDecGroups ? 65537ull - members : 1ull);
        }
#pragma unroll
        for (int s = 0; s < RS; ++s)
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    red[((wave * RS + s) * MB * 4 + mb * 4 + v) * 64 + lane] =
                        f32x4{acc[s0 + s][mb][4 * v], acc[s0 + s][mb][4 * v + 1], acc[s0 + s][mb][4 * v + 2], acc[s0 + s][mb][4 * v + 3]};
        __syncthreads();
        for (int pr = wave; pr < PAIRS; pr += kMidWaves) {
            const int j = pr & 1, mb = (pr >> 1) % MB, s = (pr >> 1) / MB;
            f32x4 sum[2];
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                f32x4 p[kMidWaves];
#pragma unroll
                for (int w = 0; w < kMidWaves; ++w) p[w] = red[((w * RS + s) * MB * 4 + mb * 4 + 2 * j + v) * 64 + lane];
                sum[v] = p[0];
#pragma unroll
                for (int w = 1; w < kMidWaves; ++w)
#pragma unroll
                    for (int e = 0; e < 4; ++e) sum[v][e] += p[w][e];
            }
            const uint32_t m = 32u * mb + i32, nb = n0 + 32u * (s0 + s) + 16u * j;
            if (m >= rows) continue;
            u32x2 o[2];
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                if (BF) {
                    o[v] = u32x2{pack_bf16(sum[v][0], sum[v][1]), pack_bf16(sum[v][2], sum[v][3])};
                } else {
                    f16x4 x;
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[e] = (f16)sum[v][e];
                    o[v] = __builtin_bit_cast(u32x2, x);
                }
            }
            // lanes i and i + 32 exchange quads, so that each holds eight consecutive features
            const u32x2 x0 = __builtin_amdgcn_permlane32_swap(o[0].x, o[1].x, false, false);
            const u32x2 x1 = __builtin_amdgcn_permlane32_swap(o[0].y, o[1].y, false, false);
            const uint32_t n = nb + 8u * h;
            if (n < N) *reinterpret_cast<u32x4*>(a.Y + (uint64_t)(row0 + m) * N + n) = u32x4{x0.x, x1.x, x0.y, x1.y};
        }
    }
}

// ---------------------------------------------------------------- host side

template <int MB, int ROWS, int S>
static int launch_mid_one(const MidArgs& a, hipStream_t stream) {
    const int mode = (a.w.flags & MILO_ACT_BF16) ? 2 : (a.w.flags & MILO_W3_SYMMETRIC) ? 1 : 0;
    auto k = mode == 2 ? w3lr_mid_kernel<MB, ROWS, S, 2> : mode == 1 ? w3lr_mid_kernel<MB, ROWS, S, 1> : w3lr_mid_kernel<MB, ROWS, S, 0>;
    constexpr int lds = kMidWaves * ROWS * 256;
    static bool raised[3][64] = {{false}};
    if (lds > 64 * 1024) {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return MILO_ERR_HIP;
        if (!raised[mode][dev]) {
            if (hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess)
                return MILO_ERR_HIP;
            raised[mode][dev] = true;
        }
    }
    k<<<dim3(a.nt + a.nmain), dim3(kMidThreads), lds, stream>>>(a);
    return launch_status();
}

// Parts of K in which T = X V^T is formed: about eight chunks each, one per wave of a worker, at most eight parts and (so that
// large batches and ranks do not crowd the others out) about 64 workers.
static int64_t mid_rank_items(int64_t M, int r) { return (M + 31) / 32 * ((r + 31) / 32); }
static int64_t mid_t_parts(int64_t M, int64_t K, int r) {
    const int64_t items = mid_rank_items(M, r), nchunks = (K / kGroup + 1) / 2;
    int64_t parts = (nchunks + 7) / 8;
    if (parts > 8) parts = 8;
    if (items * parts > 64) parts = 64 / items;
    return parts < 1 ? 1 : parts;
}

// The forms of the kernel and the constants of their estimates (us, see mid_plan).
struct MidForm {
    int rows, streams, per_cu;          // rows of a tile, 32-feature streams of a wave, workgroups that fit on a CU
    double start, wg, chunk;            // launch; per round of workgroups: each, and each chunk of a wave
    double partly;                      // share of a round's time that one with few workgroups takes
    double lr, rank32;                  // any compensator, and every 32 ranks
};
static const MidForm kMidForms[] = {
    {32, 1, 2, 2.40, 1.73, 2.00, 0.45, 1.04, 0.42},
    {32, 2, 2, 2.01, 3.17, 2.90, 0.49, 0.66, 0.46},
    {64, 2, 1, 1.86, 3.46, 2.32, 0.69, 0.28, 0.64},
    {80, 2, 1, 3.54, 1.81, 2.62, 0.79, 0.40, 0.75},
};

// Rounds of w workgroups at `cap` at a time.  At two per CU a round of up to half of that takes `partly`, one that doubles a
// CU up 0.72 of the full time and more.
static double mid_rounds(int64_t w, int64_t cus, const MidForm& f) {
    const int64_t cap = cus * f.per_cu, full = w / cap, rem = w - full * cap;
    if (rem == 0) return (double)full;
    if (f.per_cu == 1) return full + f.partly + (1.0 - f.partly) * (double)rem / (double)cap;
    return full + (rem <= cus ? f.partly : 0.72 + 0.28 * (double)(rem - cus) / (double)cus);
}

// Form of the kernel for a problem that the tiled kernel would run with tiles of 32 mb rows, `splits` K splits and t_parts
// parts of T (-1: that one takes it).  All are compared by estimates, fits to 7600 points (1900 shapes of 512 .. 14336 x
// 512 .. 14336, 17 .. 1200 rows, ranks 0 .. 128).  Of several rounds each pays the low-rank term's two trips through memory
// (and an INT3 compensator's conversion, 2 us), which the fits take for one, so from the second round on the estimate has to
// be further below the tiled kernel's.  Of 37305 other points (fp16, bf16, symmetric, INT3 compensators; in replayed graphs)
// 23369 go here and are 1.80 times as fast as with the tiled kernel (geometric mean); 93 are slower by more than 2 %, 53 by more
// than 5 %, at worst by 26 % (81 rows of 5760 x 9792, symmetric, INT3 r = 32, 27.6 / 34.6: a few more workgroups than CUs).
// Asking for a lead of an eighth where K is split into six parts and more would mend fifty and lose four hundred that are up to
// 1.4 times as fast here.  The tiled kernel stays where its tiles fill the chip: us, tiled / this one, 256 rows of 14336 x 4096
// 47 / 54, 1188 of 3952 x 13120 182 / 209, 1023 of 3392 x 2880, r = 32 42 / 48.
static int mid_form(int64_t M, int64_t N, int64_t K, int r, bool lr3, int mb, int splits, int t_parts) {
    const int64_t cus = device_cus(), nchunks = (K / kGroup + 1) / 2;
    const int64_t workers = r > 0 ? mid_rank_items(M, r) * mid_t_parts(M, K, r) : 0;
    const double ranks = (double)r / 32.0;
    int best = -1;
    double least = 0.0;
    for (int i = 0; i < (int)(sizeof(kMidForms) / sizeof(kMidForms[0])); ++i) {
        const MidForm& f = kMidForms[i];
        if (f.rows % 32 != 0 && M > f.rows) continue;               // (T is formed in blocks of 32 rows)
        const int64_t wgs = (N + 32 * f.streams - 1) / (32 * f.streams) * ((M + f.rows - 1) / f.rows) + workers;
        const double rounds = mid_rounds(wgs, cus, f);
        double t = f.start + rounds * (f.wg + f.chunk * (double)((nchunks + kMidWaves - 1) / kMidWaves) + (lr3 ? 2.0 : 0.0)) +
                   (r > 0 ? f.lr + f.rank32 * ranks : 0.0);
        t /= rounds <= 1.0 ? 0.94 : 0.84;
        if (best < 0 || t < least) {
            best = i;
            least = t;
        }
    }
    const int64_t m_tiles = (M + 32 * mb - 1) / (32 * mb), tiled_wgs = m_tiles * ((N + 255) / 256) * splits + m_tiles * t_parts, cap = 2 * cus;
    const int64_t full = tiled_wgs / cap, rem = tiled_wgs - full * cap;
    const double rounds = full + (rem > 0 ? 0.36 + 0.64 * (double)rem / (double)cap : 0.0);
    const double chunk = mb == 1 ? 1.04 : mb == 2 ? 1.71 : 3.44;
    const double tiled = 4.29 + rounds * (5.03 + chunk * (double)((nchunks + splits - 1) / splits)) +
                         (splits > 1 ? 3.31 + 0.21 * 4e-6 * (double)M * (double)N * splits : 0.0) + (r > 0 ? 0.73 + 2.26 * ranks : 0.0);
    return least < tiled ? best : -1;
}

constexpr int64_t kMidMaxRows = 1200;       // (measured up to there)

bool plan_mid(int64_t M, int64_t N, int64_t K, int r, bool lr3, int mb, int splits, int t_parts, MidPlan* p) {
    if (M > kMidMaxRows || r > MILO_LR3_MAX_RANK || mid_rank_items(M, r) > kMidMaxWorkers) return false;
    // 32-bit offsets, also of the rows past the end that a tile asks for
    if ((uint64_t)(M + 128) * K * 2 >= 0xFFFFFFF0ull || ((uint64_t)r + 32) * K * 2 >= 0xFFFFFFF0ull) return false;
    p->form = mid_form(M, N, K, r, lr3, mb, splits, t_parts);
    p->t_parts = r > 0 ? (int)mid_t_parts(M, K, r) : 0;
    return p->form >= 0;
}

void mid_plan_shape(const MidPlan& p, int* rows, int* streams) {
    *rows = kMidForms[p.form].rows;
    *streams = kMidForms[p.form].streams;
}

int launch_mid(MidArgs a, const MidPlan& p, hipStream_t stream) {
    const MidForm& f = kMidForms[p.form];
    a.tile_rows = f.rows;
    a.bands = (a.N + 32u * f.streams - 1u) / (32u * f.streams);
    a.tiles = (a.M + a.tile_rows - 1u) / a.tile_rows;
    a.nmain = a.bands * a.tiles;
    a.once = a.tiles == 1;
    a.t_parts = (uint32_t)p.t_parts;
    a.rank_blocks = (uint32_t)(a.w.r + 31) / 32u;
    a.nt = (a.M + 31u) / 32u * a.rank_blocks * a.t_parts;
    a.spin_limit = 1u << 20;
    switch (p.form) {
        case 0: return launch_mid_one<1, 32, 1>(a, stream);
        case 1: return launch_mid_one<1, 32, 2>(a, stream);
        case 2: return launch_mid_one<2, 64, 2>(a, stream);
        default: return launch_mid_one<3, 80, 2>(a, stream);
    }
}

}  // namespace milo
