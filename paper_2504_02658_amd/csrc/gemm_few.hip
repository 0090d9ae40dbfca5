// Weight-streaming kernel for the grouped linears of an MoE layer whose experts get a few rows each (decode-sized
// batches): the gate and up projections with SwiGLU (NW = 2), the down projection (NW = 1).
//
// Work split.  An item is one expert with up to sixteen of its rows.  A workgroup of four waves streams a band of the
// expert's weight rows over the whole K for one item: K goes in chunks of 256 columns, dealt to the waves (chunk c to
// wave c mod 4).  A wave holds R 16-row blocks of each of its NW weights: per chunk and
// block one unit per lane (a 16- and a 12-byte load), converted in registers and multiplied with the chunk's
// activations (mfma 16x16x32), which the wave gathers into an LDS slot of its own.  The partial sums of the four
// waves meet in LDS and are added in wave order.  No K split crosses workgroups.
//
// What bounds it: HBM and the vector units together (125 vector instructions convert 1.8 KB).  Every weight is read once
// per sixteen rows of its expert.  Four small workgroups fit on a CU, so that while one starts (two round trips to
// memory) or ends, others convert; with eight waves each, two on a CU, they do so in step.  The gate/up launch of eight
// experts of 14336 x 4096 at 16 tokens, 411 MB, us on average and at least: 86 / 80 against 92 / 85 with eight waves (the
// down launch, whose waves hold one weight, 49 / 46 against 48 / 45).  Its loads alone take 68 / 66 (6.1 TB/s), and the vector
// units are busy for 71 % of it.  The tiled kernel, which took such batches before, walks 32-row tiles with 128 columns a step
// and two steps of requests in flight: 102 / 97 there, and 38 against 16 at 4 tokens of a layer of 66 experts of 1408 x 2048.
//
// Low-rank term.  T = X V^T of an item is formed inside the launch by the first workgroups of the grid, one per block of
// 16 ranks (and, in the down projection, K part of 16 chunks), and handed over in tagged
// granules: 8 bytes of values and a tag, polled as single 64-bit accesses, so that the data is its own flag.  The
// routing kernel clears the granules of a forward, the two launches use different tags.  A T of one part is rounded by its
// worker, two values to a granule; several parts travel as fp32 and the streaming workgroups add them, in
// part order, before the one rounding.  Workers never wait and have the lowest workgroup ids.
// (One workgroup per 32 ranks over the whole K was the longest chain of a launch: K = 14336,
// rank 64, 62 -> 48 us.)
#include "milo_host.h"
#include "milo_kernels.h"
#include "stream_device.h"

namespace milo {



template <bool BF>
__device__ __forceinline__ f32x4 few_mfma(u32x4 a, u32x4 b, f32x4 c) {
    if constexpr (BF) return mfma16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c);
    else return mfma16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c);
}
template <bool BF>
__device__ __forceinline__ u32x2 few_pack4(f32x4 v) {
    if constexpr (BF) return u32x2{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
    f16x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = (f16)v[e];
    return __builtin_bit_cast(u32x2, o);
}

constexpr int kFewWaves = 4, kFewThreads = 64 * kFewWaves;
constexpr int kFewTLds = kFewWaves * kStreamSlotBytes;         // T fragments behind the slots: [fragment][64 lanes] x 16 B

// Granules of fragment i (32 ranks) of K part `part` of an item's weight: [4][64 lanes], or [8][64 lanes] with several parts.
__device__ __forceinline__ unsigned long long* few_fragment(const FewArgs& a, uint32_t weight, int part, int i) {
    return a.granules + ((size_t)(weight * a.t_frags + i) * a.t_parts + part) * (a.t_parts > 1u ? 512u : 256u);
}

// Byte offset in X of the item's row j (kOobRow: no such row; stays past every buffer when a column is added).
constexpr uint32_t kOobRow = 0x80000000u;
template <int NW>
__device__ __forceinline__ uint32_t few_row_offset(const FewArgs& a, const FewItem& it, int j) {
    const int row = NW == 2 ? it.token[j] : it.row0 + j;
    return j < it.rows ? (uint32_t)row * (2u * a.K) : kOobRow;
}

// T worker: block jb of 16 ranks of weight `w` of the item over K part `part` (kFewTChunks chunks, or all: there is no room
// for adding parts up beside the accumulators of two weights); both operands go straight from
// memory to registers (16 rows x 64 contiguous bytes per load), and the partial sums of the waves are added in wave order.
template <int NW, bool BF>
__device__ __forceinline__ void few_t_worker(const FewArgs& a, const FewItem& it, const WeightDev& w, uint32_t item, int which,
                                             int jb, int part, unsigned char* smem) {
    if (16 * jb >= w.r) return;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, j16 = lane & 15, q = lane >> 4;
    const uint32_t K = a.K, G = K / kGroup;
    const uint32_t c_lo = (uint32_t)(part * kFewTChunks), c_hi = NW == 2 ? (K + 255u) / 256u : c_lo + kFewTChunks;
    const BufRsrc xb = make_rsrc(a.X, a.x_bytes);
    const uint32_t xo = few_row_offset<NW>(a, it, j16);
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    if (!BF && (w.flags & MILO_LR_INT3)) {
        // V is a blob [pad16(r) x K] in the layout of a weight: unit of rank 16 jb + j16, group 4 c + q
        const W3Buf vq = make_w3buf(w.V, (w.r + 15) & ~15, K);
        for (uint32_t c = c_lo + wave; c < c_hi && c * 256u < K; c += kFewWaves) {
            const bool ok = 4u * c + q < G;
            const RawUnit u = load_unit_buf(vq, ok ? ((uint32_t)jb * G + 4u * c) * 16u + lane : (1u << 27));
            u32x4 b[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) b[t] = buf_load16(xb, ok ? xo + c * 512u + q * 128u + t * 16u : kOobOffset);
            dequant_unit_steps<true>(u, [&](int t, f16x8 frag) { acc = mfma16(frag, __builtin_bit_cast(f16x8, b[t]), acc); });
        }
    } else {
        const BufRsrc vb = make_rsrc(w.V, (uint64_t)w.r * K * 2u);
        const uint32_t vo = 16 * jb + j16 < w.r ? (uint32_t)(16 * jb + j16) * (2u * K) : kOobOffset;
        for (uint32_t c = c_lo + wave; c < c_hi && c * 256u < K; c += kFewWaves) {
            u32x4 v[8], b[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const uint32_t col = c * 512u + t * 64u;        // (K is a multiple of 64: 32 columns are there or not)
                const bool ok = col < 2u * K;
                v[t] = buf_load16(vb, ok && vo != kOobOffset ? vo + col + q * 16u : kOobOffset);
                b[t] = buf_load16(xb, ok ? xo + col + q * 16u : kOobOffset);
            }
#pragma unroll
            for (int t = 0; t < 8; ++t) acc = few_mfma<BF>(v[t], b[t], acc);
        }
    }
    f32x4* const red = reinterpret_cast<f32x4*>(smem);
    red[wave * 64 + lane] = acc;
    __syncthreads();
    if (wave != 0) return;
    f32x4 sum = red[lane];
#pragma unroll
    for (int k = 1; k < kFewWaves; ++k) {
        const f32x4 p = red[k * 64 + lane];
#pragma unroll
        for (int e = 0; e < 4; ++e) sum[e] += p[e];
    }
    // element v = rank 16 jb + 4 q + v, row j16: element 4 (q % 2) + v of lane (j16, 2 (jb % 2) + q / 2) in the fragment of
    // k-step jb / 2
    if (NW == 1 && a.t_parts > 1u) {
        unsigned long long* const frag = few_fragment(a, item * NW + which, part, jb >> 1);
        const uint32_t at = 4u * (q & 1) * 64u + (2u * (jb & 1) + (q >> 1)) * 16u + j16;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            __hip_atomic_store(frag + at + 64 * e, (unsigned long long)a.tag << 32 | __builtin_bit_cast(uint32_t, (float)sum[e]),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }
    const u32x2 ob = few_pack4<BF>(sum);
    unsigned long long* const frag = few_fragment(a, item * NW + which, part, jb >> 1);
    const uint32_t at = 2u * (q & 1) * 64u + (2u * (jb & 1) + (q >> 1)) * 16u + j16;
    __hip_atomic_store(frag + at, (unsigned long long)a.tag << 32 | ob.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(frag + at + 64, (unsigned long long)a.tag << 32 | ob.y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One fragment of T (32 ranks x 16 rows) as an MFMA B fragment to LDS, polled until every granule carries the
// launch's tag; a wait that gives up sets the status word.  `none`: this lane's ranks do not exist.
template <int NW, bool BF>
__device__ __forceinline__ void few_fetch_t(const FewArgs& a, const unsigned long long* frag, bool none, int lane, unsigned char* dst) {
    if (NW == 1 && a.t_parts > 1u) {
        constexpr int PT = 2;       // parts per trip to memory
        f32x4 lo = {0.0f, 0.0f, 0.0f, 0.0f}, hi = {0.0f, 0.0f, 0.0f, 0.0f};
        for (uint32_t p = 0; p < a.t_parts; p += PT) {
            const bool two = p + 1u < a.t_parts;
            const unsigned long long* const f[2] = {frag + p * 512u, frag + (two ? p + 1u : p) * 512u};
            for (uint32_t spins = 0;; ++spins) {
                unsigned long long g[PT][8];
                bool ok = true;
#pragma unroll
                for (int k = 0; k < PT; ++k)
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        g[k][e] = __hip_atomic_load(f[k] + e * 64 + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                for (int k = 0; k < PT; ++k)
#pragma unroll
                    for (int e = 0; e < 8; ++e) ok = ok && (uint32_t)(g[k][e] >> 32) == a.tag;
                if (__builtin_amdgcn_ballot_w64(!(ok || none)) == 0ull || spins > a.spin_limit) {
#pragma unroll
                    for (int k = 0; k < PT; ++k)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            if (none || (k == 1 && !two)) continue;
                            lo[e] += __builtin_bit_cast(float, (uint32_t)g[k][e]);
                            hi[e] += __builtin_bit_cast(float, (uint32_t)g[k][4 + e]);
                        }
                    if (spins > a.spin_limit && lane == 0) atomicOr(a.status, 1u);
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
        }
        const u32x2 l = few_pack4<BF>(lo), h = few_pack4<BF>(hi);
        *reinterpret_cast<u32x4*>(dst + lane * 16) = u32x4{l.x, l.y, h.x, h.y};
        return;
    }
    for (uint32_t spins = 0;; ++spins) {
        unsigned long long g[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) g[e] = __hip_atomic_load(frag + e * 64 + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        bool ok = true;
        u32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            ok = ok && (uint32_t)(g[e] >> 32) == a.tag;
            v[e] = none ? 0u : (uint32_t)g[e];
        }
        if (__builtin_amdgcn_ballot_w64(!(ok || none)) == 0ull || spins > a.spin_limit) {
            *reinterpret_cast<u32x4*>(dst + lane * 16) = v;
            if (spins > a.spin_limit && lane == 0) atomicOr(a.status, 1u);
            break;
        }
        __builtin_amdgcn_s_sleep(1);
    }
}

// The stream of one wave.  Request order and counts are those of the decode kernel's stream (gemm_decode.hip), with
// U = NW R units per chunk: X0 W00 .. W0(U-1) | X1 W10 | W11 | ..; the build script checks them.
//   unit (j, 0): 2 (U - 1) younger operations; unit (j, b > 0): 2 (U - 1) + XC; last chunk: 2 (U - 1 - b)
template <int NW, int R, int XC, bool BF>
struct FewStream {
    static constexpr int U = NW * R;
    const W3Buf (&wb)[NW];
    BufRsrc xb;
    uint32_t row[2 * XC];       // byte offsets of the item's rows (scalars)
    unsigned char* slot;
    uint32_t K, G, NB, rb0, first, lane;

    __device__ __forceinline__ uint32_t chunk_of(uint32_t j) const { return first + kFewWaves * j; }
    __device__ __forceinline__ void issue_x(uint32_t j) const {
        const uint32_t kc = chunk_of(j) * 256u;
        const uint32_t lim = K - kc >= 256u ? 512u : 2u * (K - kc);         // (kc < K: a wave walks its own chunks only)
        const uint32_t crow = lane >> 5, cp = lane & 31u;
#pragma unroll
        for (int i = 0; i < XC; ++i) {
            const uint32_t seg = (cp ^ (2u * i + crow)) << 4;               // slot position p of row j holds segment p ^ j
            const uint32_t off = (crow ? row[2 * i + 1] : row[2 * i]) + (2u * kc + seg), o = seg < lim ? off : kOobOffset;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(xb, (LdsPtr)(slot + i * 1024), 16, o, 0, 0, 0);
        }
        asm volatile("" ::: "memory");
    }
    __device__ __forceinline__ void issue_w(uint32_t j, int b, RawUnit& u) const {
        const uint32_t c = chunk_of(j), rb = rb0 + (uint32_t)(b % R);
        const bool ok = 4u * c + (lane >> 4) < G && rb < NB;
        u = load_unit_buf_once(wb[b / R], ok ? (rb * G + 4u * c) * 16u + lane : (1u << 27));
        asm volatile("" ::: "memory");
    }
    template <bool LAST>
    __device__ __forceinline__ void chunk(uint32_t j, RawUnit (&u)[U], f32x4 (&acc)[U]) const {
        f16x8 bfrag[8];
        static_for<0, U>([&](auto b_c) {
            constexpr int b = decltype(b_c)::value;
            __builtin_amdgcn_sched_barrier(0);
            MILO_WAIT_VMEM(LAST ? 2 * (U - 1 - b) : (b == 0 ? 2 * (U - 1) : 2 * (U - 1) + XC));
            __builtin_amdgcn_sched_barrier(0);
            if (b == 0) {
                read_bfrags(slot, (int)(lane & 15u), (int)(lane >> 4), bfrag);
                if (!LAST) {
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // the slot is free again
                    issue_x(j + 1);
                }
            }
            pin_unit_params(u[b]);
            if constexpr (BF)
                dequant_unit_steps_bf16(u[b], [&](int t, bf16x8 frag) {
                    acc[b] = mfma16_bf16(frag, __builtin_bit_cast(bf16x8, bfrag[t]), acc[b]);
                });
            else
                dequant_unit_steps<false>(u[b], [&](int t, f16x8 frag) { acc[b] = mfma16(frag, bfrag[t], acc[b]); });
            if (!LAST) {
                __builtin_amdgcn_sched_barrier(0);
                issue_w(j + 1, b, u[b]);
            }
        });
    }
    // the wave's chunks 0 .. C - 1 (C >= 1)
    __device__ __forceinline__ void run(uint32_t C, f32x4 (&acc)[U]) const {
        RawUnit u[U];
        issue_x(0);
#pragma unroll
        for (int b = 0; b < U; ++b) issue_w(0, b, u[b]);
        for (uint32_t j = 0; j + 1 < C; ++j) chunk<false>(j, u, acc);
        chunk<true>(C - 1, u, acc);
    }
};

template <int NW, int R, bool BF>
__global__ __launch_bounds__(kFewThreads, 4) void w3lr_few_kernel(const FewArgs a) {
    constexpr int U = NW * R;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const uint32_t per_item = NW * a.t_frags * 2u * a.t_parts, nt = a.n_items * per_item;
    const bool worker = blockIdx.x < nt;
    const uint32_t idx = worker ? blockIdx.x : blockIdx.x - nt;
    const uint32_t item = idx / (worker ? per_item : a.bands), rest = idx - item * (worker ? per_item : a.bands);
    const FewItem& it = a.items[item];
    if (it.rows <= 0) return;
    const WeightDev w0 = it.w[NW == 2 ? 0 : 2], w1 = it.w[NW == 2 ? 1 : 2];
    if (worker) {
        const uint32_t per_weight = per_item / NW, which = rest / per_weight, r2 = rest - which * per_weight;
        const uint32_t jb = r2 / a.t_parts;
        few_t_worker<NW, BF>(a, it, which == 0 ? w0 : w1, item, (int)which, (int)jb, (int)(r2 - jb * a.t_parts), smem);
        return;
    }
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t chunks = (a.K + 255u) / 256u;
    const uint32_t NB = a.N >> 4, rb0 = rest * R;
    W3Buf wb[NW];
    wb[0] = make_w3buf(w0.q3, a.N, a.K);
    wb[NW - 1] = make_w3buf(w1.q3, a.N, a.K);
    const uint32_t my_row = few_row_offset<NW>(a, it, threadIdx.x & 15);
    unsigned char* const slot = smem + wave * kStreamSlotBytes;
    f32x4 acc[U];
#pragma unroll
    for (int b = 0; b < U; ++b) acc[b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    // One instance of the stream per number of activation copies: rows that the item does not have are not copied (what the
    // slot held there only reaches output columns that are not stored).
    auto stream = [&](auto xc) {
        constexpr int XC = decltype(xc)::value;
        FewStream<NW, R, XC, BF> st{wb, make_rsrc(a.X, a.x_bytes), {}, slot, a.K, a.K / kGroup, NB, rb0, (uint32_t)wave, threadIdx.x & 63u};
#pragma unroll
        for (int i = 0; i < 2 * XC; ++i) st.row[i] = (uint32_t)__builtin_amdgcn_readlane((int)my_row, i);
        if ((uint32_t)wave < chunks) st.run((chunks - wave + kFewWaves - 1u) / kFewWaves, acc);
    };
    if (it.rows <= 4) stream(std::integral_constant<int, 2>{});
    else if (it.rows <= 8) stream(std::integral_constant<int, 4>{});
    else stream(std::integral_constant<int, 8>{});
    // the epilogue's lane number, counted anew: carried across the streaming loop, it and what is derived from it spill there
    uint32_t every = ~0u;
    asm volatile("" : "+s"(every));
    const int lane = (int)__builtin_amdgcn_mbcnt_hi(every, __builtin_amdgcn_mbcnt_lo(every, 0u)), j16 = lane & 15, q = lane >> 4;
    f32x4* const red = reinterpret_cast<f32x4*>(smem);         // wave w, unit b at 512 w + 64 b
#pragma unroll
    for (int b = 0; b < U; ++b) red[wave * (kStreamSlotBytes / 16) + b * 64 + lane] = acc[b];

    // What the epilogue needs besides the partial sums: the fragments of T, dealt to the waves, and for wave b < R, which
    // finishes row block b, the U rows.  (Asked for before the last unit is converted they gained nothing.)
    const int r0 = w0.r, r1 = NW == 2 ? w1.r : 0;
    const int ks0 = (r0 + 31) >> 5, ks1 = (r1 + 31) >> 5;
    for (int f = wave; f < ks0 + ks1; f += kFewWaves) {
        const bool second = f >= ks0;
        const int i = f - (second ? ks0 : 0);
        // an odd number of 16-rank blocks leaves the upper half of the last k-step without ranks
        const bool none = ((((second ? r1 : r0) + 15) >> 4) & 1) != 0 && lane >= 32 && i == (second ? ks1 : ks0) - 1;
        few_fetch_t<NW, BF>(a, few_fragment(a, item * NW + (second ? 1u : 0u), 0, i), none, lane, smem + kFewTLds + f * 1024);
    }
    const uint32_t blk = rb0 + (uint32_t)wave, nb16 = blk * 16u;
    const bool finish = wave < R && blk < NB;
    f16x8 uf[NW][kStreamKS];
#pragma unroll
    for (int s = 0; s < NW; ++s) {
        const WeightDev& w = s == 0 ? w0 : w1;
#pragma unroll
        for (int i = 0; i < kStreamKS; ++i) {
            const int k0 = 32 * i + 8 * q;
            uf[s][i] = zero_f16x8();
            if (finish && (BF || !(w.flags & MILO_LR_INT3)) && k0 < w.r)
                uf[s][i] = load_row8(w.U + (size_t)(nb16 + j16) * w.r, k0, w.r, (w.r & 7) == 0);
        }
    }
    int64_t orow = 0;
    float scale = 1.0f;
    if (finish && j16 < it.rows) {
        orow = it.row0 + j16;
        if (NW == 1) {
            orow = a.out_rows[orow];
            scale = a.out_scale[orow];
        }
    }
    __syncthreads();
    if (!finish) return;
    f32x4 sum[NW];
#pragma unroll
    for (int s = 0; s < NW; ++s) {
        f32x4 part[kFewWaves];
#pragma unroll
        for (int k = 0; k < kFewWaves; ++k) part[k] = red[k * (kStreamSlotBytes / 16) + (s * R + wave) * 64 + lane];
        sum[s] = part[0];
#pragma unroll
        for (int k = 1; k < kFewWaves; ++k)
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[s][e] += part[k][e];
    }
    const u32x4* const tl = reinterpret_cast<const u32x4*>(smem + kFewTLds);
#pragma unroll
    for (int s = 0; s < NW; ++s) {
        const WeightDev& w = s == 0 ? w0 : w1;
        const int ks = s == 0 ? ks0 : ks1;
        if (!BF && (w.flags & MILO_LR_INT3)) {
            // INT3 U: the blob holds U^T [pad16(r) x N] with groups of 64 along N; lane l takes rank l (then l + 64), one unit,
            // and scatters its 16 features of this block into fragments in the half of the wave's slot that no partial sum uses.
            unsigned char* const uf_lds = slot + kStreamSlotBytes / 2;
            const int rp = (w.r + 15) & ~15;
            const W3Buf ub = make_w3buf(w.U, rp, a.N);
            const uint32_t GN = a.N >> 6, g = blk >> 2, o16 = blk & 3u;
            for (int j = lane; j < 32 * ks; j += 64) {
                const RawUnit u = load_unit_buf(ub, j < rp ? ((uint32_t)(j >> 4) * GN + g) * 16u + (uint32_t)(j & 15) : (1u << 27));
                uint32_t wv[32];
                dequant_unit<true>(u, wv);
                unsigned char* const frag0 = uf_lds + (((j >> 5) * 64 + ((j & 31) >> 3) * 16) * 16 + (j & 7) * 2);
                if (o16 == 0) scatter_u_rank<1, 0>(wv, frag0);
                else if (o16 == 1) scatter_u_rank<1, 1>(wv, frag0);
                else if (o16 == 2) scatter_u_rank<1, 2>(wv, frag0);
                else scatter_u_rank<1, 3>(wv, frag0);
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            for (int i = 0; i < ks; ++i)
                sum[s] = few_mfma<BF>(reinterpret_cast<const u32x4*>(uf_lds)[i * 64 + lane], tl[((s ? ks0 : 0) + i) * 64 + lane], sum[s]);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // (read before the next weight's fragments land there)
        } else {
#pragma unroll
            for (int i = 0; i < kStreamKS; ++i)
                if (i < ks) sum[s] = few_mfma<BF>(__builtin_bit_cast(u32x4, uf[s][i]), tl[((s ? ks0 : 0) + i) * 64 + lane], sum[s]);
        }
    }
    // element v: feature nb16 + 4 q + v, row j16
    if (j16 >= it.rows) return;
    const size_t at = (size_t)orow * a.N + nb16 + 4 * q;
    f32x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = NW == 2 ? silu<BF>(sum[0][e]) * sum[NW - 1][e] : scale * sum[0][e];
    if (NW == 2) *reinterpret_cast<u32x2*>(static_cast<f16*>(a.out) + at) = few_pack4<BF>(o);
    else *reinterpret_cast<f32x4*>(static_cast<float*>(a.out) + at) = o;
}

template <int NW, int R, bool BF>
static int few_launch(const FewArgs& a, unsigned grid, hipStream_t stream) {
    const int lds = kFewTLds + (int)(NW * a.t_frags) * 1024;
    static bool raised[64] = {false};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return MILO_ERR_HIP;
    if (!raised[dev]) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(w3lr_few_kernel<NW, R, BF>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, kFewTLds + 2 * kStreamKS * 1024) != hipSuccess)
            return MILO_ERR_HIP;
        raised[dev] = true;
    }
    w3lr_few_kernel<NW, R, BF><<<dim3(grid), dim3(kFewThreads), lds, stream>>>(a);
    return launch_status();
}
int few_t_parts(int64_t K) { return (int)((K + 256 * kFewTChunks - 1) / (256 * kFewTChunks)); }

int launch_few(FewArgs a, int nw, bool bf, hipStream_t stream) {
    // Four row blocks per wave share a chunk's activations (two of the gate and two of the up projection).  A down projection
    // with few items and a long K takes two: it has too few bands otherwise (K = 14336, 2 items: 22.8 -> 19.5 us, 5
    // items 97 -> 93 us per layer; at K = 1408 the two are equal).
    int R = 4 / nw;
    if (nw == 1 && a.K >= 4096u && (uint64_t)a.n_items * ((a.N + 63u) / 64u) < 2u * (uint32_t)device_cus()) R = 2;
    a.t_parts = nw == 2 ? 1u : (uint32_t)few_t_parts(a.K);
    a.bands = (a.N + 16u * R - 1u) / (16u * R);
    const uint64_t grid = (uint64_t)a.n_items * ((uint64_t)nw * 2 * a.t_frags * a.t_parts + a.bands);
    if (grid > 0x7fffffffull) return MILO_ERR_SHAPE;
    if (nw == 2) return bf ? few_launch<2, 2, true>(a, (unsigned)grid, stream) : few_launch<2, 2, false>(a, (unsigned)grid, stream);
    if (R == 2) return bf ? few_launch<1, 2, true>(a, (unsigned)grid, stream) : few_launch<1, 2, false>(a, (unsigned)grid, stream);
    return bf ? few_launch<1, 4, true>(a, (unsigned)grid, stream) : few_launch<1, 4, false>(a, (unsigned)grid, stream);
}

}  // namespace milo
