// milo_moe_w3lr_forward: top-k routed SwiGLU experts over compensated W3A16 linears.
//
// Launch sequence on the caller's stream (no host synchronisation in between):
//   route     group the (token, slot) pairs per expert: stable placement by counting and scans,
//             and each expert's M-tiles in its own slots of a tile list
//   order     work list = the filled slots, full tiles first, then the partly filled ones
//             (batches of up to 512 pairs: both in one launch)
//   gate/up   H = SiLU(lin_w1(x)) * lin_w3(x), both projections in one grouped launch, which
//             also forms T1 = X V1^T and T3 = X V3^T (low-rank inputs) in its leading columns
//   down      O[split][pair] = gate_weight * lin_w2(H) over the split's share of K (fp16, or fp32 from gemm_few.hip; one row
//             per routed pair); T2 = H V2^T is formed inside this launch as well
//             (a few rows per expert: the two launches are gemm_few.hip's, else gemm_tiled.hip's)
//   combine   y_t = fp16( sum over the token's slots and the K splits, in a fixed order, of O )
#include <math.h>
#include <stdlib.h>

#include <type_traits>

#include "milo_host.h"
#include "milo_kernels.h"

namespace milo {

constexpr int kRouteThreads = 1024;

struct RouteArgs {
    const int32_t* ids;     // [P] expert id per (token, slot) pair, pair index p = t*topk + j
    int32_t P;
    int32_t E;
    int32_t bm;             // rows per M-tile
    int32_t topk;
    int32_t* sorted;        // [P] pair indices grouped by expert, original order inside a group
    int32_t* sorted_token;  // [P] token of each sorted pair (pair / topk)
    TileDesc* tiles;
    int32_t* header;        // [0] routing status, [1] number of tiles, [3] wait status (a wait gave up)
    uint32_t* flags;        // per-tile control words of the GEMM kernels, cleared here
    int32_t n_flags;
    int32_t max_tiles;      // slots of the tile list: ceil(P / bm) + E
};

// One workgroup per expert; no workgroup depends on another one, so a single launch suffices.
// A wave owns a contiguous range of the pairs, 256 of them per step (a lane four neighbours, one 16-byte load) and eight steps
// of them in registers, and finds its expert's pairs with one ballot per lane slot: the stable position of a pair inside
// the expert's group is the number of matches in the waves before, in the steps before and, by bit counts, in the lanes before;
// the group starts at the number of ids below the expert.  No histogram over all experts is needed (LDS atomics of a
// whole workgroup on the few popular experts serialize badly): expert e places its tiles from slot floor(start_e / bm) + e of
// the tile list, which never overlaps the next expert's first slot, and marks the slots up to there as empty.
// Bound by latency (the loads, one exchange between the waves) and by the stores of the popular experts, 4 bytes per lane and two
// per pair: 32768 pairs of 66 experts 14 us, 1024 of 8 7.9 (20 and 8.7 when a thread walked its range twice, with a
// division per pair).
__global__ __launch_bounds__(kRouteThreads) void route_kernel(const RouteArgs a) {
    constexpr int kWaves = kRouteThreads / 64, kHeld = 8;
    __shared__ int32_t s_eq[kWaves], s_less[kWaves], s_bad[kWaves];

    const int e = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int steps = (a.P + 256 * kWaves - 1) / (256 * kWaves);        // 256 pairs each
    const int lo = wave * steps * 256 + 4 * lane;
    // (a pair past the end reads as an id of nobody)
    auto load = [&](int i0) {
        int4 v = {-1, -1, -1, -1};
        if (i0 + 4 <= a.P) {
            v = *reinterpret_cast<const int4*>(a.ids + i0);
        } else {
            if (i0 < a.P) v.x = a.ids[i0];
            if (i0 + 1 < a.P) v.y = a.ids[i0 + 1];
            if (i0 + 2 < a.P) v.z = a.ids[i0 + 2];
        }
        return v;
    };
    int n_eq = 0, n_less = 0;
    bool bad = false;
    auto count = [&](int i0, const int4& v) {
        const int id[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            n_eq += __popcll(__builtin_amdgcn_ballot_w64(id[j] == e));
            n_less += (uint32_t)id[j] < (uint32_t)e;
        }
        if (e == 0) {
#pragma unroll
            for (int j = 0; j < 4; ++j) bad = bad || ((uint32_t)id[j] >= (uint32_t)a.E && i0 + j < a.P);
        }
    };
    int4 held[kHeld];
#pragma unroll
    for (int s = 0; s < kHeld; ++s)
        if (s < steps) held[s] = load(lo + 256 * s);
#pragma unroll
    for (int s = 0; s < kHeld; ++s)
        if (s < steps) count(lo + 256 * s, held[s]);
    for (int s = kHeld; s < steps; ++s) count(lo + 256 * s, load(lo + 256 * s));
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) n_less += __shfl_xor(n_less, d, 64);
    const bool any_bad = __builtin_amdgcn_ballot_w64(bad) != 0ull;
    if (lane == 0) {
        s_eq[wave] = n_eq;
        s_less[wave] = n_less;
        s_bad[wave] = any_bad;
    }
    __syncthreads();
    int before = 0, off_e = 0, count_e = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        before += w < wave ? s_eq[w] : 0;
        count_e += s_eq[w];
        off_e += s_less[w];
    }
    // stable scatter of the pairs routed to expert e
    int at = off_e + before;
    const unsigned long long below = (1ull << lane) - 1ull;
    // pair / topk from the upper half of a product: short by at most one for pairs below 2^30
    const uint32_t magic = a.topk > 1 ? (uint32_t)((1ull << 32) / (uint32_t)a.topk) : 0xffffffffu;
    auto token_of = [&](int i) {
        const uint32_t t = __umulhi((uint32_t)i, magic);
        return (int)(t + ((uint32_t)i - t * (uint32_t)a.topk >= (uint32_t)a.topk ? 1u : 0u));
    };
    auto scatter = [&](int i0, const int4& v) {
        const int id[4] = {v.x, v.y, v.z, v.w};
        unsigned long long m[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) m[j] = __builtin_amdgcn_ballot_w64(id[j] == e);
        if ((m[0] | m[1] | m[2] | m[3]) == 0ull) return;
        int pos = at;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            pos += __popcll(m[j] & below);
            at += __popcll(m[j]);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (id[j] == e) {
                a.sorted[pos] = i0 + j;
                a.sorted_token[pos] = token_of(i0 + j);
                ++pos;
            }
    };
    if (n_eq) {
#pragma unroll
        for (int s = 0; s < kHeld; ++s)
            if (s < steps) scatter(lo + 256 * s, held[s]);
        for (int s = kHeld; s < steps; ++s) scatter(lo + 256 * s, load(lo + 256 * s));
    }
    // this expert's slots of the tile list: its tiles, then empty slots up to the next expert's first
    const int tile0 = off_e / a.bm + e;
    const int tile1 = (e + 1 < a.E) ? (off_e + count_e) / a.bm + e + 1 : a.max_tiles;
    const int nt = (count_e + a.bm - 1) / a.bm;
    for (int i = tid; i < tile1 - tile0; i += kRouteThreads) {
        TileDesc td;
        td.expert = e;
        td.row0 = off_e + (i < nt ? i * a.bm : 0);
        td.rows = i < nt ? ((count_e - i * a.bm) < a.bm ? (count_e - i * a.bm) : a.bm) : 0;
        td.pad = 0;
        a.tiles[tile0 + i] = td;
    }
    if (e == 0) {
        // every workgroup has looked at all ids; this one reports the ones out of range
        for (int i = tid; i < a.n_flags; i += kRouteThreads) a.flags[i] = 0u;
        if (tid == 0) {
            int32_t found = 0;
            for (int w = 0; w < kWaves; ++w) found |= s_bad[w];
            a.header[0] = found ? MILO_ERR_ROUTING : MILO_OK;
            a.header[1] = a.max_tiles;
            a.header[3] = 0;
        }
    }
}

// Work list of the grouped GEMMs: the slots the experts filled, compacted (empty slots dropped) and
// put longest first: a tile costs about what its number of 32-row blocks says, and more with a
// compensator of high rank, so tiles go by that number, most blocks first, within it those of
// experts with a rank above 32 first, in expert order within a class.  The dispatcher hands out workgroups
// in list order, so the launch ends with the short items.  One workgroup; a wave owns a contiguous range of slots, counts
// each class with a ballot, and one scan over (class, wave) gives every wave the place of its first tile of each class.
// Latency-bound (slots, ranks of their experts, the scan, the stores): 5.4 us, also in a trace that gave the form with a scan
// per class over all threads and a second pass over the slots 13.
__global__ __launch_bounds__(kRouteThreads) void order_tiles_kernel(const TileDesc* __restrict__ slots,
                                                                    int n_slots, int bm,
                                                                    TileDesc* __restrict__ tiles,
                                                                    int32_t* __restrict__ header,
                                                                    const milo_w3lr_expert* __restrict__ experts) {
    constexpr int NC = 8, kWaves = kRouteThreads / 64;  // classes: bm / 32 blocks down to one, x rank
    static_assert(NC * kWaves == 128, "two entries per lane of the scan");
    __shared__ int32_t s_at[NC * kWaves + 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int steps = (n_slots + kRouteThreads - 1) / kRouteThreads;
    const int lo = wave * steps * 64 + lane;
    const int mb = bm / 32;
    auto load = [&](int i) {
        TileDesc td = {0, 0, 0, 0};
        if (i < n_slots) td = slots[i];
        return td;
    };
    auto cls = [&](const TileDesc& td) {                // 0: as many blocks as a full tile, high rank; -1: no tile
        const int nb = (td.rows + 31) / 32;
        const milo_w3lr_expert& ex = experts[td.expert];
        const int low = (ex.w1.r <= 32 && ex.w3.r <= 32 && ex.w2.r <= 32) ? 1 : 0;
        return td.rows > 0 ? 2 * (mb - (nb < mb ? nb : mb)) + low : -1;
    };
    int cnt[NC] = {0, 0, 0, 0, 0, 0, 0, 0};
    TileDesc td = load(lo);
    int c = cls(td);
    for (int s = 0; s < steps; ++s) {
        if (s > 0) c = cls(load(lo + 64 * s));
#pragma unroll
        for (int k = 0; k < NC; ++k) cnt[k] += __popcll(__builtin_amdgcn_ballot_w64(c == k));
    }
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < NC; ++k) s_at[k * kWaves + wave] = cnt[k];
    }
    __syncthreads();
    if (wave == 0) {
        const int x = s_at[2 * lane], y = s_at[2 * lane + 1];
        int sum = x + y;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int v = __shfl_up(sum, d, 64);
            if (lane >= d) sum += v;
        }
        s_at[2 * lane] = sum - x - y;
        s_at[2 * lane + 1] = sum - y;
        if (lane == 63) s_at[NC * kWaves] = sum;
    }
    __syncthreads();
    // From kXcdPlacementTiles tiles on, the tiled kernel reads the list as eight contiguous ranges,
    // one per sequence of workgroups (range k starts at k * (n / 8) + min(k, n % 8)).  Position p of
    // the order goes to range p % 8, place p / 8, so that every range gets the same mix and ends
    // with its short items.
    const int n = s_at[NC * kWaves], base = n >> 3, rem = n & 7;
    auto place = [&](int p) {
        if (n < (int)kXcdPlacementTiles) return p;          // the kernel takes the list in order
        const int k = p & 7;
        return k * base + (k < rem ? k : rem) + (p >> 3);
    };
    int pos[NC];
#pragma unroll
    for (int k = 0; k < NC; ++k) pos[k] = s_at[k * kWaves + wave];
    const unsigned long long below = (1ull << lane) - 1ull;
    for (int s = 0; s < steps; ++s) {
        if (steps > 1) {
            td = load(lo + 64 * s);
            c = cls(td);
        }
        int p = 0;
#pragma unroll
        for (int k = 0; k < NC; ++k) {
            const unsigned long long m = __builtin_amdgcn_ballot_w64(c == k);
            if (c == k) p = pos[k] + __popcll(m & below);
            pos[k] += __popcll(m);
        }
        if (c >= 0) tiles[place(p)] = td;
    }
    if (tid == 0) header[1] = n;
}

// Routing and work list in one launch for decode-sized batches (at most kSmallPairs routed pairs and
// kSmallExperts experts): with a handful of tokens the two kernels above are all latency, and so is
// the launch between them.  One workgroup routes; thread p owns pair p, thread e expert e.  The group of an expert
// starts at the number of pairs with a smaller id, a pair's place inside it is the number of earlier pairs with
// the same id, which is the same stable order as route_kernel's.  Tiles are written straight into the final list: tiles of
// experts with a rank above 32 first, then the others, in expert order (order_tiles_kernel's order for tiles of one height
// class).  `items` given: the list is the weight-streaming kernel's, `n_items` slots with the expert's weights beside the rows
// and no rows in those that stay empty, and the other workgroups of the launch clear the granules of T.
// Latency-bound; every thread has its expert's ranks on the way before the ids arrive and no loop goes to memory.
// FEW (up to kFewPairs pairs): every thread counts from a copy of the ids in LDS, four per read.  That loop grows with the
// pairs; more of them are counted per wave: the lanes whose ids agree in all nine bits come from one ballot per bit, the
// lowest lane of each id writes the wave's count (nothing is added atomically), and scans over waves and experts do the rest.
// us, all ids per thread / per wave: 2 pairs 4.1 / 5.0, 32 5.0 / 4.9, 60 6.2 / 5.3, 128 8.9 / 5.3, 512 22.0 / 5.4 (the two
// general kernels take 12.9 for those).  In one kernel the two cost each other 0.5 us, code that is fetched and not run.
constexpr int kSmallPairs = 512, kSmallExperts = 512, kFewPairs = 32;
template <bool FEW>
__global__ __launch_bounds__(kSmallPairs) void route_small_kernel(const RouteArgs a, TileDesc* __restrict__ list,
                                                                  const milo_w3lr_expert* __restrict__ experts,
                                                                  FewItem* __restrict__ items, int n_items,
                                                                  u32x4* __restrict__ granules, uint32_t granules16) {
    constexpr int kWaves = kSmallPairs / 64, kIdBits = 9;
    static_assert(kSmallExperts == 1 << kIdBits && kSmallExperts == kSmallPairs, "a thread per expert, ids of kIdBits bits");
    __shared__ __attribute__((aligned(16))) int32_t s_id[FEW ? kSmallPairs : 4];
    __shared__ int32_t s_wave[FEW ? 1 : kWaves][kSmallExperts];     // pairs of a wave per expert, then those of the waves before it
    __shared__ int32_t s_start[kSmallExperts], s_tile0[kSmallExperts];
    __shared__ int32_t s_hi[kWaves], s_lo[kWaves], s_cnt[kWaves];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (blockIdx.x > 0) {
        for (uint32_t i = (blockIdx.x - 1) * kSmallPairs + tid; i < granules16; i += (gridDim.x - 1) * kSmallPairs)
            granules[i] = u32x4{0u, 0u, 0u, 0u};
        return;
    }
    int id = -1;
    if (tid < a.P) {
        id = a.ids[tid];
        if (id < 0 || id >= a.E) id = -1;
    }
    const WeightDev* const ew = reinterpret_cast<const WeightDev*>(experts + (tid < a.E ? tid : 0));
    const WeightDev w0 = ew[0], w1 = ew[1], w2 = ew[2];
    // pair p = tid: earlier pairs of its expert; expert e = tid: its pairs and those before its group
    int before = 0, cnt = 0, less = 0;
    if constexpr (FEW) {
        s_id[tid] = id;
    } else {
#pragma unroll
        for (int w = 0; w < kWaves; ++w) s_wave[w][tid] = 0;
    }
    const bool bad = __syncthreads_or(tid < a.P && id < 0) != 0;
    if constexpr (FEW) {
#pragma unroll 4
        for (int p = 0; p < a.P; p += 4) {
            const int4 v4 = *reinterpret_cast<const int4*>(s_id + p);       // (entries from P on are -1)
            const int v[4] = {v4.x, v4.y, v4.z, v4.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                before += v[i] == id && p + i < tid;
                cnt += v[i] == tid;
                less += (uint32_t)v[i] < (uint32_t)tid;
            }
        }
    } else {
        unsigned long long same = __builtin_amdgcn_ballot_w64(id >= 0);
#pragma unroll
        for (int b = 0; b < kIdBits; ++b) {
            const bool set = (id >> b & 1) != 0;
            const unsigned long long m = __builtin_amdgcn_ballot_w64(set);
            same &= set ? m : ~m;
        }
        before = __popcll(same & ((1ull << lane) - 1ull));
        if (id >= 0 && before == 0) s_wave[wave][id] = __popcll(same);
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const int n = s_wave[w][tid];
            s_wave[w][tid] = cnt;
            cnt += n;
        }
        less = cnt;                                         // (scanned over the wave's experts, then over the waves)
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int c = __shfl_up(less, d, 64);
            if (lane >= d) less += c;
        }
        if (lane == 63) s_cnt[wave] = less;
        less -= cnt;
    }
    // tiles of the experts before this one, those with a high rank ahead of all others
    const bool low = w0.r <= 32 && w1.r <= 32 && w2.r <= 32;
    const int nt = tid < a.E ? (cnt + a.bm - 1) / a.bm : 0;
    int hi = low ? 0 : nt, lo = low ? nt : 0;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int h = __shfl_up(hi, d, 64), l = __shfl_up(lo, d, 64);
        if (lane >= d) {
            hi += h;
            lo += l;
        }
    }
    if (lane == 63) {
        s_hi[wave] = hi;
        s_lo[wave] = lo;
    }
    if constexpr (FEW) s_start[tid] = less;
    __syncthreads();
    if constexpr (!FEW) {
#pragma unroll
        for (int w = 0; w < kWaves; ++w) less += w < wave ? s_cnt[w] : 0;
        s_start[tid] = less;
    }
    int total_hi = 0, total = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        if (w < wave) {
            hi += s_hi[w];
            lo += s_lo[w];
        }
        total_hi += s_hi[w];
        total += s_hi[w] + s_lo[w];
    }
    const int tile0 = (low ? total_hi + lo : hi) - nt;
    s_tile0[tid] = tile0;
    for (int i = 0; i < nt; ++i) {
        const int row0 = less + i * a.bm, rows = cnt - i * a.bm < a.bm ? cnt - i * a.bm : a.bm;
        if (items) {
            FewItem& it = items[tile0 + i];
            it.expert = tid; it.row0 = row0; it.rows = rows; it.pad = 0;
            it.w[0] = w0; it.w[1] = w1; it.w[2] = w2;
        } else {
            list[tile0 + i] = TileDesc{tid, row0, rows, 0};
        }
    }
    if (items)
        for (int i = total + tid; i < n_items; i += kSmallPairs) items[i].rows = 0;
    if (!FEW || items) __syncthreads();
    if (id >= 0) {
        if constexpr (!FEW) before += s_wave[wave][id];
        const int pos = s_start[id] + before, token = tid / a.topk;
        a.sorted[pos] = tid;
        if (items) items[s_tile0[id] + before / kFewRows].token[before % kFewRows] = token;
        else a.sorted_token[pos] = token;
    }
    for (int i = tid; i < a.n_flags; i += kSmallPairs) a.flags[i] = 0u;
    if (tid == 0) {
        a.header[0] = bad ? MILO_ERR_ROUTING : MILO_OK;
        a.header[1] = total;
        a.header[3] = 0;
    }
}

// y[t, h..h+3] = fp16( sum_j O[t*topk + j, h..h+3] ), slots in order, invalid ids skipped.  BF: rows
// and result are bfloat16.  WIDE: the rows are fp32 (decode-sized batches, where they are a few hundred KB).
template <bool BF, bool WIDE>
__global__ __launch_bounds__(256) void combine_kernel(const void* __restrict__ O, int splits,
                                                      int64_t split_stride,
                                                      const int32_t* __restrict__ ids, int E,
                                                      int topk, int64_t T, int64_t H,
                                                      f16* __restrict__ Y) {
    const int64_t t = blockIdx.y;
    const int64_t h = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
    if (h >= H) return;
    // rows are added slot by slot, split by split; eight loads are in flight at a time
    f32x4 sum = {0.0f, 0.0f, 0.0f, 0.0f};
    const int total = topk * splits;
    for (int base = 0; base < total; base += 8) {
        typename std::conditional<WIDE, f32x4, u32x2>::type v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int q = base + i;
            const int j = q / splits, s = q - j * splits;
            bool ok = q < total;
            if (ok) {
                const int id = ids[t * topk + j];
                ok = id >= 0 && id < E;
            }
            const int64_t at = s * split_stride + (t * topk + j) * H + h;
            v[i] = {};
            if (ok) {
                if constexpr (WIDE) v[i] = *reinterpret_cast<const f32x4*>(static_cast<const float*>(O) + at);
                else v[i] = *reinterpret_cast<const u32x2*>(static_cast<const f16*>(O) + at);
            }
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if constexpr (WIDE) {
#pragma unroll
                for (int e = 0; e < 4; ++e) sum[e] += v[i][e];
            } else if constexpr (BF) {       // a bfloat16 is the upper half of the binary32 with the same value
                sum[0] += __builtin_bit_cast(float, v[i].x << 16);
                sum[1] += __builtin_bit_cast(float, v[i].x & 0xffff0000u);
                sum[2] += __builtin_bit_cast(float, v[i].y << 16);
                sum[3] += __builtin_bit_cast(float, v[i].y & 0xffff0000u);
            } else {
                const f16x4 f = __builtin_bit_cast(f16x4, v[i]);
#pragma unroll
                for (int e = 0; e < 4; ++e) sum[e] += (float)f[e];
            }
        }
    }
    u32x2 ob;
    if (BF) {
        ob = u32x2{pack_bf16(sum[0], sum[1]), pack_bf16(sum[2], sum[3])};
    } else {
        f16x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (f16)sum[e];
        ob = __builtin_bit_cast(u32x2, o);
    }
    *reinterpret_cast<u32x2*>(Y + t * H + h) = ob;
}

struct MoeLayout {
    int bm;
    int max_tiles;
    int64_t ldt;
    int parts_up, parts_down;   // parts of T = X V^T for the gate/up and the down projection
    int splits_down;            // K splits of the down projection
    size_t off_header, off_flags, off_sorted, off_token, off_slots, off_tiles, off_t1, off_t3, off_tp1, off_tp3, off_h, off_o, total;
    int64_t max_tiles32;
    // the weight-streaming kernel
    int few_items;              // slots of its item list (0: the tiled kernel runs)
    int few_frags;              // fragments of 32 ranks of T
    size_t off_items, off_granules, granule_bytes;
};

// Tiles of b rows that P evenly spread pairs give E experts, on average: sum over the row counts n of ceil(n / b), n Poisson
// and cut at P (which for one to three experts takes up to half off both numbers that moe_takes_few compares).
static double expected_tiles(int64_t P, int E, int b) {
    const double mean = (double)P / E;
    double p = exp(-mean), tiles = 0.0;
    for (int n = 1; n <= (int)P && (n <= mean || p > 1e-9); ++n) {
        p *= mean / n;
        tiles += p * ((n + b - 1) / b);
    }
    return tiles * E;
}

static bool moe_few_possible(int64_t H, int64_t F, int E, int r_max) {
    return E <= kSmallExperts && r_max <= kFewMaxRank && few_t_parts(H) <= kFewMaxParts && few_t_parts(F) <= kFewMaxParts;
}

// Whether the weight-streaming kernel takes a batch (else the tiled one).  Estimates per layer in us: the streaming one takes
// 14 + 0.17 per MB of weight it reads, once per item of 16 rows, + 0.007 per workgroup; the tiled one 45 + 0.19 per MB, once per
// 32-row tile.  So it is the number of rows per expert that decides, later where the weights are small.  Measured, streamed /
// tiled: 14336 x 4096, 8 experts, 4 rows each 133 / 168, 12 rows 162 / 176, 16 rows 204 / 181; 3584 x 1024, 16 experts, 16 rows
// 48 / 51, 24 rows 61 / 52; 1408 x 2048, 64 + 2 experts, 0.5 rows 41 / 76, 8 rows 90 / 107; 1024 x 512, 8 experts, 24 rows 21 / 38.
// The counts are those of evenly spread pairs.  Popular experts need more items for the tiles they save, but unpopular ones
// neither: with popularity falling as rank^-1.2 the first two layers take 118 / 149, 194 / 198, 220 / 208 and 51 / 63, 62 / 66.
// Of 2875 points measured (158 shapes, both kinds of routing) 2163 are streamed; 19 of them are slower than tiled, by 2 to
// 12 % and in one layer by 21 % (two experts of 13120 x 2112, each with 25 rows: two items for one tile, 60 / 50), and 409 of the
// others would be faster streamed.
static bool moe_takes_few(int64_t T, int64_t H, int64_t F, int E, int topk, int r_max) {
    const int64_t P = T * topk;
    if (P > kSmallPairs || !moe_few_possible(H, F, E, r_max)) return false;
    const double mb = 3.0 * 0.4375e-6 * (double)H * (double)F, groups = (double)((F + 31) / 32 + (H + 63) / 64);
    return 14.0 + expected_tiles(P, E, kFewRows) * (0.17 * mb + 0.007 * groups) < 45.0 + 0.19 * mb * expected_tiles(P, E, 32);
}

// Layout of the weight-streaming kernel; grows with T.
static void moe_few_layout(int64_t T, int64_t H, int64_t F, int E, int topk, int r_max, MoeLayout* L) {
    const int64_t P = T * topk;
    // every expert with rows may have one item that is not full
    const int64_t used = P < E ? P : E, items = used + P / kFewRows;
    L->bm = kFewRows;
    L->few_items = (int)(items < P ? items : P);
    L->few_frags = (r_max + 31) / 32;
    // granules of a fragment of T: two values each, or one each of several parts
    const int parts = few_t_parts(F), up = 2 * 256, down = parts > 1 ? 512 * parts : 256;
    L->granule_bytes = (size_t)L->few_items * L->few_frags * (up > down ? up : down) * 8;
    L->splits_down = 1;
    size_t off = 0;
    L->off_header = off; off = align_up(off + 64, 256);
    L->off_sorted = off; off = align_up(off + (size_t)P * 4, 256);
    L->off_token = 0;
    L->off_items = off;  off = align_up(off + (size_t)L->few_items * sizeof(FewItem), 256);
    L->off_granules = off; off = align_up(off + L->granule_bytes, 256);
    L->off_h = off;      off = align_up(off + (size_t)P * F * 2, 256);
    L->off_o = off;      off = align_up(off + (size_t)P * H * 4, 256);       // (fp32)
    L->total = off;
}

// The layout of a call with a workspace of `have` bytes.  With too few for the weight-streaming kernel the call goes to the
// tiled one, which for some shapes needs less (66 experts of 1408 x 2048, 62 tokens: 7.2 MB against 10.6).
static bool moe_layout(int64_t T, int64_t H, int64_t F, int E, int topk, int r_max, size_t have, MoeLayout* L) {
    if (T <= 0 || E <= 0 || topk <= 0 || r_max < 0) return false;
    if (!weight_shape_ok(F, H) || !weight_shape_ok(H, F)) return false;
    if (H % 4 != 0) return false;
    const int64_t P = T * topk;
    if (P > (int64_t)0x3fffffff || E > 65536) return false;
    if (((uint64_t)r_max + 256) * (uint64_t)(H > F ? H : F) * 2 >= 0xFFFFFFF0ull) return false;
    // activations are addressed with 32-bit offsets inside the kernels
    if ((uint64_t)T * H * 2 >= 0x80000000ull || (uint64_t)P * F * 2 >= 0x80000000ull) return false;
    // tuning override, read once per process so that the workspace query and the call agree
    static const int bm_override = [] {
        const char* e = getenv("MILO_MOE_BM");
        const int v = e ? atoi(e) : 0;
        return (v == 32 || v == 64 || v == 128) ? v : 0;
    }();
    if (!bm_override && moe_takes_few(T, H, F, E, topk, r_max)) {
        moe_few_layout(T, H, F, E, topk, r_max, L);
        if (have >= L->total) return true;
    }
    L->few_items = 0;
    const int64_t avg = P / E;
    // Tile height: an expert whose rows do not fit one tile streams its weights once more, a
    // taller tile costs more activation copies and a shallower pipeline; measured on the Mixtral
    // shape the crossovers lie near 26 and 56 rows per expert.
    L->bm = avg >= 56 ? 128 : (avg >= 26 ? 64 : 32);
    if (bm_override) L->bm = bm_override;
    const int64_t max_tiles32 = (P + 31) / 32 + E;      // bound for the smallest tile height
    const int64_t max_tiles = (P + L->bm - 1) / L->bm + E;
    if (max_tiles > 65535) return false;
    L->max_tiles = (int)max_tiles;
    L->ldt = ((int64_t)r_max + 15) / 16 * 16;
    L->parts_up = r_max > 0 ? tiled_t_parts(H) : 0;
    L->parts_down = r_max > 0 ? tiled_t_parts(F) : 0;
    const int parts = L->parts_up > L->parts_down ? L->parts_up : L->parts_down;
    if ((uint64_t)(parts > 0 ? parts : 1) * (uint64_t)P * (uint64_t)L->ldt * 4 >= 0xFFFFFFF0ull) return false;
    // the down projection has few column tiles (hidden / 256): split K when they do not fill the chip
    // (counted in full tiles: the partly filled last tile of an expert is cheap)
    int64_t est_tiles = (P + L->bm - 1) / L->bm;
    int split_cap = 64;
    if (L->bm == 32) {
        // Small batches: nearly every tile is an expert's only, partly filled one, and it costs a
        // full pass over the expert's weight whatever its rows, so the tiles to count are the experts
        // that receive anything: E (1 - (1 - 1/E)^P) for evenly spread pairs.  Measured on the Mixtral
        // shape (16, 4 and 1 tokens), splits beyond eight lose more to short workgroups than they gain.
        const double used = (double)E * (1.0 - pow(1.0 - 1.0 / (double)E, (double)P));
        if ((int64_t)(used + 0.5) > est_tiles) est_tiles = (int64_t)(used + 0.5);
        split_cap = 8;
    }
    L->splits_down = tiled_k_splits(est_tiles * ((H + 255) / 256), F, 0);
    if (L->splits_down > split_cap) L->splits_down = split_cap;
    static const int splits_override = [] {
        const char* e = getenv("MILO_MOE_SPLITS");
        const int v = e ? atoi(e) : 0;
        return (v >= 1 && v <= 16) ? v : 0;
    }();
    if (splits_override) L->splits_down = splits_override;
    size_t off = 0;
    L->off_header = off; off = align_up(off + 64, 256);
    L->max_tiles32 = max_tiles32;
    L->off_flags = off;  off = align_up(off + 2 * (size_t)max_tiles32 * 16, 256);   // gate/up launch, down launch
    L->off_sorted = off; off = align_up(off + (size_t)P * 4, 256);
    L->off_token = off;  off = align_up(off + (size_t)P * 4, 256);
    L->off_slots = off;  off = align_up(off + (size_t)max_tiles32 * sizeof(TileDesc), 256);
    L->off_tiles = off;  off = align_up(off + (size_t)max_tiles32 * sizeof(TileDesc), 256);
    L->off_t1 = off;     off = align_up(off + (size_t)P * L->ldt * 2, 256);
    L->off_t3 = off;     off = align_up(off + (size_t)P * L->ldt * 2, 256);
    L->off_tp1 = off;    off = align_up(off + (size_t)parts * P * L->ldt * 4, 256);
    L->off_tp3 = off;    off = align_up(off + (size_t)L->parts_up * P * L->ldt * 4, 256);
    L->off_h = off;      off = align_up(off + (size_t)P * F * 2, 256);
    L->off_o = off;      off = align_up(off + (size_t)L->splits_down * P * H * 2, 256);
    L->total = off;
    return true;
}

// Sums the rows of every token's pairs (and K splits) into Y.
static int launch_combine(const void* O, bool wide, int splits, int64_t split_stride, const int32_t* ids, int E, int topk, int64_t T,
                          int64_t H, f16* Y, bool bf, hipStream_t stream) {
    const unsigned gx = (unsigned)((H / 4 + 255) / 256);
    auto kern = wide ? (bf ? combine_kernel<true, true> : combine_kernel<false, true>)
                     : (bf ? combine_kernel<true, false> : combine_kernel<false, false>);
    for (int64_t t0 = 0; t0 < T; t0 += 65535) {         // (grid.y limit)
        const int64_t nt = (T - t0) < 65535 ? (T - t0) : 65535;
        kern<<<dim3(gx, (unsigned)nt), dim3(256), 0, stream>>>(static_cast<const char*>(O) + t0 * topk * H * (wide ? 4 : 2), splits,
                                                               split_stride, ids + t0 * topk, E, topk, nt, H, Y + t0 * H);
    }
    return launch_status();
}

static int check_weight(const milo_w3lr_weight& w, int64_t N, int64_t K) {
    if (!w.q3) return MILO_ERR_NULL;
    if (w.r < 0 || w.r > N || w.r > K) return MILO_ERR_RANK;
    if (w.r > 0 && (!w.U || !w.V)) return MILO_ERR_RANK;
    if (w.flags & ~(MILO_W3_SYMMETRIC | MILO_LR_INT3)) return MILO_ERR_SHAPE;
    if (w.r > 0 && (w.flags & MILO_LR_INT3)) {
        if (w.r > MILO_LR3_MAX_RANK) return MILO_ERR_RANK;
        if ((N % kGroup) != 0) return MILO_ERR_SHAPE;
    }
    if (!aligned16(w.q3) || !aligned16(w.U) || !aligned16(w.V))
        return MILO_ERR_ALIGN;
    return MILO_OK;
}

}  // namespace milo

using namespace milo;

extern "C" int milo_moe_w3lr_check_experts(const milo_w3lr_expert* experts, int E, int64_t H,
                                           int64_t F, int* r_max_out) {
    return milo_moe_w3lr_check_experts_flags(experts, E, H, F, 0u, r_max_out);
}

extern "C" int milo_moe_w3lr_check_experts_flags(const milo_w3lr_expert* experts, int E, int64_t H,
                                                 int64_t F, unsigned flags, int* r_max_out) {
    if (!experts) return MILO_ERR_NULL;
    if (flags & ~MILO_ACT_BF16) return MILO_ERR_SHAPE;
    if (E <= 0 || !weight_shape_ok(F, H) || !weight_shape_ok(H, F)) return MILO_ERR_SHAPE;
    int r_max = 0;
    for (int e = 0; e < E; ++e) {
        const milo_w3lr_weight* ws[3] = {&experts[e].w1, &experts[e].w3, &experts[e].w2};
        for (int i = 0; i < 3; ++i) {
            const int64_t N = (i < 2) ? F : H, K = (i < 2) ? H : F;
            const int st = check_weight(*ws[i], N, K);
            if (st != MILO_OK) return st;
            // the bf16 kernels read U and V as bf16 arrays: no INT3 compensators there
            if ((flags & MILO_ACT_BF16) && ws[i]->r > 0 && (ws[i]->flags & MILO_LR_INT3)) return MILO_ERR_SHAPE;
            if (ws[i]->r > r_max) r_max = ws[i]->r;
        }
        // gate and up projection share a launch: their compensators are both INT3 or both fp16
        if (experts[e].w1.r > 0 && experts[e].w3.r > 0 &&
            ((experts[e].w1.flags ^ experts[e].w3.flags) & MILO_LR_INT3))
            return MILO_ERR_SHAPE;
    }
    if (r_max_out) *r_max_out = r_max;
    return MILO_OK;
}

extern "C" size_t milo_moe_w3lr_workspace(int64_t T, int64_t H, int64_t F, int E, int topk,
                                          int r_max) {
    MoeLayout L;
    if (!moe_layout(T, H, F, E, topk, r_max, SIZE_MAX, &L)) return 0;
    size_t bytes = L.total;
    // A workspace sized for a batch that is tiled serves smaller, streamed ones at full speed as well: room for the
    // largest of those.
    if (L.few_items == 0 && moe_few_possible(H, F, E, r_max) && topk <= kSmallPairs) {
        MoeLayout S;
        moe_few_layout(T < kSmallPairs / topk ? T : kSmallPairs / topk, H, F, E, topk, r_max, &S);
        if (S.total > bytes) bytes = S.total;
    }
    return bytes;
}

extern "C" int milo_moe_w3lr_forward(const milo_half* X, int64_t T, int64_t H, int64_t F,
                                     const milo_w3lr_expert* experts, int E, int r_max,
                                     const int32_t* topk_ids, const float* topk_weights, int topk,
                                     milo_half* Y, void* workspace, size_t workspace_bytes,
                                     void* stream_) {
    return milo_moe_w3lr_forward_flags(X, T, H, F, experts, E, r_max, topk_ids, topk_weights, topk, 0u, Y, workspace,
                                       workspace_bytes, stream_);
}

extern "C" int milo_moe_w3lr_forward_flags(const milo_half* X, int64_t T, int64_t H, int64_t F,
                                           const milo_w3lr_expert* experts, int E, int r_max,
                                           const int32_t* topk_ids, const float* topk_weights, int topk,
                                           unsigned call_flags, milo_half* Y, void* workspace, size_t workspace_bytes,
                                           void* stream_) {
    if (!X || !experts || !topk_ids || !topk_weights || !Y) return MILO_ERR_NULL;
    if (call_flags & ~MILO_ACT_BF16) return MILO_ERR_SHAPE;
    const int bf = (call_flags & MILO_ACT_BF16) ? 1 : 0;
    MoeLayout L;
    if (!moe_layout(T, H, F, E, topk, r_max, workspace_bytes, &L)) return MILO_ERR_SHAPE;
    if (r_max > H || r_max > F) return MILO_ERR_RANK;
    if (!workspace || workspace_bytes < L.total) return MILO_ERR_WORKSPACE;
    if (!aligned16(X) || !aligned16(Y) || !aligned16(workspace) || !aligned16(experts) ||
        !aligned16(topk_ids) || !aligned16(topk_weights))
        return MILO_ERR_ALIGN;
    hipStream_t stream = (hipStream_t)stream_;
    char* ws = reinterpret_cast<char*>(workspace);
    int32_t* header = reinterpret_cast<int32_t*>(ws + L.off_header);
    int32_t* sorted = reinterpret_cast<int32_t*>(ws + L.off_sorted);
    int32_t* sorted_token = reinterpret_cast<int32_t*>(ws + L.off_token);
    f16* Hbuf = reinterpret_cast<f16*>(ws + L.off_h);
    void* O = ws + L.off_o;
    const int P = (int)(T * topk);
    RouteArgs ra;
    ra.ids = topk_ids; ra.P = P; ra.E = E; ra.bm = L.bm;
    ra.topk = topk; ra.sorted = sorted; ra.sorted_token = sorted_token; ra.header = header;
    int st;
    if (L.few_items > 0) {
        FewItem* items = reinterpret_cast<FewItem*>(ws + L.off_items);
        u32x4* granules = reinterpret_cast<u32x4*>(ws + L.off_granules);
        ra.tiles = nullptr; ra.flags = nullptr; ra.n_flags = 0; ra.max_tiles = 0;
        const size_t clear_blocks = (L.granule_bytes / 16 + 4 * kSmallPairs - 1) / (4 * kSmallPairs);
        const auto route = P <= kFewPairs ? route_small_kernel<true> : route_small_kernel<false>;
        route<<<dim3(1u + (unsigned)(clear_blocks < 128 ? clear_blocks : 128)), dim3(kSmallPairs), 0, stream>>>(
            ra, nullptr, experts, items, L.few_items, granules, (uint32_t)(L.granule_bytes / 16));
        st = launch_status();
        if (st != MILO_OK) return st;
        FewArgs fa;
        fa.items = items; fa.n_items = (uint32_t)L.few_items;
        fa.t_parts = 0; fa.bands = 0;
        fa.N = (uint32_t)F; fa.K = (uint32_t)H;
        fa.X = reinterpret_cast<const f16*>(X); fa.x_bytes = (uint32_t)(T * H * 2);
        fa.granules = reinterpret_cast<unsigned long long*>(granules); fa.t_frags = (uint32_t)L.few_frags; fa.tag = 1u;
        fa.spin_limit = 1u << 20; fa.status = reinterpret_cast<uint32_t*>(header + 3);
        fa.out = Hbuf; fa.out_rows = nullptr; fa.out_scale = nullptr;
        st = launch_few(fa, 2, bf != 0, stream);
        if (st != MILO_OK) return st;
        fa.N = (uint32_t)H; fa.K = (uint32_t)F;
        fa.X = Hbuf; fa.x_bytes = (uint32_t)((int64_t)P * F * 2);
        fa.tag = 2u;
        fa.out = O; fa.out_rows = sorted; fa.out_scale = topk_weights;
        st = launch_few(fa, 1, bf != 0, stream);
        if (st != MILO_OK) return st;
        return launch_combine(O, true, 1, (int64_t)P * H, topk_ids, E, topk, T, H, reinterpret_cast<f16*>(Y), bf != 0, stream);
    }
    TileDesc* slots = reinterpret_cast<TileDesc*>(ws + L.off_slots);
    TileDesc* tiles = reinterpret_cast<TileDesc*>(ws + L.off_tiles);
    f16* T1 = reinterpret_cast<f16*>(ws + L.off_t1);
    f16* T3 = reinterpret_cast<f16*>(ws + L.off_t3);
    float* Tp1 = reinterpret_cast<float*>(ws + L.off_tp1);
    float* Tp3 = reinterpret_cast<float*>(ws + L.off_tp3);
    uint32_t* flags = reinterpret_cast<uint32_t*>(ws + L.off_flags);
    ra.tiles = slots;
    ra.flags = flags; ra.n_flags = (int32_t)(2 * 4 * L.max_tiles32);
    ra.max_tiles = L.max_tiles;
    if (P <= kSmallPairs && E <= kSmallExperts && L.bm == 32) {
        const auto route = P <= kFewPairs ? route_small_kernel<true> : route_small_kernel<false>;
        route<<<dim3(1), dim3(kSmallPairs), 0, stream>>>(ra, tiles, experts, nullptr, 0, nullptr, 0u);
        st = launch_status();
        if (st != MILO_OK) return st;
    } else {
        route_kernel<<<dim3((unsigned)E), dim3(kRouteThreads), 0, stream>>>(ra);
        st = launch_status();
        if (st != MILO_OK) return st;
        order_tiles_kernel<<<dim3(1), dim3(kRouteThreads), 0, stream>>>(slots, L.max_tiles, L.bm, tiles, header, experts);
        st = launch_status();
        if (st != MILO_OK) return st;
    }

    RowSpace rs;
    rs.tiles = tiles; rs.n_tiles = header + 1; rs.experts = experts;
    rs.M = P;
    const int mb = L.bm / 32;
    // with few rows per expert nearly every expert is a single tile: its weights are read once
    const int once = L.bm < 64 ? 1 : 0;

    // gate / up projection
    rs.which[0] = 0; rs.which[1] = 1;
    rs.x_rows = sorted_token;
    {
        TiledArgs ga;
        ga.rs = rs; ga.X = reinterpret_cast<const f16*>(X); ga.ldx = H; ga.x_bytes = (uint64_t)T * H * 2;
        ga.N = F; ga.K = H;
        ga.T[0] = T1; ga.T[1] = T3; ga.ldt = L.ldt; ga.t_bytes = (uint64_t)P * L.ldt * 2;
        ga.Tp[0] = Tp1; ga.Tp[1] = Tp3; ga.tp_bytes = (uint64_t)L.parts_up * P * L.ldt * 4;
        ga.t_part_stride = (int64_t)P * L.ldt; ga.t_parts = L.parts_up; ga.v_tiles = L.parts_up; ga.ksplit = 1;
        ga.out_split_stride = 0; ga.flags = flags; ga.self_clean = 0; ga.weights_once = once;
        ga.t_dist = 0; ga.lr_splits = 1; ga.lr_step = 0; ga.act_bf16 = bf;
        ga.flags_status = reinterpret_cast<uint32_t*>(header + 3);
        ga.lr3_rank = bf ? 0 : (r_max < MILO_LR3_MAX_RANK ? r_max : MILO_LR3_MAX_RANK);    // (any weight's compensator may be INT3)
        ga.out = Hbuf; ga.ldo = F; ga.out_rows = nullptr; ga.out_scale = nullptr;
        st = launch_tiled(ga, 2, mb, EPI_SWIGLU, L.max_tiles, stream);
        if (st != MILO_OK) return st;
    }
    // down projection (T2 reuses the T1 buffer: T1 is dead once the gate/up kernel has run)
    rs.which[0] = 2; rs.which[1] = 2;
    rs.x_rows = nullptr;
    {
        TiledArgs da;
        da.rs = rs; da.X = Hbuf; da.ldx = F; da.x_bytes = (uint64_t)P * F * 2;
        da.N = H; da.K = F;
        da.T[0] = T1; da.T[1] = T1; da.ldt = L.ldt; da.t_bytes = (uint64_t)P * L.ldt * 2;
        da.Tp[0] = Tp1; da.Tp[1] = Tp1; da.tp_bytes = (uint64_t)L.parts_down * P * L.ldt * 4;
        da.t_part_stride = (int64_t)P * L.ldt; da.t_parts = L.parts_down; da.v_tiles = L.parts_down;
        da.ksplit = L.splits_down; da.out_split_stride = (int64_t)P * H; da.flags = flags + 4 * L.max_tiles32;
        da.self_clean = 0; da.weights_once = once;
        da.t_dist = 0; da.lr_splits = 1; da.lr_step = 0; da.act_bf16 = bf;
        da.flags_status = reinterpret_cast<uint32_t*>(header + 3);
        da.lr3_rank = bf ? 0 : (r_max < MILO_LR3_MAX_RANK ? r_max : MILO_LR3_MAX_RANK);
        da.out = O; da.ldo = H; da.out_rows = sorted; da.out_scale = topk_weights;
        st = launch_tiled(da, 1, mb, EPI_SCALE_SCATTER, L.max_tiles, stream);
        if (st != MILO_OK) return st;
    }
    return launch_combine(O, false, L.splits_down, (int64_t)P * H, topk_ids, E, topk, T, H, reinterpret_cast<f16*>(Y), bf != 0, stream);
}

extern "C" int milo_moe_w3lr_routing_status(const void* workspace, void* stream) {
    if (!workspace) return MILO_ERR_NULL;
    int32_t header[4] = {0, 0, 0, 0};
    if (hipMemcpyAsync(header, workspace, sizeof(header), hipMemcpyDeviceToHost,
                       (hipStream_t)stream) != hipSuccess)
        return MILO_ERR_HIP;
    if (hipStreamSynchronize((hipStream_t)stream) != hipSuccess) return MILO_ERR_HIP;
    if (header[3] != 0) return MILO_ERR_WAIT;       // a wait inside a kernel gave up
    return header[0] == MILO_OK ? MILO_OK : MILO_ERR_ROUTING;
}
