// Weight-streaming kernel for the compensated W3A16 linear at M <= 16 (decode): ONE launch that
// streams the packed weight once from HBM, forms T = X V^T cooperatively and adds T U^T.
//
// Weight stream (w3lr_decode_kernel; for K beyond sixteen chunks see also w3lr_decode_split_kernel).  A workgroup of sixteen
// waves owns 16*R output features over the whole K.  K is
// cut into chunks of 256 columns; wave w takes chunks w, w + 16, ... for all R 16-row blocks.  For
// a chunk a lane loads one unit per 16-row block (24 bytes of codes, fp16 scale and zero-point)
// with fully coalesced 16- and 12-byte buffer loads and no branches (lanes without data read out
// of range and get zeros), converts it in registers and feeds it as the A operand of
// v_mfma_f32_16x16x32_f16 (lane quad q = group 4c+q, eight steps of eight codes).
// The activations of a chunk, X[0..15][256c .. 256c+255], are the B operand of every block.  A wave
// copies them into its own 8-KB LDS slot with up to eight coalesced 1-KB buffer-to-LDS loads (two
// full 512-byte row pieces each, no registers involved); the 16-byte segment that sits at slot
// position p of row j is segment p ^ j of the row, which makes the later per-lane ds_read_b128 of
// the B fragments conflict free although the 16 lanes of a quad read 16 rows.  A slot is written
// and read by one wave only, so the main loop takes no barrier; the waves' partial sums are added
// in a fixed order at the very end.
//
// Why sixteen waves.  A CU accepts vector memory requests only as fast as earlier ones return, and
// a wave cannot convert anything while it is queueing requests.  Timestamps inside an eight-wave
// version (two chunks per wave, everything requested up front) showed the first wave of every SIMD
// queueing for 3 us and converting for 3.5 us, the second one queueing for 5.3 us and converting
// after that: half of the conversion ran after the last byte had arrived.  With sixteen waves of
// half the work each, a wave is through with its requests after a quarter of the stream and
// converts while the later waves of its SIMD still queue.
//
// Low-rank term.  The first `nt` workgroups do no streaming: each computes whole blocks of 16
// ranks of T = X V^T over a part of K (the parts are never added up across workgroups).  The
// streaming workgroups only need T in their epilogue, where they add T U^T with a few more MFMAs.
// Wave 0 of a streaming workgroup, whose requests are accepted first and which is therefore done
// long before the others, fetches the U rows into LDS, the other waves fetch a fragment of T each as
// they finish.  The workers never wait for anything, they have the lowest workgroup ids, and the grid
// never exceeds what the device keeps resident, so that wait always ends.  Data that crosses
// workgroups is written and read with device-coherent accesses.
//
// The hand-over of T (where it can be staged, see decode_t_plan) takes one trip through memory: T travels in 8-byte granules of
// two values and a 32-bit tag that names the launch, stored and polled as single 64-bit accesses, so
// a consumer polls the data itself.  (Stores, their acknowledgement, a counter, a poll of the counter
// and then the loads were five trips of 0.7 to 2 us, the longest chain of every decode launch, and
// clearing the counter at the end waited for every consumer to sign off.)  The tag comes from
// counters that only ever grow: each launch adds exactly 2^16 to every one of them, a consumer adds
// its share after it has read T, so whoever reads a counter before that finds the number of launches
// before this one in its upper bits.  Nothing has to be cleared between launches, in a replayed
// graph neither.
//
// What the hand-over costs beside the poll is kept off the path to the output: one wave polling all fragments
// took a trip through memory per four of them (eight in flight at once cost as much in instruction fetches: code that
// a launch runs once comes from memory too), its share of the counter was waited for at the next barrier, and the
// arguments of either branch were loaded before the first request of every wave (see late_args).  Against that
// form and the one with a counter of finished workers, us: M = 16, N = 14336, K = 512, r = 32 8.4 and 8.0, now 7.9;
// N = 2048, K = 8192, r = 128 10.7 and 8.8, now 8.3; M = 1, N = 1024, K = 14336, r = 64 10.7 and 9.1, now 8.8; M = 16,
// N = K = 4096, r = 64 6.8 and 7.6, now 6.3.
#include <stddef.h>
#include <stdlib.h>

#include <type_traits>

#include "milo_host.h"
#include "milo_kernels.h"
#include "stream_device.h"

namespace milo {

constexpr int kDecWaves = 16;                               // waves of a workgroup
constexpr int kDecThreads = 64 * kDecWaves;
constexpr int kDecTWaves = 8;                               // waves of a T worker that take a chunk each
constexpr int kDecSlotBytes = kStreamSlotBytes;
constexpr int kDecLdsBytes = kDecWaves * kDecSlotBytes;     // 128 KB

__device__ __forceinline__ void buf_store8_coherent(BufRsrc r, uint32_t off, u32x2 v) {
    __builtin_amdgcn_raw_buffer_store_b64(v, r, off, 0, 17);
}
// Staging of one chunk of X (16 rows x 256 columns, the B operand of every row block) in an
// 8-KB LDS slot: copy i moves rows 2i, 2i+1 with one coalesced 1-KB buffer-to-LDS load, lane l ->
// row 2i + l/32, slot position p = l%32, which receives segment p ^ row of the row's 32 segments of
// 8 columns.  Only the first XC copies are issued, XC = ceil(M / 2) rounded up to a power of two:
// rows beyond them keep whatever the slot held, which only reaches output columns (tokens) >= M,
// and those are never stored.  Rows >= M inside the copies lie past the end of X and read as zero.
struct XCopy {
    uint32_t xseg, xrow;
    __device__ __forceinline__ XCopy(int lane, uint32_t K) {
        const uint32_t crow = (uint32_t)lane >> 5, cp = (uint32_t)lane & 31u;
        xseg = (cp ^ crow) << 4;
        xrow = crow * 2u * K;
    }
    // kc = first column of the chunk; a chunk that reaches beyond K (the last one when K is not a
    // multiple of 256, or one past the end) must not wrap into the next row: only the first `lim`
    // bytes of its 512-byte row pieces exist.  lim is a multiple of 128, so whether a lane's segment
    // exists depends on its 128-byte quarter only, which the xor with 2i changes for i >= 4.
    // `base` is added to every offset (the first row of a block of V rows).
    template <int XC>
    __device__ __forceinline__ void issue(BufRsrc xb, unsigned char* slot, uint32_t kc, uint32_t K, bool valid,
                                          uint32_t base = 0u) const {
        const uint32_t lim = (!valid || kc >= K) ? 0u : (K - kc >= 256u ? 512u : 2u * (K - kc));
        const bool ok_lo = (xseg & 0x180u) < lim;
        const bool ok_hi = ((xseg & 0x180u) ^ 0x80u) < lim;
#pragma unroll
        for (int i = 0; i < XC; ++i) {
            // (the constant goes through an opaque scalar so that the per-lane offsets are formed
            // here, four cheap operations per copy, instead of living in registers across the loop)
            uint32_t flip = 32u * i, uni = __builtin_amdgcn_readfirstlane(4u * i * K + 2u * kc + base);
            asm volatile("" : "+s"(flip), "+s"(uni));
            const uint32_t off = ((xseg ^ flip) + xrow) + uni;
            const uint32_t o = (i < 4 ? ok_lo : ok_hi) ? off : kOobOffset;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(xb, (LdsPtr)(slot + i * 1024), 16, o, 0, 0, 0);
        }
        asm volatile("" ::: "memory");
    }
};

// The tag of this launch, from counter `group`: to be read before this workgroup's own contribution.
__device__ __forceinline__ uint32_t decode_tag(const DecodeArgs& a, uint32_t group) {
    const unsigned long long v =
        __hip_atomic_load(a.epoch + group * kDecGroupStride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return (uint32_t)(v >> 16) + 1u;
}

// T worker.  Work item (jb, h) = rank block jb (16 ranks) over K part h (kDecTWaves x t_chunks
// chunks of 256 columns, t_chunks per wave): T_h[m][j] = sum over the part of X[m][k] V[j][k].  The parts are NOT
// added up: the streaming workgroups multiply every T_h with U, which gives the same sum without
// a reduction across workgroups.  Both operands are staged like the activations of the main
// path (coalesced 1-KB buffer-to-LDS copies into a wave-private slot, xor-swizzled), and all
// copies of an item are requested at once.  The upper half of the workgroup's waves has no work
// here and only takes part in the barriers.
// Q: V is the INT3 blob of milo_pack_lr3, [16 rblocks x K] in the layout of a weight: a lane loads
// the unit of rank 16 jb + lane % 16, group 4c + lane / 16, exactly as a streaming wave does for a
// row block, and converts it with the zero-point-free conversion (the quantizer is symmetric).
// BF: activations, V and T are bf16 (MILO_ACT_BF16).
// TAG: T leaves as tagged granules (see the head of this file), else as plain 16-bit rows with a
// counter of finished workers.
// COUNT: the worker adds 1 to counter 0 once it has read the tag from it (the long-K kernel, where a streaming workgroup
// may add its share without having waited for T).
template <int XC, bool Q, bool BF, bool TAG, bool COUNT = false>
__device__ __forceinline__ void decode_t_worker(const DecodeArgs& a, unsigned char* smem) {
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const bool active = wave < kDecTWaves;
    const int j16 = lane & 15, q = lane >> 4;
    const int M = a.M, r = a.w.r;
    const uint32_t K = (uint32_t)a.K;
    const BufRsrc xb = make_rsrc(a.X, (uint64_t)M * K * 2u);
    const BufRsrc vb = make_rsrc(a.w.V, (uint64_t)r * K * 2u);      // < 4 GiB (checked on the host)
    const BufRsrc tb = make_rsrc(a.T, (uint64_t)a.kh * 16u * (uint64_t)a.ldt * 2u);
    uint32_t tag = 0u;
    if (TAG && wave == 0) tag = decode_tag(a, 0u);
    if (COUNT && tid == 0) {
        asm volatile("" : "+v"(tag) :: "memory");           // (the tag has been read)
        atomicAdd(a.epoch, 1ull);
    }
    unsigned char* const xs = smem + (wave & (kDecTWaves - 1)) * 2 * kDecSlotBytes;     // X chunk, then V chunk
    unsigned char* const vs = xs + kDecSlotBytes;
    f32x4* const red = reinterpret_cast<f32x4*>(smem);              // [wave][64 lanes], after a barrier
    const XCopy xc(lane, K);

    const int chunks = TAG ? a.t_chunks : 1;
    for (int item = blockIdx.x; item < a.rblocks * a.kh; item += a.nt) {
        const int jb = item / a.kh, h = item - jb * a.kh;
        f32x4 tacc = {0.0f, 0.0f, 0.0f, 0.0f};
        for (int ci = 0; active && ci < chunks; ++ci) {
            const uint32_t c = (uint32_t)((h * chunks + ci) * kDecTWaves + wave), kc = c * 256u;
            if (ci > 0) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // the slots have been read
            xc.issue<XC>(xb, xs, kc, K, true);
            if (Q) {
                const uint32_t G = K / kGroup;
                const W3Buf vq = make_w3buf(a.w.V, a.ldt, a.K);
                const RawUnit u = load_unit_buf(vq, 4u * c + q < G ? ((uint32_t)jb * G + 4u * c) * 16u + lane : (1u << 27));
                wait_vmem();
                f16x8 bfrag[8];
                read_bfrags(xs, j16, q, bfrag);
                dequant_unit_steps<true>(u, [&](int t, f16x8 frag) { tacc = mfma16(frag, bfrag[t], tacc); });
            } else {
                // rows >= r lie past the end of V and read as zero
                xc.issue<8>(vb, vs, kc, K, true, (uint32_t)(16 * jb) * K * 2u);
                wait_vmem();
                f16x8 bfrag[8], afrag[8];
                read_bfrags(xs, j16, q, bfrag);
                read_bfrags(vs, j16, q, afrag);
#pragma unroll
                for (int t = 0; t < 8; ++t)
                    tacc = BF ? mfma16_bf16(__builtin_bit_cast(bf16x8, afrag[t]), __builtin_bit_cast(bf16x8, bfrag[t]), tacc)
                              : mfma16(afrag[t], bfrag[t], tacc);
            }
        }
        __syncthreads();                                    // every wave has read its slots
        if (active) red[wave * 64 + lane] = tacc;
        __syncthreads();
        if (wave == 0) {
            f32x4 part[kDecTWaves];
#pragma unroll
            for (int p = 0; p < kDecTWaves; ++p) part[p] = red[p * 64 + lane];
            __builtin_amdgcn_sched_barrier(0);
            f32x4 sum = part[0];
#pragma unroll
            for (int p = 1; p < kDecTWaves; ++p)
#pragma unroll
                for (int x = 0; x < 4; ++x) sum[x] += part[p][x];
            // element v of lane l = rank 16*jb + 4*(l/16) + v, token l%16
            u32x2 ob;
            if (BF) {
                ob = u32x2{pack_bf16(sum[0], sum[1]), pack_bf16(sum[2], sum[3])};
            } else {
                f16x4 o;
#pragma unroll
                for (int x = 0; x < 4; ++x) o[x] = (f16)sum[x];
                ob = __builtin_bit_cast(u32x2, o);
            }
            if (TAG) {
                // ranks 16 jb + 4 q + 0..3 = granules 2 (q % 2) and the next of lane (j16, 2 (jb % 2) + q / 2)
                // in the fragment of k-step jb / 2
                const uint32_t at = (((uint32_t)(h * a.nks + (jb >> 1)) * 4u + 2u * (q & 1u)) * 64u) +
                                    ((2u * (jb & 1u) + ((uint32_t)q >> 1)) * 16u + j16);
                __hip_atomic_store(a.tg + at, (uint64_t)tag << 32 | ob.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(a.tg + at + 64, (uint64_t)tag << 32 | ob.y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            } else {
                buf_store8_coherent(tb, (uint32_t)(((h * 16 + j16) * a.ldt + 16 * jb + 4 * q) * 2), ob);
            }
        }
        __syncthreads();                                    // red is read before the slots are refilled
    }
    if (TAG) {
        // counters without a consumer in this launch move on here
        if (blockIdx.x == 0 && (uint32_t)tid < kDecGroups && (uint32_t)tid >= a.nmain)
            atomicAdd(a.epoch + (uint32_t)tid * kDecGroupStride, 65536ull);
        return;
    }
    // all T stores of this workgroup are complete before it is counted
    wait_vmem();
    __syncthreads();
    if (tid == 0) atomicAdd(a.ctrl + 0, 1u);
}

// Bounded wait until every T worker has been counted; a wait that gives up sets an error word.
__device__ __forceinline__ void decode_wait_t(const DecodeArgs& a) {
    for (uint32_t spins = 0;
         __hip_atomic_load(a.ctrl + 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < (uint32_t)a.nt; ++spins) {
        __builtin_amdgcn_s_sleep(1);
        if (spins > a.spin_limit) {
            atomicOr(a.ctrl + 3, 1u);
            break;
        }
    }
}

// Fetches the fragments f0, f0 + step, .. of T into LDS as MFMA B fragments (K part h, k-step i -> fragment
// h * nks + i), polling each granule until its tag is this launch's; a wait that gives up sets an error word.
// One wave, one fragment: at most 16 fragments over 15 waves, all on their way at once, in a few instructions.
__device__ __forceinline__ void decode_fetch_tagged(const DecodeArgs& a, unsigned char* tlds, int lane, uint32_t tag, uint32_t f0, uint32_t step) {
    const uint32_t nks = (uint32_t)a.nks, frags = (uint32_t)a.kh * nks;
#pragma unroll 1
    for (uint32_t f = f0; f < frags; f += step) {
        // an odd number of 16-rank blocks leaves the upper half of a K part's last k-step without ranks
        const bool none = (a.rblocks & 1) != 0 && lane >= 32 && f % nks == nks - 1u;
#pragma unroll 1
        for (uint32_t spins = 0;; ++spins) {
            unsigned long long g[4];
#pragma unroll
            for (uint32_t e = 0; e < 4; ++e)
                g[e] = __hip_atomic_load(a.tg + (f * 4u + e) * 64u + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            bool ok = true;
            u32x4 v;
#pragma unroll
            for (uint32_t e = 0; e < 4; ++e) {
                ok = ok && (uint32_t)(g[e] >> 32) == tag;
                v[e] = none ? 0u : (uint32_t)g[e];
            }
            *reinterpret_cast<u32x4*>(tlds + f * 1024u + lane * 16) = v;
            if (__builtin_amdgcn_ballot_w64(!(ok || none)) == 0ull) break;
            if (spins > (a.spin_limit >> 4)) {
                if (lane == 0) atomicOr(a.ctrl + 3, 1u);
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
    }
}
// The same with the tag read from counter `group`.
__device__ __forceinline__ void decode_fetch_t(const DecodeArgs& a, unsigned char* tlds, int lane, uint32_t group, uint32_t f0, uint32_t step) {
    asm volatile("" : "+v"(lane), "+s"(group), "+s"(f0));      // (what depends on them is formed here, not kept through the stream)
    if (f0 >= (uint32_t)a.kh * (uint32_t)a.nks) return;
    decode_fetch_tagged(a, tlds, lane, decode_tag(a, group), f0, step);
}

// LR: 0 = no low-rank term, 1 = U and T fragments come through LDS, 2 = more ranks or more parts of T than
// that holds (plain loads in the epilogue).
constexpr int kDecKS = kStreamKS;                               // k-steps of 32 ranks, LR == 1
constexpr int kDecULds = kDecLdsBytes;                          // U fragments [R][kDecKS][64] x 16 B
constexpr int kDecTLds = kDecULds + 4 * kDecKS * 1024;          // T fragments [kDecTFrags][64] x 16 B
constexpr int kDecTFrags = 16;                                  // (K parts) x (k-steps used) at most, LR == 1
constexpr int kDecLdsTotal = kDecTLds + kDecTFrags * 1024;      // 160 KB, all a workgroup can have

// One turn of a streaming wave: R row blocks x the wave's chunks of K (chunks wave, wave + 16, ...,
// rotated per workgroup so that the workgroups, which all read the same X, do not walk the same
// L2 channels in step).
//
// The first chunk is requested up front: its activations, then its R units.  While unit (j, b) is
// converted, unit (j + 1, b) is requested into the registers it frees, and the activations of
// chunk j + 1 right after those of chunk j have been read into registers (one slot per wave).
// Vector memory operations complete in order, so "unit (j, b) and the activations of chunk j have
// arrived" is a fixed count of younger operations (the build script checks that the compiler adds
// no memory operation of its own and keeps the order):
//   request order   X0 W00 .. W0(R-1) | X1 W10 | W11 | ... | X2 W20 | ...
//   unit (j, 0):    2 (R - 1)              (the other units of chunk j)
//   unit (j, b>0):  2 (R - 1) + XC         (the rest of chunk j, X(j+1), the first b units of chunk j + 1)
//   last chunk:     2 (R - 1 - b)          (nothing is requested any more)
// For K up to 4096 a wave has a single chunk and everything is requested up front.
template <int R, int XC, bool SYM, bool BF>
struct DecodeStream {
    const W3Buf& wb;
    BufRsrc xb;
    XCopy xc;
    unsigned char* slot;        // the wave's slot
    uint32_t K, G, NB, C, span, first, lane, q, j16;

    __device__ __forceinline__ uint32_t chunk_of(uint32_t j) const {
        uint32_t idx = first + kDecWaves * j;
        if (idx >= span) idx -= span;
        return idx;
    }
    __device__ __forceinline__ void issue_x(uint32_t j) const {
        xc.issue<XC>(xb, slot, chunk_of(j) * 256u, K, true);
    }
    __device__ __forceinline__ void issue_w(uint32_t j, uint32_t rb, RawUnit& u) const {
        const uint32_t c = chunk_of(j);
        // (an index of 2^27 is past the end of every weight the host accepts, and 16 * 2^27 does not wrap)
        const bool ok = 4u * c + q < G && rb < NB;
        u = load_unit_buf_once(wb, ok ? (rb * G + 4u * c) * 16u + lane : (1u << 27));
        asm volatile("" ::: "memory");      // the loads keep this order (the waits count them)
    }

    template <bool LAST>
    __device__ __forceinline__ void chunk(uint32_t j, uint32_t rb0, RawUnit (&u)[R], f32x4 (&acc)[R]) const {
        f16x8 bfrag[8];
        static_for<0, R>([&](auto b_c) {
            constexpr int b = decltype(b_c)::value;
            __builtin_amdgcn_sched_barrier(0);      // nothing of this unit moves above its wait
            MILO_WAIT_VMEM(LAST ? 2 * (R - 1 - b) : (b == 0 ? 2 * (R - 1) : 2 * (R - 1) + XC));
            __builtin_amdgcn_sched_barrier(0);
            if (b == 0) {
                read_bfrags(slot, (int)j16, (int)q, bfrag);
                if (!LAST) {
                    // the slot is free once its fragments are in registers
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                    issue_x(j + 1);
                }
            }
            pin_unit_params(u[b]);          // nothing is computed from this unit before the wait
            if (BF)
                dequant_unit_steps_bf16(u[b], [&](int t, bf16x8 frag) {
                    acc[b] = mfma16_bf16(frag, __builtin_bit_cast(bf16x8, bfrag[t]), acc[b]);
                });
            else
                dequant_unit_steps<SYM>(u[b], [&](int t, f16x8 frag) { acc[b] = mfma16(frag, bfrag[t], acc[b]); });
            if (!LAST) {
                __builtin_amdgcn_sched_barrier(0);
                issue_w(j + 1, rb0 + b, u[b]);
            }
        });
    }

    __device__ __forceinline__ void run(uint32_t rb0, f32x4 (&acc)[R]) const {
        RawUnit u[R];
        issue_x(0);
#pragma unroll
        for (int b = 0; b < R; ++b) issue_w(0, rb0 + b, u[b]);
        for (uint32_t j = 0; j + 1 < C; ++j) chunk<false>(j, rb0, u, acc);
        chunk<true>(C - 1, rb0, u, acc);
    }
};


// The argument block behind the kernel's leading scalar arguments, through an address the compiler knows nothing about:
// its loads stay where the values are needed.  Read through the parameter itself, whatever any branch needs is loaded at
// the kernel's first instructions, and every wave's first request to memory waits for it: 0.3 to 0.7 us of a launch
// whose stream is short.  The other variants keep the parameter: without T there is little to load (K = 14336, M = 8
// loses 1.5 % by the later loads), and with LR == 2 the longest chain is T itself.
struct DecodeKernargs {         // (the kernel's parameters in order: the layout of the argument segment)
    const void* q3; const f16* X; uint32_t units, K, nb; int M, nt; uint32_t nmain, cpw, rot_mask, x_bytes;
    DecodeArgs args;
};
__device__ __forceinline__ const DecodeArgs& late_args() {
    typedef const __attribute__((address_space(4))) char* Segment;
    Segment p = (Segment)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(DecodeKernargs, args);
    asm volatile("" : "+s"(p));
    return *(const DecodeArgs*)p;
}

// U rows of the R row blocks from rb0 on as MFMA A fragments to LDS (k-step i of block b, lane (j16, q) =
// U[n][32i + 8q ..]), by one wave; its direct copies are still on their way when it returns.
template <int R, bool Q>
__device__ __forceinline__ void decode_fetch_u(const DecodeArgs& a, unsigned char* smem, uint32_t rb0, uint32_t NB, int r, int ksu,
                                               int lane, int j16, int q) {
    if (Q) {
        // INT3 U: the blob holds U^T [ldt x N] with groups of 64 along N, and these
        // 16 R rows lie inside one group.  Lane l takes rank l (then l +
        // 64): one unit, converted, and scattered into the fragment layout the
        // epilogue reads.  Ranks past the compensator's read as zero units, which
        // also clears the rest of the last k-step.
        const W3Buf uq = make_w3buf(a.w.U, a.ldt, a.N);
        const uint32_t GN = (uint32_t)(a.N >> 6), g = rb0 >> 2, o16 = rb0 & 3u;
        for (uint32_t j = (uint32_t)lane; j < 32u * (uint32_t)ksu; j += 64u) {
            const bool ok = j < (uint32_t)a.ldt && rb0 < NB;
            const RawUnit u = load_unit_buf(uq, ok ? ((j >> 4) * GN + g) * 16u + (j & 15u) : (1u << 27));
            uint32_t w[32];
            dequant_unit<true>(u, w);
            unsigned char* const frag0 =
                smem + kDecULds + (((j >> 5) * 64u + ((j & 31u) >> 3) * 16u) * 16u + (j & 7u) * 2u);
            if (R == 4) scatter_u_rank<R, 0>(w, frag0);
            else if (R == 2) { if (o16 == 0) scatter_u_rank<R, 0>(w, frag0); else scatter_u_rank<R, 2>(w, frag0); }
            else {
                if (o16 == 0) scatter_u_rank<R, 0>(w, frag0);
                else if (o16 == 1) scatter_u_rank<R, 1>(w, frag0);
                else if (o16 == 2) scatter_u_rank<R, 2>(w, frag0);
                else scatter_u_rank<R, 3>(w, frag0);
            }
        }
    } else {
        const BufRsrc ub = make_rsrc(a.w.U, (uint64_t)a.u_bytes);
#pragma unroll 1
        for (int b = 0; b < R; ++b) {
            const uint32_t nrow = (rb0 + b) * 16u + j16;
#pragma unroll 1
            for (int i = 0; i < ksu; ++i) {
                const uint32_t k0 = 32u * i + 8u * q;
                unsigned char* const dst = smem + kDecULds + (b * kDecKS + i) * 1024;
                if ((r & 7) == 0) {
                    const uint32_t off =
                        (rb0 + b < NB && k0 < (uint32_t)r) ? (nrow * r + k0) * 2u : kOobOffset;
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(ub, (LdsPtr)dst, 16, off, 0, 0, 0);
                } else {        // rows that are not 16-byte aligned: element by element
                    uint32_t e[8];
#pragma unroll
                    for (uint32_t v = 0; v < 8; ++v)
                        e[v] = __builtin_amdgcn_raw_buffer_load_b16(
                            ub, (rb0 + b < NB && k0 + v < (uint32_t)r) ? (nrow * r + k0 + v) * 2u : kOobOffset, 0, 0);
                    int l16 = lane * 16;
                    asm volatile("" : "+v"(l16));
                    *reinterpret_cast<u32x4*>(dst + l16) =
                        u32x4{e[0] | e[1] << 16, e[2] | e[3] << 16, e[4] | e[5] << 16, e[6] | e[7] << 16};
                }
            }
        }
    }
}

// SYM: the weight blob is symmetric (zero-point-free conversion).  Q (with LR == 1): the compensator
// is the pair of INT3 blobs of milo_pack_lr3.
template <int R, int LR, int XC, bool SYM, bool Q, bool BF>
__global__ __launch_bounds__(kDecThreads) void w3lr_decode_kernel(const void* q3_, const f16* X_, uint32_t units_, uint32_t K_,
                                                                  uint32_t nb_, int M_, int nt_, uint32_t nmain_, uint32_t cpw_,
                                                                  uint32_t rot_mask_, uint32_t x_bytes_, const DecodeArgs a_) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    // What a streaming wave needs for its first requests comes as leading scalar arguments, which the
    // hardware places in registers when it starts the wave (the build asks for that with
    // -amdgpu-kernarg-preload-count); everything else is read from the argument block when it is
    // needed (LR == 1: late_args).  The values are the same as the block's.
    DecodeArgs pa = a_;
    pa.w.q3 = q3_; pa.X = X_; pa.units = units_; pa.K = (int64_t)K_; pa.nb = nb_; pa.M = M_; pa.nt = nt_; pa.nmain = nmain_;
    pa.chunks_per_wave = cpw_; pa.rot_mask = rot_mask_; pa.x_bytes = x_bytes_;

    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int nworkers = LR > 0 ? nt_ : 0;
    if (LR > 0 && (int)blockIdx.x < nworkers) {
        DecodeArgs a = LR == 1 ? late_args() : pa;
        a.X = X_; a.K = (int64_t)K_; a.M = M_; a.nt = nt_; a.nmain = nmain_;        // (in registers already)
        decode_t_worker<XC, Q, BF, LR == 1>(a, smem);
    } else {
        const int j16 = lane & 15, q = lane >> 4;
        const int M = M_;
        const uint32_t K = K_;                              // < 2^27 (checked on the host)
        const uint32_t G = K / kGroup;
        const uint32_t NB = nb_;                            // 16-row blocks
        W3Buf wb;
        wb.a = make_rsrc(q3_, (uint64_t)(units_ * 16u));                // (units <= 2^26)
        wb.b = make_rsrc(reinterpret_cast<const char*>(q3_) + (uint64_t)units_ * 16u, (uint64_t)(units_ * 12u));
        const uint32_t nmain = nmain_;

        const int wave_s = __builtin_amdgcn_readfirstlane(wave);        // known to be uniform
        DecodeStream<R, XC, SYM, BF> st{wb,
                               make_rsrc(X_, (uint64_t)x_bytes_),
                               XCopy(lane, K),
                               smem + wave_s * kDecSlotBytes,
                               K, G, NB, 0u, 0u, 0u, (uint32_t)lane, (uint32_t)q, (uint32_t)j16};
        st.C = cpw_;
        st.span = st.C * kDecWaves;
        // (rotation by a masked product instead of a remainder: no division before the first request)
        st.first = (uint32_t)wave_s + ((blockIdx.x * 5u) & rot_mask_);
        if (st.first >= st.span) st.first -= st.span;

        // (every streaming workgroup has at least one turn: the number of turns is first looked at after it)
        uint32_t turn = 0, turns, blk = blockIdx.x - nworkers;
        do {
            const uint32_t rb0 = blk * R;
            f32x4 acc[R];
#pragma unroll
            for (int b = 0; b < R; ++b) acc[b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            f32x4* const red = reinterpret_cast<f32x4*>(smem);          // wave w, block b at 512 w + 64 b
            u32x4* const ulds = reinterpret_cast<u32x4*>(smem + kDecULds);
            u32x4* const tbuf = reinterpret_cast<u32x4*>(smem + kDecTLds);

            if (rb0 < NB) st.run(rb0, acc);
            // each wave leaves its partial sums in its own slot, which it has finished reading
#pragma unroll
            for (int b = 0; b < R; ++b) red[wave * (kDecSlotBytes / 16) + b * 64 + lane] = acc[b];
            const DecodeArgs& a = LR == 1 ? late_args() : pa;
            const int r = a.w.r;
            const int ksu = (r + 31) >> 5;                  // k-steps of 32 ranks in use
            // (T fragments in LDS: K part h, k-step i -> h * ksu + i)
            turns = a.turns;
            int kh = a.kh;
            const BufRsrc tb = make_rsrc(LR == 2 ? a.T : nullptr, LR == 2 ? (uint64_t)a.t_bytes : 0u);
            if (LR > 0 && wave == 0) {
                // Everything the epilogue needs besides the partial sums, fetched by the wave that
                // is done first, while the others still stream; its requests go ahead of theirs.
                // U rows of the R row blocks as MFMA A fragments (k-step i, lane (j16, q) =
                // U[n][32i + 8q ..]); LR == 2: nothing but the wait for T.
                __builtin_amdgcn_s_setprio(3);
                if (LR == 1) decode_fetch_u<R, Q>(a, smem, rb0, NB, r, ksu, lane, j16, q);
                if (LR == 2 && turn == 0) decode_wait_t(a);
                wait_vmem();
                __builtin_amdgcn_s_setprio(0);
            }
            if (LR == 1 && turn == 0 && wave >= 1) {
                __builtin_amdgcn_s_setprio(3);
                decode_fetch_t(a, smem + kDecTLds, lane, (blockIdx.x - nworkers) % kDecGroups, (uint32_t)wave_s - 1u, kDecWaves - 1);
                __builtin_amdgcn_s_setprio(0);
            }
            uint32_t n_out = (uint32_t)a.N;
            f16* const y_out = a.Y;
            if (LR == 1) asm volatile("" : "+s"(n_out), "+s"(turns), "+s"(kh) : "s"(y_out));       // (loaded before the barrier)
            __syncthreads();                                       // partial sums, U and T are in LDS
            // T has been read: this workgroup's share of its counter, by a wave without a part in the epilogue and after
            // the barrier, which would wait for the atomic's way to memory and back
            if (LR == 1 && turn == 0 && wave == kDecWaves - 1 && lane == 0) {
                const uint32_t wg = blockIdx.x - nworkers;
                const uint32_t members = (nmain - wg % kDecGroups + kDecGroups - 1u) / kDecGroups;
                atomicAdd(a.epoch + (wg % kDecGroups) * kDecGroupStride, wg < kDecGroups ? 65537ull - members : 1ull);
            }
            if (wave < R) {
                // wave b finishes row block b: sum of the waves' partials in wave order
                const int b = wave;
                // (all partials are requested before the first addition: one LDS round trip, not sixteen)
                f32x4 part[kDecWaves];
#pragma unroll
                for (int pw = 0; pw < kDecWaves; ++pw) part[pw] = red[pw * (kDecSlotBytes / 16) + b * 64 + lane];
                __builtin_amdgcn_sched_barrier(0);
                f32x4 sum = part[0];
#pragma unroll
                for (int pw = 1; pw < kDecWaves; ++pw)
#pragma unroll
                    for (int e = 0; e < 4; ++e) sum[e] += part[pw][e];
                const uint32_t nb = (rb0 + b) * 16u;
                if (LR == 1) {
                    int f = 0;
#pragma unroll 1
                    for (int h = 0; h < kh; ++h) {
#pragma unroll 1
                        for (int i = 0; i < ksu; ++i, ++f)
                            sum = BF ? mfma16_bf16(__builtin_bit_cast(bf16x8, ulds[(b * kDecKS + i) * 64 + lane]),
                                                   __builtin_bit_cast(bf16x8, tbuf[f * 64 + lane]), sum)
                                     : mfma16(__builtin_bit_cast(f16x8, ulds[(b * kDecKS + i) * 64 + lane]),
                                              __builtin_bit_cast(f16x8, tbuf[f * 64 + lane]), sum);
                    }
                } else if (LR == 2) {
                    const int64_t nrow = (int64_t)nb + j16;
                    for (int ks = 0; ks < r; ks += 32) {
                        const int k0 = ks + 8 * q;
                        f16x8 av = zero_f16x8();
                        if (nrow < a.N) av = load_row8(a.w.U + nrow * r, k0, r, (r & 7) == 0);
                        for (int h = 0; h < kh; ++h) {
                            const f16x8 bv = __builtin_bit_cast(
                                f16x8, buf_load16_coherent(tb, k0 < a.ldt ? (uint32_t)(((h * 16 + j16) * a.ldt + k0) * 2)
                                                                          : kOobOffset));
                            sum = BF ? mfma16_bf16(__builtin_bit_cast(bf16x8, av), __builtin_bit_cast(bf16x8, bv), sum)
                                     : mfma16(av, bv, sum);
                        }
                    }
                }
                // D[v]: feature nb + 4q + v, token j16.  (The output address is formed here, from
                // scalars the compiler cannot move: formed at the top of the kernel it would sit in
                // registers through the whole stream, or in scratch memory, a round trip to memory
                // right before the store.)
                uint32_t m_out = (uint32_t)M;
                asm volatile("" : "+s"(n_out), "+s"(m_out));
                const uint32_t n = nb + 4u * q;
                if ((uint32_t)j16 < m_out && n < n_out) {
                    u32x2 ob;
                    if (BF) {
                        ob = u32x2{pack_bf16(sum[0], sum[1]), pack_bf16(sum[2], sum[3])};
                    } else {
                        f16x4 o;
#pragma unroll
                        for (int e = 0; e < 4; ++e) o[e] = (f16)sum[e];
                        ob = __builtin_bit_cast(u32x2, o);
                    }
                    *reinterpret_cast<u32x2*>(y_out + ((uint64_t)j16 * n_out + n)) = ob;
                }
            }
            if (turn + 1 < turns) __syncthreads();      // slots, U and the partial sums are reused
            blk += nmain;
        } while (++turn < turns);
    }

    // LR == 2: the streaming workgroups read T from memory in their epilogue, so they sign off last.
    if (LR == 2 && (int)blockIdx.x >= nworkers) {
        __syncthreads();
        if (tid == 0)
            __hip_atomic_store(pa.done + (blockIdx.x - nworkers), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // Worker 0 stays until every streaming workgroup has signed off (which each does only after
    // it has seen all workers counted), then restores the control words for the next launch.
    // No returning atomic on a shared word is involved: hundreds of those on one address
    // serialize for several microseconds.
    if (LR == 2 && blockIdx.x == 0 && wave == 0) {
        const DecodeArgs& a = pa;
        const uint32_t nmain = nmain_;
        bool all = false;
        for (uint32_t spins = 0; !all; ++spins) {
            all = true;
            for (uint32_t base = 0; base < nmain; base += 64) {
                const uint32_t idx = base + (uint32_t)lane;
                const uint32_t v =
                    idx < nmain ? __hip_atomic_load(a.done + idx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 1u;
                all = all && (__builtin_amdgcn_ballot_w64(v != 0u) == ~0ull);
            }
            if (!all) {
                __builtin_amdgcn_s_sleep(8);
                if (spins > (a.spin_limit >> 2)) {
                    atomicOr(a.ctrl + 3, 2u);
                    break;
                }
            }
        }
        if (all) {
            for (uint32_t base = 0; base < nmain; base += 64)
                if (base + (uint32_t)lane < nmain)
                    __hip_atomic_store(a.done + base + lane, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (lane == 0) __hip_atomic_store(a.ctrl + 0, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// Long K (more than sixteen chunks): the sixteen waves of a workgroup take sixteen consecutive (band, chunk) pairs of the
// launch's list, band by band, one chunk each with everything requested up front.  A band of 16 R features so spreads over
// several workgroups, every CU streams, and X is staged once per R row blocks and chunk by all of them together.  (In the
// other kernel a row block belongs to one workgroup: 4096 x 14336 ran on half the CUs, four chunks per wave in turn.)
//
// The workgroup that holds a band's last chunk finishes it; the ones before hand their partial sums over as granules of 4 bytes of
// value and 4 of mark, and the finisher adds its own and theirs in workgroup order.  It only waits for workgroups with
// lower ids, which never wait for anything but T and lower ones before they publish.  The granules are scratch that may
// hold anything, also this launch's mark, so their owner clears them first, while its later waves still stream, and says so with a
// tagged word among the granules of T, whose contents the library owns; the finisher looks at that word, also
// under the stream, before it looks at the granules.  So the path to the output has one trip through memory.
//
// 4096 x 14336, r = 32, us per launch, chunks in turn -> here: M = 16 15.5 -> 11.5, M = 1 12.2 -> 10.1, bf16 13.3 -> 10.7.
template <int R, int LR, bool Q, bool BF>
__global__ __launch_bounds__(kDecThreads) void w3lr_decode_split_kernel(const void* q3_, const f16* X_, uint32_t units_, uint32_t K_,
                                                                        uint32_t nb_, int M_, int nt_, uint32_t nmain_, uint32_t nchunks_,
                                                                        uint32_t magic_, uint32_t x_bytes_, const DecodeArgs) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int nworkers = LR > 0 ? nt_ : 0;
    if (LR > 0 && (int)blockIdx.x < nworkers) {
        DecodeArgs a = late_args();
        a.X = X_; a.K = (int64_t)K_; a.M = M_; a.nt = nt_; a.nmain = nmain_;        // (in registers already)
        decode_t_worker<8, Q, BF, true, true>(a, smem);
        return;
    }
    const int j16 = lane & 15, q = lane >> 4;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t K = K_, NB = nb_, nchunks = nchunks_;
    W3Buf wb;
    wb.a = make_rsrc(q3_, (uint64_t)(units_ * 16u));                // (units <= 2^26)
    wb.b = make_rsrc(reinterpret_cast<const char*>(q3_) + (uint64_t)units_ * 16u, (uint64_t)(units_ * 12u));
    // pairs 16 wg .. 16 wg + 15: chunks from c0 of band `band0` on, and, past its last one, of the next band (there are
    // more than sixteen chunks, so never of a third)
    const uint32_t wg = blockIdx.x - (uint32_t)nworkers;
    const uint32_t band0 = (uint32_t)(((uint64_t)(wg * kDecWaves) * magic_) >> 32), c0 = wg * kDecWaves - band0 * nchunks;
    const uint32_t left = nchunks - c0;                             // waves from here on belong to the next band
    const bool next = wave >= left;
    const uint32_t rb0 = (band0 + (next ? 1u : 0u)) * R;            // (past the last band: no data, zero sums)
    const DecodeStream<R, 8, false, BF> st{wb, make_rsrc(X_, (uint64_t)x_bytes_), XCopy(lane, K), smem + wave * kDecSlotBytes, K,
                                           K / kGroup, NB, 1u, ~0u, next ? wave - left : c0 + wave, (uint32_t)lane, (uint32_t)q, (uint32_t)j16};
    // (the number of activation copies does not enter the waits of a single chunk: they are older than every unit)
    {
        const uint32_t kc = st.first * 256u;
        if (M_ <= 2) st.xc.template issue<1>(st.xb, st.slot, kc, K, true);
        else if (M_ <= 4) st.xc.template issue<2>(st.xb, st.slot, kc, K, true);
        else if (M_ <= 8) st.xc.template issue<4>(st.xb, st.slot, kc, K, true);
        else st.xc.template issue<8>(st.xb, st.slot, kc, K, true);
    }
    f32x4 acc[R];
    RawUnit u[R];
#pragma unroll
    for (int b = 0; b < R; ++b) {
        acc[b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        st.issue_w(0, rb0 + b, u[b]);
    }
    st.template chunk<true>(0, rb0, u, acc);
    f32x4* const red = reinterpret_cast<f32x4*>(smem);              // wave w, block b at 512 w + 64 b
#pragma unroll
    for (int b = 0; b < R; ++b) red[wave * (kDecSlotBytes / 16) + b * 64 + lane] = acc[b];

    const DecodeArgs& a = late_args();
    const bool finishes = left <= kDecWaves;                        // the last chunk of band0 is here
    const uint32_t group = wg % kDecGroups;
    const bool hands_over = !finishes || (left < kDecWaves && (band0 + 1u) * R < NB);
    const bool live = j16 < M_;                                     // this lane's token exists
    const uint32_t first_wg = (band0 * nchunks) / kDecWaves;        // (the first one with a chunk of band0)
    unsigned long long* const pg = a.pg;                            // [workgroup][R][4][64 lanes]
    unsigned long long* const cleared = a.tg + kDecSplitFrags * 256;        // one word per workgroup, its tag in the upper half
    constexpr uint32_t kTagWave = 5, kClearWave = 3;                // (waves that are done early)
    uint32_t* const tag_lds = reinterpret_cast<uint32_t*>(smem + (kTagWave + 1) * kDecSlotBytes - 16);     // (its own slot, not read any more)
    if (wave == kClearWave && hands_over) {
        if (live)
#pragma unroll
            for (uint32_t i = 0; i < 4 * R; ++i)
                __hip_atomic_store(pg + (size_t)wg * (R * 256u) + i * 64u + lane, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t t = decode_tag(a, group);
        wait_vmem();
        if (lane == 0) __hip_atomic_store(cleared + wg, (unsigned long long)t << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (wave == kTagWave) {
        const uint32_t t = decode_tag(a, group);
        if (lane == 0) *tag_lds = t;
        if (finishes)
#pragma unroll 1
            for (uint32_t p0 = first_wg; p0 < wg; p0 += 64)
#pragma unroll 1
                for (uint32_t spins = 0;; ++spins) {
                    const unsigned long long v = __hip_atomic_load(cleared + (p0 + lane < wg ? p0 + lane : wg - 1u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (__builtin_amdgcn_ballot_w64((uint32_t)(v >> 32) != t) == 0ull) break;
                    if (spins > (a.spin_limit >> 4)) {
                        if (lane == 0) atomicOr(a.ctrl + 3, 1u);
                        break;
                    }
                    __builtin_amdgcn_s_sleep(1);
                }
    }
    const int r = a.w.r, ksu = (r + 31) >> 5;
    if (LR > 0 && finishes && wave == 0) {
        __builtin_amdgcn_s_setprio(3);
        decode_fetch_u<R, Q>(a, smem, band0 * R, NB, r, ksu, lane, j16, q);
        wait_vmem();
        __builtin_amdgcn_s_setprio(0);
    }
    __syncthreads();                                                // partial sums, the tag and U are in LDS; granules are clear
    const uint32_t tag = (uint32_t)__builtin_amdgcn_readfirstlane((int)*tag_lds);
    // waves 0 .. R-1 finish the blocks of band0, waves R .. 2R-1 hand the other partial sums over (before anything is
    // waited for: no finisher waits for T through another one), the rest fetch T
    const bool fin = wave < R;
    const uint32_t b = fin ? wave : wave - R;
    if (wave >= 2 * R) {
        if (LR > 0 && finishes) {
            decode_fetch_tagged(a, smem + kDecTLds, lane, tag, wave - 2 * R, kDecWaves - 2 * R);
            __syncthreads();
        }
        // the tag has been read: this workgroup's share of its counter (after the barrier, which would wait for the atomic)
        if (wave == kDecWaves - 1 && lane == 0) {
            const uint32_t members = (nmain_ - group + kDecGroups - 1u) / kDecGroups + (group == 0u ? (uint32_t)nworkers : 0u);
            atomicAdd(a.epoch + group * kDecGroupStride, wg < kDecGroups ? 65537ull - members : 1ull);
        }
        return;
    }
    if (!finishes && fin) return;
    if (!fin && !hands_over) {
        if (LR > 0) __builtin_amdgcn_s_barrier();
        return;
    }
    const uint32_t lo = !fin && finishes ? left : 0u, hi = fin ? left : (uint32_t)kDecWaves;
    f32x4 part[kDecWaves];
#pragma unroll
    for (int pw = 0; pw < kDecWaves; ++pw) part[pw] = red[pw * (kDecSlotBytes / 16) + b * 64 + lane];
    __builtin_amdgcn_sched_barrier(0);
    f32x4 sum = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int pw = 0; pw < kDecWaves; ++pw)
        if ((uint32_t)pw >= lo && (uint32_t)pw < hi)
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[e] += part[pw][e];
    const uint32_t mark = tag | 0x80000000u;                        // (never the zero of a cleared granule)
    if (!fin) {
        unsigned long long* const at = pg + (size_t)(wg * R + b) * 256u + lane;
        if (live)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float v = sum[e];         // (a bit cast of the vector's element itself takes element 0)
                __hip_atomic_store(at + e * 64, (unsigned long long)mark << 32 | __builtin_bit_cast(uint32_t, v), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            }
        if (LR > 0 && finishes) __builtin_amdgcn_s_barrier();       // (nothing of this wave's is behind it: no wait for the stores)
        return;
    }
    // four workgroups' partial sums in one trip
    constexpr uint32_t kBatch = 4;
#pragma unroll 1
    for (uint32_t p0 = first_wg; p0 < wg; p0 += kBatch) {
        unsigned long long g[kBatch][4];
#pragma unroll 1
        for (uint32_t spins = 0;; ++spins) {
            bool ok = true;
            if (live)
#pragma unroll
                for (uint32_t i = 0; i < kBatch; ++i)
#pragma unroll
                    for (uint32_t e = 0; e < 4; ++e)                // (past the last one: the last one again)
                        g[i][e] = __hip_atomic_load(pg + (size_t)((p0 + i < wg ? p0 + i : wg - 1u) * R + b) * 256u + e * 64u + lane, __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_AGENT);
            if (live)
#pragma unroll
                for (uint32_t i = 0; i < kBatch; ++i)
#pragma unroll
                    for (uint32_t e = 0; e < 4; ++e) ok = ok && (uint32_t)(g[i][e] >> 32) == mark;
            if (__builtin_amdgcn_ballot_w64(!ok) == 0ull) break;
            if (spins > (a.spin_limit >> 4)) {
                if (lane == 0) atomicOr(a.ctrl + 3, 1u);
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
#pragma unroll
        for (uint32_t i = 0; i < kBatch; ++i)
            if (p0 + i < wg)
#pragma unroll
                for (uint32_t e = 0; e < 4; ++e) sum[e] += live ? __builtin_bit_cast(float, (uint32_t)g[i][e]) : 0.0f;
    }
    if (LR > 0) {
        __syncthreads();                                            // T is in LDS
        const u32x4* const ulds = reinterpret_cast<const u32x4*>(smem + kDecULds);
        const u32x4* const tbuf = reinterpret_cast<const u32x4*>(smem + kDecTLds);
        const int kh = a.kh;
        int f = 0;
#pragma unroll 1
        for (int h = 0; h < kh; ++h) {
#pragma unroll 1
            for (int i = 0; i < ksu; ++i, ++f)
                sum = BF ? mfma16_bf16(__builtin_bit_cast(bf16x8, ulds[(b * kDecKS + i) * 64 + lane]),
                                       __builtin_bit_cast(bf16x8, tbuf[f * 64 + lane]), sum)
                         : mfma16(__builtin_bit_cast(f16x8, ulds[(b * kDecKS + i) * 64 + lane]),
                                  __builtin_bit_cast(f16x8, tbuf[f * 64 + lane]), sum);
        }
    }
    const uint32_t n_out = (uint32_t)a.N, n = (band0 * R + b) * 16u + 4u * q;
    if (live && n < n_out) {
        u32x2 ob;
        if (BF) {
            ob = u32x2{pack_bf16(sum[0], sum[1]), pack_bf16(sum[2], sum[3])};
        } else {
            f16x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (f16)sum[e];
            ob = __builtin_bit_cast(u32x2, o);
        }
        *reinterpret_cast<u32x2*>(a.Y + ((uint64_t)j16 * n_out + n)) = ob;
    }
}

// Workgroups the device keeps resident at once (one 128-KB-LDS workgroup per CU), cached per
// device; also raises the kernels' dynamic LDS limit once.
typedef void (*DecodeKernel)(const void*, const f16*, uint32_t, uint32_t, uint32_t, int, int, uint32_t, uint32_t, uint32_t, uint32_t,
                             const DecodeArgs);
// Variants: R x LR x XC for plain weights with an fp16 compensator (the generic path LR == 2 is not
// specialised by XC); with an INT3 compensator R x XC (LR == 1); with the symmetric conversion the
// shape that matters for speed, R == 4 with LR 0 or 1 (other shapes take the plain conversion, which
// gives the same bits).
template <int R, int LR, bool SYM, bool Q>
static DecodeKernel decode_variant_xc(int xc) {
    if constexpr (LR == 2) {
        return w3lr_decode_kernel<R, LR, 8, false, false, false>;
    } else {
        if (xc == 1) return w3lr_decode_kernel<R, LR, 1, SYM, Q, false>;
        if (xc == 2) return w3lr_decode_kernel<R, LR, 2, SYM, Q, false>;
        if (xc == 4) return w3lr_decode_kernel<R, LR, 4, SYM, Q, false>;
        return w3lr_decode_kernel<R, LR, 8, SYM, Q, false>;
    }
}
template <int LR, bool SYM, bool Q>
static DecodeKernel decode_variant_r(int R, int xc) {
    if (R == 4) return decode_variant_xc<4, LR, SYM, Q>(xc);
    if constexpr (SYM) {
        return nullptr;
    } else {
        if (R == 2) return decode_variant_xc<2, LR, SYM, Q>(xc);
        return decode_variant_xc<1, LR, SYM, Q>(xc);
    }
}
// bf16 activations: R x LR x XC
template <int R, int LR>
static DecodeKernel decode_variant_bf_xc(int xc) {
    if constexpr (LR == 2) {
        return w3lr_decode_kernel<R, LR, 8, false, false, true>;
    } else {
        if (xc == 1) return w3lr_decode_kernel<R, LR, 1, false, false, true>;
        if (xc == 2) return w3lr_decode_kernel<R, LR, 2, false, false, true>;
        if (xc == 4) return w3lr_decode_kernel<R, LR, 4, false, false, true>;
        return w3lr_decode_kernel<R, LR, 8, false, false, true>;
    }
}
template <int LR>
static DecodeKernel decode_variant_bf(int R, int xc) {
    if (R == 4) return decode_variant_bf_xc<4, LR>(xc);
    if (R == 2) return decode_variant_bf_xc<2, LR>(xc);
    return decode_variant_bf_xc<1, LR>(xc);
}
static DecodeKernel decode_variant(int R, int lr, int xc, bool sym, bool q, bool bf = false) {
    if (bf) return q ? nullptr : lr == 0 ? decode_variant_bf<0>(R, xc) : lr == 1 ? decode_variant_bf<1>(R, xc) : decode_variant_bf<2>(R, xc);
    if (q) return lr == 1 ? decode_variant_r<1, false, true>(R, xc) : nullptr;
    if (sym && R == 4 && lr < 2) return lr == 0 ? decode_variant_r<0, true, false>(R, xc) : decode_variant_r<1, true, false>(R, xc);
    if (lr == 0) return decode_variant_r<0, false, false>(R, xc);
    if (lr == 1) return decode_variant_r<1, false, false>(R, xc);
    return decode_variant_r<2, false, false>(R, xc);
}
template <int R>
static DecodeKernel decode_split_variant_r(bool lr, bool q, bool bf) {
    if (bf) return lr ? w3lr_decode_split_kernel<R, 1, false, true> : w3lr_decode_split_kernel<R, 0, false, true>;
    if (q) return w3lr_decode_split_kernel<R, 1, true, false>;
    return lr ? w3lr_decode_split_kernel<R, 1, false, false> : w3lr_decode_split_kernel<R, 0, false, false>;
}
static DecodeKernel decode_split_variant(int R, bool lr, bool q, bool bf) {
    return R == 4 ? decode_split_variant_r<4>(lr, q, bf) : R == 2 ? decode_split_variant_r<2>(lr, q, bf) : decode_split_variant_r<1>(lr, q, bf);
}
static int decode_capacity() {
    static int cached[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
    if (cached[dev] == 0) {
        int cus = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
            return 0;
        for (int R = 1; R <= 4; R *= 2)
            for (int lr = 0; lr < 3; ++lr)
                for (int xc = 1; xc <= 8; xc *= 2)
                    for (int v = 0; v < 4; ++v) {       // plain, symmetric, INT3 compensator, bf16
                        const DecodeKernel k = decode_variant(R, lr, xc, v == 1, v == 2, v == 3);
                        if (k && hipFuncSetAttribute(reinterpret_cast<const void*>(k),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize,
                                                     kDecLdsTotal) != hipSuccess)
                            return 0;
                    }
        for (int R = 1; R <= 4; R *= 2)
            for (int v = 0; v < 5; ++v)                 // no compensator, plain, INT3; bf16 without and with
                if (hipFuncSetAttribute(reinterpret_cast<const void*>(decode_split_variant(R, v == 1 || v == 2 || v == 4, v == 2, v >= 3)),
                                        hipFuncAttributeMaxDynamicSharedMemorySize, kDecLdsTotal) != hipSuccess)
                    return 0;
        cached[dev] = cus;
    }
    return cached[dev];
}

// K parts of the T workers: kDecTWaves chunks of 256 columns each, or twice that.  Two chunks per wave cost a worker a
// second round trip and halve the fragments every streaming workgroup fetches: from five fragments on that is
// the faster side (M = 16, us: N = 4096, K = 14336, r = 32, 7 or 4 fragments, 16.3 -> 16.1; r = 64, 14 or 8, 17.1 -> 16.3;
// N = 2048, K = 8192, r = 64, 8 or 4, 8.4 -> 8.0; N = K = 4096, r = 128, 8 or 4, 6.7 -> 6.6), with up to four there
// is nothing to gain, and beyond 16, all that the LDS holds, it is the only one (r = 128 beyond K = 8192).
static int decode_k_parts(int64_t K, int chunks) { return (int)((K + 256 * kDecTWaves * chunks - 1) / (256 * kDecTWaves * chunks)); }
struct DecodeT {
    bool staged;        // granules and the staged path (LR == 1)
    int chunks, kh, nks;
};
static DecodeT decode_t_plan(int64_t N, int64_t K, int r) {
    DecodeT t;
    t.nks = (r + 31) / 32;
    t.chunks = decode_k_parts(K, 1) * t.nks > 4 ? 2 : 1;
    t.kh = decode_k_parts(K, t.chunks);
    t.staged = r > 0 && r <= 32 * kDecKS && t.kh * t.nks <= kDecTFrags && (uint64_t)N * (uint64_t)r * 2u < 0xFFFFFFF0ull;
    if (!t.staged) {
        t.chunks = 1;
        t.kh = decode_k_parts(K, 1);
    }
    return t;
}

static_assert(kDecTFrags * 2048 == kDecGranuleBytes, "granules of all fragments");

// T workers of a launch: one per block of 16 ranks and K part, at most kDecMaxWorkers and never more than
// a quarter of the resident workgroups (a worker then takes several items in turn).
static int decode_workers(int rblocks, int kh, int cap) {
    int nt = rblocks * kh;
    if (nt > kDecMaxWorkers) nt = kDecMaxWorkers;
    if (nt > cap / 4) nt = cap / 4 > 0 ? cap / 4 : 1;
    return nt;
}

// Row blocks per wave with which the long-K kernel (w3lr_decode_split_kernel) can run a problem in one round: the fewest, so
// that all CUs stream (0: it cannot).
static int decode_split_rows(int64_t N, int64_t K, int r, int cap) {
    const int64_t nchunks = (K + 255) / 256;
    if (nchunks <= kDecWaves) return 0;
    int64_t slots = cap < kDecSplitMax ? cap : kDecSplitMax;
    if (r > 0) {
        const DecodeT t = decode_t_plan(N, K, r);
        if (!t.staged || t.kh * t.nks > kDecSplitFrags) return 0;
        const int64_t room = cap - decode_workers((r + 15) / 16, t.kh, cap);
        if (room < slots) slots = room;
    }
    for (int R = 1; R <= 4; R *= 2) {
        const int64_t wgs = ((N + 16 * R - 1) / (16 * R) * nchunks + kDecWaves - 1) / kDecWaves;
        if (wgs <= slots) return wgs >= (int64_t)kDecGroups ? R : 0;
    }
    return 0;
}

// Granules of the long-K kernel, behind the head.
static size_t decode_split_bytes(int64_t N, int64_t K, int R) {
    const int64_t nchunks = (K + 255) / 256;
    return (size_t)(((N + 16 * R - 1) / (16 * R) * nchunks + kDecWaves - 1) / kDecWaves) * R * 2048;
}

size_t decode_workspace_min(int64_t N, int64_t K, int r) {
    if (r <= 0) return 256;
    const size_t rblocks = ((size_t)r + 15) / 16;
    const DecodeT t = decode_t_plan(N, K, r);
    // head | T 16-bit [K parts][16 x ldt] of the other path
    return kGemmHeadBytes + (t.staged ? 0 : align_up((size_t)t.kh * 16 * rblocks * 16 * 2, 256));
}

// Row blocks per workgroup (16 R rows).  Every workgroup stages all of X once per turn and streams
// R row blocks; a CU takes in activations (from L2) roughly five times as fast as weights (from
// HBM), and the launch takes as long as its busiest CU: `turns` rounds of that.  The estimate picks
// R = 4 for the wide up projections, R = 1 for small weights, and for a long-K down projection whose
// R = 1 grid would exceed the resident workgroups by a few (a second round for a handful of
// blocks) the next R, which fits in one round.
static int decode_rows_per_workgroup(int64_t N, int64_t K, int slots) {
    const double x_bytes = 32.0 * (double)K, blk_bytes = 7.0 * (double)K;       // 16 rows of fp16 / of 3.5 bit
    int best = 1;
    double best_cost = 0.0;
    for (int R = 1; R <= 4; R *= 2) {
        const int64_t blocks = (N + 16 * R - 1) / (16 * R);
        const int64_t turns = (blocks + slots - 1) / slots;
        const double cost = (double)turns * (x_bytes / 130.0 + R * blk_bytes / 25.0);
        if (R == 1 || cost < best_cost) {
            best = R;
            best_cost = cost;
        }
    }
    return best;
}

// Whether the long-K kernel, with Rs row blocks per wave, is the faster one for a problem that the other would walk with R
// of them.  The other one walks ceil(chunks / 16) chunks per wave in turn and copies each workgroup's chunks of X; the long-K
// kernel walks one, but hands partial sums over.  Both estimates (us) are fits to 37 shapes from 512 x 4160 to 12000 x 4864 and
// 4096 x 14336 at M = 1 .. 16, and were checked on 69 drawn ones: of those 276 points one was spread although it is
// slower, by 2 %, and 17 were not although they would be 2 to 13 % faster.  The copies count with the chunks there are, not
// with whole rounds of sixteen: with seventeen to 24 chunks M = 5 .. 8 was spread at a loss (512 x 4160, M = 8, 5.5 in
// turn against 5.8; 752 x 4160, M = 5, 5.9 / 6.3).  Measured, chunks in turn -> spread: M = 16, r = 32, 4096 x 14336 15.6 -> 11.4;
// 1024 x 14336 12.1 -> 6.9; 2816 x 11008 10.3 -> 8.3; 12000 x 4864 13.5 -> 11.9; 512 x 8192 7.5 -> 6.4; M = 1, 4096 x 14336
// 12.0 -> 10.2.  Where it stays: M = 1, 3920 x 8128 6.2 -> 7.2, 1440 x 4608 5.4 -> 6.0; M = 8, 4096 x 8192 8.6 -> 9.4;
// M = 16, 3008 x 6016 7.6 -> 7.8.
static bool decode_split_faster(int64_t N, int64_t K, int xc, int R, int Rs, int slots) {
    const int64_t nchunks = (K + 255) / 256, blocks = (N + 16 * R - 1) / (16 * R), bands = (N + 16 * Rs - 1) / (16 * Rs);
    const double turns = (double)((blocks + slots - 1) / slots), rounds = (double)((nchunks + kDecWaves - 1) / kDecWaves);
    const double per_wave = (double)nchunks / kDecWaves;
    const double other = 2.9 + turns * (rounds * (0.02 + 1.1 * R) + 0.179 * xc * per_wave);
    const double split = 5.5 + 1.3 * (Rs - 1) + 0.05 * xc + 0.0013 * (double)bands * per_wave;
    return split + 0.46 < other;
}

// Tuning override of the row blocks per workgroup, read once per process (it also keeps the long-K kernel out).
static int decode_row_override() {
    static const int rows = [] {
        const char* e = getenv("MILO_DEC_R");
        const int v = e ? atoi(e) : 0;
        return (v == 1 || v == 2 || v == 4) ? v : 0;
    }();
    return rows;
}

// Row blocks per wave with which a launch of `xc` activation copies per chunk takes the long-K kernel (0: the other one), where
// that one would take R and `slots` workgroups stream.
static int decode_split_choice(int64_t N, int64_t K, int r, int xc, int R, int slots, int cap) {
    const int rows = decode_row_override() ? 0 : decode_split_rows(N, K, r, cap);
    return rows > 0 && decode_split_faster(N, K, xc, R, rows, slots) ? rows : 0;
}

// Room for the granules where any launch of up to sixteen rows takes the long-K kernel.  The more activation copies, the
// further that one is ahead (a copy more costs it 0.05 us, the other kernel 0.179 us for each chunk of a wave), so eight copies
// decide.
size_t decode_workspace_bytes(int64_t N, int64_t K, int r) {
    const size_t least = decode_workspace_min(N, K, r);
    const int cap = device_cus();
    const int slots = cap - (r > 0 ? decode_workers((r + 15) / 16, decode_t_plan(N, K, r).kh, cap) : 0);
    if (slots <= 0) return least;
    const int rows = decode_split_choice(N, K, r, 8, decode_rows_per_workgroup(N, K, slots), slots, cap);
    return rows > 0 ? kGemmHeadBytes + decode_split_bytes(N, K, rows) : least;
}

int launch_decode(DecodeArgs a, void* workspace, size_t workspace_bytes, hipStream_t stream) {
    const int cap = decode_capacity();
    if (cap <= 0) return MILO_ERR_HIP;
    const int r = a.w.r;
    a.rblocks = (r + 15) / 16;
    a.ldt = (int64_t)a.rblocks * 16;
    // V (padded to whole rank blocks) is addressed with 32-bit byte offsets
    if ((uint64_t)a.ldt * (uint64_t)a.K * 2u >= 0xFFFFFFF0ull) return MILO_ERR_SHAPE;
    char* ws = reinterpret_cast<char*>(workspace);
    a.ctrl = reinterpret_cast<uint32_t*>(ws);
    a.done = reinterpret_cast<uint32_t*>(ws + kGemmDoneAt);
    a.epoch = reinterpret_cast<unsigned long long*>(ws + kGemmCountersAt);
    a.tg = reinterpret_cast<unsigned long long*>(ws + kGemmGranulesAt);
    a.T = reinterpret_cast<f16*>(ws + kGemmHeadBytes);
    const DecodeT tp = decode_t_plan(a.N, a.K, r);
    a.kh = tp.kh;
    a.nks = tp.nks;
    a.t_chunks = tp.chunks;
    a.spin_limit = 1u << 24;
    const int nt = decode_workers(a.rblocks, a.kh, cap);
    a.nt = nt;
    const int workers = r > 0 ? nt : 0;
    if (cap <= workers || (size_t)cap * 4 > kDecDoneBytes) return MILO_ERR_HIP;
    int R = decode_rows_per_workgroup(a.N, a.K, cap - workers);
    if (decode_row_override()) R = decode_row_override();
    const int xc = a.M <= 2 ? 1 : a.M <= 4 ? 2 : a.M <= 8 ? 4 : 8;    // activation copies per chunk: rows 2i, 2i+1
    int split_rows = decode_split_choice(a.N, a.K, r, xc, R, cap - workers, cap);
    // (a workspace that has no room for the granules is one for the other kernel)
    if (split_rows > 0 && workspace_bytes < kGemmHeadBytes + decode_split_bytes(a.N, a.K, split_rows)) split_rows = 0;
    if (split_rows > 0) R = split_rows;
    const int rows = 16 * R;
    const int64_t blocks = (a.N + rows - 1) / rows;
    const int grid = (int)(blocks < cap - workers ? blocks : cap - workers) + workers;
    const int lr = r == 0 ? 0 : tp.staged ? 1 : 2;
    const bool q = r > 0 && (a.w.flags & MILO_LR_INT3) != 0;
    // an INT3 compensator only runs on the staged path; the limit is the one of its fragments at one chunk per wave
    if (q && (lr != 1 || decode_k_parts(a.K, 1) * tp.nks > kDecTFrags)) return MILO_ERR_SHAPE;
    const bool bf = (a.w.flags & MILO_ACT_BF16) != 0;
    if (bf && q) return MILO_ERR_SHAPE;
    a.units = (uint32_t)(a.N * (a.K / kGroup));
    a.nb = (uint32_t)(a.N >> 4);
    a.x_bytes = (uint32_t)((uint64_t)a.M * (uint64_t)a.K * 2u);            // (< 2^32: checked by the caller)
    a.t_bytes = (uint32_t)((uint64_t)a.kh * 16u * (uint64_t)a.ldt * 2u);
    a.u_bytes = (uint32_t)((uint64_t)a.N * (uint64_t)(r > 0 ? r : 0) * 2u);   // (fp16 U; < 2^32 on the staged path)
    const uint32_t nchunks = (uint32_t)((a.K + 255) / 256);
    if (split_rows > 0) {
        a.nmain = (uint32_t)((blocks * nchunks + kDecWaves - 1) / kDecWaves);
        a.pg = reinterpret_cast<unsigned long long*>(ws + kGemmHeadBytes);
        // quotient by nchunks as the upper half of a product: exact while dividend x divisor stays below 2^32
        const uint32_t magic = (uint32_t)((uint64_t(1) << 32) / nchunks) + 1u;
        decode_split_variant(R, r > 0, q, bf)<<<dim3(a.nmain + (uint32_t)workers), dim3(kDecThreads), kDecLdsTotal, stream>>>(
            a.w.q3, a.X, a.units, (uint32_t)a.K, a.nb, a.M, a.nt, a.nmain, nchunks, magic, a.x_bytes, a);
        return launch_status();
    }
    const DecodeKernel kernel = decode_variant(R, lr, xc, (a.w.flags & MILO_W3_SYMMETRIC) != 0, q, bf);
    if (!kernel) return MILO_ERR_HIP;
    a.nmain = (uint32_t)(grid - workers);
    a.turns = (uint32_t)((blocks + a.nmain - 1) / a.nmain);
    a.chunks_per_wave = (nchunks + kDecWaves - 1) / kDecWaves;
    uint32_t pow2 = kDecWaves;
    while (pow2 * 2u <= a.chunks_per_wave * kDecWaves) pow2 *= 2u;
    a.rot_mask = pow2 - 1u;
    kernel<<<dim3((unsigned)grid), dim3(kDecThreads), lr == 1 ? kDecLdsTotal : kDecLdsBytes, stream>>>(
        a.w.q3, a.X, a.units, (uint32_t)a.K, a.nb, a.M, a.nt, a.nmain, a.chunks_per_wave, a.rot_mask, a.x_bytes, a);
    return launch_status();
}

}  // namespace milo
