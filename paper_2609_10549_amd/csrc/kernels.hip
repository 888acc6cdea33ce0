// gfx950 kernels of the Compass hot path.
//
// gemm_kernel<BM, BN, DW, RS, WT>: persistent bf16 GEMM, C = A * W^T with fp32
// accumulation on the CDNA4 matrix cores (v_mfma_f32_16x16x32_bf16) and one
// bf16 round-to-nearest-even store. Workgroups take BM x BN output tiles in
// the order the host chose (ring-arrival order for TA-IntraFusion, Section
// III-B) and, depending on the gate mode, wait on the per-partition arrival
// flags published for the copy engines before reading A (AllGather) or before
// adding the incoming partial sum (ReduceScatter).
//
// Tile distribution: launches whose tiles do not wait for one another, and
// fused ones of one round, take fixed positions (static_position). The others
// take tickets from atomic queues: the ready order of tiles is cut into
// super-blocks; queue v (one per XCD: workgroups are dispatched round-robin
// over the 8 XCDs, so workgroup b serves queue b % 8) takes super-blocks v,
// v + 8, ... Inside the order, positions walk a group of row tiles before
// moving to the next column tile, so the tiles one XCD holds at a time share A
// rows and W rows in that XCD's L2.
//
// Data path per tile: 4 waves split the tile 2 x 2; each wave holds
// (BM/2) x (BN/2) fp32 accumulators as 16 x 16 MFMA blocks. A and W stream
// through LDS in stages of K = 64 (rows of 128 bytes, whole cache lines per
// load: the texture path's cost grows with the lines a load touches), DW + 1
// buffers of A and DW of W (with DW = 2 all 160 KiB for a 256 x 256 tile), with
// buffer_load ... lds (no register staging; out-of-range rows or K columns
// read as zero through the buffer bound). The 16-byte chunks of LDS row r are
// XOR-permuted with (r >> 1) & 7, so a fragment read hits distinct banks.
//
// What bounds it: the large tiles, the matrix cores at the clock the chip's
// power allows (1.5 - 1.7 GHz under this load, 2.4 GHz nominal), so what
// counts is energy per flop and cycles lost to waits. 8192 x 6144 x 12288,
// 256 x 256 tiles, each step against the one before it on one box:
//  - three A buffers in place of two (loads have 1 to 1.75 stages to land; one
//    barrier per stage): 942 -> 925 us;
//  - LDS reads and global loads one at a time between the MFMAs in place of
//    bursts of eight, which filled their queues and held up the MFMAs behind
//    them: 925 -> 908 us;
//  - v_mfma_f32_16x16x32_bf16 in place of 32x32x16: half the accumulator
//    traffic per flop (each accumulator is read and written once per 32 of K
//    in place of 16), a higher clock and shorter stalls: 908 -> 834 us
//    (1.48 PFLOP/s; stage time 1.46 -> 1.38 us);
//  - consecutive MFMAs always sharing an operand (slot_row): 845 -> 832 us.
// The small tiles are bound by the latency of a stage (barrier, LDS, loads),
// for which DW = 3 or 4 keeps the loads of that many stages in flight: 48 rows
// x 8192 x 3072 in 128 x 64 tiles, a stage 0.32 us with DW = 2, 0.205 with 4.
//
// skinny_kernel: the GEMM for at most 64 rows.
//
// join_kernel: one wave that (optionally) marks the start of a transfer job
// and waits for a list of flags, putting the end of the copy side onto the
// stream.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernel_params.h"

namespace compass {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

#define LDS_AS(p) ((__attribute__((address_space(3))) void *)(p))

// Buffer loads of a tile go through a resource based at the tile's first
// row (A, the partial) or first column (W), bounded by the bytes left in the
// operand, at most kTileSpanMax; offsets are relative to that base. An
// out-of-range row or column takes an offset at or beyond the bound:
// kOOBRow = 2^31 for a row, kOOBCol = 2^30 for a K column. A valid row offset
// plus a valid column offset stays below the 2^30 bound (the host checks the
// tile's span), a valid one plus an out-of-range one reaches it, and two
// out-of-range ones sum to 3 * 2^30, below 2^32, so no sum wraps.
constexpr uint32_t kOOBRow = 0x80000000u;
constexpr uint32_t kOOBCol = 0x40000000u;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_rsrc(const void *base, uint64_t total, uint64_t off) {
    const uint64_t left = total > off ? total - off : 0;
    const uint32_t bound = (uint32_t)(left < kTileSpanMax ? left : kTileSpanMax);
    return __builtin_amdgcn_make_buffer_rsrc((void *)((const char *)base + off), (short)0, (int)bound, 0x00020000);
}

__device__ __forceinline__ uint32_t ld_flag(const uint32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

__device__ __forceinline__ uint32_t ld_dev(const uint32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Poll *w until it reaches epoch; false on the bound or a raised error word.
__device__ __forceinline__ bool poll_epoch(const uint32_t *w, bool host, uint32_t epoch, uint32_t limit,
                                           uint32_t *err, int sleep_code) {
    uint32_t polls = 0;
    while ((int32_t)((host ? ld_flag(w) : ld_dev(w)) - epoch) < 0) {
        if (++polls > limit) {
            __hip_atomic_fetch_or(err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            return false;
        }
        if ((polls & 255u) == 0 && ld_flag(err) != 0) return false;
        if (sleep_code == 4) __builtin_amdgcn_s_sleep(4);
        else __builtin_amdgcn_s_sleep(16);
    }
    return true;
}

// Wait of wave 0 for every partition in `mask` (bit q: partition q, at most
// 64): lane q handles partition q, so the flags are polled in parallel. Per
// partition and epoch one workgroup (the first to claim `leader`) polls the
// host-memory arrival flag and forwards it to `mirror` in device memory;
// every other workgroup polls the mirror. A system-scope acquire follows, so
// that the rows the copy engines wrote are read from memory, not from stale
// cache lines. True when every partition arrived (false: bound or error).
__device__ bool wait_flags(const GemmParams &p, uint64_t mask, int lane) {
    bool ok = true;
    if ((mask >> lane) & 1ull) {
        const int f = p.flag_base + lane;
        if ((int32_t)(ld_dev(&p.mirror[f]) - p.epoch) < 0) {
            uint32_t cur = ld_dev(&p.leader[f]);
            bool lead = false;
            while ((int32_t)(cur - p.epoch) < 0) {
                uint32_t expect = cur;
                if (__hip_atomic_compare_exchange_strong(&p.leader[f], &expect, p.epoch, __ATOMIC_RELAXED,
                                                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                    lead = true;
                    break;
                }
                cur = expect;
            }
            if (lead) {
                ok = poll_epoch(&p.flags[f], true, p.epoch, p.spin_limit, p.err_word, 16);
                if (ok) __hip_atomic_store(&p.mirror[f], p.epoch, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
            } else {
                ok = poll_epoch(&p.mirror[f], false, p.epoch, p.spin_limit, p.err_word, 4);
            }
        }
    }
    const bool all_ok = __ballot(!ok) == 0ull;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "");
    return all_ok;
}

__device__ __forceinline__ uint32_t rtc32() { return (uint32_t)__builtin_amdgcn_s_memrealtime(); }

__device__ __forceinline__ uint32_t hw_id() {
    uint32_t v;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_HW_ID)" : "=s"(v));
    return v;
}

__device__ __forceinline__ uint32_t xcc_id() {
    uint32_t v;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(v));
    return v;
}

// Order of this workgroup among the workgroups of this launch on its CU
// (0 for the first): a claim word per (XCC, SE, SH, CU) holds
// launch_seq << 8 | count.
__device__ uint32_t claim_cu_slot(const GemmParams &p) {
    const uint32_t key = ((xcc_id() & 7u) << 8) | ((hw_id() >> 8) & 0xFFu);
    uint32_t *w = p.cu_slots + key;
    const uint32_t tag = p.launch_seq & 0xFFFFFFu;
    uint32_t cur = ld_dev(w);
    for (;;) {
        const bool same = (cur >> 8) == tag;
        const uint32_t want = same ? cur + 1u : ((tag << 8) | 1u);
        uint32_t expect = cur;
        if (__hip_atomic_compare_exchange_strong(w, &expect, want, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT))
            return same ? (cur & 0xFFu) : 0u;
        cur = expect;
    }
}

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    const __bf16 a = (__bf16)lo, b = (__bf16)hi;   // round to nearest even
    return (uint32_t)__builtin_bit_cast(uint16_t, a) | ((uint32_t)__builtin_bit_cast(uint16_t, b) << 16);
}

__device__ __forceinline__ int map_row(const GemmParams &p, int i) {
    if (p.piece == 0) return i;
    const int q = i / p.piece;
    return q * p.pstride + p.poff + (i - q * p.piece);
}

__device__ __forceinline__ uint64_t range_mask(int lo, int hi) {
    const uint64_t upto = hi >= 63 ? ~0ull : ((2ull << hi) - 1ull);
    return upto & ~((1ull << lo) - 1ull);
}

// Position in the ready order of local ticket c of queue v.
__device__ __forceinline__ int ticket_position(const GemmParams &p, int v, uint32_t c) {
    const int k = (int)(c / (uint32_t)p.q_size);
    const int i = (int)(c - (uint32_t)k * (uint32_t)p.q_size);
    return (v + p.nq * k) * p.q_size + i;
}

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// At most VM vector-memory operations (and no LDS read) still in flight.
template <int VM>
__device__ __forceinline__ void wait_vm_lgkm0() {
    static_assert(VM >= 0 && VM < 64, "vmcnt range");
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(VM) : "memory");
}

// Workgroup barrier with no memory fence: the caller has already waited for
// the LDS traffic that must be complete (s_waitcnt), and the scheduling
// barriers keep the compiler from moving LDS accesses across it.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// Buffer resource words of tile_rsrc as plain scalars, for dma16.
__device__ __forceinline__ i32x4 tile_rsrc4(const void *base, uint64_t total, uint64_t off) {
    const uint64_t left = total > off ? total - off : 0;
    const uint32_t bound = (uint32_t)(left < kTileSpanMax ? left : kTileSpanMax);
    const uint64_t a = (uint64_t)base + off;
    i32x4 r;
    r[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)a);
    r[1] = __builtin_amdgcn_readfirstlane((int)((uint32_t)(a >> 32) & 0xFFFFu));
    r[2] = __builtin_amdgcn_readfirstlane((int)bound);
    r[3] = 0x00020000;
    return r;
}

// One global -> LDS load: 16 bytes per lane from rsrc + voff to LDS byte
// address lds + 16 * lane. It has no register result, so nothing of it is
// live in a register while it is in flight; it is written as an instruction
// because the compiler, which cannot see that two halves of one LDS array
// are different buffers, would otherwise wait for every load in flight before
// each LDS read. The waits are wait_vm_lgkm0's, counted where they are made.
// (s_nop: a scalar write of M0 needs a wait state before the load reads it.)
__device__ __forceinline__ void dma16(i32x4 rsrc, uint32_t voff, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 :
                 : "s"(lds), "v"(voff), "s"(rsrc)
                 : "memory");
}

// `CNT` loads of one operand into the 1 KiB blocks j * 4 + wave of the LDS
// buffer at `lds`.
template <int CNT>
__device__ __forceinline__ void load_blocks(i32x4 rsrc, uint32_t lds, const uint32_t *off, uint32_t kc2, int wave) {
#pragma unroll
    for (int j = 0; j < CNT; ++j) dma16(rsrc, off[j] + kc2, lds + (uint32_t)((j * 4 + wave) * 1024));
}

// Fragment F of an MFMA substep in the order the substep needs them (b[0],
// a[0 .. FM), b[1 .. FN)): 16 rows of 128 bytes each; fa / fw: this lane's
// row and 16-byte chunk in the stage's buffers.
template <int F, int FM, int FN>
__device__ __forceinline__ void read_frag(const char *fa, const char *fw, bf16x8 (&a)[FM], bf16x8 (&b)[FN]) {
    if constexpr (F >= 1 && F <= FM)
        a[F - 1] = *reinterpret_cast<const bf16x8 *>(fa + (F - 1) * 16 * 128);
    else
        b[F == 0 ? 0 : F - FM] = *reinterpret_cast<const bf16x8 *>(fw + (F == 0 ? 0 : F - FM) * 16 * 128);
}

// Where operation `k` of n falls among MFMA slots [lo, hi).
constexpr int slot_of(int k, int n, int lo, int hi) { return lo + k * (hi - lo) / n; }

// The reads that fall into slot I.
template <int F, int I, int R0, int R1, int FM, int FN>
__device__ __forceinline__ void read_slot(const char *fa, const char *fw, bf16x8 (&a)[FM], bf16x8 (&b)[FN]) {
    if constexpr (F < FM + FN) {
        if constexpr (slot_of(F, FM + FN, R0, R1) == I) read_frag<F, FM, FN>(fa, fw, a, b);
        read_slot<F + 1, I, R0, R1, FM, FN>(fa, fw, a, b);
    }
}

// Block row of MFMA slot i (block column i / FM): down one column of blocks, up
// the next, so that consecutive MFMAs always share an operand. The operand that
// stays costs no switching in the matrix core, and power is what bounds these
// GEMMs: 8192 x 6144 x 12288 845 -> 832 us, 8192 x 12288 x 6144 with partial
// 906 -> 897 (going down every column before).
template <int FM>
constexpr int slot_row(int i) { return i / FM % 2 ? FM - 1 - i % FM : i % FM; }

// MFMAs [I0, I1) of a substep on (a, b) (block acc[i / FM][slot_row(i)]), with
// the next substep's fragment reads into (na, nb) spread over MFMA slots
// [R0, R1) and loads [L0, L0 + LC) of one operand over slots [D0, D1), in
// exactly this order: an LDS read and a global load each occupy a unit that
// the four waves share for about one MFMA's time, so a burst of either fills
// its queue and holds up the MFMAs behind it.
template <int I, int I1, int R0, int R1, int L0, int LC, int D0, int D1, int FM, int FN>
__device__ __forceinline__ void mfma_slots(f32x4 (&acc)[FN][FM], const bf16x8 (&a)[FM], const bf16x8 (&b)[FN],
                                           bf16x8 (&na)[FM], bf16x8 (&nb)[FN], const char *fa, const char *fw,
                                           i32x4 rsrc, uint32_t lds, const uint32_t *off, uint32_t kc2) {
    if constexpr (I < I1) {
        constexpr int NI = I / FM, MI = slot_row<FM>(I);
        acc[NI][MI] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[NI], a[MI], acc[NI][MI], 0, 0, 0);
        read_slot<0, I, R0, R1, FM, FN>(fa, fw, na, nb);
#pragma unroll
        for (int j = 0; j < LC; ++j)
            if (slot_of(j, LC, D0, D1) == I) dma16(rsrc, off[L0 + j] + kc2, lds + (uint32_t)((L0 + j) * 4096));
        __builtin_amdgcn_sched_barrier(0);
        mfma_slots<I + 1, I1, R0, R1, L0, LC, D0, D1, FM, FN>(acc, a, b, na, nb, fa, fw, rsrc, lds, off, kc2);
    }
}

constexpr int kBK = 64;   // K depth of one LDS stage

// RS = false: optional main-loop gate (AllGather), plain store.
// RS = true: optional epilogue gate, fp32 partial add, chunk-done signalling;
// WT = true (a launch whose finished chunks the copy engines send on): the
// partial-add epilogue stores every tile with system-scope write-through.
// DW: W stage buffers (DW + 1 of A). The loads of a stage go out DW - 1 to DW
// stages before their use.
template <int BM, int BN, int DW, bool RS, bool WT = false>
__global__ __launch_bounds__(kThreads, (160 << 10) / (((DW + 1) * BM + DW * BN) * 128))
void gemm_kernel(const GemmParams p) {
    constexpr int WM = BM / 2, WN = BN / 2;
    constexpr int FM = WM / 16, FN = WN / 16;
    constexpr int LA = BM / 32, LW = BN / 32;   // loads per wave and stage of A, W
    constexpr int SA = BM * 128, SW = BN * 128; // bytes of one stage buffer
    constexpr bool kSplits = BM > 64;           // (the host never splits K of the smallest tile)
    constexpr int NA = DW + 1;
    constexpr bool kAcc = NA * SA + DW * SW > (80 << 10);   // one workgroup per CU
    // the A buffers, then the W buffers
    __shared__ __attribute__((aligned(1024))) char smem[NA * SA + DW * SW];
    // control words in the tail of the last A buffer: the first load that
    // lands there is issued in stage 0 of a tile, behind the prologue's
    // barrier, which every wave reaches after it read them
    int &s_pos = reinterpret_cast<int *>(smem + NA * SA)[-1];
    int &s_ok = reinterpret_cast<int *>(smem + NA * SA)[-2];
    int &s_last = reinterpret_cast<int *>(smem + NA * SA)[-3];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm0 = (wave >> 1) * WM;
    const int wn0 = (wave & 1) * WN;
    const int total = work_items(p);
    const int v = p.nq > 1 ? (int)(blockIdx.x % (uint32_t)p.nq) : 0;


    // loader geometry: load q of this wave covers tile rows 32 q + 8 wave +
    // (lane >> 3), 128 bytes (K = 64) each; the lane loads the logical chunk
    // that the permutation (row >> 1) & 7 puts at its physical chunk lane & 7
    const int lrow0 = 8 * wave + (lane >> 3);
    const int cchunk = (lane & 7) ^ ((4 * wave + (lane >> 4)) & 7);
    const int r = lane & 15;                       // fragment row
    const int kq = lane >> 4;                      // fragment K quarter
    const int swz = (r >> 1) & 7;

    uint64_t known = 0;   // partitions already acquired by this workgroup
    bool failed = false;

    int pos, round = 0;
    if (p.fixed) {
        pos = static_position(p, (int)blockIdx.x, 0);
        if (pos == 0 && p.start_word && tid == 0)
            __hip_atomic_store(p.start_word, p.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    } else {
        if (tid == 0) {
            if (p.spread_wait > 0 && claim_cu_slot(p) > 0) {
                // bounded: a scheduling preference, never a dependency
                const uint32_t t_end = rtc32() + 1000u;   // 10 us of the 100 MHz counter
                while ((int)ld_dev(&p.ctrl[v]) < p.spread_wait && (int32_t)(rtc32() - t_end) < 0)
                    __builtin_amdgcn_s_sleep(2);
            }
            const uint32_t c = __hip_atomic_fetch_add(&p.ctrl[v], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const int first = ticket_position(p, v, c);
            if (first == 0 && p.start_word)
                __hip_atomic_store(p.start_word, p.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            s_pos = first;
        }
        __syncthreads();
        pos = __builtin_amdgcn_readfirstlane(s_pos);
    }

    while (pos >= 0 && pos < total) {
        // work position -> (tile position, K slice); `split`: this tile's K
        // is split into `ns` slices, counted by split_cnt[uc], its partials
        // at workspace tiles [wsf, wsf + ns)
        const WorkItem wi = decode_item(p, pos);
        const bool split = kSplits && wi.split;
        const int tpos = wi.tpos, slice = wi.slice, ns = wi.ns, uc = wi.uc, wsf = wi.wsf, ksl = wi.ksl;
        const int kb = split ? slice * ksl : 0;
        const int ke = split ? min(p.K, kb + ksl) : p.K;
        // tile position -> (row-tile ordinal, column tile): group_m rows at a time
        int ti, tn;
        tile_of(p, tpos, &ti, &tn);
        const int rt = p.rt_order[ti];
        const int m0 = rt * BM;
        const int n0 = tn * BN;
        const uint64_t touch = range_mask(p.rt_lo[rt], p.rt_hi[rt]);
        const uint64_t need = touch & ~p.resident_mask & ~known;
        const bool traced = p.tile_trace && p.trace_base + (uint32_t)pos < p.trace_cap;
        uint32_t t_tick = 0, t_gate = 0, t_loop = 0;
        if (traced && tid == 0) t_tick = rtc32();

        if (!RS && p.gate == kGateMain && need) {
            if (wave == 0) {
                const bool ok = wait_flags(p, need, lane);
                if (lane == 0) s_ok = ok;
            }
            __syncthreads();
            if (!s_ok) failed = true;
            known |= need;
        }
        if (!RS && traced && tid == 0) t_gate = rtc32();

        f32x4 acc[FN][FM];
#pragma unroll
        for (int ni = 0; ni < FN; ++ni)
#pragma unroll
            for (int mi = 0; mi < FM; ++mi)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[ni][mi][e] = 0.0f;

        {   // a timed-out tile still runs (its loads stay in bounds); only its
            // stores are dropped
            // A from the tile's first (mapped) row, W from its first column
            const int row0 = map_row(p, m0);
            const i32x4 rA0 = tile_rsrc4(p.A, p.a_bytes, (uint64_t)row0 * (uint64_t)p.lda * 2u);
            const i32x4 rW0 = tile_rsrc4(p.W, p.w_bytes, (uint64_t)n0 * (uint64_t)p.ldw * 2u);
            uint32_t offA[LA], offW[LW];
#pragma unroll
            for (int q = 0; q < LA; ++q) {
                const int ia = m0 + 32 * q + lrow0;
                offA[q] = ia < p.M ? (uint32_t)(map_row(p, ia) - row0) * (uint32_t)p.lda * 2u : kOOBRow;
            }
#pragma unroll
            for (int q = 0; q < LW; ++q) {
                const int iw = n0 + 32 * q + lrow0;
                offW[q] = iw < p.N ? (uint32_t)(iw - n0) * (uint32_t)p.ldw * 2u : kOOBRow;
            }
            auto kcol = [&](int st) -> uint32_t {   // byte offset of this lane's K chunk in stage st
                const int kc = kb + st * kBK + cchunk * 8;
                return kc < ke ? (uint32_t)kc * 2u : kOOBCol;
            };
            const int KT = (ke - kb + kBK - 1) / kBK;
            // LDS byte offsets of the buffers, rings of NA and DW
            const uint32_t lds0 = (uint32_t)(uintptr_t)LDS_AS(smem);
            const uint32_t ldsW = lds0 + NA * SA, ldsE = ldsW + DW * SW;
            // prologue: stages 0 to DW - 1 in flight; stage 0 landed, its first
            // fragments read (s_nop: resource words that came out of vector
            // registers need five wait states before a load reads them)
            i32x4 rA = rA0, rW = rW0;
            asm volatile("s_nop 4" : "+s"(rA), "+s"(rW));
#pragma unroll
            for (int i = 0; i < DW; ++i) {
                load_blocks<LA>(rA, lds0 + i * SA, offA, kcol(i), wave);
                load_blocks<LW>(rW, ldsW + i * SW, offW, kcol(i), wave);
            }
            wait_vm_lgkm0<(DW - 1) * (LA + LW)>();
            lds_barrier();
            bf16x8 a0[FM], b0[FN], a1[FM], b1[FN];
            const char *fa = smem + (wm0 + r) * 128;       // this lane's fragment rows, relative
            const char *fw = smem + (wn0 + r) * 128;       // to a buffer at smem + 0
            const int coff0 = (kq ^ swz) << 4, coff1 = ((4 + kq) ^ swz) << 4;
            {
                const char *ca = fa + coff0, *cw = fw + NA * SA + coff0;
#pragma unroll
                for (int mi = 0; mi < FM; ++mi) a0[mi] = *reinterpret_cast<const bf16x8 *>(ca + mi * 16 * 128);
#pragma unroll
                for (int ni = 0; ni < FN; ++ni) b0[ni] = *reinterpret_cast<const bf16x8 *>(cw + ni * 16 * 128);
            }
            constexpr int NM = FM * FN;
            constexpr int RE = NM - NM / 4;     // substep 0's reads end here, ahead of the barrier's wait
            constexpr int B1 = NM / 16;         // MFMAs of substep 1 before the barrier
            const uint32_t wb = (uint32_t)wave * 1024u;
            // Stage st on (aC, wC), its substep-0 fragments in (a0, b0), stage
            // st + 1 in flight in (aN, wN). Substep 0 (the first 32 of K) reads
            // substep 1's fragments and issues the A loads of stage st + DW into
            // aF, which stage st - 1 freed. Substep 1 waits for all of stage
            // st + 1 (the loads of later stages stay in flight), joins the
            // barrier, reads stage st + 1's first fragments and issues stage
            // st + DW's W loads into wC, whose fragments every wave has read.
            uint32_t aC = lds0, aF = lds0 + DW * SA, wC = ldsW;
            for (int st = 0; st < KT; ++st) {
                const uint32_t aN = aC + SA == ldsW ? lds0 : aC + SA, wN = wC + SW == ldsE ? ldsW : wC + SW;
                const char *ca = fa + (aC - lds0), *cw = fw + (wC - lds0);
                const uint32_t kcf = kcol(st + DW);
                // with one workgroup per CU the accumulators live in the
                // accumulation registers: saying so here keeps every one of
                // them in its own register around the loop (the compiler had
                // MFMAs write a neighbouring one and moved up to 68 registers
                // back per stage: 8192 x 6144 x 12288 855 against 811 us);
                // in the MFMAs' order
                if constexpr (kAcc) {
#pragma unroll
                    for (int i = 0; i < NM; ++i) asm volatile("" : "+a"(acc[i / FM][slot_row<FM>(i)]));
                }
                mfma_slots<0, NM, 0, RE, 0, LA, 0, NM, FM, FN>(acc, a0, b0, a1, b1, ca + coff1, cw + coff1, rA, aF + wb,
                                                             offA, kcf);
                const char *na = fa + (aN - lds0) + coff0, *nw = fw + (wN - lds0) + coff0;
                mfma_slots<0, B1, NM, NM + 1, 0, 0, 0, 1, FM, FN>(acc, a1, b1, a0, b0, na, nw, rW, 0u, offW, 0u);
                wait_vm_lgkm0<(DW - 1) * LA + (DW - 2) * LW>();
                lds_barrier();
                mfma_slots<B1, NM, B1, NM, 0, LW, B1, B1 + (NM - B1) * 3 / 4, FM, FN>(acc, a1, b1, a0, b0, na, nw, rW,
                                                                                    wC + wb, offW, kcf);
                aF = aC;
                aC = aN;
                wC = wN;
            }
            // the loads issued past the end (zeros) land before the buffers
            // are reused
            wait_vm_lgkm0<0>();
            __syncthreads();
        }

        if (traced && tid == 0) t_loop = rtc32();
        // The next ticket is fetched while the epilogue runs, but behind its gate:
        // a workgroup that waits for a late partition would hold back a tile that
        // others are free to take (ReduceScatter 6144 x 3000 x 5000, 8 ranks at
        // 100 / 50 GB/s: 751 us with the ticket taken before the gate, 665 behind)
        auto next_ticket = [&]() {
            if (!p.fixed && tid == 0) {
                const uint32_t c = __hip_atomic_fetch_add(&p.ctrl[v], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                s_pos = ticket_position(p, v, c);
            }
        };
        if (!RS) next_ticket();

        // thread coordinates the compiler cannot see to be the same for every
        // tile: addresses derived from them are computed where they are used,
        // not kept (spilled) over the main loop
        int et = tid;
        asm volatile("" : "+v"(et));
        const int er = et & 15, eq = (et >> 4) & 3;
        const int mlim = failed ? 0 : p.M;   // a failed tile stores nothing
        // the tile's partial sum: from P, or, for the rows of an aliased
        // range (a whole number of tiles), from that range's own buffer
        const float *pbase = p.P;
        int plo = 0;
        uint64_t pbytes = p.p_bytes;
        if (RS) {
            const int pm0 = map_row(p, m0);
#pragma unroll
            for (int i = 0; i < 2; ++i)
                if (pm0 >= p.palt_lo[i] && pm0 < p.palt_hi[i]) {
                    pbase = p.palt[i];
                    plo = p.palt_lo[i];
                    pbytes = (uint64_t)(p.palt_hi[i] - plo) * (uint64_t)p.ldp * 4u;
                }
        }
        // a tile of a chunk that is sent on (ReduceScatter) stores with
        // system-scope write-through, so that no L2 write-back is needed
        // before the copy engines read it
        const bool wt = RS && p.done_host != nullptr && (touch & p.send_mask) != 0;
        // 8 consecutive columns of row m from n, 16 bytes of C
        auto store8 = [&](int m, int n, u32x4 o) {
            if (m < mlim && n < p.N) {
                uint16_t *dst = p.C + (size_t)map_row(p, m) * p.ldc + n;
                if (wt) {   // written through to memory: the copy engines read it
                    __hip_atomic_store(reinterpret_cast<uint64_t *>(dst), (uint64_t)o[0] | ((uint64_t)o[1] << 32),
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                    __hip_atomic_store(reinterpret_cast<uint64_t *>(dst) + 1, (uint64_t)o[2] | ((uint64_t)o[3] << 32),
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                } else {
                    *reinterpret_cast<u32x4 *>(dst) = o;
                }
            }
        };
        // Of a 16 x 16 block in the accumulators' layout, lane (r, q) holds row
        // r, columns 4 q + 0..3. Exchanging the packed values of blocks ni and
        // ni + 1 between the 16-lane rows of the wave leaves each lane 8
        // consecutive columns, those from 8 (q / 2) of block ni + q % 2.
        auto store_pair = [&](int mi, int ni, f32x4 x, f32x4 y) {
            const u32x2 s0 = __builtin_amdgcn_permlane16_swap(pack_bf16x2(x[0], x[1]), pack_bf16x2(y[0], y[1]), false, false);
            const u32x2 s1 = __builtin_amdgcn_permlane16_swap(pack_bf16x2(x[2], x[3]), pack_bf16x2(y[2], y[3]), false, false);
            store8(m0 + wm0 + mi * 16 + er, n0 + wn0 + (ni + (eq & 1)) * 16 + 8 * (eq >> 1),
                   u32x4{s0[0], s1[0], s0[1], s1[1]});
        };
        const bool has_p = RS && p.P != nullptr;

        // split K: every slice stores its partial tile (fp32);
        // the slice that completes the tile's count sums all of them in
        // slice order, so the result does not depend on which one was last
        bool finish = true;
        if (split) {
            // in the accumulators' own layout: 4 consecutive values of every
            // thread of the workgroup, 4 KiB contiguous per store
            f32x4 *ws = reinterpret_cast<f32x4 *>(p.split_ws + (size_t)(wsf + slice) * (BM * BN)) + et;
#pragma unroll
            for (int ni = 0; ni < FN; ++ni)
#pragma unroll
                for (int mi = 0; mi < FM; ++mi) ws[(ni * FM + mi) * kThreads] = acc[ni][mi];
            // The workspace is uncached device memory: a store acknowledged
            // to the wave is in memory, visible to every XCD, and loads read
            // memory. So ordering needs no cache maintenance: each wave waits
            // for its stores, the barrier joins the waves, then the count.
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
            if (tid == 0) {
                const uint32_t old = __hip_atomic_fetch_add(&p.split_cnt[uc], 1u, __ATOMIC_RELAXED,
                                                            __HIP_MEMORY_SCOPE_AGENT);
                const bool last = old + 1u == (uint32_t)ns;
                if (last) __hip_atomic_store(&p.split_cnt[uc], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                s_last = last;
            }
            __syncthreads();   // the partial loads below are issued after the count
            finish = s_last != 0;
        }

        if (RS && finish && p.gate == kGateEpilogue && need) {
            if (wave == 0) {
                const bool ok = !failed && wait_flags(p, need, lane);
                if (lane == 0) s_ok = ok;
            }
            __syncthreads();
            if (!s_ok) failed = true;
            known |= need;
        }
        if (RS) next_ticket();
        if (RS && traced && tid == 0) t_gate = rtc32();

        if (finish) {
            if (split) {
                const f32x4 *ws0 = reinterpret_cast<const f32x4 *>(p.split_ws + (size_t)wsf * (BM * BN)) + et;
                // B pairs of blocks at a time, all their slices' loads (and the
                // partial sum's) in flight at once, then each summed in slice
                // order: the workspace is uncached, so every load costs a memory
                // round trip, and 2 B S of them overlap. The slice count is a
                // compile-time constant: the loads carry no branch, and the
                // waits before the sums count them exactly.
                auto finish_split = [&](auto b_const, auto s_const) {
                    constexpr int S = decltype(s_const)::value;
                    constexpr int NP = FM * FN / 2;   // pairs (mi, 2 nj), (mi, 2 nj + 1)
                    constexpr int WANT = decltype(b_const)::value, B = NP % WANT == 0 ? WANT : 2;
                    static_assert(NP % B == 0, "whole batches");
#pragma unroll 1
                    for (int u0 = 0; u0 < NP; u0 += B) {
                        f32x4 part[B][2][S];
                        f32x4 pv[B][2];
#pragma unroll
                        for (int b = 0; b < B; ++b) {
                            const int mi = (u0 + b) % FM, nj = (u0 + b) / FM;
                            const int m = m0 + wm0 + mi * 16 + er;
#pragma unroll
                            for (int h = 0; h < 2; ++h) {
                                const int ni = 2 * nj + h;
#pragma unroll
                                for (int jj = 0; jj < S; ++jj)
                                    part[b][h][jj] = ws0[(size_t)jj * (BM * BN / 4) + (ni * FM + mi) * kThreads];
                                const int n = n0 + wn0 + ni * 16 + 4 * eq;
                                pv[b][h] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                                if (has_p && m < p.M && n < p.N)
                                    pv[b][h] = *reinterpret_cast<const f32x4 *>(
                                        pbase + (size_t)(map_row(p, m) - plo) * p.ldp + n);
                            }
                        }
#pragma unroll
                        for (int b = 0; b < B; ++b) {
                            const int mi = (u0 + b) % FM, nj = (u0 + b) / FM;
                            f32x4 x[2];
#pragma unroll
                            for (int h = 0; h < 2; ++h) {
                                x[h] = part[b][h][0];
#pragma unroll
                                for (int jj = 1; jj < S; ++jj) x[h] += part[b][h][jj];
                                x[h] += pv[b][h];
                            }
                            store_pair(mi, 2 * nj, x[0], x[1]);
                        }
                    }
                };
                // The host splits a tile into 2 to kMaxSplit slices: each count
                // has its own branch-free instance, with batches that keep the
                // loads within the registers the main loop leaves.
                static_assert(kMaxSplit == 8, "one instance per slice count");
                using std::integral_constant;
                switch (ns) {
                case 2: finish_split(integral_constant<int, 4>{}, integral_constant<int, 2>{}); break;
                case 3: finish_split(integral_constant<int, 2>{}, integral_constant<int, 3>{}); break;
                case 4: finish_split(integral_constant<int, 2>{}, integral_constant<int, 4>{}); break;
                case 5: finish_split(integral_constant<int, 2>{}, integral_constant<int, 5>{}); break;
                case 6: finish_split(integral_constant<int, 2>{}, integral_constant<int, 6>{}); break;
                case 7: finish_split(integral_constant<int, 2>{}, integral_constant<int, 7>{}); break;
                case 8:
                default: finish_split(integral_constant<int, 2>{}, integral_constant<int, 8>{}); break;
                }
            } else {
                // Each wave turns 32 rows of its accumulators at a time to row
                // order through a region of the freed stage buffers (FN * 2 KiB
                // per wave: in the A and in the W buffers by turns; 16-byte chunk c
                // of row r at chunk c ^ (r & 7)): written straight from the
                // accumulation registers, read back 8 consecutive columns per
                // lane, one 16-byte store of C each, whole rows of the wave's
                // FN * 16 columns per instruction. The regions are the wave's
                // own, and a wave's LDS operations run in order, so nothing
                // waits between the write and the read but the read itself;
                // the next 32 rows are written while these are stored.
                constexpr int CPR = 2 * FN;         // 8-column pieces per row
                constexpr int NIT = 32 * CPR / 64;  // read-back rounds per 32 rows
                constexpr int RB = FN * 64;         // bytes of one row in the region
                static_assert(4 * 32 * RB <= NA * SA - 16 && 4 * 32 * RB <= DW * SW, "a region fits its buffers");
                char *const region[2] = {smem + wave * 32 * RB, smem + NA * SA + wave * 32 * RB};
                const int el = et & 63;
                auto to_lds = [&](int mi) {
                    char *w = region[mi & 1] + er * RB;
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int ni = 0; ni < FN; ++ni)
                            *reinterpret_cast<f32x4 *>(w + h * 16 * RB + (((4 * ni + eq) ^ (er & 7)) << 4)) =
                                acc[ni][2 * mi + h];
                    asm volatile("" ::: "memory");
                };
                // round `it` of rows mi: this lane's row and first column in the tile
                auto piece_row = [&](int mi, int it) { return wm0 + mi * 32 + (it * 64 + el) / CPR; };
                auto piece_col = [&](int it) { return wn0 + ((it * 64 + el) % CPR) * 8; };
                auto from_lds = [&](int mi, int it, float (&x)[8]) {
                    const int row = (it * 64 + el) / CPR, j = (it * 64 + el) % CPR;
                    const char *w = region[mi & 1] + row * RB;
                    // half of the lanes take their two chunks in the other
                    // order, so that 8 lanes read 8 different bank groups
                    const int sw = (j >> 2) & 1;
                    const f32x4 u = *reinterpret_cast<const f32x4 *>(w + (((2 * j + sw) ^ (row & 7)) << 4));
                    const f32x4 v = *reinterpret_cast<const f32x4 *>(w + (((2 * j + 1 - sw) ^ (row & 7)) << 4));
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        x[e] = sw ? v[e] : u[e];
                        x[4 + e] = sw ? u[e] : v[e];
                    }
                };
                if (has_p) {
                    // The fp32 partial (two 16-byte loads per piece, whole lines)
                    // is loaded 8 pieces ahead. Loads and stores go through
                    // buffer resources whose bound reads zeros / drops stores for
                    // rows or columns outside C (or all of a failed tile), so the
                    // waits count them exactly (no branch between them).
                    const int prow0 = map_row(p, m0);
                    const __amdgpu_buffer_rsrc_t rP =
                        tile_rsrc(pbase, pbytes, (uint64_t)(prow0 - plo) * (uint64_t)p.ldp * 4u);
                    const __amdgpu_buffer_rsrc_t rC =
                        tile_rsrc(p.C, p.c_bytes, (uint64_t)prow0 * (uint64_t)p.ldc * 2u);
                    constexpr int NP = FM / 2 * NIT, AHEAD = NP < 8 ? NP : 8;
                    u32x4 pv[AHEAD][2];
                    auto load_p = [&](int i) {
                        const int mi = i / NIT, it = i % NIT;
                        const int m = m0 + piece_row(mi, it), n = n0 + piece_col(it);
                        const uint32_t off = (m < p.M && n < p.N)
                                                 ? ((uint32_t)(map_row(p, m) - prow0) * (uint32_t)p.ldp + (uint32_t)n) * 4u
                                                 : kOOBRow;
                        pv[i % AHEAD][0] = __builtin_amdgcn_raw_buffer_load_b128(rP, off, 0, 0);
                        pv[i % AHEAD][1] = __builtin_amdgcn_raw_buffer_load_b128(rP, off, 16, 0);
                    };
#pragma unroll
                    for (int i = 0; i < AHEAD; ++i) load_p(i);
                    to_lds(0);
#pragma unroll
                    for (int mi = 0; mi < FM / 2; ++mi) {
                        if (mi + 1 < FM / 2) to_lds(mi + 1);
#pragma unroll
                        for (int it = 0; it < NIT; ++it) {
                            float x[8];
                            from_lds(mi, it, x);
#pragma unroll
                            for (int e = 0; e < 8; ++e)
                                x[e] += __builtin_bit_cast(float, (uint32_t)pv[(mi * NIT + it) % AHEAD][e >> 2][e & 3]);
                            if (mi * NIT + it + AHEAD < NP) load_p(mi * NIT + it + AHEAD);
                            const u32x4 o = {pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]), pack_bf16x2(x[4], x[5]),
                                             pack_bf16x2(x[6], x[7])};
                            const int m = m0 + piece_row(mi, it), n = n0 + piece_col(it);
                            const uint32_t off = (m < mlim && n < p.N)
                                                     ? ((uint32_t)(map_row(p, m) - prow0) * (uint32_t)p.ldc + (uint32_t)n) * 2u
                                                     : kOOBRow;
                            // sc0 sc1: written through to memory, the copy engines read it
                            // (a per-tile choice would be a branch around each store)
                            __builtin_amdgcn_raw_buffer_store_b128(o, rC, off, 0, WT ? 17 : 0);
                        }
                    }
                } else {
                    to_lds(0);
#pragma unroll
                    for (int mi = 0; mi < FM / 2; ++mi) {
                        if (mi + 1 < FM / 2) to_lds(mi + 1);
#pragma unroll
                        for (int it = 0; it < NIT; ++it) {
                            float x[8];
                            from_lds(mi, it, x);
                            const u32x4 o = {pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]), pack_bf16x2(x[4], x[5]),
                                             pack_bf16x2(x[6], x[7])};
                            store8(m0 + piece_row(mi, it), n0 + piece_col(it), o);
                        }
                    }
                }
            }
        }

        if (wt) __builtin_amdgcn_s_waitcnt(0);   // write-through stores acknowledged
        __syncthreads();   // stores issued and complete; LDS free for the next tile
        if (RS && finish && p.done_host && !failed && tid < 64) {
            // lane q counts for partition q, so that the counts' round trips
            // overlap: a tile of an InterDecom sub-operator counts for every
            // partition that is sent (4096 x 2048 x 4096, 8 ranks, double ring,
            // d = 4, 128 x 64 tiles: 370 -> 242 us)
            if (((touch & p.send_mask) >> lane) & 1ull) {
                const int f = p.flag_base + lane;
                const uint32_t old = __hip_atomic_fetch_add(&p.done_cnt[f], 1u, __ATOMIC_RELAXED,
                                                            __HIP_MEMORY_SCOPE_AGENT);
                if (old + 1u == p.done_expect[lane])
                    __hip_atomic_store(&p.done_host[f], p.epoch, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
            }
        }
        if (traced && tid == 0) {
            uint4 *rec = reinterpret_cast<uint4 *>(p.tile_trace + (size_t)(p.trace_base + (uint32_t)pos) * kTraceWords);
            rec[0] = make_uint4((uint32_t)pos, ((uint32_t)rt << 16) | (uint32_t)tn, hw_id(), xcc_id());
            rec[1] = make_uint4(t_tick, t_gate, t_loop, rtc32());
        }
        if (p.fixed) {
            pos = static_position(p, (int)blockIdx.x, ++round);
        } else {
            pos = __builtin_amdgcn_readfirstlane(s_pos);
        }
    }

    // exit: the last workgroup out resets the shared counters
    if (p.fixed && !(RS && p.done_host)) return;
    __syncthreads();
    if (tid == 0) {
        const uint32_t old = __hip_atomic_fetch_add(&p.ctrl[kCtrlExit], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (old == (uint32_t)p.grid - 1u) {
            if (RS && p.done_host)
                for (int q = 0; q < p.nparts; ++q)
                    __hip_atomic_store(&p.done_cnt[p.flag_base + q], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            for (int q = 0; q < p.nq; ++q)
                __hip_atomic_store(&p.ctrl[q], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&p.ctrl[kCtrlExit], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// Few rows (at most 16 MT): C of 16 columns per workgroup, K dealt to its NW
// waves one stage (64) at a time. Each wave streams its own stages of A and W
// through a ring of NST buffers of its own in LDS, so no barrier joins the
// waves before their partial sums are added (in wave order) at the end.
//
// What bounds it: the bytes a CU can pull through its L1 (64 per clock), A's
// rows once per 16 columns beside W's: hence the narrow tile, which spreads W
// over N / 16 CUs, and NST - 1 stages of loads in flight per wave. 48 x 3072 x
// 8192: 25.2 us in 64 x 64 tiles (48 CUs busy, a barrier per stage), 15.8
// here (50 MB of W at 3.2 TB/s with the launch, 4.6 TB/s without).
template <int MT, int NW, int NST>
__global__ __launch_bounds__(NW * 64) void skinny_kernel(const SkinnyParams p) {
    constexpr int SB = (MT + 1) * 2048;   // A rows, then W rows, 128 bytes each
    constexpr int L = 2 * MT + 2;         // loads per stage
    static_assert(NW * NST * SB <= (160 << 10) && NW * MT * 1024 <= NW * NST * SB, "LDS");
    __shared__ __attribute__((aligned(1024))) char smem[NW * NST * SB];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n0 = (int)blockIdx.x * 16;
    i32x4 rA = tile_rsrc4(p.A, (uint64_t)p.M * (uint64_t)p.K * 2u, 0);
    i32x4 rW = tile_rsrc4(p.W, (uint64_t)p.N * (uint64_t)p.K * 2u, (uint64_t)n0 * (uint64_t)p.K * 2u);
    asm volatile("s_nop 4" : "+s"(rA), "+s"(rW));   // as in gemm_kernel
    // load j covers rows 8 j + (lane >> 3); the lane takes the chunk that the
    // permutation (row >> 1) & 7 puts at its physical chunk lane & 7
    uint32_t offA[2 * MT], offW[2];
#pragma unroll
    for (int j = 0; j < 2 * MT; ++j) {
        const int row = 8 * j + (lane >> 3);
        offA[j] = row < p.M ? (uint32_t)row * (uint32_t)p.K * 2u : kOOBRow;
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int row = 8 * j + (lane >> 3);
        offW[j] = n0 + row < p.N ? (uint32_t)row * (uint32_t)p.K * 2u : kOOBRow;
    }
    const int c0 = (lane & 7) ^ (lane >> 4), c1 = (lane & 7) ^ (4 + (lane >> 4));
    const uint32_t ring = (uint32_t)(uintptr_t)LDS_AS(smem) + (uint32_t)(wave * NST * SB);
    const int KT = (p.K + kBK - 1) / kBK;
    auto load_stage = [&](int st, uint32_t buf) {
        const int k0 = st * kBK + c0 * 8, k1 = st * kBK + c1 * 8;
        const uint32_t q0 = k0 < p.K ? (uint32_t)k0 * 2u : kOOBCol, q1 = k1 < p.K ? (uint32_t)k1 * 2u : kOOBCol;
#pragma unroll
        for (int j = 0; j < 2; ++j) dma16(rW, offW[j] + (j & 1 ? q1 : q0), buf + (2 * MT + j) * 1024);
#pragma unroll
        for (int j = 0; j < 2 * MT; ++j) dma16(rA, offA[j] + (j & 1 ? q1 : q0), buf + j * 1024);
    };
    f32x4 acc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[mt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const int r = lane & 15, kq = lane >> 4, swz = (r >> 1) & 7;
    const char *frag = smem + wave * NST * SB + r * 128;
#pragma unroll
    for (int i = 0; i < NST; ++i) load_stage(wave + i * NW, ring + i * SB);   // (past the end: zeros)
    uint32_t slot = 0;
    for (int st = wave; st < KT; st += NW) {
        wait_vm_lgkm0<(NST - 1) * L>();
        bf16x8 a[2][MT], b[2];
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            const char *f = frag + slot + (((4 * kk + kq) ^ swz) << 4);
            b[kk] = *reinterpret_cast<const bf16x8 *>(f + MT * 2048);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) a[kk][mt] = *reinterpret_cast<const bf16x8 *>(f + mt * 2048);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the stage is in registers before its buffer is refilled
        load_stage(st + NST * NW, ring + slot);
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
                acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[kk], a[kk][mt], acc[mt], 0, 0, 0);
        slot = slot + SB == NST * SB ? 0u : slot + SB;
    }
    wait_vm_lgkm0<0>();   // the loads issued past the end have landed
    __syncthreads();
    // partial sums [wave][row][16 columns]
    f32x4 *sum = reinterpret_cast<f32x4 *>(smem);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) sum[(wave * MT * 16 + mt * 16 + r) * 4 + kq] = acc[mt];
    __syncthreads();
    if (tid < MT * 64) {
        const int row = tid >> 2, n = n0 + (tid & 3) * 4;
        if (row < p.M && n < p.N) {
            f32x4 x = sum[tid];
#pragma unroll
            for (int w = 1; w < NW; ++w) x += sum[w * MT * 64 + tid];
            const size_t o = (size_t)row * p.N + n;
            if (p.P) x += *reinterpret_cast<const f32x4 *>(p.P + o);
            *reinterpret_cast<u32x2 *>(p.C + o) = u32x2{pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3])};
        }
    }
}

hipError_t launch_skinny(const SkinnyParams &p, hipStream_t stream) {
    const dim3 grid((p.N + 15) / 16);
    if (p.M <= 16)
        hipLaunchKernelGGL((skinny_kernel<1, 8, 4>), grid, dim3(512), 0, stream, p);
    else if (p.M <= 32)
        hipLaunchKernelGGL((skinny_kernel<2, 8, 3>), grid, dim3(512), 0, stream, p);
    else if (p.M <= 48)
        hipLaunchKernelGGL((skinny_kernel<3, 4, 5>), grid, dim3(256), 0, stream, p);
    else
        hipLaunchKernelGGL((skinny_kernel<4, 4, 4>), grid, dim3(256), 0, stream, p);
    return hipGetLastError();
}

__global__ __launch_bounds__(64) void join_kernel(const JoinParams j) {
    if (threadIdx.x != 0) return;
    if (j.start_word) __hip_atomic_store(j.start_word, j.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    for (int i = 0; i < j.count; ++i) {
        const uint32_t *f = j.flags + j.idx[i];
        uint32_t polls = 0;
        while ((int32_t)(ld_flag(f) - j.epoch) < 0) {
            if (++polls > j.spin_limit) {
                __hip_atomic_fetch_or(j.err_word, 2u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                return;
            }
            if ((polls & 255u) == 0 && ld_flag(j.err_word) != 0) return;
            __builtin_amdgcn_s_sleep(8);
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "");
}

// Matrix-core probe: every wave issues `iters` rounds of 8 independent
// v_mfma_f32_32x32x16_bf16 and reads the shader-clock counter (s_memtime)
// and the 100 MHz real-time counter before and after them; out[3 w ..] gets
// wave w's two deltas and a value that keeps the products live. The 96 KiB
// LDS reservation leaves room for one workgroup (8 waves, two per SIMD) per
// CU, so a grid of one workgroup per CU runs all waves at once.
__global__ __launch_bounds__(kProbeThreads) void mfma_probe_kernel(uint64_t *out, int iters) {
    __shared__ float reserve[24 * 1024];
    const int tid = threadIdx.x;
    bf16x8 a, b;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        a[i] = (__bf16)(0.001f * (float)((tid + i) & 15));
        b[i] = (__bf16)(0.002f * (float)(i + 1));
    }
    f32x16 acc[8];
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[j][e] = 0.0f;
    const uint64_t t0 = __builtin_amdgcn_s_memtime();
    const uint64_t r0 = __builtin_amdgcn_s_memrealtime();
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[j], 0, 0, 0);
    }
    const uint64_t t1 = __builtin_amdgcn_s_memtime();
    const uint64_t r1 = __builtin_amdgcn_s_memrealtime();
    float sum = 0.0f;
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) sum += acc[j][e];
    // one exchange through the reservation keeps it allocated
    reserve[tid] = sum;
    __syncthreads();
    const float other = reserve[tid ^ 64];
    const size_t w = (size_t)blockIdx.x * (kProbeThreads / 64) + (tid >> 6);
    if ((tid & 63) == 0) {
        out[3 * w + 0] = t1 - t0;
        out[3 * w + 1] = r1 - r0;
        out[3 * w + 2] = (uint64_t)__builtin_bit_cast(uint32_t, sum + other);
    }
}

hipError_t launch_mfma_probe(uint64_t *out, int grid, int iters, hipStream_t stream) {
    hipLaunchKernelGGL(mfma_probe_kernel, dim3(grid), dim3(kProbeThreads), 0, stream, out, iters);
    return hipGetLastError();
}

template <int BM, int BN, int DW>
static void launch_tile(const GemmParams &p, bool rs, hipStream_t stream) {
    if (rs && p.done_host)
        hipLaunchKernelGGL((gemm_kernel<BM, BN, DW, true, true>), dim3(p.grid), dim3(kThreads), 0, stream, p);
    else if (rs)
        hipLaunchKernelGGL((gemm_kernel<BM, BN, DW, true>), dim3(p.grid), dim3(kThreads), 0, stream, p);
    else
        hipLaunchKernelGGL((gemm_kernel<BM, BN, DW, false>), dim3(p.grid), dim3(kThreads), 0, stream, p);
}

hipError_t launch_gemm(const GemmParams &p, int cfg, bool rs, hipStream_t stream) {
    switch (cfg) {
    case kTile256: launch_tile<256, 256, 2>(p, rs, stream); break;
    case kTile256x192: launch_tile<256, 192, 2>(p, rs, stream); break;
    case kTile256x128: launch_tile<256, 128, 2>(p, rs, stream); break;
    case kTile128: launch_tile<128, 128, 2>(p, rs, stream); break;
    case kTile128Deep: launch_tile<128, 128, 4>(p, rs, stream); break;
    case kTile128x64: launch_tile<128, 64, 2>(p, rs, stream); break;
    case kTile128x64Deep: launch_tile<128, 64, 4>(p, rs, stream); break;
    case kTile64: launch_tile<64, 64, 4>(p, rs, stream); break;
    case kTile192: launch_tile<192, 192, 2>(p, rs, stream); break;
    case kTile128x192: launch_tile<128, 192, 3>(p, rs, stream); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_join(const JoinParams &j, hipStream_t stream) {
    hipLaunchKernelGGL(join_kernel, dim3(1), dim3(64), 0, stream, j);
    return hipGetLastError();
}

}  // namespace compass
