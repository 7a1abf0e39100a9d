// Persistent, grouped 256 x 256 MFMA contraction with a four-stage direct-to-LDS pipeline (gfx950) for contraction-strided
// operands: fused wgrad + SGD update (paper section 3.2 / Algorithm 1) and the squared-norm pass (section 3.3.1).  Products with
// a contraction-contiguous operand: lomo_gemm_wide.hip.
//
// Same mathematics and epilogues as the other contraction kernels.  One launch covers
// the output tiles of up to MAX_GROUP tensors: one workgroup per CU walks the concatenated tile list
// with a fixed stride, so there is one ramp-up per pass instead of one per tensor and partial last
// rounds of one tensor are filled with tiles of the next.
//
// Shapes need not be whole tiles.  Every access goes through a buffer descriptor whose range ends where the
// tensor ends, so the hardware's range check returns zeros for what lies behind the last row, and lanes whose
// columns lie outside are given an offset no descriptor covers (loads return zero, stores are dropped; each
// wave still issues the same number of vector-memory instructions, which the counted waits rely on).  The
// contraction is cut into slices of 32 and walked from the first to the last, which may be short: the operands end with their
// ranges there.  Slices beyond the last one (their number is rounded up to a multiple of four) and the
// prefetches past the end are out of range as a whole and move no data.
// An operand may be larger than a descriptor covers (3.5 GiB: the output gradient of a projection to a
// vocabulary of 32000 from 58 500 tokens on): the descriptor's base then moves on with the walk, once per GiB, in an
// instantiation of its own.
// Measured: a 7B layer's step at 2999 tokens 6.36 -> 3.20 ms (567 -> 1138 TFLOP/s; the register-staged kernel of
// lomo_gemm.hip had every shape that was not whole tiles), at 4096 tokens 4.14 -> 4.13 ms: the descriptors' scalar offsets
// also take half of the scalar instructions out of the main loop (120 -> 58 per four slices).
//
// Data movement per tile:
//   * global -> LDS without passing through registers: buffer_load_dwordx4 ... lds writes lane L's
//     16 bytes to M0 + 16 L, and each lane may fetch any address of the buffer, so a wave instruction
//     fills 1 KiB of LDS with the 16-byte chunks of two tile rows in swizzled order;
//   * four 32 KiB stages: the loads for slice kt+3 are issued while slice kt is multiplied (one
//     load instruction after every fourth MFMA, so the loads never queue up behind each other),
//     which covers memory latency and needs no staging registers;
//   * LDS -> MFMA operands with the transposing read ds_read_b64_tr_b16; the fragments of the
//     next half-slice are read while the current one is multiplied, across the barrier;
//   * one barrier per slice.  The vector-memory counter is managed by hand because the compiler
//     would otherwise drain it before every LDS read;
//   * the first slices of the next tile are requested before the epilogue of the current one runs.
#include "lomo_gemm_common.h"
#include "lomo_gemm_persistent.h"

namespace lomo {

namespace dma {

// Soft alignment of the workgroups of one XCD between rounds of the update kernels (timing only, no effect on results).
// The 32 tiles that an XCD works on in a round share operand panels through its L2 as long as they walk the
// contraction roughly in step; the update epilogue takes a different time on every CU (it waits for HBM), and without
// anything that pulls them together again the workgroups drift apart over the rounds until a panel has left the L2
// before its last reader asks for it (measured on the 7B stack: 22 GiB fetched per launch instead of 15.6).  Every
// workgroup that has finished the main loop of a round adds one to the counter of (next round, XCD) and, before it
// enters the next main loop, waits a bounded time until the others of its XCD have done so.  The counters are cleared
// by a small kernel in front of every launch of more than one round.  Launches that overlap on one GPU share them: a workgroup may then
// wait less, or up to the bound once (after which it stops waiting), never for ever.
constexpr int SYNC_ROUNDS = 512;        // rounds beyond this run free
constexpr int SYNC_POLLS = 24;          // x 2048 clocks: the longest wait, about 30 us
__device__ int32_t g_round_arrive[SYNC_ROUNDS][8];

__global__ void clear_round_counters(int rounds) {
    const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i < rounds * 8) (&g_round_arrive[0][0])[i] = 0;
}

}  // namespace dma

// MOVE: an operand is larger than a descriptor covers.
template <int EPI, bool MOVE>
__global__ __launch_bounds__(NT) void lomo_contract_dma_kernel(dma::GroupArgs ga) {
    using namespace dma;
    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];

    if (EPI == EPI_UPDATE && ga.flag_in != nullptr && *ga.flag_in != 0) return;   // step dropped

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave & 1, wn = wave >> 1;
    const int G = gridDim.x;

    // round alignment (update kernels): how many workgroups of this XCD have a tile in round k
    constexpr bool ALIGN_ROUNDS = EPI == EPI_UPDATE || EPI == EPI_CLIPV;
    const int xcd = (int)(blockIdx.x & 7);
    auto xcd_tiles_in_round = [&](int k) {
        return xcd_run(xcd, round_tiles(k, G, ga.total_tiles), G, ga.deal != 0).count;
    };
    bool align_rounds = ALIGN_ROUNDS;      // cleared after a wait that ran into its bound
    int round = 0;

    const uint32_t lds0 = (uint32_t)(uintptr_t)smem;
    const uint32_t lds_wave = lds0 + (uint32_t)wave * 4096u;   // this wave's first KiB slot in a tile
    uint16_t* red_scratch = smem + NS * STAGE_HALVES;

    // ---- fragment read offsets (halves): fixed for the whole kernel
    const int g4 = lane >> 4, j16 = lane & 15;
    const int mhalf = g4 & 1, kh = g4 >> 1, rib = j16 >> 2, piece = j16 & 3;
    const int a_rd = (8 * kh + rib) * BM + (((wm * (BM / 16) + 2 * mhalf + (piece >> 1)) ^ swz_s(rib)) * 8) + (piece & 1) * 4;
    const int b_rd = (8 * kh + rib) * BN + (((wn * (BN / 16) + 2 * mhalf + (piece >> 1)) ^ swz_s(rib)) * 8) + (piece & 1) * 4;

    // ---- per-tile state of the loads
    uint32_t a_voff[4], b_voff[4];
    int4v a_srd{}, b_srd{};
    uint32_t a_step = 0, b_step = 0;       // bytes from one slice to the next
    uint32_t a_next = 0, b_next = 0;       // byte offset of the slice to be requested next
    uint32_t a_end = 0, b_end = 0;         // offsets from here on are behind the last slice
    // MOVE only: bytes from an operand's base to its end, and the slice offset from which on the base moves
    int64_t a_left = 0, b_left = 0;
    uint32_t a_move = ~0u, b_move = ~0u;
    int KT = 0;                            // slices walked: a multiple of 4

    // Locate tile number w of the concatenated list; set up the load state; return its coordinates.
    // A workgroup's tile numbers only grow, so the search for the tile's tensor resumes at the previous tile's.
    auto setup = [&](int w, int& tensor, int64_t& m0, int64_t& n0) {
        locate_tile(ga, w, tensor, m0, n0);
        const GroupTensor& T = ga.t[tensor];
        const int m_left = T.M - (int)m0, n_left = T.Nn - (int)n0;
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int q = wave * 4 + it;
            const int r = 2 * q + (lane >> 5), col = ((lane & 31) ^ swz_s(r)) * 8;
            a_voff[it] = ((uint32_t)(r * T.lda + col) * 2u) | (col < m_left ? 0u : OUTSIDE);
            b_voff[it] = ((uint32_t)(r * T.ldb + col) * 2u) | (col < n_left ? 0u : OUTSIDE);
        }
        a_srd = make_srd(T.A + m0, range_bytes((int64_t)T.C * T.lda - m0));
        b_srd = make_srd(T.B + n0, range_bytes((int64_t)T.C * T.ldb - n0));
        a_step = (uint32_t)BK * (uint32_t)T.lda * 2u;
        b_step = (uint32_t)BK * (uint32_t)T.ldb * 2u;
        KT = ((T.C + BK - 1) / BK + 3) & ~3;
        a_next = b_next = 0;
        a_end = (uint32_t)a_srd[2];
        b_end = (uint32_t)b_srd[2];
        if constexpr (MOVE) {
            a_left = 2 * ((int64_t)T.C * T.lda - m0);
            a_move = a_left > (int64_t)MAX_RANGE ? MOVE_BASE : ~0u;
            b_left = 2 * ((int64_t)T.C * T.ldb - n0);
            b_move = b_left > (int64_t)MAX_RANGE ? MOVE_BASE : ~0u;
        }
    };

    // One DMA instruction of the slice to be requested next: part 0 = A tile, part 1 = B tile; `it` selects this
    // wave's KiB slot.  The last of a slice's four moves on; behind the last slice the whole slice is out of range.
    auto issue1 = [&](int buf, int part, int it) {
        const uint32_t l = lds_wave + (uint32_t)buf * (STAGE_HALVES * 2u) + (uint32_t)part * (A_HALVES * 2u) +
                           (uint32_t)it * 1024u;
        if (part == 0) {
            dma16(a_voff[it], a_srd, a_next, l);
            if (it == 3) {
                a_next += a_step;
                if (a_next >= a_end) a_next = (uint32_t)a_srd[2];
            }
        } else {
            dma16(b_voff[it], b_srd, b_next, l);
            if (it == 3) {
                b_next += b_step;
                if (b_next >= b_end) b_next = (uint32_t)b_srd[2];
            }
        }
    };
    // Slices 0..2 and the A part of slice 3 of the tile that `setup` selected.
    auto issue_prologue = [&] {
#pragma unroll
        for (int st = 0; st < 3; ++st) {
#pragma unroll
            for (int it = 0; it < 4; ++it) issue1(st, 0, it);
#pragma unroll
            for (int it = 0; it < 4; ++it) issue1(st, 1, it);
        }
#pragma unroll
        for (int it = 0; it < 4; ++it) issue1(3, 0, it);
    };

    // ---- fragment reads, in the order the MFMAs consume them: a0, b0..b3, a1..a3
    auto read_a = [&](half8 (&a)[4], int buf, int kk, int i) {
        const uint16_t* p = smem + buf * STAGE_HALVES + ((a_rd ^ (i << 5)) + kk * 16 * BM);
        a[i] = read_tr8(p, p + 4 * BM);
    };
    auto read_b = [&](half8 (&b)[4], int buf, int kk, int j) {
        const uint16_t* p = smem + buf * STAGE_HALVES + A_HALVES + ((b_rd ^ (j << 5)) + kk * 16 * BN);
        b[j] = read_tr8(p, p + 4 * BN);
    };
    // Fragment groups.  EARLY packs the eight fragments into the first three groups, so that every
    // read has completed when the half-slice ends at a barrier.
    auto read_group = [&](half8 (&a)[4], half8 (&b)[4], int buf, int kk, int q, bool early) {
        if (early) {
            if (q == 0) { read_a(a, buf, kk, 0); read_b(b, buf, kk, 0); read_b(b, buf, kk, 1); }
            if (q == 1) { read_b(b, buf, kk, 2); read_b(b, buf, kk, 3); read_a(a, buf, kk, 1); }
            if (q == 2) { read_a(a, buf, kk, 2); read_a(a, buf, kk, 3); }
        } else {
            if (q == 0) { read_a(a, buf, kk, 0); read_b(b, buf, kk, 0); }
            if (q == 1) { read_b(b, buf, kk, 1); read_b(b, buf, kk, 2); }
            if (q == 2) { read_b(b, buf, kk, 3); read_a(a, buf, kk, 1); }
            if (q == 3) { read_a(a, buf, kk, 2); read_a(a, buf, kk, 3); }
        }
    };
    constexpr int READS_EARLY[4] = {6, 6, 4, 0}, READS_EVEN[4] = {4, 4, 4, 4};      // LDS read instructions, two per fragment

    floatx16 acc[4][4];
    auto zero_acc = [&] {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    };

    // Half a slice: 16 MFMAs on (ua, ub) in four groups; each group is preceded by the reads of one
    // fragment group of the next half-slice and followed by one direct-to-LDS load, so that LDS reads,
    // global loads and MFMAs overlap instead of queueing behind each other.
    auto half_slice = [&](const half8 (&ua)[4], const half8 (&ub)[4], half8 (&la)[4], half8 (&lb)[4], int lbuf, int lkk,
                          bool early, int dbuf, int dpart) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            read_group(la, lb, lbuf, lkk, q, early);
#pragma unroll
            for (int j = 0; j < 4; ++j)
                acc[q][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ua[q], ub[j], acc[q][j], 0, 0, 0);
            {   // spread this group's reads in front of its four MFMAs
                int left = early ? READS_EARLY[q] : READS_EVEN[q];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int now = (left + (3 - j)) / (4 - j);
                    if (now == 1) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // DS reads
                    if (now == 2) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                    if (now == 3) __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    left -= now;
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            issue1(dbuf, dpart, q);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // ---- walk the tile list, one tile a round; every workgroup leaves through `break`
    int w = round_tile(0, G, ga.total_tiles, ga.deal != 0);
    if (w >= ga.total_tiles) return;   // cannot happen with grid <= total_tiles; nothing was issued yet
    int tensor = 0;
    int64_t m0, n0;
    setup(w, tensor, m0, n0);
    issue_prologue();
    zero_acc();

    while (true) {
        if constexpr (ALIGN_ROUNDS) {
            if (round >= 1 && round < SYNC_ROUNDS && tid == 0 && align_rounds) {
                const int need = xcd_tiles_in_round(round);
                int polls = 0;
                while (__hip_atomic_load(&g_round_arrive[round][xcd], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < need &&
                       polls < SYNC_POLLS) {
                    __builtin_amdgcn_s_sleep(32);
                    ++polls;
                }
                if (polls == SYNC_POLLS) align_rounds = false;     // something else holds CUs: stop waiting
            }
        }
        // every load of this tile's first slices has landed and is visible to all waves (and thread 0 is back); the last
        // tile's stores, issued behind them, may still be on their way
        if (EPI == EPI_SQNORM || round == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(RowEpilogue::OPS<EPI>) : "memory");
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        half8 fa0[4], fb0[4], fa1[4], fb1[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) read_group(fa0, fb0, 0, 0, q, false);

        // KT is a multiple of 4: the body is unrolled over the four LDS stages so that every LDS
        // address is a register plus an immediate.
        for (int kt = 0; kt < KT; kt += 4) {
            if constexpr (MOVE) {
                if (__builtin_expect(a_next >= a_move, 0)) move_base(a_srd, a_left, a_next, a_end, a_move);
                if (__builtin_expect(b_next >= b_move, 0)) move_base(b_srd, b_left, b_next, b_end, b_move);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                // first half of slice kt+u; reads its second half's fragments; loads the B part of slice kt+u+3
                half_slice(fa0, fb0, fa1, fb1, u, 1, true, (u + 3) & 3, 1);
                // own loads of slice kt+u+1 landed (two younger slices may still fly); own LDS reads done
                asm volatile("s_waitcnt vmcnt(16) lgkmcnt(0)\n\ts_barrier" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
                // second half; reads the first fragments of the next slice; loads the A part of slice
                // kt+u+4 into the buffer of slice kt+u, which nobody reads any more
                half_slice(fa1, fb1, fa0, fb0, (u + 1) & 3, 0, false, u, 0);
            }
        }
        // drain: the loads past the end (zeros) have landed, all waves are done with the LDS stages
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");

        // epilogue arguments of the tile just finished
        GemmArgs g;
        g.Out = ga.t[tensor].Out;
        g.Res = nullptr;
        g.ldo = ga.t[tensor].ldo;
        g.M = ga.t[tensor].M;
        g.Nn = ga.t[tensor].Nn;
        g.s = ga.s;
        g.s_dev = ga.s_dev;
        g.lr = ga.lr;
        g.inv_s = ga.inv_s;
        g.clipv = ga.clipv;
        g.acc = ga.acc;
        g.flag_out = ga.t[tensor].flag_out;
        const int64_t em0 = m0, en0 = n0;

        // request the first blocks of W (update), then the first slices of the next tile, then finish this one
        ++round;
        w = next_tile(w, round, G, ga.total_tiles, ga.deal != 0);
        const bool more = w < ga.total_tiles;
        if constexpr (ALIGN_ROUNDS) {
            if (more && round < SYNC_ROUNDS && tid == 0) atomicAdd(&g_round_arrive[round][xcd], 1);
        }
        if constexpr (EPI != EPI_SQNORM) {
            const RowEpilogue re(g, smem, wave, em0, en0);
            re.fill(0);
            re.fill(1);
            re.fill(2);
            if (more) {
                setup(w, tensor, m0, n0);
                issue_prologue();
            }
            re.template run<EPI, 28>(acc, g, more);
        } else {
            if (more) {
                setup(w, tensor, m0, n0);
                issue_prologue();
            }
            epilogue<BM, BN, EPI>(acc, g, red_scratch, em0, en0, BM, BN);      // elements outside the tensor are zero
        }
        if (!more) break;
        zero_acc();
    }
}

// ---- host side ----------------------------------------------------------------------------

int cu_count() {
    static const int n = [] {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) != hipSuccess) return 256;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0) return 256;
        return v;
    }();
    return n;
}

// What the kernels' 32-bit offsets can address: of a contraction-strided operand the slices requested between two moves of its
// base (rows of up to 8 million elements), of everything else a tile's rows.
template <bool B_STRIDED, bool A_STRIDED>
bool dma_eligible(const GemmArgs& a) {
    using namespace dma;
    const int64_t span = (int64_t)MAX_RANGE / 2, run = ((int64_t)MAX_RANGE - (int64_t)MOVE_BASE) / 2;
    return a.M > 0 && a.Nn > 0 && a.C > 0 && a.M < (1 << 30) && a.Nn < (1 << 30) && a.C < (1 << 30) &&
           (A_STRIDED ? 5 * BK * a.lda < run : (int64_t)BM * a.lda + a.C + 8 * BK < span) &&
           (B_STRIDED ? 5 * BK * a.ldb < run : (int64_t)BN * a.ldb + a.C + 8 * BK < span) && (int64_t)BN * a.ldo < span &&
           ((a.M + BM - 1) / BM) * ((a.Nn + BN - 1) / BN) < (1 << 24);
}
template bool dma_eligible<true, true>(const GemmArgs&);
template bool dma_eligible<false, true>(const GemmArgs&);
template bool dma_eligible<false, false>(const GemmArgs&);

// A contraction-strided operand is larger than a descriptor covers (8 slices more than it has, so that no slice offset
// wraps around): the persistent kernel moves its base, the others cannot.
template <bool B_STRIDED, bool A_STRIDED>
bool beyond_descriptor(const GemmArgs& a) {
    const int64_t span = (int64_t)dma::MAX_RANGE / 2, rows = a.C + 8 * dma::BK;
    return (A_STRIDED && rows * a.lda >= span) || (B_STRIDED && rows * a.ldb >= span);
}
template bool beyond_descriptor<true, true>(const GemmArgs&);
template bool beyond_descriptor<false, true>(const GemmArgs&);
template bool beyond_descriptor<false, false>(const GemmArgs&);

template <int EPI, bool MOVE>
static hipError_t launch_dma(const GemmArgs* list, int n, hipStream_t st) {
    using namespace dma;
    auto kern = lomo_contract_dma_kernel<EPI, MOVE>;
    // thread-safe one-time set-up (initialisation of a function-local static)
    static const hipError_t cfg0 = allow_dynamic_lds(kern, LDS_BYTES);
    if (cfg0 != hipSuccess) return cfg0;
    for (int first = 0; first < n; first += MAX_GROUP) {
        const int cnt = (n - first < MAX_GROUP) ? (n - first) : MAX_GROUP;
        GroupArgs ga{};
        fill_group(ga, list + first, cnt, BM, BN);
        const int tiles = ga.total_tiles;
        const int grid = tiles < cu_count() ? tiles : cu_count();
        ga.deal = choose_deal(ga, grid);
        // the kernels that align their rounds; a single round reads no counter
        if ((EPI == EPI_UPDATE || EPI == EPI_CLIPV) && tiles > grid) {
            int rounds = (tiles + grid - 1) / grid;
            if (rounds > SYNC_ROUNDS) rounds = SYNC_ROUNDS;
            hipLaunchKernelGGL(clear_round_counters, dim3((unsigned)((rounds * 8 + 255) / 256)), dim3(256), 0, st, rounds);
        }
        hipError_t e = launch_timed(list[first].family, kern, dim3((unsigned)grid), dim3(NT), (size_t)LDS_BYTES, st, ga);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <int EPI>
hipError_t launch_dma_group(const GemmArgs* list, int n, hipStream_t st) {
    for (int i = 0; i < n; ++i)
        if (beyond_descriptor<true, true>(list[i])) return launch_dma<EPI, true>(list, n, st);
    return launch_dma<EPI, false>(list, n, st);
}

template hipError_t launch_dma_group<EPI_UPDATE>(const GemmArgs*, int, hipStream_t);
template hipError_t launch_dma_group<EPI_CLIPV>(const GemmArgs*, int, hipStream_t);
template hipError_t launch_dma_group<EPI_SQNORM>(const GemmArgs*, int, hipStream_t);

}  // namespace lomo
