// Persistent, grouped 256 x 256 MFMA contraction with a four-stage direct-to-LDS pipeline (gfx950).
//
// Same mathematics and epilogues as the other contraction kernels (fused wgrad + SGD update of
// paper section 3.2 / Algorithm 1, squared-norm pass of section 3.3.1, dgrad).  One launch covers
// the output tiles of up to MAX_GROUP tensors: one workgroup per CU walks the concatenated tile list
// with a fixed stride, so there is one ramp-up per pass instead of one per tensor and partial last
// rounds of one tensor are filled with tiles of the next.
//
// Shapes need not be whole tiles.  Every access goes through a buffer descriptor whose range ends where the
// tensor ends, so the hardware's range check returns zeros for what lies behind the last row, and lanes whose
// columns lie outside are given an offset no descriptor covers (loads return zero, stores are dropped; each
// wave still issues the same number of vector-memory instructions, which the counted waits rely on).  The
// contraction is cut into slices of 32 and walked from the first to the last, which may be short: the rows of a
// contraction-strided operand end with its range there, the lanes of a contraction-contiguous one are masked (its memory
// goes on with the next row).  Slices beyond the last one (their number is rounded up to a multiple of four) and the
// prefetches past the end are out of range as a whole and move no data.
// A contraction-strided operand may be larger than a descriptor covers (3.5 GiB: the output gradient of a projection to a
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
//   * LDS -> MFMA operands with the transposing read ds_read_b64_tr_b16 (contraction-strided
//     operands) or ds_read_b128 (contraction-contiguous operand of dgrad); the fragments of the
//     next half-slice are read while the current one is multiplied, across the barrier;
//   * one barrier per slice.  The vector-memory counter is managed by hand because the compiler
//     would otherwise drain it before every LDS read;
//   * the first slices of the next tile are requested before the epilogue of the current one runs.
#include "lomo_gemm_common.h"
#include "lomo_gemm_dma_common.h"

namespace lomo {

namespace dma {

constexpr int BM = 256, BN = 256, NS = 4;
constexpr int A_HALVES = BK * BM, B_HALVES = BK * BN, STAGE_HALVES = A_HALVES + B_HALVES;
constexpr int EPI_UNIT_HALVES = 32 * 64;                 // staging block of the row epilogue: 32 rows x 64 columns (4 KiB)
// four stages + 32 KiB behind them: two staging blocks per wave for the row epilogue (update, store), whose first
// 256 bytes serve as the reduction scratch of the norm epilogue.  160 KiB in all, the whole LDS of a CU.
constexpr int LDS_BYTES = NS * STAGE_HALVES * 2 + 8 * EPI_UNIT_HALVES * 2;
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

__device__ __forceinline__ int swz_s(int r) { return ((r & 1) * 10) + ((r & 2) * 2); }

// ---- row epilogue (update / store) --------------------------------------------------------------------
// The accumulator layout gives a lane 16 bytes of one output row at a time, so a wave instruction on global
// memory would touch 32 rows x 32 bytes.  Here each wave stages 32 x 64 blocks of its 128 x 128 sub-tile in
// LDS: the old W block arrives row-contiguous by direct-to-LDS loads (8 rows x 128 bytes per instruction),
// lanes pick their 16-byte pieces out of it, update, put the results back in the same places, and the block
// leaves row-contiguous again.  Three blocks per wave rotate; the first three loads are issued right after
// the tile's last slice, ahead of the next tile's first slices, and block u + 3 is requested as soon as block u
// is in registers.  16-byte chunk c of row r sits at chunk position c ^ (r & 7): the LDS serves eight lanes of a
// 16-byte access per clock (128 bytes), and eight consecutive lanes are either eight consecutive rows at one
// chunk (pieces) or the eight chunks of one row (rows), so both patterns are conflict-free.
__device__ __forceinline__ int swz_e(int r) { return r & 7; }

struct RowEpilogue {
    uint16_t* buf[3];
    uint32_t voff[4];
    uint32_t outside[2];      // OUTSIDE where this lane's chunk of an even / odd block lies behind the last column
    int4v old_srd;
    __amdgpu_buffer_rsrc_t out_rsrc;
    uint32_t range, row_bytes;      // bytes from this wave's 128 x 128 sub-tile to the end of the tensor; of one row

    __device__ __forceinline__ RowEpilogue(const GemmArgs& g, uint16_t* smem, int wave, int64_t m0, int64_t n0) {
        const int lane = threadIdx.x & 63;
        const int wm = wave & 1, wn = wave >> 1;
        // two blocks per wave behind the stages, the third in the B part of stage 3, which is idle between the last
        // slice of a tile and the first half-slice of the next
        buf[0] = smem + NS * STAGE_HALVES + wave * EPI_UNIT_HALVES;
        buf[1] = buf[0] + 4 * EPI_UNIT_HALVES;
        buf[2] = smem + 3 * STAGE_HALVES + A_HALVES + wave * EPI_UNIT_HALVES;
        const int64_t mw = m0 + wm * (BM / 2), nw = n0 + wn * (BN / 2);
        const int64_t origin = nw * g.ldo + mw;
        range = range_bytes((int64_t)g.Nn * g.ldo - origin);
        row_bytes = (uint32_t)g.ldo * 2u;
        old_srd = make_srd(((g.Res != nullptr) ? g.Res : g.Out) + origin, range);
        out_rsrc = __builtin_amdgcn_make_buffer_rsrc(g.Out + origin, 0, range, BUFFER_WORD3);
        // row-contiguous mapping inside a block: instruction q covers rows 8 q .. 8 q + 7, eight lanes per row
        const int rr = lane >> 3, slot = lane & 7;
        const int col = (slot ^ swz_e(rr)) * 8;                  // swz_e(8 q + rr) = swz_e(rr)
#pragma unroll
        for (int q = 0; q < 4; ++q) voff[q] = (uint32_t)(8 * q + rr) * row_bytes + (uint32_t)col * 2u;
#pragma unroll
        for (int ih = 0; ih < 2; ++ih) outside[ih] = (mw + 64 * ih + col < g.M) ? 0u : OUTSIDE;
    }
    __device__ __forceinline__ uint32_t unit_off(int u) const {
        const uint32_t o = (uint32_t)(32 * (u >> 1)) * row_bytes + (uint32_t)(128 * (u & 1));
        return o < range ? o : range;
    }
    __device__ __forceinline__ void fill(int u) const {
        const uint32_t l = (uint32_t)(uintptr_t)buf[u % 3], o = unit_off(u);
#pragma unroll
        for (int q = 0; q < 4; ++q) dma16(voff[q] | outside[u & 1], old_srd, o, l + (uint32_t)q * 1024u);
    }

    // `ahead`: vector-memory operations issued between the first three fills and this call (the next tile's first slices)
    template <int EPI>
    __device__ __forceinline__ void run(floatx16 (&acc)[4][4], const GemmArgs& g, bool ahead) const {
        constexpr bool RMW = (EPI == EPI_UPDATE || EPI == EPI_CLIPV);
        const float s = g.s_dev != nullptr ? *g.s_dev : g.s;
        uint32_t worst = 0u;      // largest exponent field seen (EPI_CLIPV)
        typedef uint32_t u32x2v __attribute__((ext_vector_type(2)));
        const int lane = threadIdx.x & 63;
        const int l32 = lane & 31, lh = lane >> 5;
        int poff[2][2];     // accumulator-layout mapping: this lane's piece (il, a) of row l32
#pragma unroll
        for (int il = 0; il < 2; ++il)
#pragma unroll
            for (int a = 0; a < 2; ++a) poff[il][a] = l32 * 64 + (((4 * il + 2 * a + lh) ^ swz_e(l32)) * 8);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int j = u >> 1, ih = u & 1;
            uint16_t* b = buf[u % 3];
            half8 w[2][2];
            if constexpr (RMW) {
                // Vector-memory operations complete in issue order.  Issued after this block's four loads: blocks 0-2,
                // the 28 loads of the next tile's first slices (if any), then per block u its stores and the loads of
                // block u + 3.  Wait until only those may still be outstanding.
                if (u == 0) { if (ahead) asm volatile("s_waitcnt vmcnt(36)" ::: "memory"); else asm volatile("s_waitcnt vmcnt(8)" ::: "memory"); }
                else if (u == 1) { if (ahead) asm volatile("s_waitcnt vmcnt(40)" ::: "memory"); else asm volatile("s_waitcnt vmcnt(12)" ::: "memory"); }
                else if (u == 2) { if (ahead) asm volatile("s_waitcnt vmcnt(44)" ::: "memory"); else asm volatile("s_waitcnt vmcnt(16)" ::: "memory"); }
                else if (u <= 5) asm volatile("s_waitcnt vmcnt(20)" ::: "memory");
                else if (u == 6) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
                else asm volatile("s_waitcnt vmcnt(12)" ::: "memory");
#pragma unroll
                for (int il = 0; il < 2; ++il)
#pragma unroll
                    for (int a = 0; a < 2; ++a) w[il][a] = *reinterpret_cast<const half8*>(b + poff[il][a]);
            }
#pragma unroll
            for (int il = 0; il < 2; ++il)
#pragma unroll
                for (int a = 0; a < 2; ++a) {
                    const int i = 2 * ih + il;
                    float v[8];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const u32x2v sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[i][j][8 * a + e]),
                                                                           __float_as_uint(acc[i][j][8 * a + 4 + e]), false, false);
                        v[e] = __uint_as_float(sw[0]);
                        v[4 + e] = __uint_as_float(sw[1]);
                    }
                    half8 out;
                    if constexpr (EPI == EPI_UPDATE) {
#pragma unroll
                        for (int e = 0; e < 8; ++e) out[e] = (_Float16)fmaf(-s, v[e], (float)w[il][a][e]);
                    } else if constexpr (EPI == EPI_CLIPV) {
                        // clip by value (section 3.3.1): clamp each unscaled gradient element, then update; a
                        // non-finite element raises the flag and leaves its weight alone
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const float gq = v[e] * g.inv_s;
                            const uint32_t ex = __float_as_uint(gq) & 0x7f800000u;
                            const float gc = fminf(fmaxf(gq, -g.clipv), g.clipv);
                            out[e] = ex < 0x7f800000u ? (_Float16)fmaf(-g.lr, gc, (float)w[il][a][e]) : w[il][a][e];
                            worst = ex > worst ? ex : worst;
                        }
                    } else {
#pragma unroll
                        for (int e = 0; e < 8; ++e) out[e] = (_Float16)v[e];
                    }
                    *reinterpret_cast<half8*>(b + poff[il][a]) = out;
                }
            half8 rows[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) rows[q] = *reinterpret_cast<const half8*>(b + q * 512 + lane * 8);
            if constexpr (RMW) {
                if (u + 3 < 8) {
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // the block is in registers: its buffer is free
                    fill(u + 3);
                }
            }
            const uint32_t o = unit_off(u);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4v, rows[q]), out_rsrc, voff[q] | outside[u & 1], o, 0);
        }
        if constexpr (EPI == EPI_CLIPV) {
            if (__any(worst == 0x7f800000u) && lane == 0 && g.flag_out != nullptr) atomicOr(g.flag_out, 1);
        }
    }
};

}  // namespace dma

// A_STRIDED = false: the A operand is contraction-contiguous as well (forward product Y = X W^T with A = W),
// fetched and read like the contraction-contiguous B.
// EDGE: some tensor's contraction ends inside a slice and an operand is contraction-contiguous, or a contraction-strided operand
// is larger than a descriptor covers (checking for the former costs 0.5 % of the time of the others).
template <bool B_STRIDED, int EPI, bool A_STRIDED, bool EDGE>
__global__ __launch_bounds__(NT) void lomo_contract_dma_kernel(dma::GroupArgs ga) {
    using namespace dma;
    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];

    if (EPI == EPI_UPDATE && ga.flag_in != nullptr && *ga.flag_in != 0) return;   // step dropped

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave & 1, wn = wave >> 1;
    const int G = gridDim.x;

    // Position of this workgroup inside a window of G consecutive tiles: workgroups of one XCD
    // (blockIdx % 8) take a contiguous run, which the band order below turns into an 8 x 4 block of
    // tiles that share operand panels in that XCD's L2.
    int pos;
    {
        const int x = (int)(blockIdx.x & 7), local = (int)(blockIdx.x >> 3);
        const int q = G >> 3, r = G & 7;
        pos = x * q + (x < r ? x : r) + local;
    }

    // round alignment (update kernels): this XCD's run of positions and how many of them have a tile in round k
    constexpr bool ALIGN_ROUNDS = (EPI == EPI_UPDATE || EPI == EPI_CLIPV) && A_STRIDED && B_STRIDED;
    const int xcd = (int)(blockIdx.x & 7);
    const int xcd_first = xcd * (G >> 3) + (xcd < (G & 7) ? xcd : (G & 7));
    const int xcd_count = (G >> 3) + (xcd < (G & 7) ? 1 : 0);
    auto xcd_tiles_in_round = [&](int k) {
        const int v = ga.total_tiles - k * G - xcd_first;
        return v < 0 ? 0 : (v > xcd_count ? xcd_count : v);
    };
    bool align_rounds = ALIGN_ROUNDS;      // cleared after a wait that ran into its bound
    int round = 0;

    const uint32_t lds0 = (uint32_t)(uintptr_t)smem;
    const uint32_t lds_wave = lds0 + (uint32_t)wave * 4096u;   // this wave's first KiB slot in a tile
    uint16_t* red_scratch = smem + NS * STAGE_HALVES;

    // ---- fragment read offsets (halves): fixed for the whole kernel
    const int g4 = lane >> 4, j16 = lane & 15;
    const int mhalf = g4 & 1, kh = g4 >> 1, rib = j16 >> 2, piece = j16 & 3;
    int a_rd;
    if constexpr (A_STRIDED) {
        a_rd = (8 * kh + rib) * BM + (((wm * (BM / 16) + 2 * mhalf + (piece >> 1)) ^ swz_s(rib)) * 8) + (piece & 1) * 4;
    } else {
        const int ml = wm * (BM / 2) + (lane & 31), lh = lane >> 5;
        a_rd = ml * BK + ((lh ^ swz_c(ml)) * 8);
    }
    int b_rd;
    if constexpr (B_STRIDED) {
        b_rd = (8 * kh + rib) * BN + (((wn * (BN / 16) + 2 * mhalf + (piece >> 1)) ^ swz_s(rib)) * 8) + (piece & 1) * 4;
    } else {
        const int nl = wn * (BN / 2) + (lane & 31), lh = lane >> 5;
        b_rd = nl * BK + ((lh ^ swz_c(nl)) * 8);
    }

    // ---- per-tile state of the loads
    uint32_t a_voff[4], b_voff[4];
    int4v a_srd{}, b_srd{};
    uint32_t a_step = 0, b_step = 0;       // bytes from one slice to the next
    uint32_t a_next = 0, b_next = 0;       // byte offset of the slice to be requested next
    uint32_t a_end = 0, b_end = 0;         // offsets from here on are behind the last slice
    // EDGE only: offset of a contraction-contiguous operand's last slice and this lane's mask there; bytes from a
    // contraction-strided operand's base to its end, and the slice offset from which on the base moves
    uint32_t last = 0, tail = 0;
    int64_t a_left = 0, b_left = 0;
    uint32_t a_move = ~0u, b_move = ~0u;
    int KT = 0;                            // slices walked: a multiple of 4

    // From the last slice of a contraction-contiguous operand on (nothing follows it) the lanes behind the end are masked.
    auto mask_a = [&] {
#pragma unroll
        for (int it = 0; it < 4; ++it) a_voff[it] |= tail;
    };
    auto mask_b = [&] {
#pragma unroll
        for (int it = 0; it < 4; ++it) b_voff[it] |= tail;
    };

    // Puts the base of a strided operand at its next slice.
    auto move_base = [](int4v& srd, int64_t& left, uint32_t& next, uint32_t& end, uint32_t& move) {
        left -= next;
        const uint64_t base = (((uint64_t)(uint32_t)srd[1] << 32) | (uint32_t)srd[0]) + next;
        srd = make_srd((const void*)base, range_bytes(left / 2));
        next = 0;
        end = (uint32_t)srd[2];
        move = left > (int64_t)MAX_RANGE ? MOVE_BASE : ~0u;
    };

    // Locate tile number w of the concatenated list; set up the load state; return its coordinates.
    // A workgroup's tile numbers only grow, so the search for the tile's tensor resumes at the previous tile's.
    auto setup = [&](int w, int& tensor, int64_t& m0, int64_t& n0) {
        int k = tensor;
        while (k + 1 < ga.n && w >= ga.t[k + 1].tile_begin) ++k;
        const GroupTensor& T = ga.t[k];
        const int t = w - T.tile_begin;
        constexpr int GM = 8;
        const int per_band = GM * T.tiles_n;
        const int band = t / per_band;
        const int first_m = band * GM;
        const int gsz = (T.tiles_m - first_m < GM) ? (T.tiles_m - first_m) : GM;
        const int in_band = t - band * per_band;
        const int tm = first_m + in_band % gsz;
        const int tn = in_band / gsz;
        tensor = k;
        m0 = (int64_t)tm * BM;
        n0 = (int64_t)tn * BN;
        const int m_left = T.M - (int)m0, n_left = T.Nn - (int)n0;
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int q = wave * 4 + it;
            if constexpr (A_STRIDED) {
                const int r = 2 * q + (lane >> 5), col = ((lane & 31) ^ swz_s(r)) * 8;
                a_voff[it] = ((uint32_t)(r * T.lda + col) * 2u) | (col < m_left ? 0u : OUTSIDE);
            } else {
                const int n = 16 * q + (lane >> 2), cp = lane & 3;
                a_voff[it] = (uint32_t)(n * T.lda + ((cp ^ swz_c(n)) * 8)) * 2u;
            }
            if constexpr (B_STRIDED) {
                const int r = 2 * q + (lane >> 5), col = ((lane & 31) ^ swz_s(r)) * 8;
                b_voff[it] = ((uint32_t)(r * T.ldb + col) * 2u) | (col < n_left ? 0u : OUTSIDE);
            } else {
                const int n = 16 * q + (lane >> 2), cp = lane & 3;
                b_voff[it] = (uint32_t)(n * T.ldb + ((cp ^ swz_c(n)) * 8)) * 2u;
            }
        }
        const int64_t a_org = A_STRIDED ? m0 : m0 * (int64_t)T.lda, a_rows = A_STRIDED ? T.C : T.M;
        const int64_t b_org = B_STRIDED ? n0 : n0 * (int64_t)T.ldb, b_rows = B_STRIDED ? T.C : T.Nn;
        a_srd = make_srd(T.A + a_org, range_bytes(a_rows * T.lda - a_org));
        b_srd = make_srd(T.B + b_org, range_bytes(b_rows * T.ldb - b_org));
        const uint32_t a_unit = A_STRIDED ? (uint32_t)T.lda * 2u : 2u, b_unit = B_STRIDED ? (uint32_t)T.ldb * 2u : 2u;
        a_step = (uint32_t)BK * a_unit;
        b_step = (uint32_t)BK * b_unit;
        const int used = (T.C + BK - 1) / BK;
        KT = (used + 3) & ~3;
        a_next = b_next = 0;
        a_end = A_STRIDED ? (uint32_t)a_srd[2] : (uint32_t)T.C * 2u;
        b_end = B_STRIDED ? (uint32_t)b_srd[2] : (uint32_t)T.C * 2u;
        if constexpr (EDGE) {
            if constexpr (A_STRIDED) {
                a_left = 2 * (a_rows * T.lda - a_org);
                a_move = a_left > (int64_t)MAX_RANGE ? MOVE_BASE : ~0u;
            }
            if constexpr (B_STRIDED) {
                b_left = 2 * (b_rows * T.ldb - b_org);
                b_move = b_left > (int64_t)MAX_RANGE ? MOVE_BASE : ~0u;
            }
            last = (uint32_t)(used - 1) * (BK * 2u);
            // swz_c(16 q + n) = swz_c(n): one mask for all of the lane's rows
            tail = ((lane & 3) ^ swz_c(lane >> 2)) * 8 < T.C - (used - 1) * BK ? 0u : OUTSIDE;
            if (last == 0) {
                if constexpr (!A_STRIDED) mask_a();
                if constexpr (!B_STRIDED) mask_b();
            }
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
                if constexpr (EDGE && !A_STRIDED) {
                    if (__builtin_expect(a_next >= last, 0)) {
                        if (a_next == last) mask_a();
                        else a_next = (uint32_t)a_srd[2];
                    }
                } else if (a_next >= a_end) {
                    a_next = (uint32_t)a_srd[2];
                }
            }
        } else {
            dma16(b_voff[it], b_srd, b_next, l);
            if (it == 3) {
                b_next += b_step;
                if constexpr (EDGE && !B_STRIDED) {
                    if (__builtin_expect(b_next >= last, 0)) {
                        if (b_next == last) mask_b();
                        else b_next = (uint32_t)b_srd[2];
                    }
                } else if (b_next >= b_end) {
                    b_next = (uint32_t)b_srd[2];
                }
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
        if constexpr (A_STRIDED) {
            const uint16_t* p = smem + buf * STAGE_HALVES + ((a_rd ^ (i << 5)) + kk * 16 * BM);
            a[i] = read_tr8(p, p + 4 * BM);
        } else {
            a[i] = *reinterpret_cast<const half8*>(smem + buf * STAGE_HALVES + ((a_rd ^ (kk << 4)) + i * 32 * BK));
        }
    };
    auto read_b = [&](half8 (&b)[4], int buf, int kk, int j) {
        const uint16_t* bs = smem + buf * STAGE_HALVES + A_HALVES;
        if constexpr (B_STRIDED) {
            const uint16_t* p = bs + ((b_rd ^ (j << 5)) + kk * 16 * BN);
            b[j] = read_tr8(p, p + 4 * BN);
        } else {
            b[j] = *reinterpret_cast<const half8*>(bs + ((b_rd ^ (kk << 4)) + j * 32 * BK));
        }
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
    constexpr int RA = A_STRIDED ? 2 : 1, RB = B_STRIDED ? 2 : 1;     // LDS read instructions per fragment
    constexpr int READS_EARLY[4] = {RA + 2 * RB, 2 * RB + RA, 2 * RA, 0};
    constexpr int READS_EVEN[4] = {RA + RB, 2 * RB, RB + RA, 2 * RA};

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

    // ---- walk the tile list: tile w = round * G + pos; every workgroup leaves through `break`
    int w = pos;
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
        // every load of this tile's first slices has landed and is visible to all waves (and thread 0 is back)
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        half8 fa0[4], fb0[4], fa1[4], fb1[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) read_group(fa0, fb0, 0, 0, q, false);

        // KT is a multiple of 4: the body is unrolled over the four LDS stages so that every LDS
        // address is a register plus an immediate.
        for (int kt = 0; kt < KT; kt += 4) {
            if constexpr (EDGE && A_STRIDED) {
                if (__builtin_expect(a_next >= a_move, 0)) move_base(a_srd, a_left, a_next, a_end, a_move);
            }
            if constexpr (EDGE && B_STRIDED) {
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
        g.Res = ga.t[tensor].Res;
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
        w += G;
        const bool more = w < ga.total_tiles;
        ++round;
        if constexpr (ALIGN_ROUNDS) {
            if (more && round < SYNC_ROUNDS && tid == 0) atomicAdd(&g_round_arrive[round][xcd], 1);
        }
        if constexpr (EPI != EPI_SQNORM) {
            const RowEpilogue re(g, smem, wave, em0, en0);
            if constexpr (EPI != EPI_STORE) {
                re.fill(0);
                re.fill(1);
                re.fill(2);
            }
            if (more) {
                setup(w, tensor, m0, n0);
                issue_prologue();
            }
            re.template run<EPI>(acc, g, more);
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

template <bool B_STRIDED, int EPI, bool A_STRIDED, bool EDGE>
static hipError_t launch_dma(const GemmArgs* list, int n, hipStream_t st) {
    using namespace dma;
    auto kern = lomo_contract_dma_kernel<B_STRIDED, EPI, A_STRIDED, EDGE>;
    // thread-safe one-time set-up (initialisation of a function-local static)
    static const hipError_t cfg0 = allow_dynamic_lds(kern, LDS_BYTES);
    if (cfg0 != hipSuccess) return cfg0;
    for (int first = 0; first < n; first += MAX_GROUP) {
        const int cnt = (n - first < MAX_GROUP) ? (n - first) : MAX_GROUP;
        GroupArgs ga{};
        fill_group(ga, list + first, cnt, BM, BN);
        const int tiles = ga.total_tiles;
        const int grid = tiles < cu_count() ? tiles : cu_count();
        // the kernels that align their rounds; a single round reads no counter
        if ((EPI == EPI_UPDATE || EPI == EPI_CLIPV) && A_STRIDED && B_STRIDED && tiles > grid) {
            int rounds = (tiles + grid - 1) / grid;
            if (rounds > SYNC_ROUNDS) rounds = SYNC_ROUNDS;
            hipLaunchKernelGGL(clear_round_counters, dim3((unsigned)((rounds * 8 + 255) / 256)), dim3(256), 0, st, rounds);
        }
        hipError_t e = launch_timed(list[first].family, kern, dim3((unsigned)grid), dim3(NT), (size_t)LDS_BYTES, st, ga);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <bool B_STRIDED, int EPI, bool A_STRIDED>
hipError_t launch_dma_group(const GemmArgs* list, int n, hipStream_t st) {
    for (int i = 0; i < n; ++i)
        if (((!A_STRIDED || !B_STRIDED) && list[i].C % dma::BK != 0) || beyond_descriptor<B_STRIDED, A_STRIDED>(list[i]))
            return launch_dma<B_STRIDED, EPI, A_STRIDED, true>(list, n, st);
    return launch_dma<B_STRIDED, EPI, A_STRIDED, false>(list, n, st);
}

template hipError_t launch_dma_group<true, EPI_UPDATE, true>(const GemmArgs*, int, hipStream_t);
template hipError_t launch_dma_group<true, EPI_CLIPV, true>(const GemmArgs*, int, hipStream_t);
template hipError_t launch_dma_group<true, EPI_SQNORM, true>(const GemmArgs*, int, hipStream_t);
template hipError_t launch_dma_group<false, EPI_STORE, true>(const GemmArgs*, int, hipStream_t);
template hipError_t launch_dma_group<false, EPI_STORE, false>(const GemmArgs*, int, hipStream_t);
template hipError_t launch_dma_group<false, EPI_UPDATE, false>(const GemmArgs*, int, hipStream_t);

}  // namespace lomo
