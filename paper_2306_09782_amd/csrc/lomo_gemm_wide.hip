// Persistent, grouped 256 x 256 MFMA contraction for products with a contraction-contiguous operand (gfx950): the
// forward product Y = X W^T (both operands) and dgrad dX = dY W (dY).
//
// Tiles, list walk, epilogues, edges and the order of the sums are those of lomo_gemm_dma.hip; what differs is the
// step of the operand loads.  A slice of 32 indices of a contraction-contiguous operand is 64 bytes of every row, half a
// cache line, so that kernel's loads asked the L2 for every line of such an operand twice.  Here the step is a slot of 64
// indices: 128 bytes of a row, whole lines, eight rows per wave instruction.
//   * two slots of 64 KiB in LDS; a slot is walked in four steps of 16 indices, the fragments of the next step are read
//     while the current one is multiplied.  After the third step all reads of the slot are done (one barrier per 64
//     indices) and its memory is loaded again: A during the fourth step, B during the first step of the next slot, one
//     load instruction after every second MFMA.  That leaves two steps (about 0.8 us) to the last of the loads.
//   * 16-byte chunk c of row r sits at position c ^ (r & 7).  That leaves two-way bank conflicts (rows r and r + 8 of the
//     sixteen that are read together); c ^ ((r >> 1) & 7) has none and measured 0 to 1 % slower: the LDS is a quarter busy,
//     the chip is held by its power limit (1.5 GHz with the matrix pipes 80 % busy).
// Measured, us, slices of 32 -> slots of 64 (same box, same bits):
//   Y of 4096 x 12288, C = 4096: 389 -> 356 (1157 TFLOP/s);  C = 11008, 4096 x 4096: 310 -> 272 (1357);
//   8192 x 5120, C = 13824: 1164 -> 1046;   dX of 4096 x 4096, C = 12288: 319 -> 307 (1344);  4096 x 11008, C = 4096: 328 -> 313.
#include "lomo_gemm_persistent.h"

namespace lomo {

namespace wide {

using namespace dma;
constexpr int BKW = 64;                                        // contraction indices of a slot
constexpr int OP_HALVES = BM * BKW, SLOT_HALVES = 2 * OP_HALVES;
static_assert(2 * SLOT_HALVES == NS * STAGE_HALVES, "the row epilogue's blocks lie behind and in the last quarter of the slots");
constexpr int AHEAD = 24;                                      // loads of a tile's prologue

__device__ __forceinline__ int swz_w(int r) { return r & 7; }

}  // namespace wide

// A_STRIDED: dgrad.  EDGE: some tensor's contraction ends inside a slot, or a contraction-strided operand is larger than a
// descriptor covers.
template <int EPI, bool A_STRIDED, bool EDGE>
__global__ __launch_bounds__(NT) void lomo_contract_wide_kernel(dma::GroupArgs ga) {
    using namespace wide;
    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];

    if (EPI == EPI_UPDATE && ga.flag_in != nullptr && *ga.flag_in != 0) return;   // step dropped

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave & 1, wn = wave >> 1;
    const int l32 = lane & 31, lh = lane >> 5;
    const int G = gridDim.x;

    const uint32_t lds0 = (uint32_t)(uintptr_t)smem;

    // ---- fragment read offsets (halves)
    int a_rd;
    if constexpr (A_STRIDED) {
        const int g4 = lane >> 4, j16 = lane & 15;
        const int mhalf = g4 & 1, kh = g4 >> 1, rib = j16 >> 2, piece = j16 & 3;
        a_rd = (8 * kh + rib) * BM + (((wm * (BM / 16) + 2 * mhalf + (piece >> 1)) ^ swz_s(rib)) * 8) + (piece & 1) * 4;
    } else {
        a_rd = (wm * (BM / 2) + l32) * BKW + ((lh ^ swz_w(l32)) * 8);
    }
    const int b_rd = (wn * (BN / 2) + l32) * BKW + ((lh ^ swz_w(l32)) * 8);

    // ---- per-tile state of the loads
    constexpr int NA = A_STRIDED ? 4 : 8;      // lane offsets of A: a strided slot is two slices with the same four
    uint32_t a_voff[NA], b_voff[8];
    int4v a_srd{}, b_srd{};
    uint32_t a_step = 0;                   // bytes from one slice (strided) or slot to the next
    uint32_t a_next = 0, b_next = 0;       // byte offset of the slice / slot to be requested next
    uint32_t a_end = 0, b_end = 0;         // offsets from here on are behind the last one
    // EDGE only: offset of a contraction-contiguous operand's last slot and this lane's mask there; bytes from a
    // contraction-strided operand's base to its end, and the slice offset from which on the base moves
    uint32_t last = 0, tail = 0;
    int64_t a_left = 0;
    uint32_t a_move = ~0u;
    int KT = 0;                            // slots walked: a multiple of 2

    auto mask_a = [&] {
#pragma unroll
        for (int it = 0; it < NA; ++it) a_voff[it] |= tail;
    };
    auto mask_b = [&] {
#pragma unroll
        for (int it = 0; it < 8; ++it) b_voff[it] |= tail;
    };

    auto setup = [&](int w, int& tensor, int64_t& m0, int64_t& n0) {
        locate_tile<A_STRIDED>(ga, w, tensor, m0, n0);
        const GroupTensor& T = ga.t[tensor];
        const int m_left = T.M - (int)m0;
        const int row8 = lane >> 3, chunk = (lane & 7) ^ swz_w(row8);      // of eight rows of 128 bytes
#pragma unroll
        for (int it = 0; it < NA; ++it) {
            if constexpr (A_STRIDED) {
                const int r = 2 * (wave * 4 + it) + (lane >> 5), col = ((lane & 31) ^ swz_s(r)) * 8;
                a_voff[it] = ((uint32_t)(r * T.lda + col) * 2u) | (col < m_left ? 0u : OUTSIDE);
            } else {
                a_voff[it] = (uint32_t)((8 * (wave * 8 + it) + row8) * T.lda + chunk * 8) * 2u;
            }
        }
#pragma unroll
        for (int it = 0; it < 8; ++it) b_voff[it] = (uint32_t)((8 * (wave * 8 + it) + row8) * T.ldb + chunk * 8) * 2u;
        const int64_t a_org = A_STRIDED ? m0 : m0 * (int64_t)T.lda, a_rows = A_STRIDED ? T.C : T.M;
        const int64_t b_org = n0 * (int64_t)T.ldb;
        a_srd = make_srd(T.A + a_org, range_bytes(a_rows * T.lda - a_org));
        b_srd = make_srd(T.B + b_org, range_bytes((int64_t)T.Nn * T.ldb - b_org));
        a_step = A_STRIDED ? (uint32_t)BK * (uint32_t)T.lda * 2u : (uint32_t)BKW * 2u;
        const int used = (T.C + BKW - 1) / BKW;
        KT = (used + 1) & ~1;
        a_next = b_next = 0;
        a_end = A_STRIDED ? (uint32_t)a_srd[2] : (uint32_t)T.C * 2u;
        b_end = (uint32_t)T.C * 2u;
        if constexpr (EDGE) {
            if constexpr (A_STRIDED) {
                a_left = 2 * (a_rows * T.lda - a_org);
                a_move = a_left > (int64_t)MAX_RANGE ? MOVE_BASE : ~0u;
            }
            last = (uint32_t)(used - 1) * (BKW * 2u);
            tail = chunk * 8 < T.C - (used - 1) * BKW ? 0u : OUTSIDE;      // the same chunk in all of the lane's rows
            if (last == 0) {
                if constexpr (!A_STRIDED) mask_a();
                mask_b();
            }
        }
    };

    // One of this wave's eight load instructions of an operand's next slot; behind the last slot (slice) all of it is out of
    // range.  A contraction-contiguous operand goes on with its next row behind the last index: those lanes are masked from
    // the last slot on (nothing follows it).
    auto issue_a = [&](int slot, int it) {
        const uint32_t l = lds0 + (uint32_t)slot * (SLOT_HALVES * 2u);
        if constexpr (A_STRIDED) {
            dma16(a_voff[it & 3], a_srd, a_next, l + (uint32_t)(it >> 2) * (A_HALVES * 2u) + (uint32_t)(wave * 4 + (it & 3)) * 1024u);
            if ((it & 3) == 3) {
                a_next += a_step;
                if (a_next >= a_end) a_next = (uint32_t)a_srd[2];
            }
        } else {
            dma16(a_voff[it], a_srd, a_next, l + (uint32_t)(wave * 8 + it) * 1024u);
            if (it == 7) {
                a_next += a_step;
                if constexpr (EDGE) {
                    if (__builtin_expect(a_next >= last, 0)) {
                        if (a_next == last) mask_a();
                        else a_next = (uint32_t)a_srd[2];
                    }
                } else if (a_next >= a_end) {
                    a_next = (uint32_t)a_srd[2];
                }
            }
        }
    };
    auto issue_b = [&](int slot, int it) {
        const uint32_t l = lds0 + (uint32_t)slot * (SLOT_HALVES * 2u) + OP_HALVES * 2u;
        dma16(b_voff[it], b_srd, b_next, l + (uint32_t)(wave * 8 + it) * 1024u);
        if (it == 7) {
            b_next += BKW * 2u;
            if constexpr (EDGE) {
                if (__builtin_expect(b_next >= last, 0)) {
                    if (b_next == last) mask_b();
                    else b_next = (uint32_t)b_srd[2];
                }
            } else if (b_next >= b_end) {
                b_next = (uint32_t)b_srd[2];
            }
        }
    };
    // Slot 0 and the A part of slot 1 of the tile that `setup` selected.
    auto issue_prologue = [&] {
#pragma unroll
        for (int it = 0; it < 8; ++it) issue_a(0, it);
#pragma unroll
        for (int it = 0; it < 8; ++it) issue_b(0, it);
#pragma unroll
        for (int it = 0; it < 8; ++it) issue_a(1, it);
    };

    // ---- fragments of step kk of a slot, in the order the MFMAs consume them: a0, b0..b3, a1..a3
    constexpr int RA = A_STRIDED ? 2 : 1;            // LDS read instructions per A fragment
    auto read_frag = [&](half8 (&a)[4], half8 (&b)[4], int slot, int kk, int f) {
        if (f >= 1 && f <= 4) {
            const uint16_t* bs = smem + slot * SLOT_HALVES + OP_HALVES;
            b[f - 1] = *reinterpret_cast<const half8*>(bs + ((b_rd ^ (kk << 4)) + (f - 1) * 32 * BKW));
        } else {
            const int i = f == 0 ? 0 : f - 4;
            const uint16_t* as = smem + slot * SLOT_HALVES;
            if constexpr (A_STRIDED) {
                const uint16_t* p = as + (kk >> 1) * A_HALVES + ((a_rd ^ (i << 5)) + (kk & 1) * 16 * BM);
                a[i] = read_tr8(p, p + 4 * BM);
            } else {
                a[i] = *reinterpret_cast<const half8*>(as + ((a_rd ^ (kk << 4)) + i * 32 * BKW));
            }
        }
    };
    // Fragments [FIRST[p], FIRST[p + 1]) are read in part p of a step.  EARLY: all of them in the first five parts, so that
    // every read has completed when the step ends at a barrier.
    constexpr int FIRST_EARLY[9] = {0, 2, 4, 6, 7, 8, 8, 8, 8}, FIRST_EVEN[9] = {0, 1, 2, 3, 4, 5, 6, 7, 8};

    floatx16 acc[4][4];
    auto zero_acc = [&] {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    };

    // One step of 16 indices: 16 MFMAs on (ua, ub) in eight parts of two, each with its share of the reads of the next
    // step's fragments in front of them and, where the step loads an operand (1: A, 2: B), one load behind them.
    auto step = [&](const half8 (&ua)[4], const half8 (&ub)[4], half8 (&la)[4], half8 (&lb)[4], int lslot, int lkk, bool early,
                    int load, int dslot) {
#pragma unroll
        for (int p = 0; p < 8; ++p) {
            int reads = 0;
#pragma unroll
            for (int f = 0; f < 8; ++f)
                if (f >= (early ? FIRST_EARLY[p] : FIRST_EVEN[p]) && f < (early ? FIRST_EARLY[p + 1] : FIRST_EVEN[p + 1])) {
                    read_frag(la, lb, lslot, lkk, f);
                    reads += (f >= 1 && f <= 4) ? 1 : RA;
                }
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int q = p >> 1, c = 2 * (p & 1) + j;
                acc[q][c] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ua[q], ub[c], acc[q][c], 0, 0, 0);
            }
            const int now = (reads + 1) / 2;
            if (now == 1) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // DS reads
            if (now == 2) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            if (reads - now == 1) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            if (reads - now == 2) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (load == 1) issue_a(dslot, p);
            if (load == 2) issue_b(dslot, p);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // ---- walk the tile list, one tile a round; every workgroup leaves through `break`
    int round = 0;
    int w = round_tile(round, G, ga.total_tiles, ga.deal != 0);
    if (w >= ga.total_tiles) return;   // cannot happen with grid <= total_tiles; nothing was issued yet
    int tensor = 0;
    int64_t m0, n0;
    setup(w, tensor, m0, n0);
    issue_prologue();
    zero_acc();

    for (bool first = true;; first = false) {
        // every load of this tile's first slots has landed and is visible to all waves; the last tile's stores, issued behind
        // them, may still be on their way
        if (first) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(RowEpilogue::OPS<EPI>) : "memory");
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        half8 fa0[4], fb0[4], fa1[4], fb1[4];
#pragma unroll
        for (int f = 0; f < 8; ++f) read_frag(fa0, fb0, 0, 0, f);

        // KT is a multiple of 2: the body is unrolled over the two slots
        for (int kt = 0; kt < KT; kt += 2) {
            if constexpr (EDGE && A_STRIDED) {
                if (__builtin_expect(a_next >= a_move, 0)) move_base(a_srd, a_left, a_next, a_end, a_move);
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                step(fa0, fb0, fa1, fb1, u, 1, false, 2, u ^ 1);      // B of the other slot
                step(fa1, fb1, fa0, fb0, u, 2, false, 0, 0);
                step(fa0, fb0, fa1, fb1, u, 3, true, 0, 0);
                // the other slot has landed, nobody reads this one any more
                asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
                step(fa1, fb1, fa0, fb0, u ^ 1, 0, false, 1, u);      // A into this slot
            }
        }
        // drain: the loads past the end (zeros) have landed, all waves are done with the slots
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
        const RowEpilogue re(g, smem, wave, m0, n0);
        if constexpr (EPI != EPI_STORE) {
            re.fill(0);
            re.fill(1);
            re.fill(2);
        }
        ++round;
        w = next_tile(w, round, G, ga.total_tiles, ga.deal != 0);
        const bool more = w < ga.total_tiles;
        if (more) {
            setup(w, tensor, m0, n0);
            issue_prologue();
        }
        re.template run<EPI, AHEAD>(acc, g, more);
        if (!more) break;
        zero_acc();
    }
}

// ---- host side ----------------------------------------------------------------------------

template <int EPI, bool A_STRIDED, bool EDGE>
static hipError_t launch_wide(const GemmArgs* list, int n, hipStream_t st) {
    using namespace dma;
    auto kern = lomo_contract_wide_kernel<EPI, A_STRIDED, EDGE>;
    // thread-safe one-time set-up (initialisation of a function-local static)
    static const hipError_t cfg0 = allow_dynamic_lds(kern, LDS_BYTES);
    if (cfg0 != hipSuccess) return cfg0;
    for (int first = 0; first < n; first += MAX_GROUP) {
        GroupArgs ga{};
        fill_group(ga, list + first, n - first < MAX_GROUP ? n - first : MAX_GROUP, BM, BN);
        const int grid = ga.total_tiles < cu_count() ? ga.total_tiles : cu_count();
        ga.deal = choose_deal(ga, grid);
        hipError_t e = launch_timed(list[first].family, kern, dim3((unsigned)grid), dim3(NT), (size_t)LDS_BYTES, st, ga);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <int EPI, bool A_STRIDED>
hipError_t launch_wide_group(const GemmArgs* list, int n, hipStream_t st) {
    for (int i = 0; i < n; ++i)
        if (list[i].C % wide::BKW != 0 || beyond_descriptor<false, A_STRIDED>(list[i])) return launch_wide<EPI, A_STRIDED, true>(list, n, st);
    return launch_wide<EPI, A_STRIDED, false>(list, n, st);
}

template hipError_t launch_wide_group<EPI_STORE, true>(const GemmArgs*, int, hipStream_t);
template hipError_t launch_wide_group<EPI_STORE, false>(const GemmArgs*, int, hipStream_t);
template hipError_t launch_wide_group<EPI_UPDATE, false>(const GemmArgs*, int, hipStream_t);

}  // namespace lomo
