// MFMA contraction for outputs of few tiles (gfx950): smaller tiles than the persistent kernel's, one workgroup per tile.
//
// Same mathematics, operands, order of the sums and epilogues as the persistent 256 x 256 kernel of lomo_gemm_dma.hip, for
// outputs that give that kernel too few tiles to occupy the chip (dgrad and forward products at up to about a thousand
// tokens, narrow models).
//   * The waves of a workgroup share the tile, not the contraction: every element of the output is one chain of matrix
//     instructions over the slices (32 contraction indices) from the first to the last, as in the other contraction kernels,
//     so a tensor's result has the same bits whichever kernel runs it, and the choice is free to look at the whole list.
//   * Operands arrive by direct-to-LDS loads through buffer descriptors, as in the persistent kernel: the range check
//     supplies the zeros outside the tensor, lanes behind the last column get an offset that no descriptor covers, and the
//     lanes of a contraction-contiguous operand that lie behind the last index are masked in the last slice.
//   * A ring of slices in LDS, two slices per barrier (one per barrier: 128 x 128 tiles 10 % slower); their fragments are read
//     into registers while the previous two are multiplied, so all of the ring but those two holds loads in flight.
//   * 256 x 128: eight waves of 64 x 64, two on every SIMD, 144 KiB.  128 x 128: eight waves of 64 x 32, two on every SIMD (one's LDS reads run behind the other's MFMAs), 128 KiB of LDS.
//     128 x 64: four waves of 64 x 32, 72 KiB; 64 x 64: four waves of 32 x 32, 80 KiB: two workgroups on a CU, so that
//     one's ramp-up and epilogue run behind the other's main loop.  64 x 32, for long contractions of very few tiles: two waves of
//     32 x 32, 72 KiB.
// One launch takes a list of tensors; workgroups start in list order, longest contraction first.
//
// Measured, us per call, against the same tiles with the contraction split over two or four groups of waves (which adds in
// another order) and against the persistent kernel:
//   dX of 1024 x 4096, C = 22016, 128 x 128 tiles: 178 (1037 TFLOP/s), 196, 350;  Y of 1024 x 4096, C = 11008: 95, 117, 190
//   dX of 2048 x 4096, C = 4096: 256 x 128 tiles 73, 128 x 128 83, persistent 82;  2048 x 4096, C = 11008: 170, 191, 184;
//   dX of 1024 x 5120, C = 13824: 157, 205, 244
//   dX of 777 x 2048, C = 32000, 128 x 64 tiles: 168, 166, 475;               update of 777 x 2048 x 2048: 14.6, 18, 28
//   dX of 256 x 1024, 64 x 64 / 64 x 32 tiles: C = 32000 127 / 91, C = 5632 22.9 / 18.7; of 128 x 4096, C = 32000 153 / 118
//   dX of 256 x 1024, C = 32000, 64 x 64 tiles: 127, 138, 470;                Y of 777 x 2048, C = 2048: 15.0, 19.7, 40
#include "lomo_gemm_common.h"
#include "lomo_gemm_dma_common.h"

#include <type_traits>

namespace lomo {

namespace tile {

using dma::BK;

// chunk swizzle of a contraction-strided tile row of BX columns: the four rows that one transposing read touches start in
// different quarters of the 256 bytes that the banks hold (rows of 64 columns: two rows side by side in them)
template <int BX>
__device__ __forceinline__ int swz_row(int r) {
    return BX == 64 ? (r & 2) * 2 : ((r & 1) * 10) + ((r & 2) * 2);
}

template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (N > 0) {
        static_for<N - 1>(f);
        f(std::integral_constant<int, N - 1>{});
    }
}

}  // namespace tile

// RI x RJ blocks of 32 x 32 per wave, WM x WN waves, ring of NS slices, U slices between barriers.
template <int RI, int RJ, int WM, int WN, int NS, int U, bool B_STRIDED, int EPI, bool A_STRIDED>
__global__ __launch_bounds__(64 * WM * WN) void lomo_contract_tile_kernel(dma::GroupArgs ga) {
    using namespace dma;
    using namespace tile;
    constexpr int W = WM * WN;
    constexpr int TM = 32 * RI * WM, TN = 32 * RJ * WN;
    constexpr int AH = BK * TM, BH = BK * TN, STAGE = AH + BH;                     // halves
    constexpr int NA = TM / 16 / W, NB = TN / 16 / W;                              // load instructions of a wave per slice
    static_assert(NA * W * 16 == TM && NB * W * 16 == TN && NS % U == 0 && NS / U >= 3, "");
    constexpr int R = NS / U;                                                      // slots of the ring
    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];

    if (EPI == EPI_UPDATE && ga.flag_in != nullptr && *ga.flag_in != 0) return;      // step dropped

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wn = wave / WM;

    // tile of this workgroup: each XCD (blockIdx % 8) takes a contiguous run of the tensor's band order, whose neighbours
    // share panels
    int tensor = 0;
    while (tensor + 1 < ga.n && (int)blockIdx.x >= ga.t[tensor + 1].tile_begin) ++tensor;
    const GroupTensor& g = ga.t[tensor];
    int64_t m0, n0;
    {
        const int tiles_m = g.tiles_m, tiles_n = g.tiles_n, total = tiles_m * tiles_n;
        const int l = (int)blockIdx.x - g.tile_begin;
        const int x = l & 7, local = l >> 3;
        const int q = total >> 3, r = total & 7;
        const int t = x * q + (x < r ? x : r) + local;
        constexpr int GM = 8;
        const int per_band = GM * tiles_n;
        const int first_m = t / per_band * GM;
        const int gsz = (tiles_m - first_m < GM) ? (tiles_m - first_m) : GM;
        const int in_band = t % per_band;
        m0 = (int64_t)(first_m + in_band % gsz) * TM;
        n0 = (int64_t)(in_band / gsz) * TN;
    }
    const int m_left = g.M - (int)m0, n_left = g.Nn - (int)n0;
    const int C = g.C, lda = g.lda, ldb = g.ldb;
    const int64_t ldo = g.ldo;

    // ---- loads: this wave's instructions of a slice, and what each lane fetches with them
    const uint32_t ring = (uint32_t)(uintptr_t)smem;
    uint32_t a_voff[U][NA], b_voff[U][NB];
#pragma unroll
    for (int it = 0; it < NA; ++it) {
        const int q = wave * NA + it;
        if constexpr (A_STRIDED) {
            const int r = q * (512 / TM) + lane / (TM / 8), col = ((lane % (TM / 8)) ^ swz_row<TM>(r)) * 8;
            a_voff[0][it] = ((uint32_t)(r * lda + col) * 2u) | (col < m_left ? 0u : OUTSIDE);
        } else {
            const int n = 16 * q + (lane >> 2), kc = ((lane & 3) ^ swz_c(n)) * 8;
            a_voff[0][it] = (uint32_t)(n * lda + kc) * 2u;
        }
#pragma unroll
        for (int x = 1; x < U; ++x) a_voff[x][it] = a_voff[0][it];
    }
#pragma unroll
    for (int it = 0; it < NB; ++it) {
        const int q = wave * NB + it;
        if constexpr (B_STRIDED) {
            const int r = q * (512 / TN) + lane / (TN / 8), col = ((lane % (TN / 8)) ^ swz_row<TN>(r)) * 8;
            b_voff[0][it] = ((uint32_t)(r * ldb + col) * 2u) | (col < n_left ? 0u : OUTSIDE);
        } else {
            const int n = 16 * q + (lane >> 2), kc = ((lane & 3) ^ swz_c(n)) * 8;
            b_voff[0][it] = (uint32_t)(n * ldb + kc) * 2u;
        }
#pragma unroll
        for (int x = 1; x < U; ++x) b_voff[x][it] = b_voff[0][it];
    }
    const int64_t a_org = A_STRIDED ? m0 : m0 * lda, a_rows = A_STRIDED ? C : g.M;
    const int64_t b_org = B_STRIDED ? n0 : n0 * ldb, b_rows = B_STRIDED ? C : g.Nn;
    const int4v a_srd = make_srd(g.A + a_org, range_bytes(a_rows * lda - a_org));
    const int4v b_srd = make_srd(g.B + b_org, range_bytes(b_rows * ldb - b_org));
    const uint32_t a_unit = A_STRIDED ? (uint32_t)lda * 2u : 2u, b_unit = B_STRIDED ? (uint32_t)ldb * 2u : 2u;
    const uint32_t a_step = (uint32_t)BK * a_unit, b_step = (uint32_t)BK * b_unit;
    const uint32_t a_end = A_STRIDED ? (uint32_t)a_srd[2] : (uint32_t)C * 2u;
    const uint32_t b_end = B_STRIDED ? (uint32_t)b_srd[2] : (uint32_t)C * 2u;
    const int slices = (C + BK - 1) / BK;
    const int KT = (slices + U - 1) / U;
    // offset of the next slice; the range itself: nothing there
    uint32_t a_next = 0, b_next = 0;
    // A contraction-contiguous operand goes on behind its last index with the next row: those lanes are masked from the last
    // slice on (nothing follows it).  Done for the coming slot among the matrix instructions, off the way of the loads.
    const int last_rows = C - (slices - 1) * BK;
    const uint32_t tail = ((lane & 3) ^ swz_c(lane >> 2)) * 8 < last_rows ? 0u : OUTSIDE;
    const uint32_t last = A_STRIDED && B_STRIDED ? 0u : (uint32_t)(slices - 1) * (BK * 2u);
    auto issue_slot = [&](int slot) {
#pragma unroll
        for (int x = 0; x < U; ++x) {
            const uint32_t l = ring + (uint32_t)(slot * U + x) * (STAGE * 2u);
#pragma unroll
            for (int it = 0; it < NA; ++it) dma16(a_voff[x][it], a_srd, a_next, l + (uint32_t)(wave * NA + it) * 1024u);
            a_next += a_step;
            if (a_next >= a_end) a_next = (uint32_t)a_srd[2];
        }
#pragma unroll
        for (int x = 0; x < U; ++x) {
            const uint32_t l = ring + (uint32_t)(slot * U + x) * (STAGE * 2u) + AH * 2u;
#pragma unroll
            for (int it = 0; it < NB; ++it) dma16(b_voff[x][it], b_srd, b_next, l + (uint32_t)(wave * NB + it) * 1024u);
            b_next += b_step;
            if (b_next >= b_end) b_next = (uint32_t)b_srd[2];
        }
    };

    auto mask_ahead = [&] {
#pragma unroll
        for (int x = 0; x < U; ++x) {
            if constexpr (!A_STRIDED) {
                const uint32_t m = a_next + (uint32_t)x * a_step == last ? tail : 0u;
#pragma unroll
                for (int it = 0; it < NA; ++it) a_voff[x][it] |= m;
            }
            if constexpr (!B_STRIDED) {
                const uint32_t m = b_next + (uint32_t)x * b_step == last ? tail : 0u;
#pragma unroll
                for (int it = 0; it < NB; ++it) b_voff[x][it] |= m;
            }
        }
    };

    // ---- fragment reads
    const int g4 = lane >> 4, j16 = lane & 15;
    const int mhalf = g4 & 1, kh = g4 >> 1, rib = j16 >> 2, piece = j16 & 3;
    const int l32 = lane & 31, lh = lane >> 5;
    int a_rd, b_rd;
    if constexpr (A_STRIDED) {
        a_rd = (8 * kh + rib) * TM + (((wm * 4 * RI + 2 * mhalf + (piece >> 1)) ^ swz_row<TM>(rib)) * 8) + (piece & 1) * 4;
    } else {
        const int ml = wm * 32 * RI + l32;
        a_rd = ml * BK + ((lh ^ swz_c(ml)) * 8);
    }
    if constexpr (B_STRIDED) {
        b_rd = (8 * kh + rib) * TN + (((wn * 4 * RJ + 2 * mhalf + (piece >> 1)) ^ swz_row<TN>(rib)) * 8) + (piece & 1) * 4;
    } else {
        const int nl = wn * 32 * RJ + l32;
        b_rd = nl * BK + ((lh ^ swz_c(nl)) * 8);
    }
    auto read_a = [&](int buf, int kk, int i) -> half8 {
        if constexpr (A_STRIDED) {
            const uint16_t* p = smem + buf * STAGE + ((a_rd ^ (i << 5)) + kk * 16 * TM);
            return read_tr8(p, p + 4 * TM);
        } else {
            return *reinterpret_cast<const half8*>(smem + buf * STAGE + ((a_rd ^ (kk << 4)) + i * 32 * BK));
        }
    };
    auto read_b = [&](int buf, int kk, int j) -> half8 {
        const uint16_t* bs = smem + buf * STAGE + AH;
        if constexpr (B_STRIDED) {
            const uint16_t* p = bs + ((b_rd ^ (j << 5)) + kk * 16 * TN);
            return read_tr8(p, p + 4 * TN);
        } else {
            return *reinterpret_cast<const half8*>(bs + ((b_rd ^ (kk << 4)) + j * 32 * BK));
        }
    };
    struct Frags {
        half8 a[U][2][RI], b[U][2][RJ];      // [slice][half of the slice][32 rows / columns]
    };
    constexpr int READS = U * 2 * (RI * (A_STRIDED ? 2 : 1) + RJ * (B_STRIDED ? 2 : 1));
    constexpr int MFMAS = U * 2 * RI * RJ;
    auto read_all = [&](Frags& f, int buf) {
#pragma unroll
        for (int x = 0; x < U; ++x)
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
                for (int i = 0; i < RI; ++i) f.a[x][kk][i] = read_a(buf + x, kk, i);
#pragma unroll
                for (int j = 0; j < RJ; ++j) f.b[x][kk][j] = read_b(buf + x, kk, j);
            }
    };

    floatx16 acc[RI][RJ];
#pragma unroll
    for (int i = 0; i < RI; ++i)
#pragma unroll
        for (int j = 0; j < RJ; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    auto step = [&](const Frags& use, Frags& load, int slot) {
        // the next slot is here, this one is in registers everywhere
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((R - 2) * U * (NA + NB)) : "memory");
        __builtin_amdgcn_sched_barrier(0);
        issue_slot(slot);
        __builtin_amdgcn_sched_barrier(0);
        mask_ahead();
        read_all(load, (slot + 1) % R * U);
#pragma unroll
        for (int x = 0; x < U; ++x)
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                for (int i = 0; i < RI; ++i)
#pragma unroll
                    for (int j = 0; j < RJ; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(use.a[x][kk][i], use.b[x][kk][j], acc[i][j], 0, 0, 0);
        static_for<MFMAS>([&](auto k) {      // one MFMA, then its share of the LDS reads
            constexpr int K = decltype(k)::value;
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            constexpr int now = READS * (K + 1) / MFMAS - READS * K / MFMAS;
            if constexpr (now > 0) __builtin_amdgcn_sched_group_barrier(0x100, now, 0);
        });
        __builtin_amdgcn_sched_barrier(0);
    };

#pragma unroll
    for (int st = 0; st < R; ++st) {
        mask_ahead();
        issue_slot(st);
    }
    mask_ahead();
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((R - 1) * U * (NA + NB)) : "memory");
    __builtin_amdgcn_sched_barrier(0);
    Frags f0, f1;
    read_all(f0, 0);
    for (int kt = 0; kt < KT;) {                     // slices from the last on are zeros
        static_for<(R % 2 ? R : R / 2)>([&](auto pair) {
            constexpr int u = 2 * decltype(pair)::value;
            if (kt >= KT) return;
            step(f0, f1, u % R);
            step(f1, f0, (u + 1) % R);
            kt += 2;
        });
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");      // the LDS is free
    __builtin_amdgcn_sched_barrier(0);

    // ---- epilogue
    constexpr bool RMW = (EPI == EPI_UPDATE || EPI == EPI_CLIPV);
    const uint16_t* old_base = (EPI == EPI_UPDATE && g.Res != nullptr) ? g.Res : g.Out;
    auto m_at = [&](int i, int a) { return wm * 32 * RI + 32 * i + 16 * a + 8 * lh; };
    auto n_at = [&](int j) { return wn * 32 * RJ + 32 * j + l32; };

    if constexpr (EPI == EPI_SQNORM) {
        float* xch = reinterpret_cast<float*>(smem);
        float sq = 0.f;
        uint32_t worst = 0u;
#pragma unroll
        for (int i = 0; i < RI; ++i)
#pragma unroll
            for (int j = 0; j < RJ; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) {           // elements outside the tensor are zero
                    const float v = acc[i][j][r];
                    sq = fmaf(v, v, sq);
                    const uint32_t mag = __float_as_uint(v) & 0x7fffffffu;
                    worst = mag > worst ? mag : worst;
                }
        sq = wave_sum(sq);
        const bool bad = __any(worst >= 0x7f800000u);
        if (lane == 0) {
            xch[wave] = sq;
            reinterpret_cast<int*>(smem)[16 + wave] = bad ? 1 : 0;
        }
        __syncthreads();
        if (tid == 0) {
            float total = 0.f;
            int any_bad = 0;
#pragma unroll
            for (int k = 0; k < W; ++k) {
                total += xch[k];
                any_bad |= reinterpret_cast<int*>(smem)[16 + k];
            }
            atomicAdd(ga.acc, (double)total);
            if (g.flag_out != nullptr && any_bad) atomicOr(g.flag_out, 1);
        }
    } else {
        half8 old[RI][RJ][2];
        if constexpr (RMW) {
#pragma unroll
            for (int i = 0; i < RI; ++i)
#pragma unroll
                for (int j = 0; j < RJ; ++j)
#pragma unroll
                    for (int a = 0; a < 2; ++a)
                        if (n_at(j) < n_left && m_at(i, a) < m_left)
                            old[i][j][a] = *reinterpret_cast<const half8*>(old_base + (n0 + n_at(j)) * ldo + m0 + m_at(i, a));
        }
        typedef uint32_t u32x2v __attribute__((ext_vector_type(2)));
        const float s = ga.s_dev != nullptr ? *ga.s_dev : ga.s;
        bool bad = false;
#pragma unroll
        for (int i = 0; i < RI; ++i)
#pragma unroll
            for (int j = 0; j < RJ; ++j)
#pragma unroll
                for (int a = 0; a < 2; ++a) {
                    // lanes l and l + 32 hold the two 4-row halves of every 8 rows: after the swap a lane owns 8 consecutive m
                    float v[8];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const u32x2v sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[i][j][8 * a + e]),
                                                                           __float_as_uint(acc[i][j][8 * a + 4 + e]), false, false);
                        v[e] = __uint_as_float(sw[0]);
                        v[4 + e] = __uint_as_float(sw[1]);
                    }
                    if (n_at(j) >= n_left || m_at(i, a) >= m_left) continue;
                    half8 out;
                    if constexpr (EPI == EPI_UPDATE) {
#pragma unroll
                        for (int e = 0; e < 8; ++e) out[e] = (_Float16)fmaf(-s, v[e], (float)old[i][j][a][e]);
                    } else if constexpr (EPI == EPI_CLIPV) {
                        // clip by value (section 3.3.1): a non-finite element raises the flag and leaves its weight alone
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const float gq = v[e] * ga.inv_s;
                            const bool fin = (__float_as_uint(gq) & 0x7f800000u) != 0x7f800000u;
                            const float gc = fminf(fmaxf(gq, -ga.clipv), ga.clipv);
                            out[e] = fin ? (_Float16)fmaf(-ga.lr, gc, (float)old[i][j][a][e]) : old[i][j][a][e];
                            bad |= !fin;
                        }
                    } else {
#pragma unroll
                        for (int e = 0; e < 8; ++e) out[e] = (_Float16)v[e];
                    }
                    *reinterpret_cast<half8*>(g.Out + (n0 + n_at(j)) * ldo + m0 + m_at(i, a)) = out;
                }
        if constexpr (EPI == EPI_CLIPV) {
            if (__any(bad) && lane == 0 && g.flag_out != nullptr) atomicOr(g.flag_out, 1);
        }
    }
}

// ---- host side ----------------------------------------------------------------------------

template <int RI, int RJ, int WM, int WN, int NS, int U, bool B_STRIDED, int EPI, bool A_STRIDED>
static hipError_t launch_tile(const GemmArgs* list, int n, hipStream_t st) {
    constexpr int TM = 32 * RI * WM, TN = 32 * RJ * WN, LDS = NS * (TM + TN) * dma::BK * 2;
    static_assert(LDS <= 160 * 1024, "");
    auto kern = lomo_contract_tile_kernel<RI, RJ, WM, WN, NS, U, B_STRIDED, EPI, A_STRIDED>;
    // thread-safe one-time set-up (initialisation of a function-local static)
    static const hipError_t cfg0 = allow_dynamic_lds(kern, LDS);
    if (cfg0 != hipSuccess) return cfg0;
    for (int first = 0; first < n; first += dma::MAX_GROUP) {
        dma::GroupArgs ga{};
        dma::fill_group(ga, list + first, n - first < dma::MAX_GROUP ? n - first : dma::MAX_GROUP, TM, TN);
        hipError_t e = launch_timed(list[first].family, kern, dim3((unsigned)ga.total_tiles), dim3(64 * WM * WN), (size_t)LDS, st, ga);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <bool B_STRIDED, int EPI, bool A_STRIDED>
hipError_t launch_tile_group(const GemmArgs* list, int n, int tile, hipStream_t st) {
    switch (tile) {
        case TILE_256_128: return launch_tile<2, 2, 4, 2, 6, 2, B_STRIDED, EPI, A_STRIDED>(list, n, st);
        case TILE_128: return launch_tile<2, 1, 2, 4, 8, 2, B_STRIDED, EPI, A_STRIDED>(list, n, st);
        case TILE_128_64: return launch_tile<2, 1, 2, 2, 6, 2, B_STRIDED, EPI, A_STRIDED>(list, n, st);
        case TILE_64_32:
            if constexpr (!B_STRIDED && EPI == EPI_STORE) return launch_tile<1, 1, 2, 1, 12, 2, B_STRIDED, EPI, A_STRIDED>(list, n, st);
            else return hipErrorInvalidValue;      // never chosen
        default: return launch_tile<1, 1, 2, 2, 10, 2, B_STRIDED, EPI, A_STRIDED>(list, n, st);
    }
}
template hipError_t launch_tile_group<true, EPI_UPDATE, true>(const GemmArgs*, int, int, hipStream_t);
template hipError_t launch_tile_group<true, EPI_CLIPV, true>(const GemmArgs*, int, int, hipStream_t);
template hipError_t launch_tile_group<true, EPI_SQNORM, true>(const GemmArgs*, int, int, hipStream_t);
template hipError_t launch_tile_group<false, EPI_STORE, true>(const GemmArgs*, int, int, hipStream_t);
template hipError_t launch_tile_group<false, EPI_STORE, false>(const GemmArgs*, int, int, hipStream_t);
template hipError_t launch_tile_group<false, EPI_UPDATE, false>(const GemmArgs*, int, int, hipStream_t);

}  // namespace lomo
