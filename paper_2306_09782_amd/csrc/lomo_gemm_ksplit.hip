// MFMA contraction for outputs of few tiles (gfx950): the waves of a workgroup share the contraction as well as the tile.
//
// Same mathematics, operands and epilogues as the persistent 256 x 256 kernel of lomo_gemm_dma.hip, for outputs that
// give that kernel too few tiles to occupy the chip (dgrad and forward products at up to about a thousand tokens, narrow
// models).  What bounds those is how many CUs work and how deep the serial walk over the contraction is, so
//   * the tile is 64 WM x 64 WN, and WK groups of WM x WN waves walk it together: group k takes the slices (32 contraction
//     indices) k, k + WK, ... with a ring of LDS stages and fp32 accumulators of its own, and the groups' partial sums
//     are added in fp32 through the LDS at the end.  128 x 128 x 2 puts two waves on every SIMD of a CU (one wave's LDS
//     reads run behind the other's MFMAs); 128 x 64 x 4 gives twice the workgroups and half of the serial
//     walk at nearly the rate, 64 x 64 x 4 four times and a quarter, with rings private to one wave each: no barrier;
//   * operands arrive by direct-to-LDS loads through buffer descriptors, as in the persistent kernel: the range check
//     supplies the zeros outside the tensor, lanes behind the last column get an offset that no descriptor covers,
//     the odd slice comes first and is masked by lane, slices behind the last one are out of range as a whole;
//   * the fragments of the next slice are read while the current one is multiplied, so the stage of the current slice is
//     already free when its multiplication starts: all stages hold loads in flight.
// One launch takes a list of tensors; workgroups start in list order, longest contraction first.
//
// Measured, before -> now (us per call; before: 256 x 256 tiles, or 128 x 128 with register-staged operands):
//   dX of 1024 x 4096, C = 22016: 267 -> 199 (926 TFLOP/s);  of 960 x 4096, C = 22016: 579 -> 196
//   Y of 1024 x 4096, C = 11008: 259 -> 118 (783);           dX of 256 x 4096, C = 32000: 450 -> 158
//   dX of 777 x 2048, C = 32000: 128 x 64 tiles 171 (783; 64 x 64 tiles 271, 128 x 128 tiles 260)
//   dX of 256 x 1024, C = 32000: 347 -> 138;                 Y of 256 x 1024, C = 2816: 51 -> 10 (the call's own cost)
// The 128 x 128 tile reads 4 KiB of the LDS per 128 matrix clocks of a wave, 128 bytes per clock and CU: that port, shared
// with the arriving loads, is its bound.  The 64 x 64 tile reads each operand byte from the L2 once per 64 products.
#include "lomo_gemm_common.h"
#include "lomo_gemm_dma_common.h"

#include <type_traits>

namespace lomo {

namespace ksplit {

using dma::BK;
// LDS stages of each group: as many as 160 KiB hold
constexpr int stages(int wm, int wn, int wk) { return wk * (wm + wn) > 8 ? 3 : 4; }

// chunk swizzle of a contraction-strided tile row of BX columns: the four rows that one transposing read touches start in
// different quarters of the 256 bytes that the banks hold (rows of 64 columns: two rows side by side in them)
template <int BX>
__device__ __forceinline__ int swz_row(int r) {
    return BX == 64 ? (r & 2) * 2 : ((r & 1) * 10) + ((r & 2) * 2);
}

template <int N, typename F>
__device__ __forceinline__ void static_for_pairs(F&& f) {
    if constexpr (N > 0) {
        static_for_pairs<N - 1>(f);
        f(std::integral_constant<int, N - 1>{});
    }
}

}  // namespace ksplit

template <int WM, int WN, int WK, bool B_STRIDED, int EPI, bool A_STRIDED>
__global__ __launch_bounds__(64 * WM * WN * WK) void lomo_contract_ksplit_kernel(dma::GroupArgs ga) {
    using namespace dma;
    using namespace ksplit;
    constexpr int TM = 64 * WM, TN = 64 * WN;
    constexpr int AH = BK * TM, BH = BK * TN, STAGE = AH + BH;                     // halves
    constexpr int NA = 4 / WN, NB = 4 / WM;                                        // load instructions of a wave per slice
    constexpr int NS = stages(WM, WN, WK);
    constexpr bool PRIVATE = WM * WN == 1;                                         // a ring belongs to one wave
    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];

    if (EPI == EPI_UPDATE && ga.flag_in != nullptr && *ga.flag_in != 0) return;      // step dropped

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = wave / (WM * WN), wi = wave % (WM * WN);
    const int wm = wi % WM, wn = wi / WM;

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
    const uint32_t ring = (uint32_t)(uintptr_t)smem + (uint32_t)grp * (NS * STAGE * 2u);
    uint32_t a_voff[NA], b_voff[NB];
    int a_c[NA], b_c[NB];                    // first contraction index of the lane's 16 bytes inside the slice
#pragma unroll
    for (int it = 0; it < NA; ++it) {
        const int q = wi * NA + it;
        if constexpr (A_STRIDED) {
            const int r = q * (512 / TM) + lane / (TM / 8), col = ((lane % (TM / 8)) ^ swz_row<TM>(r)) * 8;
            a_voff[it] = ((uint32_t)(r * lda + col) * 2u) | (col < m_left ? 0u : OUTSIDE);
            a_c[it] = r;
        } else {
            const int n = 16 * q + (lane >> 2), kc = ((lane & 3) ^ swz_c(n)) * 8;
            a_voff[it] = (uint32_t)(n * lda + kc) * 2u;
            a_c[it] = kc;
        }
    }
#pragma unroll
    for (int it = 0; it < NB; ++it) {
        const int q = wi * NB + it;
        if constexpr (B_STRIDED) {
            const int r = q * (512 / TN) + lane / (TN / 8), col = ((lane % (TN / 8)) ^ swz_row<TN>(r)) * 8;
            b_voff[it] = ((uint32_t)(r * ldb + col) * 2u) | (col < n_left ? 0u : OUTSIDE);
            b_c[it] = r;
        } else {
            const int n = 16 * q + (lane >> 2), kc = ((lane & 3) ^ swz_c(n)) * 8;
            b_voff[it] = (uint32_t)(n * ldb + kc) * 2u;
            b_c[it] = kc;
        }
    }
    const int64_t a_org = A_STRIDED ? m0 : m0 * lda, a_rows = A_STRIDED ? C : g.M;
    const int64_t b_org = B_STRIDED ? n0 : n0 * ldb, b_rows = B_STRIDED ? C : g.Nn;
    const int4v a_srd = make_srd(g.A + a_org, range_bytes(a_rows * lda - a_org));
    const int4v b_srd = make_srd(g.B + b_org, range_bytes(b_rows * ldb - b_org));
    const uint32_t a_unit = A_STRIDED ? (uint32_t)lda * 2u : 2u, b_unit = B_STRIDED ? (uint32_t)ldb * 2u : 2u;
    const uint32_t a_step = (uint32_t)(BK * WK) * a_unit, b_step = (uint32_t)(BK * WK) * b_unit;
    const uint32_t a_end = A_STRIDED ? (uint32_t)a_srd[2] : (uint32_t)C * 2u;
    const uint32_t b_end = B_STRIDED ? (uint32_t)b_srd[2] : (uint32_t)C * 2u;
    const int slices = (C + BK - 1) / BK;
    const int KT = (slices + WK - 1) / WK;             // slices that every group walks
    const int first_rows = C - (slices - 1) * BK;      // length of slice 0
    uint32_t a_next, b_next;                           // offset of the group's next slice; the range itself: nothing there
    {
        const uint32_t c = grp == 0 ? 0u : (uint32_t)(first_rows + (grp - 1) * BK);
        a_next = c < (uint32_t)C ? c * a_unit : (uint32_t)a_srd[2];
        b_next = c < (uint32_t)C ? c * b_unit : (uint32_t)b_srd[2];
    }
    auto issue = [&](int buf, bool first) {
        const uint32_t l = ring + (uint32_t)buf * (STAGE * 2u);
#pragma unroll
        for (int it = 0; it < NA; ++it)
            dma16(a_voff[it] | (first && grp == 0 && a_c[it] >= first_rows ? OUTSIDE : 0u), a_srd, a_next,
                  l + (uint32_t)(wi * NA + it) * 1024u);
#pragma unroll
        for (int it = 0; it < NB; ++it)
            dma16(b_voff[it] | (first && grp == 0 && b_c[it] >= first_rows ? OUTSIDE : 0u), b_srd, b_next,
                  l + AH * 2u + (uint32_t)(wi * NB + it) * 1024u);
        // slice 0 is the short one: the next slice of its group starts BK - first_rows earlier than a whole step away
        const uint32_t back = first && grp == 0 ? (uint32_t)(BK - first_rows) : 0u;
        a_next += a_step - back * a_unit;
        b_next += b_step - back * b_unit;
        if (a_next >= a_end) a_next = (uint32_t)a_srd[2];
        if (b_next >= b_end) b_next = (uint32_t)b_srd[2];
    };

    // ---- fragment reads
    const int g4 = lane >> 4, j16 = lane & 15;
    const int mhalf = g4 & 1, kh = g4 >> 1, rib = j16 >> 2, piece = j16 & 3;
    const int l32 = lane & 31, lh = lane >> 5;
    int a_rd, b_rd;
    if constexpr (A_STRIDED) {
        a_rd = (8 * kh + rib) * TM + (((wm * 8 + 2 * mhalf + (piece >> 1)) ^ swz_row<TM>(rib)) * 8) + (piece & 1) * 4;
    } else {
        const int ml = wm * 64 + l32;
        a_rd = ml * BK + ((lh ^ swz_c(ml)) * 8);
    }
    if constexpr (B_STRIDED) {
        b_rd = (8 * kh + rib) * TN + (((wn * 8 + 2 * mhalf + (piece >> 1)) ^ swz_row<TN>(rib)) * 8) + (piece & 1) * 4;
    } else {
        const int nl = wn * 64 + l32;
        b_rd = nl * BK + ((lh ^ swz_c(nl)) * 8);
    }
    const uint16_t* ring_p = smem + grp * (NS * STAGE);
    auto read_a = [&](int buf, int kk, int i) -> half8 {
        if constexpr (A_STRIDED) {
            const uint16_t* p = ring_p + buf * STAGE + ((a_rd ^ (i << 5)) + kk * 16 * TM);
            return read_tr8(p, p + 4 * TM);
        } else {
            return *reinterpret_cast<const half8*>(ring_p + buf * STAGE + ((a_rd ^ (kk << 4)) + i * 32 * BK));
        }
    };
    auto read_b = [&](int buf, int kk, int j) -> half8 {
        const uint16_t* bs = ring_p + buf * STAGE + AH;
        if constexpr (B_STRIDED) {
            const uint16_t* p = bs + ((b_rd ^ (j << 5)) + kk * 16 * TN);
            return read_tr8(p, p + 4 * TN);
        } else {
            return *reinterpret_cast<const half8*>(bs + ((b_rd ^ (kk << 4)) + j * 32 * BK));
        }
    };
    struct Frags {
        half8 a[2][2], b[2][2];      // [half of the slice][32 rows / columns]
    };
    constexpr int READS = 4 * (A_STRIDED ? 2 : 1) + 4 * (B_STRIDED ? 2 : 1);
    auto read_all = [&](Frags& f, int buf) {
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            f.a[kk][0] = read_a(buf, kk, 0);
            f.b[kk][0] = read_b(buf, kk, 0);
            f.b[kk][1] = read_b(buf, kk, 1);
            f.a[kk][1] = read_a(buf, kk, 1);
        }
    };

    floatx16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // Wait for the slice after the one about to be multiplied (`young` younger slices may be in flight) and for this wave's
    // own fragment reads; behind the barrier both hold for all waves that share the ring.
    auto arrive = [&] {
        constexpr int young = (NS - 2) * (NA + NB);
        if constexpr (PRIVATE) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(young) : "memory");
        else asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(young) : "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    auto step = [&](const Frags& use, Frags& load, int u) {
        arrive();                                   // stage u + 1 is here, stage u is in registers everywhere
        issue(u, false);
        __builtin_amdgcn_sched_barrier(0);
        read_all(load, (u + 1) % NS);
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(use.a[kk][i], use.b[kk][j], acc[i][j], 0, 0, 0);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);             // one MFMA, then its share of the LDS reads
            __builtin_amdgcn_sched_group_barrier(0x100, READS / 8, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };

#pragma unroll
    for (int st = 0; st < NS; ++st) issue(st, st == 0);
    // slice 0 has landed: NS - 1 younger ones in flight
    if constexpr (PRIVATE) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 1) * (NA + NB)) : "memory");
    else asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((NS - 1) * (NA + NB)) : "memory");
    __builtin_amdgcn_sched_barrier(0);
    Frags f0, f1;
    read_all(f0, 0);
    for (int kt = 0; kt < KT;) {                     // slices from KT on are zeros
        static_for_pairs<NS == 3 ? 3 : 2>([&](auto pair) {
            constexpr int u = 2 * decltype(pair)::value;
            if (kt >= KT) return;
            step(f0, f1, u % NS);
            step(f1, f0, (u + 1) % NS);
            kt += 2;
        });
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");      // the LDS is free
    __builtin_amdgcn_sched_barrier(0);

    // ---- epilogue.  The four 32 x 32 blocks of a wave's 64 x 64 sub-tile are shared out over the WK groups: group k adds
    // the partial sums of blocks k * PER .. and writes them out.  Block b is (i, j) = (b & 1, b >> 1).
    constexpr int PER = 4 / WK;
    constexpr bool RMW = (EPI == EPI_UPDATE || EPI == EPI_CLIPV);
    const uint16_t* old_base = (EPI == EPI_UPDATE && g.Res != nullptr) ? g.Res : g.Out;
    auto m_at = [&](int b, int a) { return wm * 64 + 32 * (b & 1) + 16 * a + 8 * lh; };
    auto n_at = [&](int b) { return wn * 64 + 32 * (b >> 1) + l32; };
    half8 old[PER][2];
    if constexpr (RMW) {                             // the old values travel while the partial sums are exchanged
#pragma unroll
        for (int p = 0; p < PER; ++p)
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                const int b = grp * PER + p;
                if (n_at(b) < n_left && m_at(b, a) < m_left)
                    old[p][a] = *reinterpret_cast<const half8*>(old_base + (n0 + n_at(b)) * ldo + m0 + m_at(b, a));
            }
    }
    typedef float floatx4 __attribute__((ext_vector_type(4)));
    float* xch = reinterpret_cast<float*>(smem);     // [source wave][block][quarter][lane][4]
    floatx16 sum[PER];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        if (b / PER != grp) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<floatx4*>(xch + (((wave * 4 + b) * 4 + q) * 64 + lane) * 4) =
                    floatx4{acc[b & 1][b >> 1][4 * q], acc[b & 1][b >> 1][4 * q + 1], acc[b & 1][b >> 1][4 * q + 2],
                            acc[b & 1][b >> 1][4 * q + 3]};
        } else {
            sum[b % PER] = acc[b & 1][b >> 1];
        }
    }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < PER; ++p)
#pragma unroll
        for (int k = 1; k < WK; ++k) {
            const int src = ((grp + k) % WK) * (WM * WN) + wi;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const floatx4 v = *reinterpret_cast<const floatx4*>(xch + (((src * 4 + grp * PER + p) * 4 + q) * 64 + lane) * 4);
#pragma unroll
                for (int e = 0; e < 4; ++e) sum[p][4 * q + e] += v[e];
            }
        }

    if constexpr (EPI == EPI_SQNORM) {
        float sq = 0.f;
        uint32_t worst = 0u;
#pragma unroll
        for (int p = 0; p < PER; ++p)
#pragma unroll
            for (int r = 0; r < 16; ++r) {           // elements outside the tensor are zero
                const float v = sum[p][r];
                sq = fmaf(v, v, sq);
                const uint32_t mag = __float_as_uint(v) & 0x7fffffffu;
                worst = mag > worst ? mag : worst;
            }
        sq = wave_sum(sq);
        const bool bad = __any(worst >= 0x7f800000u);
        __syncthreads();                             // the exchange area is free
        if (lane == 0) {
            xch[wave] = sq;
            reinterpret_cast<int*>(smem)[16 + wave] = bad ? 1 : 0;
        }
        __syncthreads();
        if (tid == 0) {
            float total = 0.f;
            int any_bad = 0;
#pragma unroll
            for (int k = 0; k < WM * WN * WK; ++k) {
                total += xch[k];
                any_bad |= reinterpret_cast<int*>(smem)[16 + k];
            }
            atomicAdd(ga.acc, (double)total);
            if (g.flag_out != nullptr && any_bad) atomicOr(g.flag_out, 1);
        }
    } else {
        typedef uint32_t u32x2v __attribute__((ext_vector_type(2)));
        const float s = ga.s_dev != nullptr ? *ga.s_dev : ga.s;
        bool bad = false;
#pragma unroll
        for (int p = 0; p < PER; ++p)
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                // lanes l and l + 32 hold the two 4-row halves of every 8 rows: after the swap a lane owns 8 consecutive m
                float v[8];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const u32x2v sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(sum[p][8 * a + e]),
                                                                       __float_as_uint(sum[p][8 * a + 4 + e]), false, false);
                    v[e] = __uint_as_float(sw[0]);
                    v[4 + e] = __uint_as_float(sw[1]);
                }
                const int b = grp * PER + p;
                if (n_at(b) >= n_left || m_at(b, a) >= m_left) continue;
                half8 out;
                if constexpr (EPI == EPI_UPDATE) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) out[e] = (_Float16)fmaf(-s, v[e], (float)old[p][a][e]);
                } else if constexpr (EPI == EPI_CLIPV) {
                    // clip by value (section 3.3.1): a non-finite element raises the flag and leaves its weight alone
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float gq = v[e] * ga.inv_s;
                        const bool fin = (__float_as_uint(gq) & 0x7f800000u) != 0x7f800000u;
                        const float gc = fminf(fmaxf(gq, -ga.clipv), ga.clipv);
                        out[e] = fin ? (_Float16)fmaf(-ga.lr, gc, (float)old[p][a][e]) : old[p][a][e];
                        bad |= !fin;
                    }
                } else {
#pragma unroll
                    for (int e = 0; e < 8; ++e) out[e] = (_Float16)v[e];
                }
                *reinterpret_cast<half8*>(g.Out + (n0 + n_at(b)) * ldo + m0 + m_at(b, a)) = out;
            }
        if constexpr (EPI == EPI_CLIPV) {
            if (__any(bad) && lane == 0 && g.flag_out != nullptr) atomicOr(g.flag_out, 1);
        }
    }
}

// ---- host side ----------------------------------------------------------------------------

template <int WM, int WN, int WK, bool B_STRIDED, int EPI, bool A_STRIDED>
static hipError_t launch_ksplit_tile(const GemmArgs* list, int n, hipStream_t st) {
    constexpr int LDS = ksplit::stages(WM, WN, WK) * WK * (64 * WM + 64 * WN) * dma::BK * 2;
    static_assert(LDS >= WM * WN * WK * 4 * 4096, "the partial sums are exchanged where the stages were");
    auto kern = lomo_contract_ksplit_kernel<WM, WN, WK, B_STRIDED, EPI, A_STRIDED>;
    // thread-safe one-time set-up (initialisation of a function-local static)
    static const hipError_t cfg0 = allow_dynamic_lds(kern, LDS);
    if (cfg0 != hipSuccess) return cfg0;
    for (int first = 0; first < n; first += dma::MAX_GROUP) {
        dma::GroupArgs ga{};
        dma::fill_group(ga, list + first, n - first < dma::MAX_GROUP ? n - first : dma::MAX_GROUP, 64 * WM, 64 * WN);
        hipError_t e = launch_timed(list[first].family, kern, dim3((unsigned)ga.total_tiles), dim3(64 * WM * WN * WK),
                                    (size_t)LDS, st, ga);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <bool B_STRIDED, int EPI, bool A_STRIDED>
hipError_t launch_ksplit_group(const GemmArgs* list, int n, int tile, hipStream_t st) {
    switch (tile) {
        case TILE_128: return launch_ksplit_tile<2, 2, 2, B_STRIDED, EPI, A_STRIDED>(list, n, st);
        case TILE_128_64: return launch_ksplit_tile<2, 1, 4, B_STRIDED, EPI, A_STRIDED>(list, n, st);
        default: return launch_ksplit_tile<1, 1, 4, B_STRIDED, EPI, A_STRIDED>(list, n, st);
    }
}

template hipError_t launch_ksplit_group<true, EPI_UPDATE, true>(const GemmArgs*, int, int, hipStream_t);
template hipError_t launch_ksplit_group<true, EPI_CLIPV, true>(const GemmArgs*, int, int, hipStream_t);
template hipError_t launch_ksplit_group<true, EPI_SQNORM, true>(const GemmArgs*, int, int, hipStream_t);
template hipError_t launch_ksplit_group<false, EPI_STORE, true>(const GemmArgs*, int, int, hipStream_t);
template hipError_t launch_ksplit_group<false, EPI_STORE, false>(const GemmArgs*, int, int, hipStream_t);
template hipError_t launch_ksplit_group<false, EPI_UPDATE, false>(const GemmArgs*, int, int, hipStream_t);

}  // namespace lomo
