// Squared gradient norm of a linear tensor without forming the gradient: Gram route (gfx950).
//
// The norm pass of paper section 3.3.1 needs ||G||_F^2 for G = dY^T X (scaled gradient, [N x K]).
// With x_t, dy_t the rows of X [T x K] and dY [T x N]:
//
//     ||G||_F^2 = sum_{t,t'} (x_t . x_t') (dy_t . dy_t') = sum_{t,t'} P[t,t'] Q[t,t'],
//     P = X X^T,  Q = dY dY^T   (both T x T, symmetric),
//
// so only the lower triangle is needed: sum_t P_tt Q_tt + 2 sum_{t > t'} P Q.  That is
// T^2 (K + N) flop instead of 2 T N K, which is less whenever T < 2 N K / (N + K) -- the case
// for the wide tensors of large models at moderate token counts.  The overflow flag keeps its
// meaning: some element of G is non-finite exactly when some input is inf/NaN, and then the
// diagonal entry of P or Q in that row is non-finite.
//
// Accuracy: P and Q are accumulated in fp32 on the MFMA units; the error of the result is of the
// order 1e-6 * sum_{t,t'} |P Q|, i.e. relative to the per-token gradient energy rather than to
// ||G||^2 itself.  When the per-token gradients nearly cancel in the sum over tokens this is less
// accurate than the direct kernel, which is why the direct route is the default.
//
// Kernel: one persistent workgroup per CU walks a list of 256 x 128 tiles of the triangle of up to
// MAX_GROUP tensors.  A tile runs K/64 slots of X rows into the P accumulators and N/64 slots of
// dY rows into the Q accumulators as one continuous direct-to-LDS pipeline (both
// operands are contraction-contiguous, so LDS reads are plain 16-byte reads), then multiplies the
// two accumulator sets element by element, applies the triangle weights and adds one double.
//
// A slot is 64 contraction indices: 128 bytes of a row, whole cache lines, where slices of 32 asked for every line twice and met
// at a barrier twice as often.  Three slots of 48 KiB rotate; a slot is walked in four steps of 16 indices, the fragments of the
// next step are read while the current one is multiplied; after the third step the slot's memory is loaded again, with the slot
// after the next two, in twelve instructions per wave over the next three steps, so that a load has more than a slot's
// time to land.  Measured, us, norm pass by this route, slices of 32 in four stages -> slots: one layer of width 8192 at 2048 tokens
// 782 -> 649 (1136 TFLOP/s of the tiles' products; the direct route 2670), at 4096 tokens 3170 -> 2459, two 5120 wide at 1024 tokens 469 -> 380,
// four 4096 wide at 512 tokens 244 -> 196.
#include "lomo_gemm_persistent.h"

#include <algorithm>

namespace lomo {
namespace gram {

constexpr int BM = 256, BN = 128, BK = 64, NS = 3;
constexpr int A_HALVES = BM * BK, B_HALVES = BN * BK, SLOT_HALVES = A_HALVES + B_HALVES;
constexpr int LDS_BYTES = NS * SLOT_HALVES * 2 + 256;
constexpr int LOADS = 12;      // instructions of a wave per slot: eight of A, four of B, eight rows each
constexpr int MAX_GROUP = 40;
constexpr int BAND = 4;   // tile rows per band: the 32 tiles an XCD holds at once form a 4 x 8 block

struct GramTensor {
    const uint16_t* X;
    const uint16_t* dY;
    int32_t* flag_out;
    int K, N, tiles_m, tile_begin;
};

struct GroupArgs {
    double* acc;
    int n, total_tiles;
    GramTensor t[MAX_GROUP];
};

// 16-byte chunk c of row r sits at position c ^ swz(r): sixteen rows read at one chunk fall on all 64 banks.
__device__ __forceinline__ int swz(int r) { return (r >> 1) & 7; }

__device__ __forceinline__ void dma16(uint32_t voff, const void* base, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :: "v"(voff), "s"(base), "s"(lds_addr) : "memory", "m0");
}

// Tile number t of the lower triangle (tile row bi covers tokens [256 bi, 256 bi + 256), tile column bj
// covers [128 bj, 128 bj + 128); valid when bj <= 2 bi + 1).  Bands of BAND tile rows, column-major
// inside a band.  The host guarantees t < tm (tm + 1).
__device__ __forceinline__ void locate(int t, int tm, int& bi, int& bj) {
    bi = 0;
    bj = 0;
    for (int r0 = 0; r0 < tm; r0 += BAND) {
        const int R = (tm - r0 < BAND) ? (tm - r0) : BAND;
        const int r1 = r0 + R - 1;
        const int cnt = R * (r0 + r1 + 2);          // sum over rows of (2 row + 2)
        if (t >= cnt) {
            t -= cnt;
            continue;
        }
        const int full = 2 * r0 + 2;                // columns that reach every row of the band
        if (t < R * full) {
            bj = t / R;
            bi = r0 + t % R;
            return;
        }
        t -= R * full;
        for (int c = full; c <= 2 * r1 + 1; ++c) {
            const int lo = c >> 1;                  // first row that reaches column c
            const int n = r1 - lo + 1;
            if (t < n) {
                bj = c;
                bi = lo + t;
                return;
            }
            t -= n;
        }
        return;
    }
}

}  // namespace gram

__global__ __launch_bounds__(NT) void lomo_gram_sqnorm_kernel(gram::GroupArgs ga) {
    using namespace gram;
    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave & 1, wn = wave >> 1;
    const int l32 = lane & 31, lh = lane >> 5;
    const int G = gridDim.x;

    const uint32_t lds0 = (uint32_t)(uintptr_t)smem;
    float* red_scratch = reinterpret_cast<float*>(smem + NS * SLOT_HALVES);

    // ---- fragment read offsets (halves)
    const int arow = wm * (BM / 2) + l32, brow = wn * (BN / 2) + l32;
    const int a_rd = arow * BK + ((lh ^ swz(arow)) * 8);
    const int b_rd = A_HALVES + brow * BK + ((lh ^ swz(brow)) * 8);

    // ---- per-tile state of the loads: phase P reads X, phase Q reads dY.  A wave instruction fetches eight rows of 128 bytes;
    // lane L takes row L / 8 and, of its chunks, the one that the swizzle assigns to LDS position L % 8.  The swizzle depends on
    // the row modulo 16: one lane offset per phase for even instructions, one for odd, and the row block goes into the base.
    uint32_t voffP[2] = {0, 0}, voffQ[2] = {0, 0};
    const uint16_t *paP = nullptr, *pbP = nullptr, *paQ = nullptr, *pbQ = nullptr;
    int KTP = 0, KT = 0, ldP = 0, ldQ = 0;

    auto setup = [&](int w, int& tensor, int& bi, int& bj) {
        int k = 0;
        while (k + 1 < ga.n && w >= ga.t[k + 1].tile_begin) ++k;
        const GramTensor& T = ga.t[k];
        locate(w - T.tile_begin, T.tiles_m, bi, bj);
        tensor = k;
        const int n = lane >> 3, cp = lane & 7;
#pragma unroll
        for (int odd = 0; odd < 2; ++odd) {
            const uint32_t c = (uint32_t)((cp ^ swz(8 * odd + n)) * 8);
            voffP[odd] = ((uint32_t)n * (uint32_t)T.K + c) * 2u;
            voffQ[odd] = ((uint32_t)n * (uint32_t)T.N + c) * 2u;
        }
        ldP = T.K;
        ldQ = T.N;
        // this wave's rows: 64 of the tile's rows, 32 of its columns
        paP = T.X + ((int64_t)bi * BM + wave * 64) * T.K;
        pbP = T.X + ((int64_t)bj * BN + wave * 32) * T.K;
        paQ = T.dY + ((int64_t)bi * BM + wave * 64) * T.N;
        pbQ = T.dY + ((int64_t)bj * BN + wave * 32) * T.N;
        KTP = T.K / BK;
        KT = KTP + T.N / BK;
    };

    // The slot being requested: its place in LDS (bytes), its rows, the distance of eight rows.
    uint32_t to = 0, v0 = 0, v1 = 0;
    const uint16_t *fa = nullptr, *fb = nullptr;
    int64_t eight = 0;
    auto request = [&](int slot, int ring) {      // slots past the end re-read the last one
        const int s = slot < KT ? slot : KT - 1;
        const bool q = s >= KTP;
        const int at = (q ? s - KTP : s) * BK;
        to = lds0 + (uint32_t)ring * (SLOT_HALVES * 2u);
        fa = (q ? paQ : paP) + at;
        fb = (q ? pbQ : pbP) + at;
        eight = 8 * (int64_t)(q ? ldQ : ldP);
        v0 = q ? voffQ[0] : voffP[0];
        v1 = q ? voffQ[1] : voffP[1];
    };
    auto load = [&](int n) {
        if (n < 8) {
            dma16(n & 1 ? v1 : v0, fa, to + (uint32_t)(wave * 8 + n) * 1024u);
            fa += eight;
        } else {
            dma16(n & 1 ? v1 : v0, fb, to + (uint32_t)(A_HALVES * 2) + (uint32_t)(wave * 4 + n - 8) * 1024u);
            fb += eight;
        }
    };
    // Slots 0 and 1, and the first four loads of slot 2.
    auto issue_prologue = [&] {
#pragma unroll
        for (int st = 0; st < 3; ++st) {
            request(st, st);
#pragma unroll
            for (int n = 0; n < (st < 2 ? LOADS : 4); ++n) load(n);
        }
    };

    auto read_a = [&](half8 (&a)[4], int ring, int kk, int i) {
        a[i] = *reinterpret_cast<const half8*>(smem + ring * SLOT_HALVES + ((a_rd ^ (kk << 4)) + i * 32 * BK));
    };
    auto read_b = [&](half8 (&b)[2], int ring, int kk, int j) {
        b[j] = *reinterpret_cast<const half8*>(smem + ring * SLOT_HALVES + ((b_rd ^ (kk << 4)) + j * 32 * BK));
    };
    // EARLY packs the six fragments into the first three groups so that every read of the slot has
    // completed when the step ends at the barrier that releases it.
    auto read_group = [&](half8 (&a)[4], half8 (&b)[2], int ring, int kk, int q, bool early) {
        if (early) {
            if (q == 0) { read_a(a, ring, kk, 0); read_b(b, ring, kk, 0); read_b(b, ring, kk, 1); }
            if (q == 1) { read_a(a, ring, kk, 1); read_a(a, ring, kk, 2); }
            if (q == 2) { read_a(a, ring, kk, 3); }
        } else {
            if (q == 0) { read_a(a, ring, kk, 0); read_b(b, ring, kk, 0); }
            if (q == 1) { read_b(b, ring, kk, 1); read_a(a, ring, kk, 1); }
            if (q == 2) { read_a(a, ring, kk, 2); }
            if (q == 3) { read_a(a, ring, kk, 3); }
        }
    };
    constexpr int READS_EARLY[4] = {3, 2, 1, 0};
    constexpr int READS_EVEN[4] = {2, 2, 1, 1};

    floatx16 accP[4][2], accQ[4][2];
    auto zero_acc = [&] {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    accP[i][j][r] = 0.f;
                    accQ[i][j][r] = 0.f;
                }
    };

    // One step of 16 indices: 8 MFMAs on (ua, ub) in four groups of two; each group is preceded by the reads of one
    // fragment group of the next step and, where the step loads (first >= 0), followed by one direct-to-LDS load.
    auto step = [&](floatx16 (&acc)[4][2], const half8 (&ua)[4], const half8 (&ub)[2], half8 (&la)[4],
                    half8 (&lb)[2], int ring, int kk, bool early, int first) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            read_group(la, lb, ring, kk, q, early);
#pragma unroll
            for (int j = 0; j < 2; ++j)
                acc[q][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ua[q], ub[j], acc[q][j], 0, 0, 0);
            {
                int left = early ? READS_EARLY[q] : READS_EVEN[q];
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const int now = (left + (1 - j)) / (2 - j);
                    if (now == 1) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // DS reads
                    if (now == 2) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                 // one MFMA
                    left -= now;
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            if (first >= 0) load(first + q);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    half8 fa0[4], fb0[2], fa1[4], fb1[2];
    int ring = 0;      // place of the current slot
    // Slot number s accumulated into `acc`.
    auto one_slot = [&](floatx16 (&acc)[4][2], int s) {
        const int next = ring == NS - 1 ? 0 : ring + 1;
        step(acc, fa0, fb0, fa1, fb1, ring, 1, false, 4);      // the rest of slot s + 2
        step(acc, fa1, fb1, fa0, fb0, ring, 2, false, 8);
        step(acc, fa0, fb0, fa1, fb1, ring, 3, true, -1);
        // slot s + 1 has landed (slot s + 2 may still fly); nobody reads slot s any more
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(LOADS) : "memory");
        __builtin_amdgcn_sched_barrier(0);
        request(s + 3, ring);
        step(acc, fa1, fb1, fa0, fb0, next, 0, false, 0);
        ring = next;
    };

    int round = 0;
    int w = dma::round_tile(round, G, ga.total_tiles, true);
    if (w >= ga.total_tiles) return;   // grid <= total_tiles: cannot happen; nothing was issued yet
    int tensor, bi, bj;
    setup(w, tensor, bi, bj);
    issue_prologue();
    zero_acc();

    while (true) {
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        ring = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) read_group(fa0, fb0, 0, 0, q, false);

        for (int s = 0; s < KTP; ++s) one_slot(accP, s);
        for (int s = KTP; s < KT; ++s) one_slot(accQ, s);
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");

        int32_t* const flag_out = ga.t[tensor].flag_out;
        const int ebi = bi, ebj = bj;

        w = dma::round_tile(++round, G, ga.total_tiles, true);
        const bool more = w < ga.total_tiles;
        if (more) {
            setup(w, tensor, bi, bj);
            issue_prologue();
        }

        // ---- sum of weight * P * Q over the tile.  Lane (l32, lh) holds, in register 4 q4 + e of MFMA
        // block (i, j), the pair (row 32 i + 8 q4 + 4 lh + e of the wave's rows, column 32 j + l32).
        const bool below = ebj < 2 * ebi;     // every pair of the tile has t > t'
        float sum = 0.f;
        uint32_t worst = 0u;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const float p = accP[i][j][r], qv = accQ[i][j][r];
                    const uint32_t mp = __float_as_uint(p) & 0x7fffffffu, mq = __float_as_uint(qv) & 0x7fffffffu;
                    worst = mp > worst ? mp : worst;
                    worst = mq > worst ? mq : worst;
                    float wgt = 2.f;
                    if (!below) {
                        const int t = ebi * BM + wm * (BM / 2) + 32 * i + 8 * (r >> 2) + 4 * lh + (r & 3);
                        const int tp = ebj * BN + wn * (BN / 2) + 32 * j + l32;
                        wgt = t > tp ? 2.f : (t == tp ? 1.f : 0.f);
                    }
                    sum = fmaf(wgt * p, qv, sum);
                }
        sum = wave_sum(sum);
        const bool bad = __any(worst >= 0x7f800000u);
        int* redflag = reinterpret_cast<int*>(red_scratch) + 8;
        if (lane == 0) {
            red_scratch[wave] = sum;
            redflag[wave] = bad ? 1 : 0;
        }
        __syncthreads();
        if (tid == 0) {
            const double total = ((double)red_scratch[0] + (double)red_scratch[1]) +
                                 ((double)red_scratch[2] + (double)red_scratch[3]);
            atomicAdd(ga.acc, total);
            if (flag_out != nullptr && (redflag[0] | redflag[1] | redflag[2] | redflag[3])) atomicOr(flag_out, 1);
        }
        if (!more) break;
        zero_acc();
    }
}

// ---- host side ----------------------------------------------------------------------------

// `a` is a norm-pass contraction (A = X [C x M], B = dY [C x Nn], dense rows).
bool gram_eligible(const GemmArgs& a) {
    using namespace gram;
    return a.C >= BM && a.C % BM == 0 && a.M >= 2 * BK && a.M % (2 * BK) == 0 && a.Nn >= 2 * BK &&
           a.Nn % (2 * BK) == 0 && a.lda == a.M && a.ldb == a.Nn && a.C <= (1 << 20) && a.M < (1 << 22) &&
           a.Nn < (1 << 22) && (a.C / BM) * (a.C / BM + 1) < (1 << 24);
}

// Estimated cost in units of one 256 x 256 x 32 slice on one CU.  32 indices of a 256 x 128 tile are half the arithmetic of that;
// a wave tile of 128 x 64 reads 1.5 times the operand bytes per flop of the direct kernel's 128 x 128.  Measured 0.60; the
// line stays at the 0.73 of the kernel before, so that no tensor leaves the direct route, which is the more accurate one, for
// a gain of a few per cent.
constexpr double kGramSlice = 0.73;
double gram_cost(const GemmArgs& a) {
    const double tm = (double)(a.C / gram::BM);
    return kGramSlice * tm * (tm + 1.0) * (double)(a.M + a.Nn) / 32.0;
}
double direct_cost(const GemmArgs& a) {
    return (double)((a.M + 255) / 256) * (double)((a.Nn + 255) / 256) * (double)a.C / 32.0;
}

// The order launch_gram_group runs its tensors in: longest tiles first, so that the static walk ends on the short ones.
static void gram_launch_order(std::vector<GemmArgs>& v) {
    std::stable_sort(v.begin(), v.end(), [](const GemmArgs& x, const GemmArgs& y) { return x.M + x.Nn > y.M + y.Nn; });
}

// When the Gram launches of these tensors finish, in the same units: workgroup p of a launch is taken to walk tiles p, p + G, ...,
// every tile of a tensor costs the same, and a launch ends with its busiest workgroup.  An approximation: the kernel deals the last round,
// whose tiles are the shortest, out to other workgroups.
// A few hundred long tiles on 256 CUs end far later than (total work) / (number of CUs) says.
static double gram_finish_time(std::vector<GemmArgs> v) {
    gram_launch_order(v);
    const int cus = cu_count();
    double total = 0.0;
    std::vector<double> load;
    for (size_t first = 0; first < v.size(); first += gram::MAX_GROUP) {
        const size_t cnt = v.size() - first < (size_t)gram::MAX_GROUP ? v.size() - first : (size_t)gram::MAX_GROUP;
        int64_t tiles = 0;
        for (size_t i = 0; i < cnt; ++i) {
            const int64_t tm = v[first + i].C / gram::BM;
            tiles += tm * (tm + 1);
        }
        const int64_t G = tiles < cus ? tiles : cus;
        load.assign((size_t)G, 0.0);
        int64_t w = 0;
        for (size_t i = 0; i < cnt; ++i) {
            const GemmArgs& a = v[first + i];
            const int64_t tm = a.C / gram::BM, n = tm * (tm + 1);
            const double tile = kGramSlice * (double)(a.M + a.Nn) / 32.0;
            for (int64_t k = 0; k < n; ++k, ++w) load[(size_t)(w % G)] += tile;
        }
        double longest = 0.0;
        for (double l : load) longest = l > longest ? l : longest;
        total += longest;
    }
    return total;
}

void choose_norm_route(int mode, const std::vector<GemmArgs>& all, std::vector<GemmArgs>& gram, std::vector<GemmArgs>& direct) {
    for (const GemmArgs& a : all) {
        const bool g = mode != LOMO_NORM_DIRECT && gram_eligible(a) && (mode == LOMO_NORM_GRAM || gram_cost(a) < direct_cost(a));
        (g ? gram : direct).push_back(a);
    }
    if (mode != LOMO_NORM_AUTO || gram.empty()) return;
    // Compare finishing times, not total work: the direct kernels' tiles are short and many (their share of the chip is
    // their work), the Gram tiles are long and few.
    double work_d = 0.0;
    for (const GemmArgs& a : gram) work_d += direct_cost(a);
    if (gram_finish_time(gram) >= work_d / (double)cu_count()) {
        direct.insert(direct.end(), gram.begin(), gram.end());
        gram.clear();
    }
}

hipError_t launch_gram_group(const GemmArgs* list, int n, hipStream_t st) {
    using namespace gram;
    auto kern = lomo_gram_sqnorm_kernel;
    // thread-safe one-time set-up (initialisation of a function-local static)
    static const hipError_t cfg0 = allow_dynamic_lds(kern, LDS_BYTES);
    if (cfg0 != hipSuccess) return cfg0;
    // Longest tiles first: the static round-robin then ends on the short ones.
    std::vector<GemmArgs> order(list, list + n);
    gram_launch_order(order);
    list = order.data();
    for (int first = 0; first < n; first += MAX_GROUP) {
        const int cnt = (n - first < MAX_GROUP) ? (n - first) : MAX_GROUP;
        GroupArgs ga{};
        ga.acc = list[first].acc;
        ga.n = cnt;
        int tiles = 0;
        for (int i = 0; i < cnt; ++i) {
            const GemmArgs& a = list[first + i];
            GramTensor& t = ga.t[i];
            t.X = a.A; t.dY = a.B; t.flag_out = a.flag_out;
            t.K = (int)a.M; t.N = (int)a.Nn;
            t.tiles_m = (int)(a.C / BM);
            t.tile_begin = tiles;
            tiles += t.tiles_m * (t.tiles_m + 1);
        }
        ga.total_tiles = tiles;
        const int grid = tiles < cu_count() ? tiles : cu_count();
        hipError_t e = launch_timed(LOMO_KERNEL_GRAM_SQNORM, kern, dim3((unsigned)grid), dim3(NT), (size_t)LDS_BYTES, st, ga);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace lomo
