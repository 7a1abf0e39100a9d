// MFMA contraction kernel of the LOMO hot path for any shape, gfx950 (CDNA4, wave64), and the choice between the kernels.
// What the direct-to-LDS kernels address with 32-bit offsets goes to them; this one serves rows too long for that (from 7 million
// elements on).
//
// One kernel template serves the three dense steps of a linear tensor:
//   * fused wgrad + SGD update (paper section 3.2, Algorithm 1: theta <- theta - lr * g, the
//     gradient never leaves the accumulators; section 3.3.2: update arithmetic in fp32),
//   * wgrad squared norm + overflow detection (section 3.3.1 / 3.3.2, first backward pass),
//   * dgrad dX = dY W for the continuing back-propagation.
//
// Layout.  The output tile is Out[n][m] with m contiguous in memory.  Operand "A" supplies the m
// index and is always stored with the contraction index as its slow dimension (X[t][k] for wgrad,
// W[n][k] for dgrad), so it has to be transposed on its way to the matrix cores: a lane fetches
// dwords (two neighbouring m) from eight consecutive contraction rows, repacks them with byte
// permutes into two 16-byte runs along the contraction, and stores those to LDS in [m][c] order.
// Operand "B" supplies n and is transposed the same way (dY[t][n] for wgrad) or copied straight
// (dY[t][n] for dgrad, where n_out is the contraction).  MFMA 32x32x16 f16 then reads 16-byte
// fragments from LDS rows of 80 bytes (64 + 16 pad), which makes ds_read_b128 conflict free.
// With A on the MFMA row side, each lane's four consecutive accumulator registers are four
// consecutive m, i.e. an 8-byte run of W / dX: the read-modify-write epilogue is vectorised.
#include "lomo_gemm_common.h"
#include "lomo_gemm_persistent.h"

#include <stdlib.h>

#include <algorithm>
#include <cmath>
#include <new>

namespace lomo {

constexpr int BK = 32;         // contraction slice per pipeline stage
constexpr int LROW = BK + 8;   // halves per LDS row

// ---- global -> registers ------------------------------------------------------------------

// Contraction-strided operand: tile of BK rows x BX columns starting at `base` (row stride ld).
// Item = (column pair p, row octet q): eight dword loads down the rows.
template <int BX, bool GUARD>
__device__ __forceinline__ void load_strided(const uint16_t* __restrict__ base, int64_t ld, int c_rem, int x_rem,
                                             uint32_t (&r)[BX / 128][8], int tid) {
#pragma unroll
    for (int it = 0; it < BX / 128; ++it) {
        const int item = tid + it * NT;
        const int p = item % (BX / 2);
        const int q = item / (BX / 2);
        const uint16_t* src = base + (int64_t)(8 * q) * ld + 2 * p;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (!GUARD || (8 * q + i < c_rem && 2 * p < x_rem))
                r[it][i] = *reinterpret_cast<const uint32_t*>(src + (int64_t)i * ld);
            else
                r[it][i] = 0u;
        }
    }
}

template <int BX>
__device__ __forceinline__ void store_strided(uint16_t* __restrict__ lds, const uint32_t (&r)[BX / 128][8], int tid) {
#pragma unroll
    for (int it = 0; it < BX / 128; ++it) {
        const int item = tid + it * NT;
        const int p = item % (BX / 2);
        const int q = item / (BX / 2);
        u32x4 lo, hi;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            lo[j] = __builtin_amdgcn_perm(r[it][2 * j + 1], r[it][2 * j], 0x05040100u);
            hi[j] = __builtin_amdgcn_perm(r[it][2 * j + 1], r[it][2 * j], 0x07060302u);
        }
        *reinterpret_cast<u32x4*>(lds + (2 * p) * LROW + 8 * q) = lo;
        *reinterpret_cast<u32x4*>(lds + (2 * p + 1) * LROW + 8 * q) = hi;
    }
}

// Contraction-contiguous operand: tile of BX rows x BK halves, 16-byte chunks.
template <int BX, bool GUARD>
__device__ __forceinline__ void load_contig(const uint16_t* __restrict__ base, int64_t ld, int c_rem, int x_rem,
                                            u32x4 (&r)[BX / 64], int tid) {
#pragma unroll
    for (int it = 0; it < BX / 64; ++it) {
        const int item = tid + it * NT;
        const int n = item / (BK / 8);
        const int q = item % (BK / 8);
        if (!GUARD || (n < x_rem && 8 * q < c_rem))
            r[it] = *reinterpret_cast<const u32x4*>(base + (int64_t)n * ld + 8 * q);
        else
            r[it] = u32x4{0u, 0u, 0u, 0u};
    }
}

template <int BX>
__device__ __forceinline__ void store_contig(uint16_t* __restrict__ lds, const u32x4 (&r)[BX / 64], int tid) {
#pragma unroll
    for (int it = 0; it < BX / 64; ++it) {
        const int item = tid + it * NT;
        const int n = item / (BK / 8);
        const int q = item % (BK / 8);
        *reinterpret_cast<u32x4*>(lds + n * LROW + 8 * q) = r[it];
    }
}

// ---- the kernel ---------------------------------------------------------------------------

// A_STRIDED = false serves the forward product Y = X W^T (both operands contraction-contiguous: A = W[n][k]
// supplies the m index, B = X[t][k] the n index), used to recompute activations from a checkpoint.
template <int BM, int BN, bool B_STRIDED, int EPI, bool A_STRIDED = true>
__global__ __launch_bounds__(NT) void lomo_contract_kernel(GemmArgs g) {
    constexpr int TM = BM / 64, TN = BN / 64;          // 32x32 MFMA tiles per wave
    constexpr int STAGE = (BM + BN) * LROW;            // halves per LDS stage
    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];

    if (EPI == EPI_UPDATE && g.flag_in != nullptr && *g.flag_in != 0) {
        return;   // overflow seen in pass 1: the step is dropped, W stays as it is
    }

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave & 1, wn = wave >> 1;
    const int l32 = lane & 31, lh = lane >> 5;

    const int tiles_m = (int)((g.M + BM - 1) / BM);
    const int64_t m0 = (int64_t)(blockIdx.x % tiles_m) * BM;
    const int64_t n0 = (int64_t)(blockIdx.x / tiles_m) * BN;
    const int m_rem = (int)((g.M - m0 < BM) ? (g.M - m0) : BM);
    const int n_rem = (int)((g.Nn - n0 < BN) ? (g.Nn - n0) : BN);
    const bool full_mn = (m_rem == BM) && (n_rem == BN);

    floatx16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    const uint16_t* pa = A_STRIDED ? (g.A + m0) : (g.A + m0 * g.lda);        // (c = 0, m0)
    const uint16_t* pb = B_STRIDED ? (g.B + n0) : (g.B + n0 * g.ldb);        // (c = 0, n0)
    const int64_t a_step = A_STRIDED ? (int64_t)BK * g.lda : (int64_t)BK;
    const int64_t b_step = B_STRIDED ? (int64_t)BK * g.ldb : (int64_t)BK;

    uint32_t ra[A_STRIDED ? BM / 128 : 1][8];
    u32x4 rac[A_STRIDED ? 1 : BM / 64];
    uint32_t rbs[B_STRIDED ? BN / 128 : 1][8];
    u32x4 rbc[B_STRIDED ? 1 : BN / 64];

    const int KT = (int)((g.C + BK - 1) / BK);

    auto fetch = [&](int kt) {
        const int c_rem = (int)(g.C - (int64_t)kt * BK);
        const bool guard = !full_mn || c_rem < BK;
        const uint16_t* a = pa + (int64_t)kt * a_step;
        const uint16_t* b = pb + (int64_t)kt * b_step;
        if (!guard) {
            if constexpr (A_STRIDED) load_strided<BM, false>(a, g.lda, c_rem, m_rem, ra, tid);
            else load_contig<BM, false>(a, g.lda, c_rem, m_rem, rac, tid);
            if constexpr (B_STRIDED) load_strided<BN, false>(b, g.ldb, c_rem, n_rem, rbs, tid);
            else load_contig<BN, false>(b, g.ldb, c_rem, n_rem, rbc, tid);
        } else {
            if constexpr (A_STRIDED) load_strided<BM, true>(a, g.lda, c_rem, m_rem, ra, tid);
            else load_contig<BM, true>(a, g.lda, c_rem, m_rem, rac, tid);
            if constexpr (B_STRIDED) load_strided<BN, true>(b, g.ldb, c_rem, n_rem, rbs, tid);
            else load_contig<BN, true>(b, g.ldb, c_rem, n_rem, rbc, tid);
        }
    };
    auto stash = [&](int buf) {
        uint16_t* as = smem + buf * STAGE;
        uint16_t* bs = as + BM * LROW;
        if constexpr (A_STRIDED) store_strided<BM>(as, ra, tid);
        else store_contig<BM>(as, rac, tid);
        if constexpr (B_STRIDED) store_strided<BN>(bs, rbs, tid);
        else store_contig<BN>(bs, rbc, tid);
    };

    if (KT > 0) {
        fetch(0);
        stash(0);
    }
    __syncthreads();

    for (int kt = 0; kt < KT; ++kt) {
        const bool more = kt + 1 < KT;
        if (more) fetch(kt + 1);

        const uint16_t* as = smem + (kt & 1) * STAGE + (wm * (BM / 2) + l32) * LROW + 8 * lh;
        const uint16_t* bs = smem + (kt & 1) * STAGE + BM * LROW + (wn * (BN / 2) + l32) * LROW + 8 * lh;
#pragma unroll
        for (int kk = 0; kk < BK / 16; ++kk) {
            half8 a[TM], b[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) a[i] = *reinterpret_cast<const half8*>(as + i * 32 * LROW + kk * 16);
#pragma unroll
            for (int j = 0; j < TN; ++j) b[j] = *reinterpret_cast<const half8*>(bs + j * 32 * LROW + kk * 16);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[i], b[j], acc[i][j], 0, 0, 0);
        }

        if (more) stash((kt + 1) & 1);
        __syncthreads();
    }

    epilogue<BM, BN, EPI>(acc, g, smem, m0, n0, m_rem, n_rem);
}

// ---- host side ----------------------------------------------------------------------------

template <int BM, int BN, bool B_STRIDED, int EPI, bool A_STRIDED = true>
static hipError_t launch_one(const GemmArgs& a, hipStream_t st) {
    if (a.M <= 0 || a.Nn <= 0) return hipSuccess;
    constexpr size_t lds = 2u * (BM + BN) * LROW * sizeof(uint16_t);
    auto kern = lomo_contract_kernel<BM, BN, B_STRIDED, EPI, A_STRIDED>;
    // thread-safe one-time set-up (initialisation of a function-local static)
    static const hipError_t cfg0 = allow_dynamic_lds(kern, (int)lds);
    if (cfg0 != hipSuccess) return cfg0;
    const int64_t tiles = ((a.M + BM - 1) / BM) * ((a.Nn + BN - 1) / BN);
    if (tiles > 0x7fffffff) return hipErrorInvalidValue;
    return launch_timed(a.family, kern, dim3((unsigned)tiles), dim3(NT), lds, st, a);
}

// Tile choice: 256 x 256 when that still gives every CU at least one tile, else 128 x 128.
template <bool B_STRIDED, int EPI, bool A_STRIDED>
static hipError_t launch_generic(const GemmArgs& a, hipStream_t st) {
    const int64_t big = ((a.M + 255) / 256) * ((a.Nn + 255) / 256);
    return big >= 192 ? launch_one<256, 256, B_STRIDED, EPI, A_STRIDED>(a, st)
                      : launch_one<128, 128, B_STRIDED, EPI, A_STRIDED>(a, st);
}

// LOMO_DISABLE_FAST=1 in the environment of the first call takes every contraction to the kernel of this file (testing aid).
static bool fast_enabled() {
    static const bool on = [] {
        const char* e = getenv("LOMO_DISABLE_FAST");
        return !(e && e[0] == '1');
    }();
    return on;
}

// ---- which kernel runs a tensor -----------------------------------------------------------
// Six shapes of workgroup: 256 x 256 (persistent, lomo_gemm_dma.hip and lomo_gemm_wide.hip), and in lomo_gemm_tile.hip 256 x 128,
// 128 x 128, 128 x 64, 64 x 64 and, for stored products of long contractions (above 4608 indices; below, 64 x 32 gains no more
// than 1 us), 64 x 32.  Larger tiles do more work per operand byte, smaller ones occupy more of the CUs and walk the
// contraction faster.
// The kernels of a pass run one behind the other, so what counts is the sum of their times over the whole list: tensors that
// would leave most of the chip idle alone fill each other's rounds in the persistent kernel, and one leaves it only where
// that makes the pass shorter (a long contraction with few tiles).  All kernels give the same bits, so the list a tensor
// comes in does not show in its result.
//
// A tile takes a fixed part (ramp-up and epilogue) and a part per contraction index; the latter is at least `latency` and, with
// every CU busy, `through` for each tile that a CU has.  Times in microseconds.
//   * Gradients: fitted to 270 shapes of output and contraction (128 to 8192 tokens of layers 1024 to 8192 wide and their
//     vocabularies); root mean square error 4 to 13 %, choosing by them costs 0.1 to 0.3 % on average over the best kernel of each.
//   * Stored products read weights, which come from HBM in every pass of a model larger than the Infinity Cache, and a workgroup
//     that waits for HBM takes 1.2 to 1.4 times as long per index: about 2.4 ns for each 128-byte line that its CU fetches, against
//     1.75 ns from the cache.  A ring twice as deep does not change that (128 x 64, 128 x 128, 64 x 64 and 64 x 32 tiles of 64 to 1024
//     tokens, one workgroup on a CU: all within 1 %), fewer lines per index and more CUs do.  So they are fitted to products that
//     go through 2 GiB of weights in turn, 77 shapes of 64 to 1024 tokens; there the choice is the fastest tile of each of
//     them (with the times from warm weights 2.4 % above it on average, 36 % at the worst: dX of 512 x 13824, C = 5120, 116 against 85).
//     Outside the fit they are less exact: dX of two layers 4096 wide with a vocabulary at 512 tokens is reckoned 600 in 256 x 128 tiles
//     and takes 677, while the choice before, 128 x 128 for all but the square tensors, takes 668.
//     Forward products with a residual are priced as updates, from warm weights.
//   * 256 x 128 tiles take the same time as the persistent kernel over several rounds, but more power: dX of a 13B layer at 874
//     tokens 655 us either way, while the norm and the update behind it go from 546 and 657 to 574 and 700.  `through` of 0.0166
//     instead of the fitted 0.0142 leaves such lists to the persistent kernel (the pass 1900 -> 1855 us).
// dX at C = 4096, warm, in the order of the table: 1024 x 4096 outputs 67, 47, 38, 47, 57;   2048 x 4096: 83, 73, 83, -, -;
// 4096 x 4096: 108, 130, 132, 166, 222.
// Lists, measured with all of one shape of tile against the choice by each tensor alone (dX, us): 7B layers at 1024
// tokens 1528 against 1960 for four, at 2048 tokens 2647 against 3642; 24 layers of width 1024 at 2048 tokens 1443 against
// 2077, their updates 1219 against 1826.
struct TileCost {
    int m, n, per_cu;             // tile; workgroups that a CU holds
    double fixed[3];              // by Product
    double latency[2], through[2];      // gradients; stored products, whose weights come from HBM in every pass
};
static const TileCost kTile[N_TILES] = {
    {256, 256, 1, {3.0, 10.0, 4.1}, {0.0140, 0.0174}, {0.0244, 0.0244}},
    {256, 128, 1, {7.0, 8.5, 5.2}, {0.0098, 0.0114}, {0.0158, 0.0166}},
    {128, 128, 1, {2.8, 4.2, 2.5}, {0.0057, 0.0075}, {0.0082, 0.0091}},
    {128, 64, 2, {1.9, 2.9, 3.0}, {0.0043, 0.0061}, {0.0055, 0.0062}},
    {64, 64, 2, {1.4, 2.0, 3.0}, {0.0027, 0.0046}, {0.0036, 0.0045}},
    {64, 32, 2, {1.4, 1e9, 1e9}, {0.0026, 0.0042}, {0.0034, 0.0037}},      // stored products only
};
constexpr int64_t kShort = 4608;         // contractions up to this length leave TILE_64_32 out
constexpr double kLaunch = 10.0;         // launch, ramp-up and drain
// A list leaves the persistent kernels for a gain that stands out from the error of the times: dX of a layer 5120 wide at 2100 tokens took
// 1320 us with two of its tensors in 256 x 128 tiles (0.7 % less by the table) against 1246.
constexpr double kLeave = 0.97;
constexpr size_t kGreedyShapes = 64;     // lists of more shapes than this take one of the starting choices as it is

namespace {
struct Shape {
    int64_t M, Nn, C;
    bool fixed;      // stays in the persistent kernel
    int tile = TILE_256;
    double n[N_TILES];      // tiles of each shape, of all tensors together
    Shape(int64_t m, int64_t nn, int64_t c, bool persistent_only) : M(m), Nn(nn), C(c), fixed(persistent_only) {
        for (int t = 0; t < N_TILES; ++t) n[t] = (double)((M + kTile[t].m - 1) / kTile[t].m) * (double)((Nn + kTile[t].n - 1) / kTile[t].n);
    }
};
}  // namespace

namespace {
// What a launch's time is reckoned from: its tiles, the contraction indices that they walk together, the longest contraction.
struct Sum {
    double tiles = 0.0, indices = 0.0, longest = 0.0;
    bool out = false;      // a tensor that TILE_64_32 leaves out
    void add(const Shape& s, int tile) {
        tiles += s.n[tile];
        indices += s.n[tile] * (double)s.C;
        longest = std::max(longest, (double)s.C);
        out |= tile == TILE_64_32 && s.C <= kShort;
    }
};
}  // namespace

// Time of the launches of a tile shape other than the persistent kernels'.
static double launch_time(const Sum& sum, int tile, int product, double cus) {
    if (sum.tiles == 0.0) return 0.0;
    if (sum.out) return 1e30;
    const TileCost& k = kTile[tile];
    const double per_cu = sum.tiles / cus, mean = sum.indices / sum.tiles, longest = sum.longest, f = k.fixed[product];
    const double latency = k.latency[product == PRODUCT_STORE], through = k.through[product == PRODUCT_STORE];
    // a partly filled round costs 0.7 of a full one, or what it has of it
    const double rounds = std::max(per_cu, floor(per_cu) + (per_cu > floor(per_cu) ? 0.7 : 0.0));
    const double waves = ceil(per_cu / k.per_cu);
    // the longest walk of a mixed list goes on alone when the rest is done
    const double busy = std::min(longest, mean * per_cu);
    return kLaunch + std::max(waves * f + mean * std::max(latency * waves, through * rounds),
                              f + (longest > mean ? through * busy + latency * (longest - busy) : longest * std::max(latency, 0.7 * through)));
}

static Sum sum_of(const Shape* shapes, size_t n_shapes, int tile) {
    Sum sum;
    for (size_t i = 0; i < n_shapes; ++i)
        if (shapes[i].tile == tile) sum.add(shapes[i], tile);
    return sum;
}

// Time of the launches of one tile shape; shapes come longest contraction first (the persistent launch, whose time depends on the order,
// mostly takes the caller's, which costs as much or less).
static double launch_time(const Shape* shapes, size_t n_shapes, int tile, int product, double cus) {
    const Sum sum = sum_of(shapes, n_shapes, tile);
    if (tile != TILE_256 || sum.tiles == 0.0) return launch_time(sum, tile, product, cus);
    const TileCost& k = kTile[tile];
    const double per_cu = sum.tiles / cus, f = k.fixed[product];
    const double latency = k.latency[product == PRODUCT_STORE], through = k.through[product == PRODUCT_STORE];
    // A workgroup walks one tile per round, so a round takes as long as its first tile; a round that is not full takes less
    // (a tile is faster when it has the memory system to itself).
    double time = kLaunch, seen = 0.0;
    for (size_t i = 0; i < n_shapes; ++i) {
        const Shape& s = shapes[i];
        if (s.tile != tile) continue;
        const double n = s.n[tile];
        const double from = ceil(seen / cus), to = ceil((seen + n) / cus);      // the rounds that begin with this shape
        const double full = std::max(0.0, std::min(to, floor(per_cu)) - from);
        time += full * (f + through * (double)s.C);
        if (to - from > full) time += f + (latency + (through - latency) * (per_cu - floor(per_cu))) * (double)s.C;
        seen += n;
    }
    return time;
}

// Contraction indices of the longest walk of G workgroups of a persistent kernel over tensors of tiles(i) tiles with contractions of
// length(i): tile t of a full round goes to the same workgroup in every one, the last round as xcd_run says.
template <typename Tiles, typename Length>
static double longest_walk(size_t n, int G, bool deal, Tiles&& tiles, Length&& length) {
    constexpr int MOST = 1024;
    if (G > MOST) G = MOST;      // no such device
    double load[MOST + 1] = {};      // in full rounds: from one workgroup to the next
    int64_t total = 0;
    for (size_t i = 0; i < n; ++i) total += tiles(i);
    const int64_t full = total / G * G;
    double all = 0.0;
    int64_t at = 0;
    size_t i = 0;
    for (; i < n; ++i) {
        const int64_t end = std::min(at + tiles(i), full), count = end - at;
        const double c = (double)length(i);
        all += c * (double)(count / G);
        const int64_t from = at % G, to = from + count % G;
        load[from] += c;
        load[to < G ? to : G] -= c;
        if (to > G) {
            load[0] += c;
            load[to - G] -= c;
        }
        if (end == full) break;
        at = end;
    }
    for (int p = 1; p < G; ++p) load[p] += load[p - 1];
    at = 0;
    for (size_t k = 0; k < i; ++k) at += tiles(k);
    const int left = (int)(total - full);
    for (int x = 0; x < 8 && i < n; ++x) {
        const dma::Run run = dma::xcd_run(x, left, G, deal);
        for (int l = 0; l < run.count; ++l) {
            while (at + tiles(i) <= full + run.first + l) at += tiles(i++);
            load[dma::xcd_run(x, G, G, true).first + l] += (double)length(i);
        }
    }
    double longest = 0.0;
    for (int p = 0; p < G; ++p) longest = std::max(longest, load[p]);
    return all + longest;
}

// Dealt out, unless that makes the longest walk longer.
int choose_deal(const dma::GroupArgs& ga, int workgroups) {
    bool same = true;
    for (int i = 1; i < ga.n; ++i) same &= ga.t[i].C == ga.t[0].C;
    if (same || ga.total_tiles % workgroups == 0) return 1;
    auto tiles = [&](size_t i) { return (int64_t)ga.t[i].tiles_m * ga.t[i].tiles_n; };
    auto length = [&](size_t i) { return ga.t[i].C; };
    return longest_walk((size_t)ga.n, workgroups, true, tiles, length) <= longest_walk((size_t)ga.n, workgroups, false, tiles, length);
}

static double pass_time(const std::vector<Shape>& shapes, int product, double cus) {
    double t = 0.0;
    for (int tile = 0; tile < N_TILES; ++tile) t += launch_time(shapes.data(), shapes.size(), tile, product, cus);
    return t;
}

static int best_alone(Shape one, int product, double cus) {
    int to = one.tile = TILE_256;
    if (one.fixed) return to;
    double best = launch_time(&one, 1, TILE_256, product, cus);
    for (one.tile = TILE_256 + 1; one.tile < N_TILES; ++one.tile) {
        const double t = launch_time(&one, 1, one.tile, product, cus);
        if (t < best) {
            best = t;
            to = one.tile;
        }
    }
    return to;
}

// Starting choices: all tensors in the persistent kernel, all in the shape of tile that is best for all together, and each in the
// one that is best for it alone; from each, one shape after the other (longest contraction first) moves to where the pass is
// shortest.  A move changes two launches of the pass, and only these are reckoned again (60 different shapes 815 -> 150 us on the host,
// two layers and a vocabulary 16 -> 12.5, the binding's part included).
void choose_tiles(const GemmArgs* list, size_t n, int product, int* tile_of) {
    const double cus = (double)cu_count();
    std::vector<Shape> shapes;
    std::vector<int> count;
    auto same = [&](const Shape& s, const GemmArgs& a) { return s.M == a.M && s.Nn == a.Nn && s.C == a.C; };
    for (size_t i = 0; i < n; ++i) {
        size_t k = 0;
        while (k < shapes.size() && !same(shapes[k], list[i])) ++k;
        if (k == shapes.size()) {
            shapes.emplace_back(list[i].M, list[i].Nn, list[i].C, list[i].persistent_only);
            count.push_back(0);
        }
        ++count[k];
    }
    std::vector<Shape> alone = shapes;      // a list of one shape is its own
    for (size_t k = 0; k < shapes.size(); ++k) {
        for (double& t : shapes[k].n) t *= (double)count[k];
        alone[k].tile = best_alone(shapes.size() > 1 ? alone[k] : shapes[k], product, cus);
        std::copy(shapes[k].n, shapes[k].n + N_TILES, alone[k].n);
    }
    auto longer = [](const Shape& x, const Shape& y) { return x.C > y.C; };
    std::stable_sort(shapes.begin(), shapes.end(), longer);
    std::stable_sort(alone.begin(), alone.end(), longer);
    auto improve = [&](std::vector<Shape>& v) {
        double launch[N_TILES];
        Sum sums[N_TILES];
        for (int tile = 0; tile < N_TILES; ++tile) {
            launch[tile] = launch_time(v.data(), v.size(), tile, product, cus);
            sums[tile] = sum_of(v.data(), v.size(), tile);
        }
        auto sum = [&](int a, double ta, int b, double tb) {
            double t = 0.0;
            for (int tile = 0; tile < N_TILES; ++tile) t += tile == a ? ta : tile == b ? tb : launch[tile];
            return t;
        };
        double best = sum(-1, 0.0, -1, 0.0);
        for (int sweep = 0; sweep < 3 && v.size() <= kGreedyShapes; ++sweep) {
            bool moved = false;
            for (Shape& s : v) {
                if (s.fixed) continue;
                const int was = s.tile;
                int to = was;
                s.tile = -1;
                const double without = launch_time(v.data(), v.size(), was, product, cus);
                double with = launch[was];
                for (int tile = 0; tile < N_TILES; ++tile) {
                    if (tile == was) continue;
                    s.tile = tile;
                    Sum more = sums[tile];
                    more.add(s, tile);
                    const double there = tile == TILE_256 ? launch_time(v.data(), v.size(), tile, product, cus)
                                                          : launch_time(more, tile, product, cus);
                    const double t = sum(was, without, tile, there);
                    if (t < best) {
                        best = t;
                        to = tile;
                        with = there;
                    }
                }
                s.tile = to;
                if (to == was) continue;
                launch[was] = without;
                launch[to] = with;
                sums[was] = sum_of(v.data(), v.size(), was);
                sums[to].add(s, to);
                moved = true;
            }
            if (!moved) break;
        }
        return best;
    };
    if (shapes.size() > 1) {
        std::vector<Shape> same_tile = shapes;
        auto all_in = [&](int tile) {
            for (Shape& s : same_tile) s.tile = s.fixed ? TILE_256 : tile;
            return pass_time(same_tile, product, cus);
        };
        int uniform = TILE_256;
        double best = all_in(TILE_256);
        for (int tile = TILE_256 + 1; tile < N_TILES; ++tile) {
            const double t = all_in(tile);
            if (t < best) {
                best = t;
                uniform = tile;
            }
        }
        all_in(uniform);
        const double in_one = uniform == TILE_256 ? 1e30 : improve(same_tile);
        best = improve(shapes);
        if (in_one < best) {
            best = in_one;
            shapes = same_tile;
        }
        const double each = improve(alone);
        if (each < best) {
            best = each;
            shapes.swap(alone);
        }
        if (best > kLeave * all_in(TILE_256)) shapes.swap(same_tile);
    } else {
        shapes.swap(alone);
    }
    for (size_t i = 0; i < n; ++i)
        tile_of[i] = std::find_if(shapes.begin(), shapes.end(), [&](const Shape& s) { return same(s, list[i]); })->tile;
}

// A last round of a few tiles takes nearly as long as a full one (the workgroups have few neighbours to share panels with and wait
// for memory, so an index takes more than `latency`), small tiles spread the same work over the chip.  Measured, us, norm of T = 4096 and 4096 columns: 512 + 16, + 32, + 64
// tiles 315, 315, 325 against 224 for the 512; a list of 12 rounds and 16 tiles 1361.
Leftover cut_leftover(const GemmArgs* list, int n, int product, bool a_strided, bool b_strided) {
    Leftover best;
    const int64_t cus = cu_count();
    auto tiles = [](int64_t x) { return (x + 255) / 256; };
    int64_t total = 0;
    for (int i = 0; i < n; ++i) total += tiles(list[i].M) * tiles(list[i].Nn);
    const int64_t left = total % cus;
    if (total < cus || left == 0 || 4 * left > cus) return best;
    double shortest = 1e30;
    for (int i = 0; i < n; ++i) {
        const GemmArgs& a = list[i];
        if (a.persistent_only) continue;
        for (bool columns : {true, false}) {
            const int64_t along = tiles(columns ? a.M : a.Nn), across = tiles(columns ? a.Nn : a.M);
            const int64_t k = (left + across - 1) / across;      // columns or rows of tiles to take away
            if (k >= along) continue;
            const int64_t at = (along - k) * 256;
            Shape piece(columns ? a.M - at : a.M, columns ? a.Nn : a.Nn - at, a.C, false);
            // the round that is saved, by the measurements above
            double time = kTile[TILE_256].fixed[product] + 0.0215 * (double)list[n - 1].C;
            int tile = TILE_256;
            for (piece.tile = TILE_256 + 1; piece.tile < N_TILES; ++piece.tile) {
                const double t = launch_time(&piece, 1, piece.tile, product, (double)cus);
                if (t < time) {
                    time = t;
                    tile = piece.tile;
                }
            }
            if (tile == TILE_256 || time >= shortest) continue;
            shortest = time;
            best.tensor = i;
            best.tile = tile;
            best.kept = best.piece = a;
            (columns ? best.kept.M : best.kept.Nn) = at;
            best.piece.M = piece.M;
            best.piece.Nn = piece.Nn;
            const int64_t m0 = columns ? at : 0, n0 = columns ? 0 : at;
            best.piece.A += a_strided ? m0 : m0 * a.lda;
            best.piece.B += b_strided ? n0 : n0 * a.ldb;
            if (a.Out != nullptr) best.piece.Out += n0 * a.ldo + m0;
            if (a.Res != nullptr) best.piece.Res += n0 * a.ldo + m0;
        }
    }
    return best;
}

void tile_size(int tile, int32_t* m, int32_t* n) {
    *m = kTile[tile].m;
    *n = kTile[tile].n;
}

template <bool B_STRIDED, int EPI, bool A_STRIDED>
static hipError_t launch_with(int tile, const GemmArgs* list, size_t n, hipStream_t st) {
    if (tile != TILE_256) return launch_tile_group<B_STRIDED, EPI, A_STRIDED>(list, (int)n, tile, st);
    constexpr int product = EPI == EPI_SQNORM ? PRODUCT_NORM : EPI == EPI_STORE ? PRODUCT_STORE : PRODUCT_UPDATE;
    GemmArgs group[dma::MAX_GROUP];
    for (size_t first = 0; first < n; first += dma::MAX_GROUP) {
        const int cnt = (int)(n - first < (size_t)dma::MAX_GROUP ? n - first : (size_t)dma::MAX_GROUP);
        std::copy(list + first, list + first + cnt, group);
        const Leftover l = cut_leftover(group, cnt, product, A_STRIDED, B_STRIDED);
        if (l.tensor >= 0) group[l.tensor] = l.kept;
        hipError_t e;
        if constexpr (B_STRIDED) e = launch_dma_group<EPI>(group, cnt, st);
        else e = launch_wide_group<EPI, A_STRIDED>(group, cnt, st);
        if (e == hipSuccess && l.tensor >= 0) e = launch_tile_group<B_STRIDED, EPI, A_STRIDED>(&l.piece, 1, l.tile, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Workgroups of the small tiles start in list order: the longest walks first.  In the persistent kernels that is done where
// it makes the longest walk shorter; otherwise the order does not matter much (dX of a 7B layer at 4096 tokens 1339 us as
// listed, 1337 sorted; at 2999 tokens 1070 and 1078; of two 13B layers at 1070 tokens 1286 and 1339).
static void order_list(int tile, std::vector<GemmArgs>& list) {
    std::vector<GemmArgs> sorted = list;
    std::stable_sort(sorted.begin(), sorted.end(), [](const GemmArgs& x, const GemmArgs& y) { return x.C > y.C; });
    auto walk = [&](const std::vector<GemmArgs>& v) {
        auto tiles = [&](size_t i) { return ((v[i].M + 255) / 256) * ((v[i].Nn + 255) / 256); };
        auto length = [&](size_t i) { return v[i].C; };
        return std::min(longest_walk(v.size(), cu_count(), true, tiles, length), longest_walk(v.size(), cu_count(), false, tiles, length));
    };
    if (tile != TILE_256 || walk(sorted) < 0.98 * walk(list)) list.swap(sorted);
}

LastRound last_round(const GemmArgs* list, size_t n, const int* tile_of, int product, bool a_strided, bool b_strided) {
    LastRound r;
    std::vector<GemmArgs> v;
    for (size_t i = 0; i < n; ++i)
        if (tile_of[i] == TILE_256) v.push_back(list[i]);
    if (v.empty()) return r;
    if (n > 1) order_list(TILE_256, v);
    const int cnt = (int)std::min(v.size(), (size_t)dma::MAX_GROUP);
    r.cut = cut_leftover(v.data(), cnt, product, a_strided, b_strided);
    if (r.cut.tensor >= 0) {
        v[r.cut.tensor] = r.cut.kept;
        r.tensor = r.cut.kept.family;      // its place in the list
    }
    dma::GroupArgs ga{};
    dma::fill_group(ga, v.data(), cnt, 256, 256);
    r.dealt = choose_deal(ga, std::min(ga.total_tiles, cu_count()));
    return r;
}

// A list of one allocates no host memory; for longer ones a failed allocation is an error code like a refused launch.
template <bool B_STRIDED, int EPI, bool A_STRIDED>
static hipError_t launch_list(const GemmArgs* list, size_t n, hipStream_t st) try {
    constexpr int product = EPI == EPI_SQNORM ? PRODUCT_NORM : EPI == EPI_STORE ? PRODUCT_STORE : PRODUCT_UPDATE;
    auto any_shape = [](const GemmArgs& a) { return !fast_enabled() || !dma_eligible<B_STRIDED, A_STRIDED>(a); };
    if (n == 1) {
        if (any_shape(*list)) return launch_generic<B_STRIDED, EPI, A_STRIDED>(*list, st);
        GemmArgs one = *list;
        one.persistent_only = beyond_descriptor<B_STRIDED, A_STRIDED>(one);
        const Shape s(one.M, one.Nn, one.C, one.persistent_only);
        return launch_with<B_STRIDED, EPI, A_STRIDED>(best_alone(s, product, (double)cu_count()), &one, 1, st);
    }
    std::vector<GemmArgs> fit, by[N_TILES];
    for (size_t i = 0; i < n; ++i) {
        if (any_shape(list[i])) {
            const hipError_t e = launch_generic<B_STRIDED, EPI, A_STRIDED>(list[i], st);
            if (e != hipSuccess) return e;
        } else {
            fit.push_back(list[i]);
            fit.back().persistent_only = beyond_descriptor<B_STRIDED, A_STRIDED>(list[i]);
        }
    }
    std::vector<int> tile_of(fit.size());
    choose_tiles(fit.data(), fit.size(), product, tile_of.data());
    for (size_t i = 0; i < fit.size(); ++i) by[tile_of[i]].push_back(fit[i]);
    for (int tile = 0; tile < N_TILES; ++tile) {
        if (by[tile].empty()) continue;
        order_list(tile, by[tile]);
        const hipError_t e = launch_with<B_STRIDED, EPI, A_STRIDED>(tile, by[tile].data(), by[tile].size(), st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
} catch (const std::bad_alloc&) {
    return hipErrorOutOfMemory;
}

hipError_t launch_wgrad_update(const GemmArgs* list, size_t n, hipStream_t st) {
    return launch_list<true, EPI_UPDATE, true>(list, n, st);
}
hipError_t launch_wgrad_update_clipv(const GemmArgs* list, size_t n, hipStream_t st) {
    return launch_list<true, EPI_CLIPV, true>(list, n, st);
}
hipError_t launch_wgrad_sqnorm(const GemmArgs* list, size_t n, int norm_route, hipStream_t st) try {
    if (norm_route == LOMO_NORM_DIRECT || !fast_enabled()) return launch_list<true, EPI_SQNORM, true>(list, n, st);
    std::vector<GemmArgs> gram, direct;
    choose_norm_route(norm_route, std::vector<GemmArgs>(list, list + n), gram, direct);
    if (!gram.empty()) {
        const hipError_t e = launch_gram_group(gram.data(), (int)gram.size(), st);
        if (e != hipSuccess) return e;
    }
    return launch_list<true, EPI_SQNORM, true>(direct.data(), direct.size(), st);
} catch (const std::bad_alloc&) {
    return hipErrorOutOfMemory;
}
hipError_t launch_dgrad(const GemmArgs* list, size_t n, hipStream_t st) {
    return launch_list<false, EPI_STORE, true>(list, n, st);
}

// Y = X W^T (EPI_STORE) or Y <- Y + X W^T rounded once (EPI_UPDATE with s = -1: the residual connection).
hipError_t launch_forward(const GemmArgs& a, bool accumulate, hipStream_t st) {
    return accumulate ? launch_list<false, EPI_UPDATE, false>(&a, 1, st) : launch_list<false, EPI_STORE, false>(&a, 1, st);
}

}  // namespace lomo
