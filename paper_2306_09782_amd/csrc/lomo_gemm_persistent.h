// What the two persistent 256 x 256 contraction kernels share: geometry, the order of the tiles, the row epilogue.
#pragma once
#include "lomo_gemm_dma_common.h"

namespace lomo {

namespace dma {

constexpr int BM = 256, BN = 256, NS = 4;
constexpr int A_HALVES = BK * BM, B_HALVES = BK * BN, STAGE_HALVES = A_HALVES + B_HALVES;
constexpr int EPI_UNIT_HALVES = 32 * 64;                 // staging block of the row epilogue: 32 rows x 64 columns (4 KiB)
// four stages (two slots in lomo_gemm_wide.hip) + 32 KiB behind them: two staging blocks per wave for the row epilogue (update, store), whose first
// 256 bytes serve as the reduction scratch of the norm epilogue.  160 KiB in all, the whole LDS of a CU.
constexpr int LDS_BYTES = NS * STAGE_HALVES * 2 + 8 * EPI_UNIT_HALVES * 2;

__device__ __forceinline__ int swz_s(int r) { return ((r & 1) * 10) + ((r & 2) * 2); }

// Tiles of round k of a list that G workgroups walk: G, in the last round what is left.
__device__ __forceinline__ int round_tiles(int k, int G, int total) {
    const int left = total - k * G;
    return left < 0 ? 0 : (left < G ? left : G);
}
// Tiles that the workgroups of XCD x (blockIdx % 8) take in a round of n, of which the first is number `first`.
struct Run {
    int first, count;
};
__host__ __device__ __forceinline__ Run xcd_run(int x, int n, int G, bool deal) {
    const int m = deal ? n : G, q = m >> 3, r = m & 7, first = x * q + (x < r ? x : r), own = q + (x < r ? 1 : 0);
    const int left = n - first;
    return {first, left < 0 ? 0 : (left < own ? left : own)};
}
// This workgroup's tile of round k, `total` where it has none.  The workgroups of one XCD take a contiguous
// run, which the band order of locate_tile turns into an 8 x 4 block of tiles that share operand panels in that XCD's L2;
// a last round is dealt out to all XCDs alike: left to the first of them, a round of 96 tiles runs at the speed of three XCDs' memory
// paths.  Measured, us, first XCDs -> all: update of 8192 x 5120 x 5120 (400 tiles) 430 -> 364, its Y and dX (640) 400 -> 354; norm of
// 4096 x 4096 x 22016 (1376) 623 -> 598, its update 654 -> 630; dX of 4096 x 11008 x 4096 (688) 325 -> 298.  Where contractions differ and
// that gives a workgroup with long tiles one more (choose_deal), it is left to the first: dX of a layer 8192 wide at 1280
// tokens 1884 dealt out, 1800 not.
__device__ __forceinline__ int round_tile(int k, int G, int total, bool deal) {
    const Run run = xcd_run((int)(blockIdx.x & 7), round_tiles(k, G, total), G, deal);
    const int local = (int)(blockIdx.x >> 3);
    return local < run.count ? k * G + run.first + local : total;
}
// The tile of round k of a workgroup that had `w` in the round before: in a full round its place is the same.
__device__ __forceinline__ int next_tile(int w, int k, int G, int total, bool deal) {
    if (__builtin_expect((k + 1) * G <= total, 1)) return w + G;
    return round_tile(k, G, total, deal);
}

// Tensor and origin of tile number w of the concatenated list.  A workgroup's tile numbers only grow, so the search for
// the tile's tensor resumes at the previous tile's.
// COLUMNS: outputs of five or six rows of tiles go column by column (dX of 1025 to 1536 tokens), so that the panel of W behind a column, which
// comes from HBM, is read by one XCD, or two; bands of 8 x 4 tiles split such outputs over two XCDs each.  Measured, us, bands -> columns: dX
// of two layers 5120 wide at 1070 tokens 1338 -> 1308, at 1280 1437 -> 1392, at 1536 1655 -> 1602, of one 8192 wide at 1280 1788 -> 1729; but
// two 4096 wide at 1792 (seven rows) 1230 -> 1237, and Y of 1536 x 22016 251 -> 255: forward products keep the bands.
template <bool COLUMNS = false>
__device__ __forceinline__ void locate_tile(const GroupArgs& ga, int w, int& tensor, int64_t& m0, int64_t& n0) {
    int k = tensor;
    while (k + 1 < ga.n && w >= ga.t[k + 1].tile_begin) ++k;
    const GroupTensor& T = ga.t[k];
    const int t = w - T.tile_begin;
    if (COLUMNS && (T.tiles_n == 5 || T.tiles_n == 6)) {
        const int m = t / T.tiles_n;
        tensor = k;
        m0 = (int64_t)m * BM;
        n0 = (int64_t)(t - m * T.tiles_n) * BN;
        return;
    }
    constexpr int GM = 8;
    const int per_band = GM * T.tiles_n;
    const int band = t / per_band;
    const int first_m = band * GM;
    const int gsz = (T.tiles_m - first_m < GM) ? (T.tiles_m - first_m) : GM;
    const int in_band = t - band * per_band;
    tensor = k;
    m0 = (int64_t)(first_m + in_band % gsz) * BM;
    n0 = (int64_t)(in_band / gsz) * BN;
}

// Puts the base of a contraction-strided operand larger than a descriptor covers at its next slice: bytes left to the operand's end, offset
// of the next slice, where the slices end, and from which offset on the base moves again.
__device__ __forceinline__ void move_base(int4v& srd, int64_t& left, uint32_t& next, uint32_t& end, uint32_t& move) {
    left -= next;
    const uint64_t base = (((uint64_t)(uint32_t)srd[1] << 32) | (uint32_t)srd[0]) + next;
    srd = make_srd((const void*)base, range_bytes(left / 2));
    next = 0;
    end = (uint32_t)srd[2];
    move = left > (int64_t)MAX_RANGE ? MOVE_BASE : ~0u;
}

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
        // two blocks per wave behind the stages, the third in the B part of the last stage (slot), which is idle between
        // the last slice of a tile and the first half-slice of the next
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

    // Vector-memory operations of `run`: the four stores of every block and, with an old value, the loads of blocks 3..7.
    template <int EPI>
    static constexpr int OPS = 8 * 4 + (EPI == EPI_UPDATE || EPI == EPI_CLIPV ? 5 * 4 : 0);

    // `ahead`: AHEAD vector-memory operations were issued between the first three fills and this call (the next tile's
    // first slices)
    template <int EPI, int AHEAD>
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
                // the loads of the next tile's first slices (if any), then per block u its stores and the loads of
                // block u + 3.  Wait until only those may still be outstanding.
                static_assert(16 + AHEAD < 64, "the counter holds six bits");
                if (u == 0) { if (ahead) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(8 + AHEAD) : "memory"); else asm volatile("s_waitcnt vmcnt(8)" ::: "memory"); }
                else if (u == 1) { if (ahead) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(12 + AHEAD) : "memory"); else asm volatile("s_waitcnt vmcnt(12)" ::: "memory"); }
                else if (u == 2) { if (ahead) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(16 + AHEAD) : "memory"); else asm volatile("s_waitcnt vmcnt(16)" ::: "memory"); }
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
}  // namespace lomo
