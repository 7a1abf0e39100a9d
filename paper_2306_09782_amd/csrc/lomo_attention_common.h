// Pieces shared by the attention forward and backward kernels: tile geometry, the chunk swizzle of the [64 x 128] LDS tiles,
// their direct-to-LDS loads, fragment reads, and the way from accumulators to fragments and to memory.
//
// All three kernels have one shape: a workgroup of four waves owns 128 rows (queries, or keys in the dk / dv kernel), 32 per
// wave, whose operands stay in registers as MFMA fragments; the waves share a pair of [64 x 128] tiles that moves along the
// sequence, double-buffered in LDS, one barrier per pair.  Scores are formed so that a lane owns one of the wave's own rows;
// what they become (probabilities, their gradients) reaches the next product through registers, so nothing but the
// moving tiles passes through LDS and waves meet only where a tile changes.
// SPLIT = 2, for calls that give too few of these: a workgroup owns 64 rows, two waves have the same 32, and each takes one half
// of every moving tile.  The forward puts their sums together at the end, as it does with the halves of one wave; the
// backward kernels hand P and dS over through LDS, each wave having a part of the sums.  Every sum has the same terms in the
// same order either way, so a call's size does not show in its results.  (The backward of sequences of one block is one kernel that does the
// same on tiles that stay where they are.)
#pragma once
#include "lomo_gemm_common.h"

namespace lomo {

typedef short short4a __attribute__((ext_vector_type(4)));

namespace attn {

constexpr int D = 128;                 // head width
template <int SPLIT>
constexpr int ROWS = 128 / SPLIT;      // rows of a workgroup
constexpr int BLK = 64;                // rows of a moving tile
constexpr int TILE = BLK * D;          // halves
constexpr int PAIR = 2 * TILE;
constexpr int LDS_BYTES = 2 * PAIR * 2;      // two pairs
constexpr float SCALE = 0.08838834764831845f;      // 1 / sqrt(128)
constexpr float LOG2E = 1.4426950408889634f;

typedef __attribute__((address_space(3))) short4a* lds_p;
// at LDS addresses
__device__ __forceinline__ half8 read_tr8(uint32_t p0, uint32_t p1) {
    const short4a lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_p)p0);
    const short4a hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_p)p1);
    return __builtin_bit_cast(half8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}
__device__ __forceinline__ half8 read8(uint32_t p) { return *(__attribute__((address_space(3))) const half8*)p; }

// Chunk swizzle of the [64 x 128] tiles: 16-byte chunk c of row r sits at position c ^ swz(r).  Rows that
// differ in their low two bits are 4 chunks apart (the four rows of a transposing read fall on disjoint banks,
// and so do its two 16-column halves), rows that differ in the next two bits are 1..3 chunks apart (sixteen
// consecutive rows read at the same column hit sixteen different chunks).
__device__ __forceinline__ int swz(int r) { return ((r & 3) << 2) | ((r >> 2) & 3); }

// 16 bytes per lane from base + voff to LDS address m0 + 16 * lane.
__device__ __forceinline__ void load_lds16(uint32_t voff, const void* base, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(base), "s"(lds_addr) : "memory", "m0");
}

// The loads of a [64 x 128] tile with rows of `ld` elements: wave w of the four fetches rows 16 w .. 16 w + 15 with four instructions of
// four rows.  A row is a multiple of 256 bytes, so the chunk's place in it is the low byte of the offset, where the swizzles
// of the four instructions differ by their number.  Four rows have to fit 32-bit offsets: up to FAR heads.
constexpr int64_t FAR = 1 << 20;
struct TileLoad {
    uint32_t voff;
    int64_t step;      // four rows
    __device__ __forceinline__ TileLoad(int64_t ld) {
        const int lane = threadIdx.x & 63, rr = lane >> 4;
        voff = (uint32_t)rr * (uint32_t)ld * 2u + (uint32_t)(((lane & 15) ^ swz(rr)) * 16);
        step = 4 * ld;
    }
    // `tile`: LDS address; `wave` uniform
    template <int WAVES = 4>
    __device__ __forceinline__ void issue(const uint16_t* base, uint32_t tile, int wave) const {
        if constexpr (WAVES == 2) issue(base, tile, wave + 2);
        base += 4 * wave * step;
        uint32_t v = voff;
        asm volatile("" : "+v"(v));      // formed again each time, not kept in registers
#pragma unroll
        for (int it = 0; it < 4; ++it) load_lds16(v ^ (uint32_t)(16 * it), base + it * step, tile + (uint32_t)(4 * wave + it) * 1024u);
    }
};

// The same for rows of any length, by 64-bit addresses.
struct TileLoadFar {
    int64_t row;       // bytes from one row to the next
    uint32_t chunk;
    __device__ __forceinline__ TileLoadFar(int64_t ld) {
        const int lane = threadIdx.x & 63, rr = lane >> 4;
        row = 2 * ld;
        chunk = (uint32_t)(((lane & 15) ^ swz(rr)) * 16);
    }
    __device__ __forceinline__ void issue(const uint16_t* base, uint32_t tile, int wave) const {
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const char* at = reinterpret_cast<const char*>(base) + (16 * wave + 4 * it + ((threadIdx.x & 63) >> 4)) * row + (chunk ^ (uint32_t)(16 * it));
            asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(at), "s"(tile + (uint32_t)(4 * wave + it) * 1024u)
                         : "memory", "m0");
        }
    }
};

// Fragment reads from a tile, by LDS address (of tiles that begin at multiples of 256 bytes).  The places of the fragments differ
// in a few low bits; they are formed again for every tile (one instruction each), which costs less than keeping them in registers.
struct TileRead {
    uint32_t row_rd, tr0, tr1;
    __device__ __forceinline__ TileRead(uint32_t tile) {
        const int lane = threadIdx.x & 63;
        const int l32 = lane & 31, lh = lane >> 5;
        const int g4 = lane >> 4, j16 = lane & 15;
        const int mhalf = g4 & 1, kh = g4 >> 1, rib = j16 >> 2, piece = j16 & 3;
        const int tr_row = 8 * kh + rib, tr_col = 16 * mhalf + 4 * piece;
        row_rd = tile + 2u * (uint32_t)(l32 * D + ((8 * lh) ^ (swz(l32) << 3)));
        tr0 = tile + 2u * (uint32_t)(tr_row * D + (tr_col ^ (swz(tr_row) << 3)));
        tr1 = tile + 2u * (uint32_t)((tr_row + 4) * D + (tr_col ^ (swz(tr_row + 4) << 3)));
    }
    // the same for a tile `halves` further on
    __device__ __forceinline__ TileRead at(int halves) const {
        TileRead t = *this;
        t.row_rd += 2u * (uint32_t)halves;
        t.tr0 += 2u * (uint32_t)halves;
        t.tr1 += 2u * (uint32_t)halves;
        asm volatile("" : "+v"(t.row_rd), "+v"(t.tr0), "+v"(t.tr1));
        return t;
    }
    __device__ __forceinline__ void move(int halves) {
        row_rd += 2u * (uint32_t)halves;
        tr0 += 2u * (uint32_t)halves;
        tr1 += 2u * (uint32_t)halves;
        asm volatile("" : "+v"(row_rd), "+v"(tr0), "+v"(tr1));
    }
    // the same with column tiles counted from `i` on
    __device__ __forceinline__ TileRead column_tile(int i) const {
        TileRead t = *this;
        t.tr0 ^= (uint32_t)(64 * i);
        t.tr1 ^= (uint32_t)(64 * i);
        return t;
    }
    // `off`: halves from the tile of this to the one that is read.
    // rows 0 .. 31, columns 16 ks .. + 15: a lane holds eight consecutive columns of its row
    __device__ __forceinline__ half8 rows(int off, int ks) const { return read8((row_rd ^ (uint32_t)(32 * ks)) + 2u * (uint32_t)off); }
    // columns 32 i .. + 31, rows 16 ks .. + 15: a lane holds eight consecutive rows of its column
    __device__ __forceinline__ half8 columns(int off, int i, int ks) const {
        const uint32_t o = 2u * (uint32_t)(off + 16 * ks * D);
        return read_tr8((tr0 ^ (uint32_t)(64 * i)) + o, (tr1 ^ (uint32_t)(64 * i)) + o);
    }
};

template <int N, typename F>
__device__ __forceinline__ void repeat(F&& f) {
    if constexpr (N > 0) {
        f();
        repeat<N - 1>(f);
    }
}
// Order of a run of matrix instructions and of the LDS reads that feed them: AHEAD reads in front, then READS behind every MFMAS.
template <int AHEAD, int MFMAS, int READS, int TIMES, int REST>
__device__ __forceinline__ void interleave() {
    __builtin_amdgcn_sched_group_barrier(0x100, AHEAD, 0);
    repeat<TIMES>([] {
        __builtin_amdgcn_sched_group_barrier(0x008, MFMAS, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, READS, 0);
    });
    __builtin_amdgcn_sched_group_barrier(0x008, REST, 0);
}

// This wave's 32 rows, straight from memory: a lane holds eight consecutive columns of its row per fragment.
__device__ __forceinline__ void load_fragments(half8 (&f)[D / 16], const uint16_t* row) {
    const int lh = (threadIdx.x & 63) >> 5;
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) f[ks] = *reinterpret_cast<const half8*>(row + 16 * ks + 8 * lh);
}

// A lane's sixteen values of a 32 x 32 block, as packed fp16 pairs of neighbouring rows of the block: pk[r / 2] holds the
// rows 8 (r / 4) + 4 lh + r % 4 and the next.  Lane halves exchange so that each holds eight consecutive rows 16 ks + 8 lh ..:
// the fragment of the next product's second operand.
__device__ __forceinline__ half8 fragment_of(const uint32_t (&pk)[8], int ks) {
    typedef uint32_t u32x2v __attribute__((ext_vector_type(2)));
    const u32x2v s0 = __builtin_amdgcn_permlane32_swap(pk[4 * ks + 0], pk[4 * ks + 2], false, false);
    const u32x2v s1 = __builtin_amdgcn_permlane32_swap(pk[4 * ks + 1], pk[4 * ks + 3], false, false);
    const u32x4 w = {s0[0], s1[0], s0[1], s1[1]};
    return __builtin_bit_cast(half8, w);
}
__device__ __forceinline__ uint32_t pack2(float a, float b) {
    typedef _Float16 half2v __attribute__((ext_vector_type(2)));
    const half2v h = {(_Float16)a, (_Float16)b};
    return __builtin_bit_cast(uint32_t, h);
}

// acc[i][r]: column 32 c + 8 (r / 4) + 4 lh + r % 4 of the lane's row, rounded once; c = i, of two accumulators first + 2 i.
template <int N>
__device__ __forceinline__ void store_rows(const floatx16 (&acc)[N], uint16_t* row, int first = 0) {
    const int lh = (threadIdx.x & 63) >> 5;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        uint32_t pk[8];
#pragma unroll
        for (int r = 0; r < 16; r += 2) pk[r >> 1] = pack2(acc[i][r], acc[i][r + 1]);
#pragma unroll
        for (int a = 0; a < 2; ++a) *reinterpret_cast<half8*>(row + 32 * (N == 4 ? i : first + 2 * i) + 16 * a + 8 * lh) = fragment_of(pk, a);
    }
}

// Waves of a call that is not split, per CU.  Below four, one for every SIMD, the chip has room for twice as many; with more a call of
// long walks still ends sooner when they are halved.
inline double waves_per_cu(int64_t B, int64_t s, int64_t nh) { return (double)(s / 32 * nh * B) / (double)cu_count(); }

// This workgroup's (sequence, head) pair and its place among the pair's `nb` blocks, 0 the first to start.  Each XCD (blockIdx % 8)
// takes a contiguous run of pairs, so that the blocks that read the same rows meet in one L2.  Where they divide evenly, the
// first blocks of all its pairs start first, the heaviest there are; pair by pair, the 32 blocks of 4096 tokens fall on
// the 32 CUs of an XCD alike for every pair, and one CU has all the heaviest.
__device__ __forceinline__ void locate_block(int nb, int& pair, int& place) {
    const int G = gridDim.x, x = (int)(blockIdx.x & 7), local = (int)(blockIdx.x >> 3);
    if (G % (8 * nb) == 0) {
        const int pairs = G / (8 * nb);
        place = local / pairs;
        pair = x * pairs + (local - place * pairs);
    } else {
        const int q = G >> 3, r = G & 7, pos = x * q + (x < r ? x : r) + local;
        pair = pos / nb;
        place = pos - pair * nb;
    }
}

}  // namespace attn

}  // namespace lomo
