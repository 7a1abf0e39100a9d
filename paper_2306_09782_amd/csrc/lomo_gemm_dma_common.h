// What the contraction kernels with direct-to-LDS operand loads share: buffer descriptors, the load itself, the swizzle of
// contraction-contiguous tiles and the transposing fragment read.
#pragma once
#include "lomo_gemm_common.h"

namespace lomo {

typedef short short4v __attribute__((ext_vector_type(4)));

namespace dma {

constexpr int BK = 32;        // contraction slice

// Buffer descriptors: word 3 asks for raw 32-bit data, `bytes` is where the range check ends.
typedef int int4v __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));
constexpr uint32_t BUFFER_WORD3 = 0x00020000u;
constexpr uint32_t MAX_RANGE = 0xE0000000u;      // no descriptor covers more than this ...
constexpr uint32_t OUTSIDE = 0xF0000000u;        // ... so a lane offset with these bits set is outside every one
constexpr uint32_t MOVE_BASE = 0x40000000u;      // the base of a larger operand moves when its slice offset reaches this
__device__ __forceinline__ int4v make_srd(const void* base, uint32_t bytes) {
    const uint64_t b = (uint64_t)(uintptr_t)base;
    return int4v{(int)(uint32_t)b, (int)((uint32_t)(b >> 32) & 0xffffu), (int)bytes, (int)BUFFER_WORD3};
}
__device__ __forceinline__ uint32_t range_bytes(int64_t halves) {
    return halves <= 0 ? 0u : (2 * halves > (int64_t)MAX_RANGE ? MAX_RANGE : (uint32_t)(2 * halves));
}

__device__ __forceinline__ int swz_c(int n) { return ((n >> 1) & 3) ^ ((n >> 3) & 1); }

// 16 bytes per lane from descriptor base + soff + voff to LDS address m0 + 16 * lane; zeros where voff is not below
// the descriptor's range - soff (callers keep soff within the range).
__device__ __forceinline__ void dma16(uint32_t voff, int4v srd, uint32_t soff, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds"
                 :: "v"(voff), "s"(srd), "s"(soff), "s"(lds_addr) : "memory", "m0");
}

__device__ __forceinline__ half8 read_tr8(const uint16_t* p0, const uint16_t* p1) {
    typedef __attribute__((address_space(3))) short4v* lds_p;
    const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_p)(p0));
    const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_p)(p1));
    return __builtin_bit_cast(half8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

constexpr int MAX_GROUP = 40;

struct GroupTensor {
    const uint16_t* A;
    const uint16_t* B;
    uint16_t* Out;
    const uint16_t* Res;
    int32_t* flag_out;
    int M, Nn, C, lda, ldb, ldo;
    int tiles_m, tiles_n, tile_begin;
};

struct GroupArgs {
    double* acc;
    const int32_t* flag_in;
    float s, lr, inv_s, clipv;
    const float* s_dev;
    int n, total_tiles;
    int deal;      // persistent kernels: the last round is dealt out to all XCDs
    GroupTensor t[MAX_GROUP];
};

// The kernel's argument table for `cnt` tensors cut into tiles of bm x bn; what the tensors share comes from the first.
inline void fill_group(GroupArgs& ga, const GemmArgs* list, int cnt, int bm, int bn) {
    ga.acc = list[0].acc;
    ga.flag_in = list[0].flag_in;
    ga.s = list[0].s;
    ga.s_dev = list[0].s_dev;
    ga.lr = list[0].lr;
    ga.inv_s = list[0].inv_s;
    ga.clipv = list[0].clipv;
    ga.n = cnt;
    int tiles = 0;
    for (int i = 0; i < cnt; ++i) {
        const GemmArgs& a = list[i];
        GroupTensor& t = ga.t[i];
        t.A = a.A; t.B = a.B; t.Out = a.Out; t.Res = a.Res; t.flag_out = a.flag_out;
        t.M = (int)a.M; t.Nn = (int)a.Nn; t.C = (int)a.C;
        t.lda = (int)a.lda; t.ldb = (int)a.ldb; t.ldo = (int)a.ldo;
        t.tiles_m = (int)((a.M + bm - 1) / bm); t.tiles_n = (int)((a.Nn + bn - 1) / bn);
        t.tile_begin = tiles;
        tiles += t.tiles_m * t.tiles_n;
    }
    ga.total_tiles = tiles;
}

}  // namespace dma
}  // namespace lomo
