// Backward of causal softmax attention with the rotary step, for the hand-on gradient of Algorithm 1
// (paper section 3.2) through the self-attention block of a LLaMA layer (the models of section 4), gfx950.
//
// Tokens t = b * s + pos; head n owns columns [128 n, 128 n + 128) of q, k, v, o.  qkv holds the rotated
// q and k and v side by side ([T x 3H]); lse[t][n] = log sum_j exp(S_tj) is saved by the forward pass.
//
//   P_ij = exp(q_i . k_j / sqrt(d) - lse_i)  (j <= i),   dP_ij = do_i . v_j,   delta_i = do_i . o_i
//   dS = P (dP - delta) / sqrt(d);   dv_j = sum_i P_ij do_i;   dk_j = sum_i dS_ij q_i;   dq_i = sum_j dS_ij k_j
//   then the rotary step backwards (rotation by the negative angle) on dq and dk.
//
// fp16 storage, fp32 accumulation on the MFMA units; P and dS pass through fp16 before the products that
// consume them (fp16 training holds them as fp16 tensors); dq, dk, dv are rounded once, after the rotation.
//
// Two deterministic kernels, no atomics.  The first: a workgroup per (sequence, head, block of queries) forms delta, walks
// the key blocks up to the diagonal and accumulates dq.  The second: a workgroup per (sequence, head, block of keys) walks
// the query blocks from the diagonal on and accumulates dk, dv.  Both recompute S, P, dP, dS, in blocks of 32 x 32 per
// wave that lie with the wave's own rows along the lanes (see lomo_attention_common.h): rotary pairs, P and dS never leave the
// lane pair that made them.  Sequences of one block have a kernel that does both from one copy of the rows in LDS.
//
// Measured, us, against 64 x 64 blocks over four waves with P and dS through LDS, tiles through registers and delta by a kernel of its
// own: 1 x 8192 tokens, 32 heads 2552 -> 1897 (724 TFLOP/s of the five products, 1013 of the seven executed); 8 x 1024, 40 heads 593 -> 455;
// 8 x 512, 32 heads 179 -> 133; 1 x 1024 93 -> 73; 3 x 320 41.8 -> 38.3; 128 x 64
// (one block) 198 -> 163.
#include "lomo_attention_common.h"

namespace lomo {

namespace attn {

constexpr int XCH_BYTES = 4 * 2 * 64 * 16;                      // SPLIT = 2: two fragments of each wave
constexpr int STAT_BYTES = 2 * 2 * BLK * 4;                     // lse and delta of a pair's queries
template <int SPLIT>
constexpr int DQ_LDS_BYTES = LDS_BYTES + (SPLIT == 2 ? XCH_BYTES : 0);
template <int SPLIT>
constexpr int DKDV_LDS_BYTES = DQ_LDS_BYTES<SPLIT> + STAT_BYTES;
constexpr int BLOCK_STAT_BYTES = 2 * BLK * 4, BLOCK_LDS_BYTES = 2 * PAIR * 2 + BLOCK_STAT_BYTES;      // both pairs of one block

struct Args {
    const uint16_t* qkv;   // [T x 3H]
    const uint16_t* o;     // [T x H]
    const uint16_t* dO;    // [T x H]
    const float* lse;      // [T x nh]
    float* delta;          // [T x nh], written by the dq kernel
    const float* cosv;     // [s x 64] or null
    const float* sinv;
    uint16_t* dqkv;        // [T x 3H]
    int s, nh, H;
};

// The rotary step backwards on the lane's row at position `pos`: the pair (c, c + 64) lies in the same register of acc[i] and
// acc[i + N / 2], which have columns 32 (first + i) and 32 (first + i) + 64.
template <int N>
__device__ __forceinline__ void rotate_back(floatx16 (&acc)[N], const Args& a, int pos, int first = 0) {
    const int lh = (threadIdx.x & 63) >> 5;
#pragma unroll
    for (int i = 0; i < N / 2; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int64_t at = (int64_t)pos * 64 + 32 * (first + i) + 8 * g + 4 * lh;
            const float4 co = *reinterpret_cast<const float4*>(a.cosv + at);
            const float4 si = *reinterpret_cast<const float4*>(a.sinv + at);
            const float cc[4] = {co.x, co.y, co.z, co.w}, ss[4] = {si.x, si.y, si.z, si.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float x1 = acc[i][4 * g + e], x2 = acc[i + N / 2][4 * g + e];
                float y1 = fmaf(x2, ss[e], x1 * cc[e]), y2 = fmaf(-x1, ss[e], x2 * cc[e]);
                asm volatile("" : "+v"(y1), "+v"(y2));      // rounded to fp32 before they are to fp16
                acc[i][4 * g + e] = y1;
                acc[i + N / 2][4 * g + e] = y2;
            }
        }
}

// dS = (p / sqrt(d)) (dP - delta) in fp16.  The product is rounded to fp32 and then to fp16, as a packed conversion does it; in
// the diagonal's blocks, where values are masked one by one, to fp16 at once.
__device__ __forceinline__ uint32_t times_once(float a, float b) {
    uint32_t x;
    asm("v_fma_mixlo_f16 %0, %1, %2, 0\n\ts_nop 1" : "=v"(x) : "v"(a), "v"(b));      // the wait: a register of which half was written is not read at once
    return x & 0xffffu;
}
// A packed pair of a diagonal block, zero where the mask takes it; the branch around it stays one (most blocks have no mask).
__device__ __forceinline__ uint32_t masked_pair(uint32_t lo, uint32_t hi, bool no_lo, bool no_hi) {
    asm volatile("" : "+v"(lo), "+v"(hi));
    uint32_t v = (no_lo ? 0u : lo) | (no_hi ? 0u : hi << 16);
    asm volatile("" : "+v"(v));
    return v;
}

// do . o of the lane's row: sums of eight columns, then in pairs.
__device__ __forceinline__ float row_product(const half8 (&fo)[D / 16], const half8 (&fd)[D / 16]) {
    float sum[D / 16];
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) {
        sum[ks] = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) sum[ks] = fmaf((float)fo[ks][e], (float)fd[ks][e], sum[ks]);
    }
#pragma unroll
    for (int n2 = D / 32; n2 > 0; n2 >>= 1)
#pragma unroll
        for (int ks = 0; ks < n2; ++ks) sum[ks] += sum[ks + n2];
    typedef uint32_t u32x2v __attribute__((ext_vector_type(2)));
    const u32x2v sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(sum[0]), __float_as_uint(sum[0]), false, false);
    return __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
}
// exp(x) is the hardware's 2^y with y = x log2(e): its relative error (about 1e-6 for |x| < 30) is far below half an fp16 ulp.
// dS of keys 32 h .. + 31 of a pair of tiles and the wave's queries qw ..; diag: the pair has the queries' positions among its own.
__device__ __forceinline__ void query_gradients(const TileRead& r0, const half8 (&fq)[D / 16], const half8 (&fd)[D / 16], float lq, float delta, int qw,
                                            int h, bool diag, half8 (&f)[2]) {
    const int l32 = threadIdx.x & 31, lh = (threadIdx.x & 63) >> 5;
    floatx16 S, P;
#pragma unroll
    for (int r = 0; r < 16; ++r) S[r] = P[r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) {
        S = __builtin_amdgcn_mfma_f32_32x32x16_f16(r0.rows(0, ks), fq[ks], S, 0, 0, 0);
        P = __builtin_amdgcn_mfma_f32_32x32x16_f16(r0.rows(TILE, ks), fd[ks], P, 0, 0, 0);
    }
    interleave<4, 2, 2, 6, 4>();
    __builtin_amdgcn_sched_barrier(0);
    uint32_t pk[8];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        S[r] = SCALE * __builtin_amdgcn_exp2f(fmaf(SCALE * LOG2E, S[r], -lq));
        P[r] -= delta;
    }
    if (diag) {
        auto ahead = [&](int r) { return 32 * h + 8 * (r >> 2) + 4 * lh + (r & 3) > (qw & 32) + l32; };
#pragma unroll
        for (int r = 0; r < 16; r += 2) pk[r >> 1] = masked_pair(times_once(S[r], P[r]), times_once(S[r + 1], P[r + 1]), ahead(r), ahead(r + 1));
    } else {
#pragma unroll
        for (int r = 0; r < 16; r += 2) pk[r >> 1] = pack2(S[r] * P[r], S[r + 1] * P[r + 1]);
    }
    __builtin_amdgcn_sched_barrier(0);
    f[0] = fragment_of(pk, 0);
    f[1] = fragment_of(pk, 1);
}
// P and dS of queries 32 h .. + 31 of a pair of tiles and the wave's keys kw ..; diag: the pair has the keys' positions among its own.
__device__ __forceinline__ void key_gradients(const TileRead& r0, const float* sL, const half8 (&fk)[D / 16], const half8 (&fv)[D / 16], int kw, int h,
                                          bool diag, uint32_t (&pp)[8], uint32_t (&pd)[8]) {
    const int l32 = threadIdx.x & 31, lh = (threadIdx.x & 63) >> 5;
    floatx16 S, P;
#pragma unroll
    for (int r = 0; r < 16; ++r) S[r] = P[r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) {
        S = __builtin_amdgcn_mfma_f32_32x32x16_f16(r0.rows(0, ks), fk[ks], S, 0, 0, 0);
        P = __builtin_amdgcn_mfma_f32_32x32x16_f16(r0.rows(TILE, ks), fv[ks], P, 0, 0, 0);
    }
    interleave<4, 2, 2, 6, 4>();
    __builtin_amdgcn_sched_barrier(0);
    // register r <-> query 8 (r / 4) + 4 lh + r % 4
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const float4 l4 = *reinterpret_cast<const float4*>(sL + 8 * g), d4 = *reinterpret_cast<const float4*>(sL + BLK + 8 * g);
        const float lq[4] = {l4.x, l4.y, l4.z, l4.w}, dq[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            S[4 * g + e] = __builtin_amdgcn_exp2f(fmaf(SCALE * LOG2E, S[4 * g + e], -lq[e]));
            P[4 * g + e] -= dq[e];
        }
        if (g == 1) __builtin_amdgcn_sched_barrier(0);
    }
    if (diag) {
        auto above = [&](int r) { return (kw & 32) + l32 > 32 * h + 8 * (r >> 2) + 4 * lh + (r & 3); };
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
            const uint32_t p2 = pack2(S[r], S[r + 1]);
            pd[r >> 1] = masked_pair(times_once(SCALE * S[r], P[r]), times_once(SCALE * S[r + 1], P[r + 1]), above(r), above(r + 1));
            pp[r >> 1] = masked_pair(p2 & 0xffffu, p2 >> 16, above(r), above(r + 1));
        }
    } else {
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
            pp[r >> 1] = pack2(S[r], S[r + 1]);
            pd[r >> 1] = pack2(SCALE * S[r] * P[r], SCALE * S[r + 1] * P[r + 1]);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
}

// The exchange of SPLIT = 2: two fragments of this wave, of its partner (the wave with the same rows and the other half).
struct Exchange {
    half8 *own, *other;
    __device__ __forceinline__ Exchange(uint16_t* lds, int wave) {
        half8* x = reinterpret_cast<half8*>(lds) + (threadIdx.x & 63);
        own = x + wave * 128;
        other = x + (wave ^ 2) * 128;
    }
    __device__ __forceinline__ void put(const half8 (&f)[2]) const {
        own[0] = f[0];
        own[64] = f[1];
    }
    __device__ __forceinline__ void get(half8 (&f)[2]) const {
        f[0] = other[0];
        f[1] = other[64];
    }
};
// LDS writes are visible to the other waves; the moving tiles' loads stay in flight
__device__ __forceinline__ void meet() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

}  // namespace attn

template <int SPLIT>
__global__ __launch_bounds__(256, 2) void attention_backward_dq_kernel(attn::Args a) {
    using namespace attn;
    extern __shared__ __attribute__((aligned(256))) uint16_t smem[];      // two pairs of tiles: K, V

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int part = SPLIT == 2 ? wave >> 1 : 0;             // which half of the tiles
    const int l32 = lane & 31, lh = lane >> 5;
    const uint32_t lds0 = (uint32_t)(uintptr_t)smem;

    const int nb = (a.s + ROWS<SPLIT> - 1) / ROWS<SPLIT>;
    int head, within;
    locate_block(nb, head, within);
    const int n = head % a.nh, b = head / a.nh;
    // heaviest blocks first, counted from the sequence's end: one that is not full has the lightest rows (of 192 tokens four pairs of tiles are
    // walked instead of five; 32 x 192 tokens, 32 heads, with the dk / dv kernel 159.5 -> 156 us, 42 x 192, 8 heads 66.6 -> 60.4)
    const int q0 = a.s - (within + 1) * ROWS<SPLIT>;
    const int qw = q0 + 32 * (SPLIT == 2 ? wave & 1 : wave);      // this wave's queries
    const bool active = qw >= 0;                             // s is a multiple of 64
    const int last = (q0 + ROWS<SPLIT> - 1) / BLK;      // key blocks of the workgroup
    const int64_t ld3 = 3 * (int64_t)a.H, ldh = a.H;
    const int64_t t0 = (int64_t)b * a.s;
    const uint16_t* gq = a.qkv + (int64_t)n * D;
    const uint16_t* gk = gq + a.H + t0 * ld3;
    const uint16_t* gv = gk + a.H;
    const int64_t t = t0 + qw + l32;                         // the lane's query

    const TileLoad load(ld3);
    const TileRead rd(lds0);
    auto fetch = [&](int blk, int buf) {
        const int64_t off = (int64_t)blk * BLK * ld3;
        load.issue(gk + off, lds0 + (uint32_t)buf * (PAIR * 2u), wave);
        load.issue(gv + off, lds0 + (uint32_t)buf * (PAIR * 2u) + TILE * 2u, wave);
    };
    fetch(0, 0);

    half8 fq[D / 16], fd[D / 16];
    float lq = 0.f, delta = 0.f;
    if (active) {
        load_fragments(fq, gq + t * ld3);
        load_fragments(fd, a.dO + t * ldh + (int64_t)n * D);
        half8 fo[D / 16];
        load_fragments(fo, a.o + t * ldh + (int64_t)n * D);
        lq = a.lse[t * a.nh + n] * LOG2E;
        delta = row_product(fo, fd);
        if (lh == 0 && part == 0) a.delta[t * a.nh + n] = delta;
    }

    constexpr int NT = 4 / SPLIT;      // dq's tiles of 32 columns: of two waves with the same rows each has part and part + 2
    floatx16 acc[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;

    constexpr int K = 0, V = TILE;      // in the pair
    auto gradients = [&](const TileRead& r0, int h, bool diag, half8 (&f)[2]) { query_gradients(r0, fq, fd, lq, delta, qw, h, diag, f); };
    // dq^T[dcol][query] += k^T[dcol][key] dS^T[key][query], 16 keys at a time
    auto multiply = [&](const TileRead& r0, const half8 (&f)[2]) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int i = 0; i < NT; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(r0.columns(K, SPLIT * i, ks), f[ks], acc[i], 0, 0, 0);
        if constexpr (SPLIT == 1) interleave<4, 1, 2, 6, 2>();
        else interleave<4, 1, 2, 2, 2>();
        __builtin_amdgcn_sched_barrier(0);
    };

    const Exchange xch(smem + 2 * PAIR, wave);
    for (int blk = 0; blk <= last; ++blk) {
        const int buf = blk & 1;
        // the block's tiles have landed; everybody is done with the other pair
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (blk < last) fetch(blk + 1, buf ^ 1);      // in flight while this block is multiplied
        if constexpr (SPLIT == 1) {
            if (!active) continue;
#pragma nounroll
            for (int h = 0; h < 2; ++h) {
                const int ahead = qw / 32 - (2 * blk + h);      // of this half's keys
                if (ahead < 0) continue;
                const TileRead r0 = rd.at(buf * PAIR + 32 * h * D);
                half8 f[2];
                gradients(r0, h, blk == qw / BLK, f);
                multiply(r0, f);
            }
        } else {
            const int ahead = qw / 32 - 2 * blk;      // of the first half's keys
            const TileRead own = rd.at(buf * PAIR + 32 * part * D), other = rd.at(buf * PAIR + 32 * (1 - part) * D);
            half8 f[2], g[2];
            if (ahead >= part) {
                gradients(own, part, blk == last, f);
                xch.put(f);
            }
            meet();
            if (part == 1) {
                xch.get(g);
                multiply(other.column_tile(1), g);
                if (ahead >= 1) multiply(own.column_tile(1), f);
            } else {
                multiply(own, f);
                if (ahead >= 1) {
                    xch.get(g);
                    multiply(other, g);
                }
            }
        }
    }
    if (!active) return;
    if (a.cosv != nullptr) rotate_back(acc, a, qw + l32, part);
    store_rows(acc, a.dqkv + t * ld3 + (int64_t)n * D, part);
}

template <int SPLIT>
__global__ __launch_bounds__(256, 2) void attention_backward_dkdv_kernel(attn::Args a) {
    using namespace attn;
    extern __shared__ __attribute__((aligned(256))) uint16_t smem[];      // lse and delta of two pairs of tiles; the pairs: Q, dO

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int part = SPLIT == 2 ? wave >> 1 : 0;             // which half of the tiles
    const int l32 = lane & 31, lh = lane >> 5;
    uint16_t* tiles = smem + STAT_BYTES / 2;
    const uint32_t lds0 = (uint32_t)(uintptr_t)tiles;
    float* stats = reinterpret_cast<float*>(smem);      // [pair][lse log2(e) | delta][64]

    const int nb = (a.s + ROWS<SPLIT> - 1) / ROWS<SPLIT>;
    int head, within;
    locate_block(nb, head, within);
    const int n = head % a.nh, b = head / a.nh;
    const int k0 = within * ROWS<SPLIT>;          // heaviest blocks first
    const int kw = k0 + 32 * (SPLIT == 2 ? wave & 1 : wave);      // this wave's keys
    const bool active = kw < a.s;                            // s is a multiple of 64
    const int first = k0 / BLK, last = a.s / BLK - 1;
    const int64_t ld3 = 3 * (int64_t)a.H, ldh = a.H;
    const int64_t t0 = (int64_t)b * a.s;
    const uint16_t* gq = a.qkv + (int64_t)n * D + t0 * ld3;
    const uint16_t* gdo = a.dO + (int64_t)n * D + t0 * ldh;
    const float* gstat = (wave == 0 ? a.lse : a.delta) + t0 * a.nh + n;      // wave 0 and 1
    const int64_t t = t0 + kw + l32;                         // the lane's key

    const TileLoad load_q(ld3), load_do(ldh);
    float stat = 0.f;
    TileRead rd(lds0);
    auto fetch = [&](int blk, int buf) {
        load_q.issue(gq + (int64_t)blk * BLK * ld3, lds0 + (uint32_t)buf * (PAIR * 2u), wave);
        load_do.issue(gdo + (int64_t)blk * BLK * ldh, lds0 + (uint32_t)buf * (PAIR * 2u) + TILE * 2u, wave);
        if (wave < 2) stat = gstat[((int64_t)blk * BLK + lane) * a.nh];
    };
    fetch(first, 0);

    half8 fk[D / 16], fv[D / 16];
    if (active) {
        load_fragments(fk, a.qkv + a.H + (int64_t)n * D + t * ld3);
        load_fragments(fv, a.qkv + 2 * (int64_t)a.H + (int64_t)n * D + t * ld3);
    }

    constexpr int Q = 0, DO = TILE;      // in the pair
    // dv, dk; SPLIT = 2: the first of two waves with the same keys has dv, the second dk
    floatx16 acc[2 / SPLIT][4];
#pragma unroll
    for (int x = 0; x < 2 / SPLIT; ++x)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[x][i][r] = 0.f;

    auto gradients = [&](const TileRead& r0, const float* sL, int h, bool diag, uint32_t (&pp)[8], uint32_t (&pd)[8]) {
        key_gradients(r0, sL, fk, fv, kw, h, diag, pp, pd);
    };

    const Exchange xch(tiles + 2 * PAIR, wave);
    int at = 0;      // where rd is (SPLIT = 1)
    for (int blk = first; blk <= last; ++blk) {
        const int buf = (blk - first) & 1;
        if (wave < 2) stats[(2 * buf + wave) * BLK + lane] = wave == 0 ? stat * LOG2E : stat;
        // the block's tiles have landed; everybody is done with the other pair
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (blk < last) fetch(blk + 1, buf ^ 1);      // in flight while this block is multiplied
        const float* sL = stats + 2 * buf * BLK + 4 * lh;
        uint32_t pp[8], pd[8];
        if constexpr (SPLIT == 1) {
            if (!active) continue;
#pragma nounroll
            for (int h = 0; h < 2; ++h) {
                const int behind = 2 * blk + h - kw / 32;      // this half's queries
                if (behind < 0) continue;
                const int to = buf * PAIR + 32 * h * D;
                rd.move(to - at);
                at = to;
                gradients(rd, sL + 32 * h, h, blk == kw / BLK, pp, pd);
                // dv^T[dcol][key] += dO^T P,  dk^T[dcol][key] += q^T dS, 16 queries at a time
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) {
                    const half8 fp = fragment_of(pp, ks), fd = fragment_of(pd, ks);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        acc[0][i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(rd.columns(DO, i, ks), fp, acc[0][i], 0, 0, 0);
                        acc[1][i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(rd.columns(Q, i, ks), fd, acc[1][i], 0, 0, 0);
                    }
                }
                interleave<4, 1, 2, 14, 2>();
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
            const int behind = 2 * blk - kw / 32;      // the first half's queries
            // half h's share in dv (of P) or dk (of dS)
            auto multiply = [&](int h, const half8 (&f)[2]) {
                const TileRead r0 = rd.at(buf * PAIR + (part == 0 ? DO : Q) + 32 * h * D);
#pragma unroll
                for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[0][i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(r0.columns(0, i, ks), f[ks], acc[0][i], 0, 0, 0);
                interleave<4, 1, 2, 6, 2>();
                __builtin_amdgcn_sched_barrier(0);
            };
            const bool computes = behind + part >= 0;
            half8 f[2], g[2];      // the fragments that this wave multiplies, its partner's
            if (computes) {
                gradients(rd.at(buf * PAIR + 32 * part * D), sL + 32 * part, part, blk == first, pp, pd);
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) {
                    f[ks] = part == 0 ? fragment_of(pp, ks) : fragment_of(pd, ks);
                    g[ks] = part == 0 ? fragment_of(pd, ks) : fragment_of(pp, ks);
                }
                xch.put(g);
            }
            meet();
            if (part == 0) {
                if (computes) multiply(0, f);
                xch.get(g);
                multiply(1, g);
            } else {
                if (behind >= 0) {
                    xch.get(g);
                    multiply(0, g);
                }
                multiply(1, f);
            }
        }
    }
    if (!active) return;
    uint16_t* out = a.dqkv + t * ld3 + (int64_t)n * D;
    if (SPLIT == 1 || part == 0) store_rows(acc[0], out + 2 * (int64_t)a.H);
    if (SPLIT == 1 || part == 1) {
        if (a.cosv != nullptr) rotate_back(acc[2 / SPLIT - 1], a, kw + l32);
        store_rows(acc[2 / SPLIT - 1], out + a.H);
    }
}

// Sequences of one block: a workgroup of two waves has q, k, v and do of a (sequence, head) pair in LDS, reads them once and does what the two
// kernels above do, in their order (the bits are theirs); two workgroups on a CU.  Bytes bound it.  Measured, us, 32 heads with the rotary
// step, the two kernels -> this: 1 x 64 tokens 17.2 -> 12.4, 32 x 64 56 -> 46, 64 x 64 89 -> 74, 128 x 64 213 -> 163 (537 MB, 3.3 TB/s; the two
// kernels read 268 MB of them again).  Whole rows stored through LDS instead of 32-byte pieces: 164, without the rotary step 138 -> 124.
__global__ __launch_bounds__(128, 1) void attention_backward_block_kernel(attn::Args a) {
    using namespace attn;
    extern __shared__ __attribute__((aligned(256))) uint16_t smem[];      // lse and delta; K, V, Q, dO

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31, lh = lane >> 5;
    float* stats = reinterpret_cast<float*>(smem);      // [lse log2(e) | delta][64]
    const uint32_t lds0 = (uint32_t)(uintptr_t)(smem + BLOCK_STAT_BYTES / 2);

    int head, within;
    locate_block(1, head, within);
    const int n = head % a.nh, b = head / a.nh;
    const int w0 = 32 * wave;                                // this wave's queries, its keys
    const int64_t ld3 = 3 * (int64_t)a.H, ldh = a.H;
    const int64_t t0 = (int64_t)b * BLK, t = t0 + w0 + l32;
    const uint16_t* gq = a.qkv + (int64_t)n * D + t0 * ld3;
    const TileLoad load(ld3), load_do(ldh);
    load.issue<2>(gq + a.H, lds0, wave);
    load.issue<2>(gq, lds0 + PAIR * 2u, wave);
    load_do.issue<2>(a.dO + (int64_t)n * D + t0 * ldh, lds0 + (PAIR + TILE) * 2u, wave);
    load.issue<2>(gq + 2 * (int64_t)a.H, lds0 + TILE * 2u, wave);
    half8 fo[D / 16];
    load_fragments(fo, a.o + t * ldh + (int64_t)n * D);
    const float lq = a.lse[t * a.nh + n] * LOG2E;
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");

    const TileRead kv(lds0), qd = kv.at(PAIR);
    half8 fx[D / 16], fy[D / 16];      // q and do, then k and v
    auto own_rows = [&](const TileRead& tile) {
        const TileRead r0 = tile.at(w0 * D);
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) {
            fx[ks] = r0.rows(0, ks);
            fy[ks] = r0.rows(TILE, ks);
        }
    };
    own_rows(qd);
    const float delta = row_product(fo, fy);
    if (lh == 0) {
        a.delta[t * a.nh + n] = delta;
        stats[w0 + l32] = lq;
        stats[BLK + w0 + l32] = delta;
    }

    floatx16 acc[2][4];
    auto clear = [&](floatx16 (&x)[4]) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) x[i][r] = 0.f;
    };
    clear(acc[0]);
#pragma nounroll
    for (int h = 0; h <= wave; ++h) {
        const TileRead r0 = kv.at(32 * h * D);
        half8 f[2];
        query_gradients(r0, fx, fy, lq, delta, w0, h, true, f);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[0][i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(r0.columns(0, i, ks), f[ks], acc[0][i], 0, 0, 0);
    }
    uint16_t* out = a.dqkv + t * ld3 + (int64_t)n * D;
    if (a.cosv != nullptr) rotate_back(acc[0], a, w0 + l32);
    store_rows(acc[0], out);

    __syncthreads();             // lse and delta of all queries
    own_rows(kv);
    clear(acc[0]);
    clear(acc[1]);
#pragma nounroll
    for (int h = wave; h < 2; ++h) {
        const TileRead r0 = qd.at(32 * h * D);
        uint32_t pp[8], pd[8];
        key_gradients(r0, stats + 32 * h + 4 * lh, fx, fy, w0, h, true, pp, pd);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const half8 fp = fragment_of(pp, ks), fd = fragment_of(pd, ks);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                acc[0][i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(r0.columns(TILE, i, ks), fp, acc[0][i], 0, 0, 0);
                acc[1][i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(r0.columns(0, i, ks), fd, acc[1][i], 0, 0, 0);
            }
        }
    }
    store_rows(acc[0], out + 2 * (int64_t)a.H);
    if (a.cosv != nullptr) rotate_back(acc[1], a, w0 + l32);
    store_rows(acc[1], out + a.H);
}

template <int SPLIT>
static hipError_t launch(const attn::Args& a, int64_t B, hipStream_t st) {
    using namespace attn;
    auto dq = attention_backward_dq_kernel<SPLIT>;
    auto dkdv = attention_backward_dkdv_kernel<SPLIT>;
    // thread-safe one-time set-up (initialisation of a function-local static)
    static const hipError_t cfg0 = allow_dynamic_lds(dq, DQ_LDS_BYTES<SPLIT>);
    if (cfg0 != hipSuccess) return cfg0;
    static const hipError_t cfg1 = allow_dynamic_lds(dkdv, DKDV_LDS_BYTES<SPLIT>);
    if (cfg1 != hipSuccess) return cfg1;
    const dim3 grid((unsigned)(((int64_t)a.s + ROWS<SPLIT> - 1) / ROWS<SPLIT> * a.nh * B));
    hipLaunchKernelGGL(dq, grid, dim3(256), DQ_LDS_BYTES<SPLIT>, st, a);
    hipLaunchKernelGGL(dkdv, grid, dim3(256), DKDV_LDS_BYTES<SPLIT>, st, a);
    return hipGetLastError();
}

static hipError_t launch_block(const attn::Args& a, int64_t B, hipStream_t st) {
    using namespace attn;
    static const hipError_t cfg = allow_dynamic_lds(attention_backward_block_kernel, BLOCK_LDS_BYTES);
    if (cfg != hipSuccess) return cfg;
    hipLaunchKernelGGL(attention_backward_block_kernel, dim3((unsigned)(a.nh * B)), dim3(128), BLOCK_LDS_BYTES, st, a);
    return hipGetLastError();
}

hipError_t launch_attention_backward(const uint16_t* qkv, const uint16_t* o, const uint16_t* dO, const float* lse,
                                     const float* cosv, const float* sinv, float* delta, uint16_t* dqkv, int64_t B, int64_t s,
                                     int64_t nh, hipStream_t st) {
    attn::Args a;
    a.qkv = qkv; a.o = o; a.dO = dO; a.lse = lse; a.delta = delta; a.cosv = cosv; a.sinv = sinv; a.dqkv = dqkv;
    a.s = (int)s; a.nh = (int)nh; a.H = (int)(nh * attn::D);
    if (s <= attn::BLK) return launch_block(a, B, st);
    // not split / split, us: 3 x 320 tokens, 32 heads 43 / 38, 8 x 128 (4 waves per CU) 30.3 / 30.9, 5 x 448, 16 heads (4.4) 51.5 / 49.4, 3 x 448, 32 heads (5.3)
    // 56 / 60;  1 x 1024 (4) 86 / 73, 1 x 1536 (6) 129 / 118, 7 x 1024, 8 heads (7) 103 / 107, 1 x 2048, 32 heads (8) 178 / 186
    const double waves = attn::waves_per_cu(B, s, nh);
    return waves < 4.0 || (s >= 384 && waves <= 5.0) || (s >= 1024 && waves < 7.0) ? launch<2>(a, B, st) : launch<1>(a, B, st);
}

}  // namespace lomo
