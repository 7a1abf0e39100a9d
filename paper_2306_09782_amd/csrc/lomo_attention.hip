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
// lane pair that made them.
//
// Measured, us, against the kernels before (64 x 64 blocks over four waves, P and dS through LDS, tiles through registers, delta
// by a kernel of its own): 1 x 8192 tokens, 32 heads 2545 -> 1945 (706 TFLOP/s of the five products, 988 of the seven executed);
// 8 x 1024, 40 heads 668 -> 554; 8 x 512, 32 heads 170 -> 140; 1 x 1024 93 -> 79; 3 x 320 41 -> 41.  At 8192 tokens the matrix pipes are
// 53 % (dq) and 49 % (dk, dv) busy at 1.85 GHz.  A quarter fewer vector instructions (scales folded into lse and delta)
// gave 1 %.
#include "lomo_attention_common.h"

namespace lomo {

namespace attn {

constexpr int BWD_LDS_BYTES = LDS_BYTES + 2 * 2 * BLK * 4;      // + lse and delta of a pair's queries

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
// acc[i + 2].
__device__ __forceinline__ void rotate_back(floatx16 (&acc)[4], const Args& a, int pos) {
    const int lh = (threadIdx.x & 63) >> 5;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const float4 co = *reinterpret_cast<const float4*>(a.cosv + (int64_t)pos * 64 + 32 * i + 8 * g + 4 * lh);
            const float4 si = *reinterpret_cast<const float4*>(a.sinv + (int64_t)pos * 64 + 32 * i + 8 * g + 4 * lh);
            const float cc[4] = {co.x, co.y, co.z, co.w}, ss[4] = {si.x, si.y, si.z, si.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float x1 = acc[i][4 * g + e], x2 = acc[i + 2][4 * g + e];
                acc[i][4 * g + e] = fmaf(x2, ss[e], x1 * cc[e]);
                acc[i + 2][4 * g + e] = fmaf(-x1, ss[e], x2 * cc[e]);
            }
        }
}

}  // namespace attn

// exp(x) is the hardware's 2^y with y = x log2(e): its relative error (about 1e-6 for |x| < 30) is far below half an fp16 ulp.

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
    const int pos = xcd_position();
    const int head = pos / nb, within = pos - head * nb;
    const int n = head % a.nh, b = head / a.nh;
    const int q0 = (nb - 1 - within) * ROWS<SPLIT>;          // heaviest blocks first
    const int qw = q0 + 32 * (SPLIT == 2 ? wave & 1 : wave);      // this wave's queries
    const bool active = qw < a.s;                            // s is a multiple of 64
    const int last = ((q0 + ROWS<SPLIT> < a.s ? q0 + ROWS<SPLIT> : a.s) - 1) / BLK;      // key blocks of the workgroup
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
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks)
#pragma unroll
            for (int e = 0; e < 8; ++e) delta = fmaf((float)fo[ks][e], (float)fd[ks][e], delta);
        typedef uint32_t u32x2v __attribute__((ext_vector_type(2)));
        const u32x2v sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(delta), __float_as_uint(delta), false, false);
        delta = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
        if (lh == 0 && part == 0) a.delta[t * a.nh + n] = delta;
    }

    const float scaled_delta = SCALE * delta;

    floatx16 acc[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;

    // Keys 32 h .. + 31 of the pair in `buf` against this wave's queries; diag: they have the queries' positions.
    auto block = [&](int buf, int h, bool diag) {
        const TileRead r0 = rd.at(buf * PAIR + 32 * h * D);
        constexpr int sK = 0, sV = TILE;      // in the pair
        floatx16 S, P;
#pragma unroll
        for (int r = 0; r < 16; ++r) S[r] = P[r] = 0.f;
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) {
            S = __builtin_amdgcn_mfma_f32_32x32x16_f16(r0.rows(sK, ks), fq[ks], S, 0, 0, 0);
            P = __builtin_amdgcn_mfma_f32_32x32x16_f16(r0.rows(sV, ks), fd[ks], P, 0, 0, 0);
        }
        interleave<4, 2, 2, 6, 4>();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float p = __builtin_amdgcn_exp2f(fmaf(SCALE * LOG2E, S[r], -lq));
            P[r] = p * fmaf(SCALE, P[r], -scaled_delta);
        }
        if (diag) {
            mask(P, [&](int r) { return 8 * (r >> 2) + 4 * lh + (r & 3) > l32; });
        }
        uint32_t pk[8];
#pragma unroll
        for (int r = 0; r < 16; r += 2) pk[r >> 1] = pack2(P[r], P[r + 1]);
        __builtin_amdgcn_sched_barrier(0);
        // dq^T[dcol][query] += k^T[dcol][key] dS^T[key][query], 16 keys at a time
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const half8 f = fragment_of(pk, ks);
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(r0.columns(sK, i, ks), f, acc[i], 0, 0, 0);
        }
        interleave<4, 1, 2, 6, 2>();
        __builtin_amdgcn_sched_barrier(0);
    };

    for (int blk = 0; blk <= last; ++blk) {
        const int buf = blk & 1;
        // the block's tiles have landed; everybody is done with the other pair
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (blk < last) fetch(blk + 1, buf ^ 1);      // in flight while this block is multiplied
        if (!active) continue;
#pragma nounroll
        for (int h = part; h < (SPLIT == 2 ? part + 1 : 2); ++h) {
            const int ahead = qw / 32 - (2 * blk + h);      // of this half's keys
            if (ahead >= 0) block(buf, h, ahead == 0);
        }
    }
    if constexpr (SPLIT == 2) {
        float* xch = reinterpret_cast<float*>(smem) + (wave & 1) * 64 * 64 + lane;
        __syncthreads();      // the tiles are free
        if (part == 1) put_registers(acc, xch);
        __syncthreads();
        if (part == 1) return;
        add_registers(acc, xch);
    }
    if (!active) return;
    if (a.cosv != nullptr) rotate_back(acc, a, qw + l32);
    store_rows(acc, 1.f, a.dqkv + t * ld3 + (int64_t)n * D);
}

template <int SPLIT>
__global__ __launch_bounds__(256, 2) void attention_backward_dkdv_kernel(attn::Args a) {
    using namespace attn;
    extern __shared__ __attribute__((aligned(256))) uint16_t smem[];      // two pairs of tiles: Q, dO; their lse and delta

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int part = SPLIT == 2 ? wave >> 1 : 0;             // which half of the tiles
    const int l32 = lane & 31, lh = lane >> 5;
    const uint32_t lds0 = (uint32_t)(uintptr_t)smem;
    float* stats = reinterpret_cast<float*>(smem + 2 * PAIR);      // [pair][lse log2(e) | delta / sqrt(d)][64]

    const int nb = (a.s + ROWS<SPLIT> - 1) / ROWS<SPLIT>;
    const int pos = xcd_position();
    const int head = pos / nb;
    const int n = head % a.nh, b = head / a.nh;
    const int k0 = (pos - head * nb) * ROWS<SPLIT>;          // heaviest blocks first
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
    const TileRead rd(lds0);
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

    floatx16 dk[4], dv[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) dk[i][r] = dv[i][r] = 0.f;

    // Queries 32 h .. + 31 of the pair in `buf` against this wave's keys; diag: they have the keys' positions.
    auto block = [&](int buf, int h, bool diag) {
        const TileRead r0 = rd.at(buf * PAIR + 32 * h * D);
        constexpr int sQ = 0, sD = TILE;      // in the pair
        const float* sL = stats + 2 * buf * BLK + 32 * h + 4 * lh;
        floatx16 S, P;
#pragma unroll
        for (int r = 0; r < 16; ++r) S[r] = P[r] = 0.f;
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) {
            S = __builtin_amdgcn_mfma_f32_32x32x16_f16(r0.rows(sQ, ks), fk[ks], S, 0, 0, 0);
            P = __builtin_amdgcn_mfma_f32_32x32x16_f16(r0.rows(sD, ks), fv[ks], P, 0, 0, 0);
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
                const int r = 4 * g + e;
                S[r] = __builtin_amdgcn_exp2f(fmaf(SCALE * LOG2E, S[r], -lq[e]));
                P[r] = S[r] * fmaf(SCALE, P[r], -dq[e]);
            }
        }
        if (diag) {
            auto above = [&](int r) { return l32 > 8 * (r >> 2) + 4 * lh + (r & 3); };
            mask(S, above);
            mask(P, above);
        }
        uint32_t pp[8], pd[8];
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
            pp[r >> 1] = pack2(S[r], S[r + 1]);
            pd[r >> 1] = pack2(P[r], P[r + 1]);
        }
        __builtin_amdgcn_sched_barrier(0);
        // dv^T[dcol][key] += dO^T P,  dk^T[dcol][key] += q^T dS, 16 queries at a time
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const half8 fp = fragment_of(pp, ks), fd = fragment_of(pd, ks);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                dv[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(r0.columns(sD, i, ks), fp, dv[i], 0, 0, 0);
                dk[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(r0.columns(sQ, i, ks), fd, dk[i], 0, 0, 0);
            }
        }
        interleave<4, 1, 2, 14, 2>();
        __builtin_amdgcn_sched_barrier(0);
    };

    for (int blk = first; blk <= last; ++blk) {
        const int buf = (blk - first) & 1;
        if (wave < 2) stats[(2 * buf + wave) * BLK + lane] = stat * (wave == 0 ? LOG2E : SCALE);
        // the block's tiles have landed; everybody is done with the other pair
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (blk < last) fetch(blk + 1, buf ^ 1);      // in flight while this block is multiplied
        if (!active) continue;
#pragma nounroll
        for (int h = part; h < (SPLIT == 2 ? part + 1 : 2); ++h) {
            const int behind = 2 * blk + h - kw / 32;      // this half's queries
            if (behind >= 0) block(buf, h, behind == 0);
        }
    }
    if constexpr (SPLIT == 2) {
        float* xch = reinterpret_cast<float*>(smem) + (wave & 1) * 128 * 64 + lane;
        __syncthreads();      // the tiles are free
        if (part == 1) {
            put_registers(dv, xch);
            put_registers(dk, xch + 64 * 64);
        }
        __syncthreads();
        if (part == 1) return;
        add_registers(dv, xch);
        add_registers(dk, xch + 64 * 64);
    }
    if (!active) return;
    uint16_t* out = a.dqkv + t * ld3 + (int64_t)n * D;
    store_rows(dv, 1.f, out + 2 * (int64_t)a.H);
    if (a.cosv != nullptr) rotate_back(dk, a, kw + l32);
    store_rows(dk, 1.f, out + a.H);
}

template <int SPLIT>
static hipError_t launch(const attn::Args& a, int64_t B, hipStream_t st) {
    using namespace attn;
    auto dq = attention_backward_dq_kernel<SPLIT>;
    auto dkdv = attention_backward_dkdv_kernel<SPLIT>;
    // thread-safe one-time set-up (initialisation of a function-local static)
    static const hipError_t cfg0 = allow_dynamic_lds(dq, LDS_BYTES);
    if (cfg0 != hipSuccess) return cfg0;
    static const hipError_t cfg1 = allow_dynamic_lds(dkdv, BWD_LDS_BYTES);
    if (cfg1 != hipSuccess) return cfg1;
    const dim3 grid((unsigned)(((int64_t)a.s + ROWS<SPLIT> - 1) / ROWS<SPLIT> * a.nh * B));
    hipLaunchKernelGGL(dq, grid, dim3(256), LDS_BYTES, st, a);
    hipLaunchKernelGGL(dkdv, grid, dim3(256), BWD_LDS_BYTES, st, a);
    return hipGetLastError();
}

hipError_t launch_attention_backward(const uint16_t* qkv, const uint16_t* o, const uint16_t* dO, const float* lse,
                                     const float* cosv, const float* sinv, float* delta, uint16_t* dqkv, int64_t B, int64_t s,
                                     int64_t nh, hipStream_t st) {
    attn::Args a;
    a.qkv = qkv; a.o = o; a.dO = dO; a.lse = lse; a.delta = delta; a.cosv = cosv; a.sinv = sinv; a.dqkv = dqkv;
    a.s = (int)s; a.nh = (int)nh; a.H = (int)(nh * attn::D);
    // below a workgroup of two waves per SIMD on every CU; not split / split, us: 1 x 1024 tokens, 32 heads (1024 waves) 88.8 / 78, 3 x 320 (960)
    // 50 / 40; 8 x 512 (4096) 145 not split
    return attn::attention_waves(B, s, nh) < 8 * cu_count() ? launch<2>(a, B, st) : launch<1>(a, B, st);
}

}  // namespace lomo
