// Forward of causal softmax attention (head width 128) on the rotated q, k and v, for recomputing the
// activations that Algorithm 1's backward loop reads from a checkpoint of the layer input (paper section 3.2;
// activation checkpointing: sections 2 and 4.1).  Produces o and lse = log sum_j exp(q_i . k_j / sqrt(d)) in
// the layout the backward kernel reads.
//
// One workgroup per (sequence, head, block of queries) walks the key blocks (64 keys) up to the diagonal; a wave owns 32
// queries.  The keys of the even and of the odd halves of the blocks (32 each) have a running maximum, a sum and an output
// accumulator of their own per query, put together at the end: with two maxima two probabilities of every query are exactly 1, which
// takes 6 to 10 % off what the roundings of the others do to o.  A workgroup of 128 queries holds both in one wave, one of 64
// has a wave for each (SPLIT = 2); the operations on a query and their order are the same, so o and lse do not depend on the
// size of the call.  The score tile is computed transposed (keys are the MFMA rows): a lane owns one query, its maximum is a
// scan of the lane's registers plus one exchange with lane + 32, and the probabilities become the B operand of o^T += v^T p^T
// through a v_permlane32_swap.  Probabilities are rounded to fp16 relative to the running maximum; accumulation is fp32; o is rounded
// once.  Deterministic.
//
// Measured, us, against a workgroup of 64 queries with the halves on different waves and tiles through registers: 1 x 8192 tokens, 32 heads
// 839 -> 673 (817 TFLOP/s); 8 x 1024, 40 heads 210 -> 172; 8 x 512, 32 heads 61 -> 43.6; 1 x 1024 31.5 -> 24.7; 3 x 320 13.2 -> 13.3.  Vector
// instructions are the limit: at short sequences most blocks move some query's maximum, which is 128 products a lane beside about
// 250 for the probabilities.
#include "lomo_attention_common.h"

namespace lomo {

namespace attn {

struct FwdArgs {
    const uint16_t* qkv;   // [T x 3H]
    uint16_t* o;           // [T x H]
    float* lse;            // [T x nh]
    int s, nh, H;
};

constexpr float C2 = SCALE * LOG2E;

}  // namespace attn

template <int SPLIT, typename Load>
__global__ __launch_bounds__(256, 2) void attention_forward_kernel(attn::FwdArgs a) {
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
    // walked instead of five; 32 x 192 tokens, 32 heads 53 -> 47 us, 42 x 192, 8 heads 23.0 -> 18.0, 12 x 448, 16 heads 33.7 -> 31.2)
    const int q0 = a.s - (within + 1) * ROWS<SPLIT>;
    const int qw = q0 + 32 * (SPLIT == 2 ? wave & 1 : wave);      // this wave's queries
    const bool active = qw >= 0;                             // s is a multiple of 64
    const int last = (q0 + ROWS<SPLIT> - 1) / BLK;      // key blocks of the workgroup, of this wave
    const int own_last = qw / BLK;
    const int64_t ld3 = 3 * (int64_t)a.H;
    const int64_t t0 = (int64_t)b * a.s;
    const uint16_t* gq = a.qkv + (int64_t)n * D;
    const uint16_t* gk = gq + a.H + t0 * ld3;
    const uint16_t* gv = gk + a.H;
    const int query = qw + l32;

    const Load load(ld3);
    const TileRead rd(lds0);
    auto fetch = [&](int blk, int buf) {
        const int64_t off = (int64_t)blk * BLK * ld3;
        load.issue(gk + off, lds0 + (uint32_t)buf * (PAIR * 2u), wave);
        load.issue(gv + off, lds0 + (uint32_t)buf * (PAIR * 2u) + TILE * 2u, wave);
    };
    fetch(0, 0);

    half8 fq[D / 16];
    if (active) load_fragments(fq, gq + (t0 + query) * ld3);

    // by half of the blocks that this wave has; log2 domain; l_run is this lane's share (its half of the keys)
    constexpr int STATES = 2 / SPLIT;
    floatx16 accO[STATES][4];
    float m_run[STATES], l_run[STATES];
#pragma unroll
    for (int h = 0; h < STATES; ++h) {
        m_run[h] = -INFINITY;
        l_run[h] = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) accO[h][i][r] = 0.f;
    }

    // Scores of keys 32 h .. + 31 of the pair in `buf` against this wave's queries.
    auto scores = [&](const TileRead& r0, floatx16& S) {
#pragma unroll
        for (int r = 0; r < 16; ++r) S[r] = 0.f;
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) S = __builtin_amdgcn_mfma_f32_32x32x16_f16(r0.rows(0, ks), fq[ks], S, 0, 0, 0);
    };
    // What they add to sum and output; diag: the block has the queries' positions among its own.
    auto half = [&](const TileRead& r0, int h, floatx16& S, floatx16 (&O)[4], float& m_run, float& l_run, bool diag) {
        // S[r] <-> key 32 h + 8 (r / 4) + 4 lh + r % 4 of the block
        float scale = C2, bmax = -INFINITY;
        if (diag) {      // scaled and masked; the branch stays one
            scale = 1.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                float x = 32 * h + 8 * (r >> 2) + 4 * lh + (r & 3) > (qw & 32) + l32 ? -INFINITY : S[r] * C2;
                asm volatile("" : "+v"(x));
                S[r] = x;
            }
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) bmax = fmaxf(bmax, S[r]);
        {
            typedef uint32_t u32x2v __attribute__((ext_vector_type(2)));
            const u32x2v sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(bmax), __float_as_uint(bmax), false, false);
            bmax = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
        }
        const float m_new = fmaxf(m_run, bmax * scale);
        const float m_ref = (m_new == -INFINITY) ? 0.f : m_new;      // a query that has seen no key yet
        float alpha = 1.f;
        if (__any(m_new > m_run)) {
            alpha = __builtin_amdgcn_exp2f(m_run - m_ref);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) O[i][r] *= alpha;
            m_run = m_new;
        }
        float psum = 0.f;
        uint32_t pk[8];
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
            const float p0 = __builtin_amdgcn_exp2f(fmaf(S[r], scale, -m_ref)), p1 = __builtin_amdgcn_exp2f(fmaf(S[r + 1], scale, -m_ref));
            psum += p0 + p1;
            pk[r >> 1] = pack2(p0, p1);
        }
        l_run = fmaf(l_run, alpha, psum);
        // o^T[dcol][query] += v^T[dcol][key] p^T[key][query], 16 keys at a time
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const half8 fp = fragment_of(pk, ks);
#pragma unroll
            for (int i = 0; i < 4; ++i) O[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(r0.columns(TILE, i, ks), fp, O[i], 0, 0, 0);
        }
    };

    for (int blk = 0; blk <= last; ++blk) {
        const int buf = blk & 1;
        // the block's tiles have landed; everybody is done with the other pair
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (blk < last) fetch(blk + 1, buf ^ 1);      // in flight while this block is multiplied
        if (!active || blk > own_last) continue;
        const bool diag = blk == own_last;      // where the even waves' queries come before the second half
        const bool second = !diag || (wave & 1) != 0;
        if constexpr (SPLIT == 1) {
            const TileRead r0 = rd.at(buf * PAIR), r1 = rd.at(buf * PAIR + 32 * D);
            floatx16 S0, S1;
            scores(r0, S0);
            scores(r1, S1);
            half(r0, 0, S0, accO[0], m_run[0], l_run[0], diag);
            if (second) half(r1, 1, S1, accO[1], m_run[1], l_run[1], diag);
        } else if (part == 0 || second) {
            const TileRead r0 = rd.at(buf * PAIR + 32 * part * D);
            floatx16 S;
            scores(r0, S);
            half(r0, part, S, accO[0], m_run[0], l_run[0], diag);
        }
    }

    // ---- the two halves' common maximum and total sum (finite: key 0 is visible to every query), then o
    typedef uint32_t u32x2v __attribute__((ext_vector_type(2)));
    float m[2], l[2];
#pragma unroll
    for (int h = 0; h < STATES; ++h) {
        const u32x2v sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(l_run[h]), __float_as_uint(l_run[h]), false, false);
        m[h] = m_run[h];
        l[h] = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
    }
    float* xch = reinterpret_cast<float*>(smem) + (wave & 1) * 66 * 64 + lane;
    if constexpr (SPLIT == 2) {
        __syncthreads();             // the tiles are free
        if (part == 1) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) xch[(16 * i + r) * 64] = accO[0][i][r];
            xch[64 * 64] = m[0];
            xch[65 * 64] = l[0];
        }
        __syncthreads();
        if (part == 1) return;
        m[1] = xch[64 * 64];
        l[1] = xch[65 * 64];
    }
    if (!active) return;
    const float mt = fmaxf(m[0], m[1]);
    const float e0 = __builtin_amdgcn_exp2f(m[0] - mt), e1 = __builtin_amdgcn_exp2f(m[1] - mt);
    const float lt = fmaf(l[0], e0, l[1] * e1);
    const float f0 = e0 / lt, f1 = e1 / lt;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            float other;
            if constexpr (SPLIT == 2) other = xch[(16 * i + r) * 64];
            else other = accO[1][i][r];
            float x = fmaf(accO[0][i][r], f0, other * f1);
            asm volatile("" : "+v"(x));      // rounded to fp32 before it is to fp16
            accO[0][i][r] = x;
        }
    store_rows(accO[0], a.o + (t0 + query) * a.H + (int64_t)n * D);
    if (lh == 0) a.lse[(t0 + query) * a.nh + n] = (mt + __builtin_amdgcn_logf(lt)) * 0.6931471805599453f;
}

template <int SPLIT, typename Load = attn::TileLoad>
static hipError_t launch(const attn::FwdArgs& a, int64_t B, hipStream_t st) {
    using namespace attn;
    auto kern = attention_forward_kernel<SPLIT, Load>;
    // thread-safe one-time set-up (initialisation of a function-local static)
    static const hipError_t cfg0 = allow_dynamic_lds(kern, LDS_BYTES);
    if (cfg0 != hipSuccess) return cfg0;
    const dim3 grid((unsigned)(((int64_t)a.s + ROWS<SPLIT> - 1) / ROWS<SPLIT> * a.nh * B));
    hipLaunchKernelGGL(kern, grid, dim3(256), LDS_BYTES, st, a);
    return hipGetLastError();
}

hipError_t launch_attention_forward(const uint16_t* qkv, uint16_t* o, float* lse, int64_t B, int64_t s, int64_t nh,
                                    hipStream_t st) {
    attn::FwdArgs a;
    a.qkv = qkv; a.o = o; a.lse = lse;
    a.s = (int)s; a.nh = (int)nh; a.H = (int)(nh * attn::D);
    if (nh > attn::FAR) return launch<1, attn::TileLoadFar>(a, B, st);
    // not split / split, us: 3 x 320 tokens, 32 heads 14.5 / 13.3, 8 x 128 (4 waves per CU) 8.9 / 10.9, 4 x 256 (4) 12.4 / 12.0, 5 x 256 (5) 14.7 / 18.0;
    // 3 x 512 (6) 23.4 / 23.8, 4 x 512 (8) 25.4 / 29.2;  1 x 1024 (4) 34.7 / 24.7, 1 x 1536 (6) 54.4 / 39.1, 1 x 2048 (8) 75 / 61, 3 x 768 (9) 33.9 / 40.2
    const double waves = attn::waves_per_cu(B, s, nh);
    return waves < 4.0 || (s >= 384 && waves <= 5.0) || (s >= 768 && waves <= 8.0) ? launch<2>(a, B, st) : launch<1>(a, B, st);
}

}  // namespace lomo
