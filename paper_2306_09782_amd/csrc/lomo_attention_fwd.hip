// Forward of causal softmax attention (head width 128) on the rotated q, k and v, for recomputing the
// activations that Algorithm 1's backward loop reads from a checkpoint of the layer input (paper section 3.2;
// activation checkpointing: sections 2 and 4.1).  Produces o and lse = log sum_j exp(q_i . k_j / sqrt(d)) in
// the layout the backward kernel reads.
//
// One workgroup per (sequence, head, block of queries) walks the key blocks (64 keys) up to the diagonal; a wave owns 32
// queries, with a running maximum, sum and output accumulator per query.  The score tile is computed transposed (keys are
// the MFMA rows): a lane owns one query, its maximum is a scan of the lane's registers plus one exchange with lane + 32, and
// the probabilities become the B operand of o^T += v^T p^T through a v_permlane32_swap.  Probabilities are rounded to fp16
// relative to the running maximum; accumulation is fp32; o is rounded once.  Deterministic.
// The first 64 queries of a sequence see so few keys that a probability's rounding shows in their outputs, which are also the
// largest: in their own block the roundings' remainders are multiplied as well (o is 2.27e-4 off a 64-bit result at 8 x 512 tokens,
// 2.46e-4 without).  They are 2 of a head's s / 32 waves.
//
// Measured, us, against the kernel before (64 queries per workgroup, keys split over the waves, tiles through registers): 1 x 8192
// tokens, 32 heads 945 -> 772 (713 TFLOP/s); 8 x 1024, 40 heads 236 -> 192; 8 x 512, 32 heads 55 -> 46; 3 x 320 13.1 -> 13.7.  At 8192
// tokens the matrix pipes are 38 % busy at 1.94 GHz: vector instructions (54 % of the issue slots) and products of a SIMD's two
// waves overlap only in part, and the clock is already lowered by the power limit.  Not leaving it to chance which wave
// issues first (s_setprio by the wave's place on its SIMD) changed nothing.
#include "lomo_attention_common.h"

#include <type_traits>

namespace lomo {

namespace attn {

struct FwdArgs {
    const uint16_t* qkv;   // [T x 3H]
    uint16_t* o;           // [T x H]
    float* lse;            // [T x nh]
    int s, nh, H;
};

}  // namespace attn

template <int SPLIT>
__global__ __launch_bounds__(256, 2) void attention_forward_kernel(attn::FwdArgs a) {
    using namespace attn;
    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];      // two pairs of tiles: K, V

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
    const int last = ((q0 + ROWS<SPLIT> < a.s ? q0 + ROWS<SPLIT> : a.s) - 1) / BLK;      // key blocks of the workgroup, of this wave
    const int own_last = qw / BLK;
    const int64_t ld3 = 3 * (int64_t)a.H;
    const int64_t t0 = (int64_t)b * a.s;
    const uint16_t* gq = a.qkv + (int64_t)n * D;
    const uint16_t* gk = gq + a.H + t0 * ld3;
    const uint16_t* gv = gk + a.H;
    constexpr float C2 = SCALE * LOG2E;
    const int query = qw + l32;

    const TileLoad load(ld3);
    const TileRead rd;
    auto fetch = [&](int blk, int buf) {
        const int64_t off = (int64_t)blk * BLK * ld3;
        load.issue(gk + off, lds0 + (uint32_t)buf * (PAIR * 2u), wave);
        load.issue(gv + off, lds0 + (uint32_t)buf * (PAIR * 2u) + TILE * 2u, wave);
    };
    fetch(0, 0);

    half8 fq[D / 16];
    if (active) load_fragments(fq, gq + (t0 + query) * ld3);

    floatx16 accO[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) accO[i][r] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;      // log2 domain; l_run is this lane's share (its half of the keys)

    // HALVES x 32 keys of the pair in `buf`, from key 32 h on, against this wave's queries; DIAG: the last 32 of them have the
    // queries' positions.
    auto block = [&](int buf, int h0, auto halves_t, auto diag_t) {
        constexpr int HALVES = decltype(halves_t)::value;
        constexpr bool DIAG = decltype(diag_t)::value;
        const TileRead r0 = rd.at(buf * PAIR + 32 * h0 * D);
        floatx16 S[HALVES];
#pragma unroll
        for (int h = 0; h < HALVES; ++h)
#pragma unroll
            for (int r = 0; r < 16; ++r) S[h][r] = 0.f;
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks)
#pragma unroll
            for (int h = 0; h < HALVES; ++h) S[h] = __builtin_amdgcn_mfma_f32_32x32x16_f16(r0.rows(smem + 32 * h * D, ks), fq[ks], S[h], 0, 0, 0);
        // S[h][r] <-> key 32 (h0 + h) + 8 (r / 4) + 4 lh + r % 4 of the block
        float bmax = -INFINITY;
#pragma unroll
        for (int h = 0; h < HALVES; ++h)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                if (DIAG && h == HALVES - 1 && 8 * (r >> 2) + 4 * lh + (r & 3) > l32) S[h][r] = -INFINITY;
                bmax = fmaxf(bmax, S[h][r]);
            }
        {
            typedef uint32_t u32x2v __attribute__((ext_vector_type(2)));
            const u32x2v sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(bmax), __float_as_uint(bmax), false, false);
            bmax = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
        }
        const float m_new = fmaxf(m_run, bmax * C2);
        const float m_ref = (m_new == -INFINITY) ? 0.f : m_new;      // a query whose scores are all -inf so far
        if (__any(m_new > m_run)) {
            const float alpha = __builtin_amdgcn_exp2f(m_run - m_ref);
            l_run *= alpha;
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) accO[i][r] *= alpha;
            m_run = m_new;
        }
        float psum = 0.f;
#pragma unroll
        for (int h = 0; h < HALVES; ++h) {
            uint32_t pk[8];
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                S[h][r] = __builtin_amdgcn_exp2f(fmaf(S[h][r], C2, -m_ref));
                S[h][r + 1] = __builtin_amdgcn_exp2f(fmaf(S[h][r + 1], C2, -m_ref));
                psum += S[h][r] + S[h][r + 1];
                pk[r >> 1] = pack2(S[h][r], S[h][r + 1]);
            }
            // o^T[dcol][query] += v^T[dcol][key] p^T[key][query], 16 keys at a time
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                const half8 fp = fragment_of(pk, ks);
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    accO[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(r0.columns(smem + TILE, i, 2 * h + ks), fp, accO[i], 0, 0, 0);
            }
            if constexpr (DIAG) {
                if (qw < BLK) {      // the roundings' remainders
#pragma unroll
                    for (int r = 0; r < 16; r += 2) pk[r >> 1] = pack2(S[h][r] - (float)(_Float16)S[h][r], S[h][r + 1] - (float)(_Float16)S[h][r + 1]);
#pragma unroll
                    for (int ks = 0; ks < 2; ++ks) {
                        const half8 fp = fragment_of(pk, ks);
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            accO[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(r0.columns(smem + TILE, i, 2 * h + ks), fp, accO[i], 0, 0, 0);
                    }
                }
            }
        }
        l_run += psum;
    };

    using one = std::integral_constant<int, 1>;
    using two = std::integral_constant<int, 2>;
    for (int blk = 0; blk <= last; ++blk) {
        const int buf = blk & 1;
        // the block's tiles have landed; everybody is done with the other pair
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (blk < last) fetch(blk + 1, buf ^ 1);      // in flight while this block is multiplied
        if (!active || blk > own_last) continue;
        if constexpr (SPLIT == 1) {
            if (blk < own_last) block(buf, 0, two{}, std::false_type{});
            else if (wave & 1) block(buf, 0, two{}, std::true_type{});
            else block(buf, 0, one{}, std::true_type{});
        } else {
            const int ahead = qw / 32 - (2 * blk + part);      // of this half's keys
            if (ahead > 0) block(buf, part, one{}, std::false_type{});
            else if (ahead == 0) block(buf, part, one{}, std::true_type{});
        }
    }

    typedef uint32_t u32x2v __attribute__((ext_vector_type(2)));
    const u32x2v sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(l_run), __float_as_uint(l_run), false, false);
    float l = __uint_as_float(sw[0]) + __uint_as_float(sw[1]), m = m_run;
    if constexpr (SPLIT == 2) {      // common maximum and total sum of the two halves
        float* xch = reinterpret_cast<float*>(smem) + (wave & 1) * 66 * 64 + lane;
        __syncthreads();             // the tiles are free
        if (part == 1) {
            put_registers(accO, xch);
            xch[64 * 64] = m_run;
            xch[65 * 64] = l;
        }
        __syncthreads();
        if (part == 1) return;
        const float m_other = xch[64 * 64], l_other = xch[65 * 64];
        m = fmaxf(m_run, m_other);
        const float m_ref = (m == -INFINITY) ? 0.f : m;
        const float f = __builtin_amdgcn_exp2f(m_run - m_ref), f_other = __builtin_amdgcn_exp2f(m_other - m_ref);
        l = fmaf(l, f, l_other * f_other);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) accO[i][r] = fmaf(accO[i][r], f, xch[(16 * i + r) * 64] * f_other);
    }
    if (!active) return;
    store_rows(accO, 1.0f / l, a.o + (t0 + query) * a.H + (int64_t)n * D);
    if (lh == 0) a.lse[(t0 + query) * a.nh + n] = (((m == -INFINITY) ? 0.f : m) + __builtin_amdgcn_logf(l)) * 0.6931471805599453f;
}

template <int SPLIT>
static hipError_t launch(const attn::FwdArgs& a, int64_t B, hipStream_t st) {
    using namespace attn;
    auto kern = attention_forward_kernel<SPLIT>;
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
    return attn::attention_waves(B, s, nh) < 4 * cu_count() ? launch<2>(a, B, st) : launch<1>(a, B, st);
}

}  // namespace lomo
