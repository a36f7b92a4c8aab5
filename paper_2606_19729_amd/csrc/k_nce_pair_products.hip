// k_nce_pair_products.hip -- stage 2 of the bfloat16 contrastive parameter
// derivative (nce_pair.hpp): the weight derivatives as products over pairs.
#include "nce_pair.hpp"

namespace voila {

namespace {

// A block streams its pair-units (64 pairs: two units of one row) through NBUF
// LDS buffers: the layer's stored operand of both units, then up to five
// kilobytes of what the rest is formed from.  Every wave issues kDma
// direct-to-LDS loads per stage, whatever the layer, so that one wait covers
// the stage (extras that another wave loads too carry the same bytes).
constexpr int kNBuf = 4, kWaves = 8, kDma = 5, kExtra = 5;
constexpr int kStage = 2 * kArr + kExtra * 1024;

struct Stages {
    char* lds;
    const char* tiles;   // the layer's stored array at the block's first pair-unit
    long last;           // last stage
    int wave, lane;
    // extra e of stage v: its source, and whether it is 16 or 4 bytes per lane
    template <class Extra>
    __device__ __forceinline__ void fetch(long stage, Extra&& extra) const {
        const long v = stage < last ? stage : last;  // past the end: the last one again (one count of loads throughout)
        char* const dst = lds + (int)(stage % kNBuf) * kStage;
        const char* const t = tiles + (size_t)v * (2 * kArr);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int off = (r * kWaves + wave) * 1024;
            __builtin_amdgcn_global_load_lds((const void*)(t + off + (uint32_t)lane * 16),
                                             (__attribute__((address_space(3))) void*)(dst + off), 16, 0, 0);
        }
        extra(v, dst + 2 * kArr);
    }
};
// body(stage's LDS) for stages 0 .. n - 1, three stages ahead in flight.
template <class Extra, class Body>
__device__ __forceinline__ void over_stages(const Stages& st, long n, Extra&& extra, Body&& body) {
#pragma unroll
    for (int k = 0; k < kNBuf - 1; ++k) st.fetch(k, extra);
    for (long v = 0; v < n; ++v) {
        // this wave's loads of stage v have landed and its reads of stage
        // v - 1 are done; then everybody's, and that buffer is free
        __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0((kNBuf - 2) * kDma));
        __builtin_amdgcn_s_barrier();
        st.fetch(v + kNBuf - 1, extra);
        body((const char*)(st.lds + (int)(v % kNBuf) * kStage + opaque_zero()));
    }
    __builtin_amdgcn_s_waitcnt(0);
}

__device__ __forceinline__ bf16x8 lds_op(const char* stage, int unit, int t, int h, int lane) {
    return *reinterpret_cast<const bf16x8*>(stage + unit * kArr + (2 * t + h) * 1024 + lane * 16);
}
__device__ __forceinline__ void sum_words(float& s, uint32_t w) { s += bf_lo(w) + bf_hi(w); }

// dst[m][n] (+)= the wave's accumulators of output tiles (r0 + a, c0 + b).
template <int RT, int CT>
__device__ __forceinline__ void put_tiles(float* dst, const f32x16 (&acc)[RT][CT], int r0, int c0, int g, int col,
                                          bool add) {
#pragma unroll
    for (int a = 0; a < RT; ++a)
#pragma unroll
        for (int b = 0; b < CT; ++b) {
            float* d = dst + (size_t)(32 * (r0 + a) + 4 * g) * kW + 32 * (c0 + b) + col;
            f32x16 v = acc[a][b];
            if (add)
#pragma unroll
                for (int r = 0; r < 16; ++r) v[r] += d[out_row(r, 0) * kW];
#pragma unroll
            for (int r = 0; r < 16; ++r) d[out_row(r, 0) * kW] = v[r];
        }
}

}  // namespace

// One layer's derivative over the block's pair-units, the 256 x 256 ones by
// eight waves of 2 x 4 or 4 x 2 tiles (128 accumulator registers, two waves
// per SIMD).  Stage 1 stores the operands as the matrix cores read them, so
// they go to LDS by direct loads and from there to the products; delta_3 is
// formed from the sign pattern of h_3, h_1 recomputed from the observations
// (a quarter more products), which cost less than 16 KB each per unit.
// Bound by memory: 16 KB per unit and layer, 25.7 GB at B = 4,096 in 6.4 ms
// (4.0 TB/s; staging through registers with feature-major operands took 17.8).
template <int D_O>
__global__ __launch_bounds__(64 * kWaves) void nce_pair_wgrad_kernel(NcePairParams p) {
    constexpr int IN_KS = in_slots(DT_BF16, D_O, 0, 0) / 8;
    static_assert(IN_KS == 2, "first-layer operands: two k-steps");
    typedef PairSeq<IN_KS> S;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int lane = threadIdx.x & 63, g = lane >> 5, col = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int layer = (int)blockIdx.x < p.wb[0] ? 3 : (int)blockIdx.x < p.wb[0] + p.wb[1] ? 2 : 1;
    const int blk = layer == 3 ? blockIdx.x : layer == 2 ? blockIdx.x - p.wb[0] : blockIdx.x - p.wb[0] - p.wb[1];
    const int nb = p.wb[3 - layer];
    const long pairs = p.u1 - p.u0;
    const long v0 = pairs * blk / nb, n = pairs * (blk + 1) / nb - v0;  // pair-units of the chunk: v0 .. v0 + n - 1
    const bool add = p.accumulate;
    const Stages st{smem, p.act + ((size_t)(3 - layer) * (p.uc + 2) + 2 * v0) * kArr, n - 1, wave, lane};
    auto row_of = [&](long v) { return (int)((uint32_t)(p.u0 + v0 + v) / (uint32_t)p.jpairs); };
    auto jt_of = [&](long v, int i) { return ((int)(p.u0 + v0 + v) - i * p.jpairs) * 2; };

    if (layer == 3) {
        // rows 2 wr, 2 wr + 1 of delta_3 against tiles 4 wc .. of h_2
        const int wr = wave >> 1, wc = wave & 1;
        f32x16 acc[2][4];
        float sd[2] = {0.0f, 0.0f}, wv[2];  // the adjoint's sums over pairs: the bias derivative
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            wv[a] = p.w_out[32 * (2 * wr + a) + col];
#pragma unroll
            for (int b = 0; b < 4; ++b) acc[a][b] = f32x16{};
        }
        __builtin_amdgcn_s_waitcnt(0);
        if (n > 0)
            over_stages(
                st, n,
                [&](long v, char* dst) {
                    const size_t u = (size_t)2 * (v0 + v);
                    if (wave % 3 < 2) load16(p.sgn + (u + wave % 3) * kSgn, dst + (wave % 3) * kSgn, lane);
                    else load4(p.gt + u * 32 + lane, dst + 2 * kSgn);
                },
                [&](const char* s) {
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        const uint32_t m =
                            *reinterpret_cast<const uint32_t*>(s + 2 * kArr + q * kSgn + lane * 16 + wr * 4);
                        const float* gt = reinterpret_cast<const float*>(s + 2 * kArr + 2 * kSgn) + 32 * q + 4 * g;
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            bf16x8 fb[4];
#pragma unroll
                            for (int b = 0; b < 4; ++b) fb[b] = lds_op(s, q, 4 * wc + b, h, lane);
                            const f32x4 x0 = *reinterpret_cast<const f32x4*>(gt + 16 * h);
                            const f32x4 x1 = *reinterpret_cast<const f32x4*>(gt + 16 * h + 8);
#pragma unroll
                            for (int a = 0; a < 2; ++a) {
                                uint32_t w[4];
#pragma unroll
                                for (int k = 0; k < 4; ++k) {
                                    const f32x4& x = k < 2 ? x0 : x1;
                                    const float e0 = x[2 * (k % 2)], e1 = x[2 * (k % 2) + 1];
                                    w[k] = bf16x2_of(wv[a] * e0, wv[a] * e1) &
                                           spread16((m >> (4 * h + k + 8 * a)) & 0x00010001u);
                                    sum_words(sd[a], w[k]);
                                }
                                const bf16x8 fa = frag_of(w);
#pragma unroll
                                for (int b = 0; b < 4; ++b) acc[a][b] = mfma(fa, fb[b], acc[a][b]);
                            }
                        }
                    }
                });
        float* const dst = p.wpart[0] + (size_t)blk * (kW * kW + kW);
        put_tiles<2, 4>(dst, acc, 2 * wr, 4 * wc, g, col, add);
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            const float v = sd[a] + __shfl_xor(sd[a], 32);
            float* d = dst + kW * kW + 32 * (2 * wr + a) + col;
            if (wc == 0 && g == 0) *d = (add ? *d : 0.0f) + v;
        }
        return;
    }
    if (layer == 2) {
        // rows 4 wr .. of delta_2 against tiles 2 wc, 2 wc + 1 of h_1
        const int wr = wave >> 2, wc = wave & 3;
        f32x16 acc[4][2];
        float sd[4];
        bf16x8 w1[IN_KS][2];  // the first layer's weights of those tiles
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            sd[a] = 0.0f;
#pragma unroll
            for (int b = 0; b < 2; ++b) acc[a][b] = f32x16{};
        }
#pragma unroll
        for (int c = 0; c < IN_KS; ++c)
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const int t = 2 * wc + b, f = (t / S::PT * IN_KS + c) * S::PT + t % S::PT;
                w1[c][b] = reinterpret_cast<const bf16x8*>(p.stream)[f * 64 + lane];
            }
        __builtin_amdgcn_s_waitcnt(0);
        if (n > 0)
            over_stages(
                st, n,
                [&](long v, char* dst) {
                    const int i = row_of(v), e = wave % 5;
                    const char* ob = p.obs_n + (size_t)jt_of(v, i) * IN_KS * 1024 + e * 1024;
                    load16(e < 4 ? ob : (const char*)(p.b0 + (size_t)i * kW), dst + e * 1024, lane);
                },
                [&](const char* s) {
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        bf16x8 in[IN_KS], fh[2][2];
#pragma unroll
                        for (int c = 0; c < IN_KS; ++c)
                            in[c] = *reinterpret_cast<const bf16x8*>(s + 2 * kArr + (q * IN_KS + c) * 1024 + lane * 16);
#pragma unroll
                        for (int b = 0; b < 2; ++b) {
                            const float bias =
                                reinterpret_cast<const float*>(s + 2 * kArr + 4096)[32 * (2 * wc + b) + col];
                            f32x16 h;
#pragma unroll
                            for (int r = 0; r < 16; ++r) h[r] = bias;
#pragma unroll
                            for (int c = 0; c < IN_KS; ++c) h = mfma(in[c], w1[c][b], h);
                            fh[b][0] = relu_bf16x8(h, 0);
                            fh[b][1] = relu_bf16x8(h, 1);
                        }
#pragma unroll
                        for (int a = 0; a < 4; ++a)
#pragma unroll
                            for (int h = 0; h < 2; ++h) {
                                const bf16x8 fa = lds_op(s, q, 4 * wr + a, h, lane);
                                if (wc == a)  // one wave of the four per row tile
#pragma unroll
                                    for (int k = 0; k < 4; ++k) sum_words(sd[a], word_of(fa, k));
#pragma unroll
                                for (int b = 0; b < 2; ++b) acc[a][b] = mfma(fa, fh[b][h], acc[a][b]);
                            }
                    }
                });
        float* const dst = p.wpart[1] + (size_t)blk * (kW * kW + kW);
        put_tiles<4, 2>(dst, acc, 4 * wr, 2 * wc, g, col, add);
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const float v = sd[a] + __shfl_xor(sd[a], 32);
            float* d = dst + kW * kW + 32 * (4 * wr + a) + col;
            if (wc == a && g == 0) *d = (add ? *d : 0.0f) + v;
        }
        return;
    }
    // first layer, one row tile per wave: columns [s', a, o] of W_1 and the
    // bias; tile 0 of the products is o, tile 1 [s', a, 1] (the same for every
    // pair of a row)
    const int na = p.d_s + (p.n_actions > 0 ? p.n_actions : p.d_a), d_in = na + D_O;
    f32x16 acc[2] = {f32x16{}, f32x16{}};
    if (n > 0)
        over_stages(
            st, n,
            [&](long v, char* dst) {
                const int i = row_of(v), e = wave % 5;
                if (e < 4) load16(p.obs_t + (size_t)jt_of(v, i) * 2048 + e * 1024, dst + e * 1024, lane);
                else load4(reinterpret_cast<const float*>(p.row_ops) + (size_t)i * 64 + lane, dst + 4096);
            },
            [&](const char* s) {
                const uint32_t w = *reinterpret_cast<const uint32_t*>(s + 2 * kArr + 4096 + lane * 4);
                const bf16x8 sa = __builtin_bit_cast(bf16x8, (u32x4){w, w, w, w});
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const bf16x8 fa = lds_op(s, q, wave, h, lane);
                        const bf16x8 fo =
                            *reinterpret_cast<const bf16x8*>(s + 2 * kArr + (q * 2 + h) * 1024 + lane * 16);
                        acc[0] = mfma(fa, fo, acc[0]);
                        acc[1] = mfma(fa, sa, acc[1]);
                    }
            });
    float* const dst = p.wpart[2] + (size_t)blk * (kW * d_in + kW);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int m = 32 * wave + out_row(r, g);
        auto put = [&](float* d, float v) { *d = (add ? *d : 0.0f) + v; };
        if (col < D_O) put(dst + (size_t)m * d_in + na + col, acc[0][r]);
        if (col < na) put(dst + (size_t)m * d_in + col, acc[1][r]);
        if (col == na) put(dst + (size_t)kW * d_in + m, acc[1][r]);
    }
}

hipError_t launch_nce_pair_wgrad(const NcePairParams& p, hipStream_t s) {
    constexpr int lds = kNBuf * kStage;
    (void)hipFuncSetAttribute((const void*)nce_pair_wgrad_kernel<32>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    hipLaunchKernelGGL(nce_pair_wgrad_kernel<32>, p.wb[0] + p.wb[1] + p.wb[2], 64 * kWaves, lds, s, p);
    return hipGetLastError();
}

}  // namespace voila
