// k_nce_pair.hip -- stage 1 of the bfloat16 contrastive parameter derivative
// (nce_pair.hpp): forward and reverse sweep of every pair, and the operands.
#include "nce_pair.hpp"

namespace voila {

namespace {
constexpr int kST = 2;    // units per wave
constexpr int kPF = 6;    // weight fragments read ahead
// The work of a finished pass at the steps of the pass after it, for tile e of
// its kST PT (tile, unit) tiles, from step kStart + kStep e on: conversion over
// four steps (two value pairs each; not at step 0, where the pass's last
// products are still under way), exchange of rows and columns in the next two,
// and a step later the transposed values over two steps, four pairs and one
// store each.
constexpr int kStart = 1, kStep = 6, kFin = 7, kEnd = 9;
template <int IN_KS>
constexpr int kWaveIn = kW * 4 + 256 + kST * IN_KS * 1024;  // LDS bytes of a wave's inputs
template <class S>
struct PairStores {
    static constexpr int in_step(int f) {  // global stores at fragment-step f
        const int q = S::gpass(f) - 1, s = f - S::pass_start(q + 1);
        if (q < S::NP || q / S::NP == 2) return 0;  // layer 0 stores nothing, layer 2 its sign pattern (not counted)
        int n = 0;
        for (int e = 0; e < kST * S::PT; ++e) {
            const int k = s - kStart - kStep * e;
            n += k >= kFin && k < kEnd;
        }
        return n;
    }
};
}  // namespace

// Bound by the matrix cores (1,184 products of 32 cycles per pair-unit of 64
// pairs) beside the vector work that converts, masks and stores: as in the
// rollout kernel, the work of each finished pass is spread over the products
// of the next one, in the order of a compile-time sequence (left
// free within a fragment-step: pacing the vector instructions by five or eight
// per product was 5 % slower).  Matrix cores busy 50 %; 68 bytes per lane are
// spilled.  B = 4,096: 9.9 ms
// for the 262,144 pair-units, where one unit per wave with 2-byte stores and
// 612 bytes of spills took 25.4 ms.
template <int D_O>
__global__ __launch_bounds__(256) void nce_pair_bwd_kernel(NcePairParams p) {
    constexpr int IN_KS = in_slots(DT_BF16, D_O, 0, 0) / 8;
    typedef PairSeq<IN_KS> S;
    typedef PairStream<S, kPF, PairStores<S>> Src;
    constexpr int ST = kST, PT = S::PT, NP = S::NP, PF = kPF, R = PF + 1;
    constexpr int LEAD = 4;  // fragment-steps the biases are read ahead
    static_assert(PT == 1, "the output weights read ahead are one tile's");
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int lane = threadIdx.x & 63, g = lane >> 5, col = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    float* const bh = reinterpret_cast<float*>(smem + Src::LDS_BYTES);
    float* const wo = bh + 2 * kW;
    // the wave's inputs of a pair-unit: bias row, G, first-layer operands
    char* const mine = reinterpret_cast<char*>(wo + kW) + wave * kWaveIn<IN_KS>;
    float* const rowb = reinterpret_cast<float*>(mine);
    float* const gl = rowb + kW;
    const bf16x8* const inl = reinterpret_cast<const bf16x8*>(gl + 64);
    for (int k = threadIdx.x; k < 2 * kW; k += blockDim.x) bh[k] = p.bh[k];
    for (int k = threadIdx.x; k < kW; k += blockDim.x) wo[k] = p.w_out[k];
    bf16x8 eye[2];  // the 0/1 operands of the exchange
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < 8; ++j) eye[h][j] = (__bf16)(out_row(8 * h + j, g) == col ? 1.0f : 0.0f);
    __syncthreads();
    Src src(smem, p.stream);
    src.start();

    float dwo[kHT], dbo = 0.0f;  // output layer: feature 32 t + col of this lane, summed over its pairs
#pragma unroll
    for (int t = 0; t < kHT; ++t) dwo[t] = 0.0f;

    // the inputs of the wave's next pair-unit, loaded into LDS during the
    // current one's last layer (no registers, no wait: the chunk boundary that
    // opens the next pair-unit covers them)
    auto next_inputs = [&](long u) {
        const long v = u < p.u1 ? u : p.u1 - 1;  // wave-uniform
        const int i = (int)((uint32_t)v / (uint32_t)p.jpairs), jt = ((int)v - i * p.jpairs) * ST;
        const char* ob = p.obs_n + (size_t)jt * IN_KS * 1024;
        load16(p.b0 + (size_t)i * kW, mine, lane);
        const int j = (jt + g) * 32 + col;
        load4(p.grad + (size_t)i * p.B + (j < p.B ? j : p.B - 1), mine + kW * 4);
#pragma unroll
        for (int c = 0; c < ST * IN_KS; ++c) load16(ob + c * 1024, mine + kW * 4 + 256 + c * 1024, lane);
    };
    next_inputs(p.u0 + (long)blockIdx.x * 4 + wave);

    // block-uniform loop: the stream's chunk barriers need every wave
    for (long ub = blockIdx.x; p.u0 + ub * 4 < p.u1; ub += gridDim.x) {
        const long u = p.u0 + ub * 4 + wave;
        const bool ok = u < p.u1;
        // first unit of the pair within the chunk; waves past its end write to
        // the two units after the arrays' last (no branch around the stores)
        const long ul = ok ? 2 * (u - p.u0) : p.uc;
        char* const out = p.act + (size_t)ul * kArr;
        char* const out_sgn = p.sgn + (size_t)ul * kSgn;
        const uint32_t lane16 = (uint32_t)lane * 16;
        const size_t arr_bytes = (size_t)(p.uc + 2) * kArr;

        Act<DT_BF16, kHT> A[2][ST];
        f32x16 acc[2][ST][PT];
        f32x16 T;
        bf16x8 ring[R], tmp[2];          // tmp: operands of the tile being transposed (h_3, delta_1)
        uint32_t sgn1[ST][kHT / 2];      // sign pattern of h_1: bits j and 16 + j (+ 8 for odd tiles) of value pair j
        uint32_t sgn3[ST][kHT / 2];      // the same of h_3, pairs along the registers
        uint32_t fw[4];
        float gc[ST];                    // G of this lane's pair in each unit
        f32x4 wq[4], gq[4];              // output weights of the tile, G of its pairs (read ahead of their use)
#pragma unroll
        for (int st = 0; st < ST; ++st)
#pragma unroll
            for (int t = 0; t < kHT / 2; ++t) sgn1[st][t] = sgn3[st][t] = 0;

        // value pair j of tile t = 2 (q % NP) + tt of the finished pass q, unit st, as operand words
        auto convert = [&](auto qi, auto sti, auto tti, auto ji) {
            constexpr int q = decltype(qi)::value, st = decltype(sti)::value, tt = decltype(tti)::value;
            constexpr int j = decltype(ji)::value, L = q / NP, t = PT * (q % NP) + tt;
            const float a = acc[q % 2][st][tt][2 * j], b = acc[q % 2][st][tt][2 * j + 1];
            bf16x8& mine = A[L % 2][st].v[2 * t + j / 4];
            if constexpr (L == 0) {
                const uint32_t w = relu_bf16x2(a, b);
                sgn1[st][t / 2] |= ones16(w) << (j + 8 * (t % 2));
                set_word(mine, j % 4, w);
            } else if constexpr (L == 1) {
                set_word(mine, j % 4, relu_bf16x2(a, b));
            } else if constexpr (L == 2) {
                // h_3 for the output layer's derivative; delta_3 = G w_out on its active units
                const uint32_t w = relu_bf16x2(a, b);
                set_word(tmp[j / 4], j % 4, w);
                const float w0 = wq[j / 2][2 * (j % 2)], w1 = wq[j / 2][2 * (j % 2) + 1];
                set_word(mine, j % 4, bf16x2_of(w0 * gc[st], w1 * gc[st]) & spread16(ones16(w)));
            } else if constexpr (L == 3) {
                // delta_2 over h_2, on h_2's active units
                set_word(mine, j % 4, bf16x2_of(a, b) & spread16(ones16(word_of(mine, j % 4))));
            } else {
                const uint32_t m = (sgn1[st][t / 2] >> (j + 8 * (t % 2))) & 0x00010001u;
                set_word(tmp[j / 4], j % 4, bf16x2_of(a, b) & spread16(m));
            }
        };
        // half h of the tile's exchange of rows and columns (an infinite value
        // times the zeros makes NaN of its pair's whole tile)
        auto transpose = [&](auto qi, auto sti, auto tti, auto hi) {
            constexpr int q = decltype(qi)::value, st = decltype(sti)::value, tt = decltype(tti)::value;
            constexpr int h = decltype(hi)::value, L = q / NP, t = PT * (q % NP) + tt;
            if constexpr (L == 2 && h == 0) {
                const float* gt = gl + 32 * st + 4 * g + opaque_zero();
#pragma unroll
                for (int m = 0; m < 4; ++m) gq[m] = *reinterpret_cast<const f32x4*>(gt + 8 * m);
            }
            const bf16x8 v = L == 2 || L == 4 ? tmp[h] : A[L % 2][st].v[2 * t + h];
            T = h == 0 ? mfma(v, eye[0], f32x16{}) : mfma(v, eye[1], T);
        };
        // values 2 j and 2 j + 1 (pairs along the registers) of the transposed tile
        auto finish = [&](auto qi, auto sti, auto tti, auto ji) {
            constexpr int q = decltype(qi)::value, st = decltype(sti)::value, tt = decltype(tti)::value;
            constexpr int j = decltype(ji)::value, L = q / NP, t = PT * (q % NP) + tt;
            const uint32_t w = bf16x2_of(T[2 * j], T[2 * j + 1]);  // exact: the values are bfloat16
            if constexpr (L == 2) {
                dwo[t] = __builtin_fmaf(gq[j / 2][2 * (j % 2)], T[2 * j], dwo[t]);
                dwo[t] = __builtin_fmaf(gq[j / 2][2 * (j % 2) + 1], T[2 * j + 1], dwo[t]);
                sgn3[st][t / 2] |= ones16(w) << (j + 8 * (t % 2));
                if constexpr (t == kHT - 1 && j == 7)
                    *reinterpret_cast<u32x4*>(out_sgn + st * kSgn + lane16) =
                        (u32x4){sgn3[st][0], sgn3[st][1], sgn3[st][2], sgn3[st][3]};
            } else {
                fw[j % 4] = w;
                if constexpr (j % 4 == 3) {
                    constexpr int arr = L == 1 ? 0 : L == 3 ? 1 : 2;  // h_2, delta_2, delta_1
                    *reinterpret_cast<bf16x8*>(out + arr * arr_bytes + (st * kArr + (2 * t + j / 4) * 1024) + lane16) =
                        frag_of(fw);
                }
            }
        };
        auto bias_of = [&](auto qi) {
            constexpr int q = decltype(qi)::value, L = q / NP;
            if constexpr (q < S::NQ && L < 3) {
                const float* bias = (L == 0 ? rowb : bh + (L - 1) * kW) + 32 * PT * (q % NP);
                init_bias<PT>(acc[q % 2][0], bias + opaque_zero(), g);
            }
        };
        // the slice of pass q's work at fragment-step s of the pass after it
        auto work = [&](auto qi, auto si) {
            constexpr int q = decltype(qi)::value, s = decltype(si)::value;
            static_for<PT * ST>([&](auto ei) {
                constexpr int e = decltype(ei)::value, k = s - kStart - kStep * e;
                typedef std::integral_constant<int, e % ST> sti;
                typedef std::integral_constant<int, e / ST> tti;
                if constexpr (k >= 0 && k < 4)
                    static_for<2>([&](auto ji) {
                        convert(qi, sti{}, tti{}, std::integral_constant<int, 2 * k + decltype(ji)::value>{});
                    });
                if constexpr (q >= NP && (k == 4 || k == 5))
                    transpose(qi, sti{}, tti{}, std::integral_constant<int, k - 4>{});
                if constexpr (q >= NP && k >= kFin && k < kEnd)
                    static_for<4>([&](auto ji) {
                        finish(qi, sti{}, tti{}, std::integral_constant<int, 4 * (k - kFin) + decltype(ji)::value>{});
                    });
            });
        };

        static_for<PF>([&](auto fi) { ring[decltype(fi)::value % R] = src.template load<decltype(fi)::value>(lane); });
        bias_of(std::integral_constant<int, 0>{});
        {
            const int j = (int)((uint32_t)(ok ? u : 0) % (uint32_t)p.jpairs) * 64 + lane;  // lane (g, col): unit g, column col
            const float x = ok && j < p.B ? gl[lane] : 0.0f;
            gl[lane] = x;
            p.gt[(size_t)ul * 32 + lane] = x;
            dbo += x;
        }
#pragma unroll
        for (int st = 0; st < ST; ++st) gc[st] = gl[st * 32 + col];
        static_for<S::NFR>([&](auto fi) {
            constexpr int f = decltype(fi)::value;
            constexpr int L = S::layer(f), c = S::kstep(f), t = S::tile(f), q = S::gpass(f);
            constexpr int s = f - S::pass_start(q);
            if constexpr (q == (S::NL - 1) * NP && s == 0) next_inputs(u + (long)gridDim.x * 4);
            if constexpr (q >= 1 && q < NP) {
                // the first layer's passes are short: a whole tile's conversion per step
                static_for<8>([&](auto ji) {
                    constexpr int e = s * PT * ST / S::pass_len(q);
                    static_assert(S::pass_len(q) == PT * ST, "one tile per step");
                    convert(std::integral_constant<int, q - 1>{}, std::integral_constant<int, e % ST>{},
                            std::integral_constant<int, e / ST>{}, ji);
                });
            } else if constexpr (q >= 1) {
                work(std::integral_constant<int, q - 1>{}, std::integral_constant<int, s>{});
            }
            // (into the registers of pass q - 1, whose first unit is converted by then)
            if constexpr (s == (S::pass_len(q) > LEAD ? S::pass_len(q) - LEAD : S::pass_len(q) - 1))
                bias_of(std::integral_constant<int, q + 1>{});
            if constexpr (L == 2 && s == S::pass_len(q) - 3) {
                const float* wt = wo + 32 * PT * (q % NP) + 4 * g + opaque_zero();
#pragma unroll
                for (int m = 0; m < 4; ++m) wq[m] = *reinterpret_cast<const f32x4*>(wt + 8 * m);
            }
            if constexpr (f + PF < S::NFR) ring[(f + PF) % R] = src.template load<f + PF>(lane);
            // the second unit first: at a pass's first k-step it adds to the
            // first unit's bias registers before they are updated
            static_for<ST>([&](auto ii) {
                constexpr int st = ST - 1 - decltype(ii)::value;
                const bf16x8 b = L == 0 ? inl[(st * IN_KS + c % IN_KS) * 64 + lane] : A[(L + 1) % 2][st].v[c];
                if constexpr (c == 0 && L >= 3)
                    acc[q % 2][st][t] = mfma(ring[f % R], b, f32x16{});
                else
                    acc[q % 2][st][t] = mfma(ring[f % R], b, acc[q % 2][c == 0 ? 0 : st][t]);
            });
            __builtin_amdgcn_sched_barrier(0);
        });
        static_for<kStart + kStep * (PT * ST - 1) + kEnd>([&](auto si) {
            work(std::integral_constant<int, S::NQ - 1>{}, si);
        });
    }
    src.finish();
    // the block's output-layer partial: lane halves, then waves in order (the
    // chunk buffers are free once every wave has left the stream)
    __syncthreads();
    float* const red = reinterpret_cast<float*>(smem);
#pragma unroll
    for (int t = 0; t < kHT; ++t) {
        const float v = dwo[t] + __shfl_xor(dwo[t], 32);
        if (g == 0) red[wave * (kW + 1) + 32 * t + col] = v;
    }
    dbo = sum32(dbo);
    dbo += __shfl_xor(dbo, 32);
    if (lane == 0) red[wave * (kW + 1) + kW] = dbo;
    __syncthreads();
    float* const part = p.part + (size_t)blockIdx.x * (kW + 1);
    for (int k = threadIdx.x; k <= kW; k += blockDim.x) {
        float v = p.accumulate ? part[k] : 0.0f;
#pragma unroll
        for (int w = 0; w < 4; ++w) v += red[w * (kW + 1) + k];
        part[k] = v;
    }
}

// Operands of the mini-batch, once per call: obs_n (observations for the
// network's first layer: features along the registers), obs_t (for the products
// over pairs: pairs along the registers), zero past the last observation; and
// row_ops, row i's [s'_i, a_i, 1] as bfloat16 pairs of the lane's column.
template <int D_O>
__global__ __launch_bounds__(64) void nce_pair_prep_kernel(NcePairParams p, const float* obs) {
    constexpr int IN_KS = in_slots(DT_BF16, D_O, 0, 0) / 8;
    static_assert(D_O <= 32, "one operand tile of observations");
    const int lane = threadIdx.x, g = lane >> 5, col = lane & 31, B = p.B;
    if ((int)blockIdx.x < B) {
        const int i = blockIdx.x, na = p.d_s + (p.n_actions > 0 ? p.n_actions : p.d_a);
        float x = col == na ? 1.0f : 0.0f;
        if (col < p.d_s) {
            x = p.states[(size_t)i * p.d_s + col];
        } else if (col < na) {
            if (p.n_actions > 0) {
                int a = reinterpret_cast<const int32_t*>(p.actions)[i];
                if (a < 0 || a >= p.n_actions) a = 0;  // as the forward pass
                x = col - p.d_s == a ? 1.0f : 0.0f;
            } else {
                x = reinterpret_cast<const float*>(p.actions)[(size_t)i * p.d_a + (col - p.d_s)];
            }
        }
        reinterpret_cast<uint32_t*>(p.row_ops)[(size_t)i * 64 + lane] = bf16x2_of(x, x);
        return;
    }
    const int jt = blockIdx.x - B, j = jt * 32 + col;
#pragma unroll
    for (int c = 0; c < IN_KS; ++c) {
        bf16x8 v;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int f = 2 * (8 * c + k) + g;
            v[k] = (__bf16)(j < B && f < D_O ? obs[(size_t)j * D_O + f] : 0.0f);
        }
        reinterpret_cast<bf16x8*>(p.obs_n)[((size_t)jt * IN_KS + c) * 64 + lane] = v;
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        bf16x8 v;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int r = jt * 32 + out_row(8 * h + k, g);
            v[k] = (__bf16)(r < B && col < D_O ? obs[(size_t)r * D_O + col] : 0.0f);
        }
        reinterpret_cast<bf16x8*>(p.obs_t)[((size_t)jt * 2 + h) * 64 + lane] = v;
    }
}

// ---------------------------------------------------------------------------
// launchers (the realistic shape: width 256, three hidden layers, d_o = 32)
// ---------------------------------------------------------------------------
namespace {
constexpr int kDO = 32;
constexpr size_t bwd_lds() {
    return (size_t)PairStream<PairSeq<2>, kPF, PairStores<PairSeq<2>>>::LDS_BYTES + (size_t)3 * kW * 4 + 4 * kWaveIn<2>;
}
}  // namespace

bool nce_pair_supported(int shape, int dt) { return shape == 1 && dt == DT_BF16; }
int nce_pair_pass_tiles() { return PairSeq<2>::PT; }
size_t nce_pair_unit_bytes() { return 3 * (size_t)kArr + kSgn + 32 * 4; }
size_t nce_pair_batch_bytes(int B, int jpairs) { return (size_t)jpairs * 2 * 1024 * 4 + (size_t)B * 256; }

void nce_pair_carve(NcePairParams& p, char* act, char* batch) {
    p.act = act;
    p.sgn = act + (size_t)3 * (p.uc + 2) * kArr;
    p.gt = reinterpret_cast<float*>(p.sgn + (size_t)(p.uc + 2) * kSgn);
    p.obs_n = batch;
    p.obs_t = batch + (size_t)p.jpairs * 2 * 2 * 1024;
    p.row_ops = p.obs_t + (size_t)p.jpairs * 2 * 2 * 1024;
}

hipError_t launch_nce_pair_prep(const NcePairParams& p, const float* obs, hipStream_t s) {
    hipLaunchKernelGGL(nce_pair_prep_kernel<kDO>, p.B + 2 * p.jpairs, 64, 0, s, p, obs);
    return hipGetLastError();
}

hipError_t launch_nce_pair_bwd(const NcePairParams& p, int blocks, hipStream_t s) {
    (void)hipFuncSetAttribute((const void*)nce_pair_bwd_kernel<kDO>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)bwd_lds());
    hipLaunchKernelGGL(nce_pair_bwd_kernel<kDO>, blocks, 256, bwd_lds(), s, p);
    return hipGetLastError();
}

}  // namespace voila
