// k_update.hip -- the belief update: action/observation folds, proposal and
// likelihood (update stage 1), single-workgroup normalisation and systematic
// resampling (stage 2), their batched forms, and the counter-based noise hook.
#include "kcommon.hpp"

namespace voila {

const ShapeInfo& shape_info(int shape) { return kShapeInfo[shape]; }

// First-layer biases with the action (then the observation) of every row
// folded in: the first layer's weight columns of those inputs times their
// values (a one-hot action selects its column), added to the bias.  Inputs are
// read from device memory; a discrete action outside [0, n_actions) or a
// non-finite action or observation value sets the status word to
// VOILA_ERR_INVALID_ARG (an out-of-range action is then taken as action 0).
__global__ __launch_bounds__(256) void fold_steps_kernel(FoldStepsParams p) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= p.width) return;
    for (int j = blockIdx.y; j < p.rows; j += gridDim.y) fold_element(p, j, r);
}

// One row of two networks in one launch (an update's transition and likelihood).
__global__ __launch_bounds__(256) void fold_pair_kernel(FoldStepsParams a, FoldStepsParams b) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    const FoldStepsParams& p = blockIdx.y ? b : a;
    if (r < p.width) fold_element(p, 0, r);
}

// fold_steps_kernel for many rows: a block stages its 256 rows of the columns in LDS,
// transposed (read once, coalesced, instead of once per row with a stride of nf
// floats), and the values of eight rows at a time, checked and rounded once
// instead of by every thread.  4,096 rows of 36 columns: 29 -> 12 us.
constexpr int kFoldRows = 8;
__global__ __launch_bounds__(256) void fold_rows_kernel(FoldStepsParams p) {
    extern __shared__ __attribute__((aligned(16))) char fold_smem[];
    float* sv = reinterpret_cast<float*>(fold_smem);  // [nf][kFoldRows] values of the rows
    float* wt = sv + p.nf * kFoldRows;                // [nf][257]: the transposing writes change banks
    const int r0 = blockIdx.x * 256, r = r0 + threadIdx.x, nr = min(256, p.width - r0);
    // element threadIdx.x + 256 k of the block's columns, its row and column stepped along
    const int dr = 256 / p.nf, dc = 256 - dr * p.nf;
    for (int e = threadIdx.x, er = e / p.nf, ec = e - er * p.nf; e < nr * p.nf; e += 256) {
        wt[ec * 257 + er] = p.w[(size_t)r0 * p.nf + e];
        er += dr;
        ec += dc;
        if (ec >= p.nf) {
            ec -= p.nf;
            ++er;
        }
    }
    const bool mine = (int)threadIdx.x < nr;
    const float bias = mine ? p.b[r] : 0.0f;
    const int na = p.n_actions > 0 ? p.n_actions : p.d_a, nc = p.obs ? p.nf : na;
    for (int j0 = blockIdx.y * kFoldRows; j0 < p.rows; j0 += gridDim.y * kFoldRows) {
        __syncthreads();
        for (int e = threadIdx.x; e < nc * kFoldRows; e += 256) {
            const int c = e / kFoldRows, j = min(j0 + e % kFoldRows, p.rows - 1);
            float v;
            bool bad;
            if (c < na && p.n_actions > 0) {
                int a = reinterpret_cast<const int32_t*>(p.cands)[j];
                bad = a < 0 || a >= p.n_actions;
                if (bad) a = 0;
                v = c == a ? 1.0f : 0.0f;
            } else {
                v = c < na ? reinterpret_cast<const float*>(p.cands)[(size_t)j * p.d_a + c]
                           : p.obs[(size_t)j * p.d_o + (c - na)];
                bad = !isfinite(v);
                if (p.bf16) v = (float)(__bf16)v;
            }
            if (bad && p.status && r0 == 0) p.status[0] = 1;
            sv[e] = v;
        }
        __syncthreads();
        if (!mine) continue;
        float acc[kFoldRows];
#pragma unroll
        for (int q = 0; q < kFoldRows; ++q) acc[q] = bias;
        for (int c = 0; c < nc; ++c) {
            const float w = wt[c * 257 + threadIdx.x];
#pragma unroll
            for (int q = 0; q < kFoldRows; ++q) acc[q] += w * sv[c * kFoldRows + q];
        }
#pragma unroll
        for (int q = 0; q < kFoldRows; ++q)
            if (j0 + q < p.rows) p.out[(size_t)(j0 + q) * p.width + r] = acc[q];
    }
}

// Per-instance first-layer bias with the instance's action (and observation)
// folded in; the fold inputs are read from device memory so the launch can be
// replayed from a graph with new actions / observations.
__global__ __launch_bounds__(256) void fold_batch_kernel(const FoldBatchItem* items, const void* actions,
                                                         const float* obs, int32_t* status) {
    const FoldBatchItem p = items[blockIdx.y];
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= p.width) return;
    float acc = p.b[r];
    int c = 0;
    if (p.n_actions > 0) {
        int a = reinterpret_cast<const int32_t*>(actions)[p.inst];
        if (a < 0 || a >= p.n_actions) {
            if (status && r == 0) status[0] = 1;
            a = 0;
        }
        acc += p.w[(size_t)r * p.nf + a];
        c = p.n_actions;
    } else {
        const float* ac = reinterpret_cast<const float*>(actions) + (size_t)p.inst * p.d_a;
        for (int j = 0; j < p.d_a; ++j, ++c) {
            float v = ac[j];
            if (p.bf16) v = (float)(__bf16)v;
            acc += p.w[(size_t)r * p.nf + c] * v;
        }
    }
    if (p.with_obs) {
        const float* ob = obs + (size_t)p.inst * p.d_o;
        for (int j = 0; j < p.d_o; ++j, ++c) {
            float v = ob[j];
            if (p.bf16) v = (float)(__bf16)v;
            acc += p.w[(size_t)r * p.nf + c] * v;
        }
    }
    p.out[r] = acc;
}

// ---------------------------------------------------------------------------
// update stage 1: proposal and likelihood
// ---------------------------------------------------------------------------
// One 32-particle tile of the update's first stage: proposal through the
// transition network, likelihood of the proposal, x = l / lambda (+ log prior).
template <int DT, int D_S, int D_W, int WIDTH, int NHID, bool SPLIT = false>
__device__ __forceinline__ void propose_tile(const NetPtrs& PT, const NetPtrs& PL, const ProposeParams& p, int tile,
                                             bool tile_ok, int lane, int g, int col, int wave = 0,
                                             char* lds = nullptr) {
    constexpr int SS = state_slots(D_S), SW = noise_slots(D_W);
    typedef Net<DT, WIDTH, NHID, in_slots(DT, D_S, 0, D_W)> NTT;
    typedef Net<DT, WIDTH, NHID, in_slots(DT, D_S, 0, 0)> NTL;
    const int i = tile * 32 + col;
    const bool valid = tile_ok && i < p.N;
    float slots[NTT::IN_SLOTS];
#pragma unroll
    for (int s = 0; s < NTT::IN_SLOTS; ++s) slots[s] = 0.0f;
    float st[SS];
#pragma unroll
    for (int s = 0; s < SS; ++s) {
        int f = 2 * s + g;
        st[s] = (valid && f < D_S) ? p.states[(size_t)i * D_S + f] : 0.0f;
        slots[s] = st[s];
    }
    if (p.noise) {
#pragma unroll
        for (int s = 0; s < SW; ++s) {
            int f = noise_feature(s, g);
            slots[SS + s] = (valid && f < D_W) ? p.noise[(size_t)i * D_W + f] : 0.0f;
        }
    } else {
        float nz[SW];
        noise_slots_philox<SW>(nz, p.key0, p.key1, (uint32_t)i, 0u, 0u, 5u, g);
#pragma unroll
        for (int s = 0; s < SW; ++s) slots[SS + s] = nz[s];
    }
    f32x16 d;
    if constexpr (SPLIT) {
        d = run_net_split<NTT>(PT, p.b0_trans, slots, lane, g, wave, lds);
    } else {
        auto srct = DirectFor<NTT>::make(PT);
        d = run_net<NTT>(srct, PT, p.b0_trans, slots, lane, g);
    }
    const bool writer = !SPLIT || wave == 0;  // a split tile is written by its first wave
    float ls[NTL::IN_SLOTS];
#pragma unroll
    for (int s = 0; s < NTL::IN_SLOTS; ++s) ls[s] = 0.0f;
#pragma unroll
    for (int s = 0; s < SS; ++s) {
        int f = 2 * s + g;
        st[s] += d[s];
        ls[s] = st[s];
        if (writer && valid && f < D_S) p.prop[(size_t)i * D_S + f] = st[s];
    }
    f32x16 lo;
    if constexpr (SPLIT) {
        lo = run_net_split<NTL>(PL, p.b0_lik, ls, lane, g, wave, lds);
    } else {
        auto srcl = DirectFor<NTL>::make(PL);
        lo = run_net<NTL>(srcl, PL, p.b0_lik, ls, lane, g);
    }
    if (writer && g == 0 && valid) {
        float l = lo[0];
        if (p.loglik) p.loglik[i] = l;
        if (!isfinite(l) && p.status) p.status[0] = 5;
        double x = (double)l / p.lambda;
        if (p.prior_w) x += log(p.prior_w[i]);
        p.x[i] = x;
    }
}

// Whether updates of a shape run this kernel: not those refused at model creation
// (binary32 wider than 256), those of the split rollout kernel's networks, and
// binary32 up to 256, which runs on half tiles at every size.
template <int DT, int WIDTH, int NHID>
constexpr bool propose_on_tiles() {
    return generic_compiled(DT, WIDTH, NHID) && !(pass_mode<WIDTH>() == kSplit && DT == DT_F32);
}

template <int DT, int D_S, int D_W, int WIDTH, int NHID, int MODE>
__global__ __launch_bounds__(256) void propose_kernel(ProposeParams p) {
    static_assert(propose_on_tiles<DT, WIDTH, NHID>(), "run by another kernel");
    constexpr bool WLDS = MODE == kResident;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    if (WLDS) {
        stage_blob(smem, p.trans.base, p.trans.bytes);
        stage_blob(smem + p.trans.bytes, p.lik.base, p.lik.bytes);
        __syncthreads();
    }
    const NetPtrs PT = net_ptrs(WLDS ? (const char*)smem : p.trans.base, p.trans);
    const NetPtrs PL = net_ptrs(WLDS ? (const char*)smem + p.trans.bytes : p.lik.base, p.lik);
    const int lane = threadIdx.x & 63, g = lane >> 5, col = lane & 31;
    const int wpb = blockDim.x >> 6;
    const int n_tiles = (p.N + 31) / 32;
    if constexpr (MODE == kSplit) {
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        for (int tile = blockIdx.x; tile < n_tiles; tile += gridDim.x)
            propose_tile<DT, D_S, D_W, WIDTH, NHID, true>(PT, PL, p, tile, true, lane, g, col, wave, smem);
    } else {
        for (int tile = blockIdx.x * wpb + (threadIdx.x >> 6); tile < n_tiles; tile += gridDim.x * wpb)
            propose_tile<DT, D_S, D_W, WIDTH, NHID>(PT, PL, p, tile, true, lane, g, col);
    }
}

// ---------------------------------------------------------------------------
// update stage 1 on half tiles
// ---------------------------------------------------------------------------
// A belief of 4,096 particles is 128 tiles of 32: half the CUs of the chip, one
// wave per SIMD.  Here a block advances 16 particles with one wave per 32 rows
// of a hidden layer (two 16x16 products per k-step; for width 256 eight waves,
// two per SIMD), on the weight fragments as the 32-row tiles are packed: lane
// (m, g4) of a product over two packed k-steps reads rows 2 m and 2 m + 1 (one
// load for both) of k-step g4 / 2, half g4 % 2.  Each product sums its k values
// in ascending order and the output layer's quarters are added in wave order,
// so the results are the tiles' bit for bit.  The weights come as one sequence
// over the layers of both networks, DEPTH k-step pairs ahead and across
// the layer barriers; the first layer's action and observation are folded by
// the block itself (256 + 256 rows by 512 threads) while the first fragments
// arrive, instead of by two launches before it.  Bound by the chain of k-steps
// of the six hidden products and the layer barriers (matrix cores 34 % busy):
// 4,096 particles in binary32 33.8 us, 76 + 10 on 32-row tiles.
template <int DT> struct HalfOps;
template <> struct HalfOps<DT_F32> {
    static constexpr int GROUP = 4;  // k-step pairs per 16-byte B operand read
    typedef f32x2 Weights;           // rows 2 m and 2 m + 1
    typedef float Fragment;
    static constexpr int DEPTH = 16;
    __device__ static __forceinline__ float row(const Weights& w, int h) { return w[h]; }
    __device__ static __forceinline__ float b(const u32x4& v, int s) { return __builtin_bit_cast(f32x4, v)[s % 4]; }
    __device__ static __forceinline__ f32x4 mul(float a, float b, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    // LDS offset of slot s of half g of particle n
    __device__ static __forceinline__ int slot(int s, int g, int n) {
        return (((s / 8) * 4 + (s % 2) * 2 + g) * 16 + n) * 16 + (s / 2) % 4 * 4;
    }
    __device__ static __forceinline__ void put(char* p, float v) { *reinterpret_cast<float*>(p) = v; }
    // ReLU of the wave's rows, stored where the next layer reads its B operands
    __device__ static __forceinline__ void store(char* act, const f32x4 (&acc)[2], int tile, int n, int g4) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int a = 0; a < 2; ++a)
                *reinterpret_cast<f32x2*>(act + (((2 * tile + g4 / 2) * 4 + 2 * h + a) * 16 + n) * 16 + 8 * (g4 % 2)) =
                    (f32x2){relu_f32(acc[h][2 * a]), relu_f32(acc[h][2 * a + 1])};
    }
};
template <> struct HalfOps<DT_BF16> {
    static constexpr int GROUP = 1;
    struct Weights {
        bf16x8 r[2];
    };
    typedef bf16x8 Fragment;
    static constexpr int DEPTH = 8;
    __device__ static __forceinline__ bf16x8 row(const Weights& w, int h) { return w.r[h]; }
    __device__ static __forceinline__ bf16x8 b(const u32x4& v, int) { return __builtin_bit_cast(bf16x8, v); }
    __device__ static __forceinline__ f32x4 mul(bf16x8 a, bf16x8 b, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    }
    __device__ static __forceinline__ int slot(int s, int g, int n) {
        return (((s / 16) * 4 + (s / 8 % 2) * 2 + g) * 16 + n) * 16 + s % 8 * 2;
    }
    __device__ static __forceinline__ void put(char* p, float v) { *reinterpret_cast<__bf16*>(p) = (__bf16)v; }
    __device__ static __forceinline__ void store(char* act, const f32x4 (&acc)[2], int tile, int n, int g4) {
#pragma unroll
        for (int a = 0; a < 2; ++a)
            *reinterpret_cast<uint2*>(act + ((tile * 4 + 2 * (g4 / 2) + a) * 16 + n) * 16 + 8 * (g4 % 2)) =
                make_uint2(relu_bf16x2(acc[0][2 * a], acc[1][2 * a]), relu_bf16x2(acc[0][2 * a + 1], acc[1][2 * a + 1]));
    }
};

template <class N> struct HalfNet {
    static constexpr int IN_S = cdiv(N::IN_KS, 2), HID_S = N::HID_KS / 2;  // k-step pairs per layer
    static constexpr int SEQ = IN_S + (N::NHID - 1) * HID_S;               // of the hidden layers
    static constexpr int OUT_S = HID_S / 4;                                // of an output quarter
    static constexpr int IN_BYTES = cdiv(IN_S, HalfOps<N::DT>::GROUP) * 1024;
    static constexpr int ACT = cdiv(HID_S, HalfOps<N::DT>::GROUP) * 1024;
    static_assert(N::CT == N::HT && N::HT % 4 == 0 && N::NO == 1, "layered networks of 4k tiles");
};
constexpr int kHalfPart = 4 * 32 * 16 * 4;  // the output quarters [quarter][feature][particle]

// The weights of k-step pair n of the networks' sequence (N, then NN if there is one).
template <class N, class NN, int n>
__device__ __forceinline__ typename HalfOps<N::DT>::Weights half_weights(const char* f0, const char* next, uint32_t off) {
    typedef typename HalfOps<N::DT>::Weights W;
    constexpr int FB = N::FRAG_BYTES * N::HT;
    if constexpr (n >= HalfNet<N>::SEQ) {
        return half_weights<NN, NN, n - HalfNet<N>::SEQ>(next, next, off);
    } else {
        constexpr int s = n < HalfNet<N>::IN_S ? 2 * n : N::IN_KS + 2 * (n - HalfNet<N>::IN_S);
        return *reinterpret_cast<const W*>(f0 + (size_t)s * FB + off);
    }
}

// One network on the block's 16 particles: inputs at `in`, first-layer bias
// `b0` (row order, LDS); the output quarters are left in `part` behind a
// barrier, for quarter_sum.  `ring` holds pairs R0 .. of the sequence.
template <class N, class NN, int R0, int D>
__device__ __forceinline__ void half_net(typename HalfOps<N::DT>::Weights (&ring)[D], const NetPtrs& P,
                                         const char* next, uint32_t off, const float* b0, const char* in, char* act,
                                         float* part, int d_out, int lane, int wave) {
    typedef HalfOps<N::DT> Ops;
    typedef HalfNet<N> HN;
    constexpr int FB = N::FRAG_BYTES;
    const int m = lane & 15, g4 = lane >> 4;
    const int quarter = wave & 3;
    const char* fo = P.f0 + (size_t)(FragIdx<N>::out(0) + quarter * (N::HID_KS / 4)) * FB;
    f32x4 acc[2];
    auto bias = [&](const float* b) {
        const f32x4 lo = *reinterpret_cast<const f32x4*>(b + 32 * wave + 8 * g4);
        const f32x4 hi = *reinterpret_cast<const f32x4*>(b + 32 * wave + 8 * g4 + 4);
        acc[0] = (f32x4){lo[0], lo[2], hi[0], hi[2]};
        acc[1] = (f32x4){lo[1], lo[3], hi[1], hi[3]};
    };
    typename Ops::Fragment of[HN::OUT_S];
    const int oh = wave >> 2;  // the output rows' half of this wave (waves 0 .. 3 take both if there are no others)
    auto out_weights = [&](int h) {
        const char* p = fo + opaque_zero();
        const int off = (g4 >> 1) * FB + (g4 & 1) * (FB / 2) + (16 * h + m) * (FB / 64);
#pragma unroll
        for (int s = 0; s < HN::OUT_S; ++s)
            of[s] = *reinterpret_cast<const typename Ops::Fragment*>(p + 2 * s * FB + off);
    };
    bias(b0);
    static_for<N::NHID>([&](auto li) {
        constexpr int l = decltype(li)::value;
        constexpr int KS = l == 0 ? HN::IN_S : HN::HID_S, n0 = l == 0 ? 0 : HN::IN_S + (l - 1) * HN::HID_S;
        constexpr int NG = cdiv(KS, Ops::GROUP);
        const char* src = l == 0 ? in : act + (l - 1) % 2 * HN::ACT;
        auto operand = [&](int q) { return *reinterpret_cast<const u32x4*>(src + (q * 64 + lane) * 16); };
        u32x4 b[2];
        b[0] = operand(0);
        f32x4 nb[2];
        if constexpr (l + 1 < N::NHID) {
            const float* bh = P.bh + l * N::WIDTH + 32 * wave + opaque_zero();
            nb[0] = *reinterpret_cast<const f32x4*>(bh + 8 * g4);
            nb[1] = *reinterpret_cast<const f32x4*>(bh + 8 * g4 + 4);
        }
        static_for<KS>([&](auto si) {
            constexpr int s = decltype(si)::value, q = s / Ops::GROUP;
            if constexpr (s % Ops::GROUP == 0 && q + 1 < NG) b[(q + 1) % 2] = operand(q + 1);
            typename Ops::Weights w = ring[(R0 + n0 + s) % D];
            // the second half of an odd last k-step pair holds other weights
            if constexpr (l == 0 && 2 * s + 1 == N::IN_KS)
                if (g4 >= 2) w = typename Ops::Weights{};
#pragma unroll
            for (int h = 0; h < 2; ++h) acc[h] = Ops::mul(Ops::row(w, h), Ops::b(b[q % 2], s), acc[h]);
            if constexpr (n0 + s + D < HN::SEQ || !std::is_same<N, NN>::value)
                ring[(R0 + n0 + s) % D] = half_weights<N, NN, n0 + s + D>(P.f0, next, off);
            if constexpr (l + 1 == N::NHID && s == KS / 2) out_weights(oh);
        });
        Ops::store(act + l % 2 * HN::ACT, acc, wave, m, g4);
        if constexpr (l + 1 < N::NHID) {
            acc[0] = (f32x4){nb[0][0], nb[0][2], nb[1][0], nb[1][2]};
            acc[1] = (f32x4){nb[0][1], nb[0][3], nb[1][1], nb[1][3]};
        }
        __syncthreads();
    });
    const char* src = act + (N::NHID - 1) % 2 * HN::ACT + quarter * (HN::ACT / 4);
    for (int h = oh; 16 * h < 2 * cdiv(d_out, 2); h += N::HT / 4) {
        if (h != oh) out_weights(h);
        f32x4 o = {};
        if (quarter == 0) o = *reinterpret_cast<const f32x4*>(P.bo + 16 * h + 4 * g4);
#pragma unroll
        for (int s = 0; s < HN::OUT_S; ++s)
            o = Ops::mul(of[s], Ops::b(*reinterpret_cast<const u32x4*>(src + (s / Ops::GROUP * 64 + lane) * 16), s), o);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            part[(quarter * 32 + 2 * (8 * h + 4 * (g4 / 2) + i) + g4 % 2) * 16 + m] = o[i];
    }
    __syncthreads();
}

__device__ __forceinline__ float quarter_sum(const float* part, int f, int n) {
    const float* p = part + f * 16 + n;
    return ((p[0] + p[512]) + p[1024]) + p[1536];
}

template <int DT, int D_S, int D_W, int WIDTH, int NHID>
struct HalfPropose {
    typedef Net<DT, WIDTH, NHID, in_slots(DT, D_S, 0, D_W)> NTT;
    typedef Net<DT, WIDTH, NHID, in_slots(DT, D_S, 0, 0)> NTL;
    static constexpr int IN_T = HalfNet<NTT>::IN_BYTES, IN_L = HalfNet<NTL>::IN_BYTES;
    static constexpr int COLS = 2 * kHalfCols * 4;  // folded values: action | action, observation
    static constexpr int LDS = IN_T + IN_L + 2 * HalfNet<NTT>::ACT + kHalfPart + 2 * WIDTH * 4 + COLS;
};

template <int DT, int D_S, int D_W, int WIDTH, int NHID>
__global__ __launch_bounds__(2 * WIDTH, 2) void propose_half_kernel(ProposeHalfParams hp) {
    if constexpr (pass_mode<WIDTH>() != kSplit) {
        return;  // the other networks run in propose_kernel or propose_split_kernel
    } else {
    typedef HalfPropose<DT, D_S, D_W, WIDTH, NHID> H;
    typedef typename H::NTT NTT;
    typedef typename H::NTL NTL;
    typedef HalfOps<DT> Ops;
    constexpr int T = 2 * WIDTH, SS = state_slots(D_S), D = Ops::DEPTH;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    char* const in_t = smem;
    char* const in_l = in_t + H::IN_T;
    char* const act = in_l + H::IN_L;
    float* const part = reinterpret_cast<float*>(act + 2 * HalfNet<NTT>::ACT);
    float* const b0 = part + kHalfPart / 4;  // [trans, lik][WIDTH]
    float* const cols = b0 + 2 * WIDTH;      // [trans, lik][kHalfCols]
    const ProposeParams& p = hp.p;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const NetPtrs PT = net_ptrs(p.trans.base, p.trans), PL = net_ptrs(p.lik.base, p.lik);
    constexpr int FB = NTT::FRAG_BYTES;
    const uint32_t off0 = (((lane >> 5) & 1) * NTT::HT + wave) * FB + ((lane >> 4) & 1) * (FB / 2) + 2 * (lane & 15) * (FB / 64);
    typename Ops::Weights ring[D];
    // addresses opaque to the compiler, or it computes every k-step's ahead of the loop
    NetPtrs QT = PT, QL = PL;
    uint32_t off;
    auto fill = [&] {
        QT.f0 = PT.f0 + opaque_zero();
        QL.f0 = PL.f0 + opaque_zero();
        off = off0;
        asm volatile("" : "+v"(off));
        static_for<D>([&](auto ni) {
            constexpr int n = decltype(ni)::value;
            ring[n] = half_weights<NTT, NTL, n>(QT.f0, QL.f0, off);
        });
    };
    fill();
    for (int e = tid; e < (H::IN_T + H::IN_L) / 4; e += T) reinterpret_cast<float*>(smem)[e] = 0.0f;
    // folded values, checked and rounded once
    if (tid < 2 * kHalfCols) {
        const FoldStepsParams& f = tid < kHalfCols ? hp.fold_trans : hp.fold_lik;
        const int c = tid % kHalfCols, na = f.n_actions > 0 ? f.n_actions : f.d_a;
        float v = 0.0f;
        bool bad = false;
        if (c < na && f.n_actions > 0) {
            int a = reinterpret_cast<const int32_t*>(f.cands)[0];
            bad = a < 0 || a >= f.n_actions;
            v = c == (bad ? 0 : a) ? 1.0f : 0.0f;
        } else if (c < na + f.d_o) {
            v = c < na ? reinterpret_cast<const float*>(f.cands)[c] : f.obs[c - na];
            bad = !isfinite(v);
            if (f.bf16) v = (float)(__bf16)v;
        }
        if (bad && f.status) f.status[0] = 1;
        cols[tid] = v;
    }
    __syncthreads();
    {
        // thread r of each half folds row r
        const int r = tid % WIDTH;
        const FoldStepsParams& f = tid < WIDTH ? hp.fold_trans : hp.fold_lik;
        const float* v = cols + (tid < WIDTH ? 0 : kHalfCols);
        const float* w = f.w + (size_t)r * f.nf;
        const int nc = (f.n_actions > 0 ? f.n_actions : f.d_a) + f.d_o;
        float a = f.b[r];
#pragma unroll 4
        for (int c = 0; c < nc; ++c) a += w[c] * v[c];
        b0[tid] = a;
    }
    const int n_half = (p.N + 15) / 16;
    for (int u = blockIdx.x; u < n_half; u += gridDim.x) {
        if (u != (int)blockIdx.x) fill();
        // inputs: states of (particle, feature), noise of (particle, block of four, half)
        float st[cdiv(32 * SS, T)];
#pragma unroll
        for (int k = 0; k < cdiv(32 * SS, T); ++k) {
            const int e = tid + k * T, f = e % (2 * SS), n = e / (2 * SS), i = u * 16 + n;
            st[k] = (n < 16 && i < p.N && f < D_S) ? p.states[(size_t)i * D_S + f] : 0.0f;
            if (n < 16) Ops::put(in_t + Ops::slot(f / 2, f % 2, n), st[k]);
        }
        for (int e = tid; e < 16 * noise_slots(D_W); e += T) {
            const int n = e % 16, g = e / 16 % 2, blk = e / 32, i = u * 16 + n, f = 4 * blk + 2 * g;
            float z0, z1;
            if (p.noise) {
                z0 = (i < p.N && f < D_W) ? p.noise[(size_t)i * D_W + f] : 0.0f;
                z1 = (i < p.N && f + 1 < D_W) ? p.noise[(size_t)i * D_W + f + 1] : 0.0f;
            } else {
                const uint4 w = philox4x32_10(make_uint4((uint32_t)i, 0u, 0u, (5u << 16) | (uint32_t)blk), p.key0, p.key1);
                box_muller(g ? w.z : w.x, g ? w.w : w.y, z0, z1);
            }
            Ops::put(in_t + Ops::slot(SS + 2 * blk, g, n), z0);
            Ops::put(in_t + Ops::slot(SS + 2 * blk + 1, g, n), z1);
        }
        __syncthreads();
        half_net<NTT, NTL, 0, D>(ring, QT, QL.f0, off, b0, in_t, act, part, D_S, lane, wave);
#pragma unroll
        for (int k = 0; k < cdiv(32 * SS, T); ++k) {
            const int e = tid + k * T, f = e % (2 * SS), n = e / (2 * SS), i = u * 16 + n;
            if (n >= 16) continue;
            const float s1 = st[k] + quarter_sum(part, f, n);
            Ops::put(in_l + Ops::slot(f / 2, f % 2, n), s1);
            if (i < p.N && f < D_S) p.prop[(size_t)i * D_S + f] = s1;
        }
        __syncthreads();
        half_net<NTL, NTL, HalfNet<NTT>::SEQ % D, D>(ring, QL, QL.f0, off, b0 + WIDTH, in_l, act, part, 1, lane, wave);
        if (tid < 16 && u * 16 + tid < p.N) {
            const int i = u * 16 + tid;
            const float l = quarter_sum(part, 0, tid);
            if (p.loglik) p.loglik[i] = l;
            if (!isfinite(l) && p.status) p.status[0] = 5;
            double x = (double)l / p.lambda;
            if (p.prior_w) x += log(p.prior_w[i]);
            p.x[i] = x;
        }
    }
    }
}

// Update stage 1 of many instances: block items (instance, first tile, tiles),
// networks restaged in LDS on an instance change.
template <int DT, int D_S, int D_W, int WIDTH, int NHID>
__global__ __launch_bounds__(512) void propose_batch_kernel(BatchProposeParams bp) {
    if constexpr (WIDTH > 64) {
        return;  // batches need networks that fit in LDS (the launcher refuses wider ones)
    } else {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    __shared__ int s_item;
    const int lane = threadIdx.x & 63, g = lane >> 5, col = lane & 31;
    const int wave = threadIdx.x >> 6;
    int loaded = -1;
    int item = blockIdx.x;
    for (int iter = 0;; ++iter) {
        if (bp.dynamic) {
            if (threadIdx.x == 0) s_item = atomicAdd(bp.counter, 1);
            __syncthreads();
            item = s_item;
            __syncthreads();
        } else if (iter > 0) {
            item += gridDim.x;
        }
        if (item >= bp.n_items) break;
        const int4 it = bp.items[item];
        ProposeParams p = bp.insts[it.x];
        p.status = bp.status;
        if (it.x != loaded) {
            __syncthreads();
            stage_blob(smem, p.trans.base, p.trans.bytes);
            stage_blob(smem + p.trans.bytes, p.lik.base, p.lik.bytes);
            __syncthreads();
            loaded = it.x;
        }
        const NetPtrs PT = net_ptrs(smem, p.trans);
        const NetPtrs PL = net_ptrs(smem + p.trans.bytes, p.lik);
        propose_tile<DT, D_S, D_W, WIDTH, NHID>(PT, PL, p, it.y + wave, wave < it.z, lane, g, col);
    }
    }
}

// Proposals of models whose transition network runs in the split evaluation
// (more than two hidden layers wider than 256): a block of kPropSplitWaves
// waves advances two 32-particle tiles, every layer split over the waves
// (run_net_split_owned); wave q forms tile q's inputs [s, w] (noise as in
// propose_tile) and writes its proposals s + f_T(s, a, w).
constexpr int kPropSplitWaves = 8, kPropSplitDepth = 3;

template <int DT, int D_S, int D_W, int WIDTH, int NHID, int ST>
__global__ __launch_bounds__(64 * kPropSplitWaves) void propose_split_kernel(ProposeParams p) {
    if constexpr (!net_compiled(DT, WIDTH) || generic_compiled(DT, WIDTH, NHID)) {
        return;  // the other networks run in propose_kernel
    } else {
    constexpr int SS = state_slots(D_S), SW = noise_slots(D_W), NO = cdiv(D_S, 32);
    constexpr int DEPTH = ST > 1 ? kPropSplitDepth : kSingleTileDepth;
    typedef Net<DT, WIDTH, NHID, in_slots(DT, D_S, 0, D_W), WIDTH / 32, NO> NT;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    char* const in_lds = smem + ST * SplitLds<NT>::ACT;
    const int lane = threadIdx.x & 63, g = lane >> 5, col = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool owner = wave < ST;
    const int n_groups = ((p.N + 31) / 32 + ST - 1) / ST;
    const NetPtrs P = net_ptrs(p.trans.base, p.trans);
    for (int u = p.tile0 / ST + blockIdx.x; u < n_groups; u += gridDim.x) {
        const int i = (u * ST + (owner ? wave : 0)) * 32 + col;
        const bool valid = owner && i < p.N;
        if (owner) {
            float slots[NT::IN_SLOTS];
#pragma unroll
            for (int s = 0; s < NT::IN_SLOTS; ++s) slots[s] = 0.0f;
#pragma unroll
            for (int s = 0; s < SS; ++s) {
                const int f = 2 * s + g;
                slots[s] = (valid && f < D_S) ? p.states[(size_t)i * D_S + f] : 0.0f;
            }
            if (p.noise) {
#pragma unroll
                for (int s = 0; s < SW; ++s) {
                    const int f = noise_feature(s, g);
                    slots[SS + s] = (valid && f < D_W) ? p.noise[(size_t)i * D_W + f] : 0.0f;
                }
            } else {
                float nz[SW];
                noise_slots_philox<SW>(nz, p.key0, p.key1, (uint32_t)i, 0u, 0u, 5u, g);
#pragma unroll
                for (int s = 0; s < SW; ++s) slots[SS + s] = nz[s];
            }
            split_stage_inputs<NT>(in_lds + wave * SplitIn<NT>::BYTES, slots, lane);
        }
        float d[NO][16];
        run_net_split_owned<NT, ST, kPropSplitWaves, DEPTH>(P, p.b0_trans, in_lds, d, lane, g, wave, smem);
        if (valid)
#pragma unroll
            for (int s = 0; s < SS; ++s) {
                const int f = 2 * s + g;
                if (f < D_S) p.prop[(size_t)i * D_S + f] = p.states[(size_t)i * D_S + f] + d[s / 16][s % 16];
            }
    }
    }
}

// The likelihood of the proposals for those models, x = l / lambda (+ log
// prior): the block's four waves split one 32-particle tile's layers
// (run_net_split), as propose_kernel does at width 256.
template <int DT, int D_S, int LW, int LNH>
__global__ __launch_bounds__(256) void lik_rows_kernel(ProposeParams p) {
    static_assert(pass_mode<LW>() == kSplit, "likelihood widths above 64 and up to 256");
    typedef Net<DT, LW, LNH, in_slots(DT, D_S, 0, 0)> NTL;
    constexpr int SS = state_slots(D_S);
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int lane = threadIdx.x & 63, g = lane >> 5, col = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const NetPtrs PL = net_ptrs(p.lik.base, p.lik);
    const int n_tiles = (p.N + 31) / 32;
    for (int tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        const int i = tile * 32 + col;
        const bool valid = i < p.N;
        float ls[NTL::IN_SLOTS];
#pragma unroll
        for (int s = 0; s < NTL::IN_SLOTS; ++s) ls[s] = 0.0f;
#pragma unroll
        for (int s = 0; s < SS; ++s) {
            const int f = 2 * s + g;
            ls[s] = (valid && f < D_S) ? p.prop[(size_t)i * D_S + f] : 0.0f;
        }
        const f32x16 lo = run_net_split<NTL>(PL, p.b0_lik, ls, lane, g, wave, smem);
        if (wave == 0 && g == 0 && valid) {
            const float l = lo[0];
            if (p.loglik) p.loglik[i] = l;
            if (!isfinite(l) && p.status) p.status[0] = 5;
            double x = (double)l / p.lambda;
            if (p.prior_w) x += log(p.prior_w[i]);
            p.x[i] = x;
        }
    }
}

__global__ __launch_bounds__(kNormResThreads) void norm_res_kernel(NormResParams p) {
    __shared__ double buf[kNormResMaxN];
    __shared__ int ids[kNormResMaxN];
    __shared__ double redd[kNRWaves];
    __shared__ int redi[kNRWaves];
    norm_res_body(p, buf, redd, redi, ids, blockIdx.x, gridDim.x);
}

// One workgroup per instance.
__global__ __launch_bounds__(kNormResThreads) void norm_res_batch_kernel(const NormResParams* ps, const uint32_t* us,
                                                                          int32_t* status) {
    __shared__ double buf[kNormResMaxN];
    __shared__ int ids[kNormResMaxN];
    __shared__ double redd[kNRWaves];
    __shared__ int redi[kNRWaves];
    NormResParams p = ps[blockIdx.x];
    if (us) p.U = us[blockIdx.x];
    p.status = status;
    norm_res_body(p, buf, redd, redi, ids);
}

__global__ __launch_bounds__(256) void philox_kernel(PhiloxParams p) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= p.n) return;
    const int nb = (p.d + 3) / 4;
    for (int b = 0; b < nb; ++b) {
        uint4 w = philox4x32_10(make_uint4(p.c0 + (uint32_t)r, p.c1, p.c2, (p.stream << 16) | (uint32_t)b), p.key0,
                                p.key1);
        if (p.words) {
            uint32_t* o = p.words + ((size_t)r * nb + b) * 4;
            o[0] = w.x; o[1] = w.y; o[2] = w.z; o[3] = w.w;
        }
        float z[4];
        box_muller(w.x, w.y, z[0], z[1]);
        box_muller(w.z, w.w, z[2], z[3]);
        for (int j = 0; j < 4; ++j)
            if (4 * b + j < p.d) p.out[(size_t)r * p.d + 4 * b + j] = z[j];
    }
}

// launchers
bool weights_in_lds(int shape) { return kShapeInfo[shape].width <= 64; }

#define VOILA_IN_SLOTS(fn, expr)                                                                   \
    int fn(int shape, int dt) {                                                                     \
        const ShapeInfo& s = kShapeInfo[shape];                                                     \
        (void)s;                                                                                    \
        return expr;                                                                                \
    }
VOILA_IN_SLOTS(plan_in_slots, in_slots(dt, s.d_s, s.n_actions > 0 ? 0 : s.d_a, s.d_w))
VOILA_IN_SLOTS(update_in_slots, in_slots(dt, s.d_s, 0, s.d_w))
VOILA_IN_SLOTS(obs_in_slots, in_slots(dt, s.d_s, 0, s.d_wz))
VOILA_IN_SLOTS(lik_in_slots, in_slots(dt, s.d_s, 0, 0))
VOILA_IN_SLOTS(nce_in_slots, in_slots(dt, s.d_o, 0, 0))
#undef VOILA_IN_SLOTS

int pass_tiles_per_block(int shape) { return pass_split(shape) ? 1 : 4; }

template <int DT, int D_S, int D_W, int W, int NH>
hipError_t launch_propose_one(const ProposeParams& p, int blocks, size_t lds, hipStream_t s) {
    if constexpr (!propose_on_tiles<DT, W, NH>()) {
        return hipErrorInvalidValue;
    } else {
        hipLaunchKernelGGL((propose_kernel<DT, D_S, D_W, W, NH, pass_mode<W>()>), blocks, 256, lds, s, p);
        return hipGetLastError();
    }
}
template <int DT, int D_S, int D_W, int W, int NH>
int propose_occupancy() {
    if constexpr (!propose_on_tiles<DT, W, NH>())
        return 1;
    else
        return occupancy(propose_kernel<DT, D_S, D_W, W, NH, pass_mode<W>()>, lds_for_width<W>() ? 2 * kLdsGuess : kSplitLds);
}

hipError_t launch_propose(int shape, int dt, const ProposeParams& p, int blocks, hipStream_t s) {
    const size_t lds = weights_in_lds(shape) ? (size_t)p.trans.bytes + p.lik.bytes : pass_split(shape) ? kSplitLds : 0;
    switch (shape * 2 + dt) {
#define X(id, ds, na, da, dw, dox, dwz, w, nh)                                      \
    case id * 2 + 0:                                                               \
        return launch_propose_one<DT_F32, ds, dw, w, nh>(p, blocks, lds, s);       \
    case id * 2 + 1:                                                               \
        return launch_propose_one<DT_BF16, ds, dw, w, nh>(p, blocks, lds, s);
        VOILA_SHAPES(X)
#undef X
    }
    return hipErrorInvalidValue;
}

#define PROPH_K(id, ds, na, da, dw, dox, dwz, w, nh, DT) propose_half_kernel<DT, ds, dw, w, nh>

template <int DT, int D_S, int D_W, int W, int NH>
constexpr size_t propose_half_lds() {
    if constexpr (pass_mode<W>() != kSplit)
        return 0;
    else
        return HalfPropose<DT, D_S, D_W, W, NH>::LDS;
}

hipError_t launch_propose_half(int shape, int dt, const ProposeHalfParams& p, int blocks, hipStream_t s) {
    if (!pass_split(shape) || p.fold_trans.nf > kHalfCols || p.fold_lik.nf > kHalfCols) return hipErrorInvalidValue;
    switch (shape * 2 + dt) {
#define X(id, ds, na, da, dw, dox, dwz, w, nh)                                                                    \
    case id * 2 + 0:                                                                                             \
        hipLaunchKernelGGL((PROPH_K(id, ds, na, da, dw, dox, dwz, w, nh, DT_F32)), blocks, 2 * w,                 \
                           (propose_half_lds<DT_F32, ds, dw, w, nh>()), s, p);                                    \
        break;                                                                                                   \
    case id * 2 + 1:                                                                                             \
        hipLaunchKernelGGL((PROPH_K(id, ds, na, da, dw, dox, dwz, w, nh, DT_BF16)), blocks, 2 * w,                \
                           (propose_half_lds<DT_BF16, ds, dw, w, nh>()), s, p);                                   \
        break;
        VOILA_SHAPES(X)
#undef X
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

int propose_blocks_per_cu(int shape, int dt) {
    switch (shape * 2 + dt) {
#define X(id, ds, na, da, dw, dox, dwz, w, nh)                     \
    case id * 2 + 0:                                              \
        return propose_occupancy<DT_F32, ds, dw, w, nh>();        \
    case id * 2 + 1:                                              \
        return propose_occupancy<DT_BF16, ds, dw, w, nh>();
        VOILA_SHAPES(X)
#undef X
    }
    return 1;
}

int lik_shape_width(int shape) {
#define X(id, ds, lw, lnh) \
    if (shape == id) return lw;
    VOILA_LIK_SHAPES(X)
#undef X
    return 0;
}
int lik_shape_hidden(int shape) {
#define X(id, ds, lw, lnh) \
    if (shape == id) return lnh;
    VOILA_LIK_SHAPES(X)
#undef X
    return 0;
}

#define PROPS_K(id, ds, na, da, dw, dox, dwz, w, nh, DT) propose_split_kernel<DT, ds, dw, w, nh, kPropSplitTiles>
#define PROPS_1(id, ds, na, da, dw, dox, dwz, w, nh, DT) propose_split_kernel<DT, ds, dw, w, nh, 1>

template <int DT, int D_S, int D_W, int W, int NH, int ST = kPropSplitTiles>
constexpr size_t propose_split_lds() {
    if constexpr (!net_compiled(DT, W) || generic_compiled(DT, W, NH)) {
        return 0;
    } else {
        typedef Net<DT, W, NH, in_slots(DT, D_S, 0, D_W), W / 32, cdiv(D_S, 32)> NT;
        return (size_t)ST * (SplitLds<NT>::ACT + SplitIn<NT>::BYTES);
    }
}

template <class K>
void launch_propose_split_one(K k, size_t lds, int blocks, const ProposeParams& p, hipStream_t s) {
    if (lds > 65536) (void)hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(k, blocks, 64 * kPropSplitWaves, lds, s, p);
}

// Rounds of tile groups over the chip's `cap` blocks, then the remaining
// tiles, singly if they are then one round.
template <class KS, class K1>
void launch_propose_groups(KS ks, K1 k1, size_t lds, size_t lds1, int cap, int cus, ProposeParams p, hipStream_t s) {
    const int n_tiles = (p.N + 31) / 32;
    const int grouped = (int)split_grouped_tiles(n_tiles, kPropSplitTiles, cap, cus);
    if (grouped > 0) {
        const int groups = (grouped + kPropSplitTiles - 1) / kPropSplitTiles;
        ProposeParams q = p;
        if (grouped < n_tiles) q.N = 32 * grouped;
        launch_propose_split_one(ks, lds, groups < cap ? groups : cap, q, s);
    }
    if (grouped < n_tiles) {
        p.tile0 = grouped;
        launch_propose_split_one(k1, lds1, n_tiles - grouped, p, s);
    }
}

hipError_t launch_propose_split(int shape, int dt, const ProposeParams& p, int cap, int cus, hipStream_t s) {
    switch (shape * 2 + dt) {
#define V(id, ds, na, da, dw, dox, dwz, w, nh, DT)                                                                 \
    if (propose_split_lds<DT, ds, dw, w, nh>() == 0) return hipErrorInvalidValue;                                  \
    launch_propose_groups(PROPS_K(id, ds, na, da, dw, dox, dwz, w, nh, DT), PROPS_1(id, ds, na, da, dw, dox, dwz, w, nh, DT), \
                          propose_split_lds<DT, ds, dw, w, nh>(), propose_split_lds<DT, ds, dw, w, nh, 1>(), cap, cus, p, s)
#define X(id, ds, na, da, dw, dox, dwz, w, nh)                    \
    case id * 2 + 0: {                                           \
        V(id, ds, na, da, dw, dox, dwz, w, nh, DT_F32);          \
        break;                                                   \
    }                                                            \
    case id * 2 + 1: {                                           \
        V(id, ds, na, da, dw, dox, dwz, w, nh, DT_BF16);         \
        break;                                                   \
    }
        VOILA_SHAPES(X)
#undef X
#undef V
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

int propose_split_blocks_per_cu(int shape, int dt) {
    switch (shape * 2 + dt) {
#define X(id, ds, na, da, dw, dox, dwz, w, nh)                                                              \
    case id * 2 + 0:                                                                                       \
        return occupancy_t(PROPS_K(id, ds, na, da, dw, dox, dwz, w, nh, DT_F32), 64 * kPropSplitWaves,       \
                           propose_split_lds<DT_F32, ds, dw, w, nh>());                                     \
    case id * 2 + 1:                                                                                       \
        return occupancy_t(PROPS_K(id, ds, na, da, dw, dox, dwz, w, nh, DT_BF16), 64 * kPropSplitWaves,      \
                           propose_split_lds<DT_BF16, ds, dw, w, nh>());
        VOILA_SHAPES(X)
#undef X
    }
    return 1;
}

hipError_t launch_lik_rows(int shape, int dt, const ProposeParams& p, int blocks, hipStream_t s) {
    switch (shape * 2 + dt) {
#define X(id, ds, lw, lnh)                                                                                 \
    case id * 2 + 0:                                                                                      \
        hipLaunchKernelGGL((lik_rows_kernel<DT_F32, ds, lw, lnh>), blocks, 256, kSplitLds, s, p);         \
        break;                                                                                            \
    case id * 2 + 1:                                                                                      \
        hipLaunchKernelGGL((lik_rows_kernel<DT_BF16, ds, lw, lnh>), blocks, 256, kSplitLds, s, p);        \
        break;
        VOILA_LIK_SHAPES(X)
#undef X
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

int lik_rows_blocks_per_cu(int shape, int dt) {
    switch (shape * 2 + dt) {
#define X(id, ds, lw, lnh)                                                          \
    case id * 2 + 0:                                                               \
        return occupancy(lik_rows_kernel<DT_F32, ds, lw, lnh>, kSplitLds);         \
    case id * 2 + 1:                                                               \
        return occupancy(lik_rows_kernel<DT_BF16, ds, lw, lnh>, kSplitLds);
        VOILA_LIK_SHAPES(X)
#undef X
    }
    return 1;
}

#define PROPB_K(id, ds, na, da, dw, dox, dwz, w, nh, DT) propose_batch_kernel<DT, ds, dw, w, nh>

hipError_t launch_propose_batch(int shape, int dt, const BatchProposeParams& p, int blocks, int wpb, size_t lds,
                                hipStream_t s) {
    if (!weights_in_lds(shape)) return hipErrorInvalidValue;
    switch (shape * 2 + dt) {
#define X(id, ds, na, da, dw, dox, dwz, w, nh)                                                                     \
    case id * 2 + 0:                                                                                              \
        hipLaunchKernelGGL((PROPB_K(id, ds, na, da, dw, dox, dwz, w, nh, DT_F32)), blocks, 64 * wpb, lds, s, p);   \
        break;                                                                                                    \
    case id * 2 + 1:                                                                                              \
        hipLaunchKernelGGL((PROPB_K(id, ds, na, da, dw, dox, dwz, w, nh, DT_BF16)), blocks, 64 * wpb, lds, s, p);  \
        break;
        VOILA_SHAPES(X)
#undef X
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

int propose_batch_blocks_per_cu(int shape, int dt, int wpb, size_t lds) {
    switch (shape * 2 + dt) {
#define X(id, ds, na, da, dw, dox, dwz, w, nh)                                                        \
    case id * 2 + 0:                                                                                 \
        return occupancy_t(PROPB_K(id, ds, na, da, dw, dox, dwz, w, nh, DT_F32), 64 * wpb, lds);      \
    case id * 2 + 1:                                                                                 \
        return occupancy_t(PROPB_K(id, ds, na, da, dw, dox, dwz, w, nh, DT_BF16), 64 * wpb, lds);
        VOILA_SHAPES(X)
#undef X
    }
    return 1;
}

hipError_t launch_fold_batch(const FoldBatchItem* d_items, int n_items, int max_width, const void* d_actions,
                             const float* d_obs, int32_t* d_status, hipStream_t s) {
    if (n_items == 0) return hipSuccess;
    hipLaunchKernelGGL(fold_batch_kernel, dim3((max_width + 255) / 256, n_items), 256, 0, s, d_items, d_actions, d_obs,
                       d_status);
    return hipGetLastError();
}

hipError_t launch_norm_res_batch(const NormResParams* d_ps, int n_inst, const uint32_t* d_u, int32_t* d_status,
                                 hipStream_t s) {
    if (n_inst == 0) return hipSuccess;
    hipLaunchKernelGGL(norm_res_batch_kernel, n_inst, kNormResThreads, 0, s, d_ps, d_u, d_status);
    return hipGetLastError();
}

// Whether the kernel for many rows folds p: from one row per CU on (below, a
// block per row fills no more CUs than this one's staging costs), and from 4,096
// rows where they are narrower than the block (calls around a width-64 fold: 640
// rows 89.4 against 90.3 us, 1,024 28.6 / 29.1, 4,096 100.5 / 98.9, 8,000 48.0 /
// 46.6); the LDS without an attribute holds 61 columns, every compiled shape's.
size_t fold_rows_lds(const FoldStepsParams& p) { return (size_t)p.nf * (257 + kFoldRows) * sizeof(float); }
bool fold_takes_rows(const FoldStepsParams& p) {
    return p.rows >= (p.width >= 256 ? 256 : 4096) && fold_rows_lds(p) <= 65536;
}

hipError_t launch_fold_steps(const FoldStepsParams& p, hipStream_t s) {
    if (p.rows == 0) return hipSuccess;
    if (fold_takes_rows(p)) {
        const int groups = (p.rows + kFoldRows - 1) / kFoldRows;
        hipLaunchKernelGGL(fold_rows_kernel, dim3((p.width + 255) / 256, groups < 512 ? groups : 512), 256,
                           fold_rows_lds(p), s, p);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(fold_steps_kernel, dim3((p.width + 255) / 256, p.rows < 65535 ? p.rows : 65535), 256, 0, s, p);
    return hipGetLastError();
}

// Workgroups of a resampling: one per kNormResShare positions, as the search and
// the gather were half of one workgroup's time (4,096 rows of 64 bytes: LDS
// search 5.0, gather 6.2 of 21.3 us; 13.0 with 16 workgroups).  One where an
// output overlaps an input, which the others may still have to read.
constexpr int kNormResShare = 256;
int norm_res_slices(const NormResParams& p) {
    if (!p.do_resample) return 1;
    const size_t n = (size_t)p.N;
    const struct {
        const void* at;
        size_t bytes;
    } in[] = {{p.x, 8 * n}, {p.loglik, 4 * n}, {p.prior_w, 8 * n}, {p.w_in, 8 * n}, {p.src, p.dst ? 4 * n * p.row_floats : 0}},
      out[] = {{p.w_out, 8 * n}, {p.stats, 16}, {p.idx_out, 4 * n}, {p.dst, p.src ? 4 * n * p.row_floats : 0}};
    for (const auto& o : out)
        for (const auto& i : in)
            if (!buffers_apart(o.at, o.bytes, i.at, i.bytes)) return 1;
    return (p.N + kNormResShare - 1) / kNormResShare;
}

hipError_t launch_fold_pair(const FoldStepsParams& a, const FoldStepsParams& b, hipStream_t s) {
    const int width = a.width > b.width ? a.width : b.width;
    hipLaunchKernelGGL(fold_pair_kernel, dim3((width + 255) / 256, 2), 256, 0, s, a, b);
    return hipGetLastError();
}

hipError_t launch_norm_res(const NormResParams& p, hipStream_t s) {
    hipLaunchKernelGGL(norm_res_kernel, norm_res_slices(p), kNormResThreads, 0, s, p);
    return hipGetLastError();
}

hipError_t launch_philox(const PhiloxParams& p, hipStream_t s) {
    if (p.n == 0) return hipSuccess;
    hipLaunchKernelGGL(philox_kernel, (p.n + 255) / 256, 256, 0, s, p);
    return hipGetLastError();
}

}  // namespace voila
