// k_plan.hip -- the persistent rollout kernel (plan), its batched form and
// the fixed-order Q reduction.
//
// plan_kernel     each wave owns a (candidate, 32-particle) tile, keeps the 32
//                 states in registers for the whole horizon and runs every
//                 transition-network layer on the matrix cores (transposed
//                 evaluation, see device.hpp), with the noise drawn in registers
//                 from Philox.  Small networks are staged in LDS once per block;
//                 wide ones stream their fragments from L2.
// plan_split_kernel  deep wide networks, each layer split over a block's waves.
// plan_half_kernel   small plans, 16 particles per block.
// q_reduce_kernel fixed-order sum of the per-tile (or per-half-tile) partial
//                 returns into Q.
#include "plan_unit.hpp"

namespace voila {

// Deep wide transition networks (more than two hidden layers wider than 256,
// the depth of the paper's distilled samplers): a block of kPlanSplitWaves
// waves advances kPlanSplitTiles 32-particle tiles of one candidate together,
// each layer split over the waves (run_net_split_owned), so that every
// weight fragment read from L2 serves all of the block's tiles.  Wave q
// carries tile q's states, noise and return, stages the tile's first-layer
// operands in LDS each step and receives the tile's output; the other waves
// hold no per-particle state.  The per-tile partial returns are those of
// plan_kernel.
#ifndef VOILA_PLAN_SPLIT_WAVES
#define VOILA_PLAN_SPLIT_WAVES 8
#endif
#ifndef VOILA_PLAN_SPLIT_TILES
#define VOILA_PLAN_SPLIT_TILES 2
#endif
#ifndef VOILA_PLAN_SPLIT_DEPTH
#define VOILA_PLAN_SPLIT_DEPTH 3
#endif
constexpr int kPlanSplitWaves = VOILA_PLAN_SPLIT_WAVES, kPlanSplitTiles = VOILA_PLAN_SPLIT_TILES,
              kPlanSplitDepth = VOILA_PLAN_SPLIT_DEPTH;

template <int DT, int WIDTH, int NHID>
constexpr bool plan_split() {
    return net_compiled(DT, WIDTH) && !generic_compiled(DT, WIDTH, NHID);
}

// LDS of the split rollout kernel beyond the activations: each owner wave's
// first-layer operands and states ([slot][lane]), then the goal.
template <class NT, int D_S, int ST>
struct PlanSplitLds {
    static constexpr int IN = ST * SplitIn<NT>::BYTES;
    static constexpr int STATE = ST * state_slots(D_S) * 64 * 4;
    static constexpr int BYTES = ST * SplitLds<NT>::ACT + IN + STATE + 64 * 4;
};

template <int DT, int D_S, int N_ACT, int D_A, int D_W, int WIDTH, int NHID, int ST>
__global__ __launch_bounds__(64 * kPlanSplitWaves) void plan_split_kernel(PlanParams p, uint32_t unit0, uint32_t n_units) {
    if constexpr (!plan_split<DT, WIDTH, NHID>()) {
        return;  // the other networks run in plan_kernel
    } else {
    constexpr int DEPTH = ST > 1 ? kPlanSplitDepth : kSingleTileDepth;
    constexpr int SS = state_slots(D_S), SA = action_slots(D_A), SW = noise_slots(D_W);
    // states wider than 32 come out of the network in two 32-row tiles: state
    // slot s is register s % 16 of output tile s / 16
    constexpr int NO = cdiv(D_S, 32);
    typedef Net<DT, WIDTH, NHID, in_slots(DT, D_S, D_A, D_W), WIDTH / 32, NO> NT;
    typedef PlanSplitLds<NT, D_S, ST> L;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    char* const in_lds = smem + ST * SplitLds<NT>::ACT;
    const int lane = threadIdx.x & 63, g = lane >> 5, col = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // wave q < ST owns sample tile q of every group: its states (kept in LDS
    // across the network, which needs every register), noise and return; the
    // other waves only evaluate the network
    const bool owner = wave < ST;
    float* const st_lds = reinterpret_cast<float*>(in_lds + L::IN) + (owner ? wave : 0) * SS * 64 + lane;
    float* const goal_lds = reinterpret_cast<float*>(in_lds + L::IN + L::STATE);
    if (threadIdx.x < 64) goal_lds[threadIdx.x] = p.goal[threadIdx.x];
    __syncthreads();
    auto goal_at = [&](int s) { return goal_lds[2 * s + g]; };
    // -|s - goal|^2 over this lane's state slots (both lane groups summed)
    auto reward = [&](const float (&x)[SS]) {
        float part = 0.0f;
#pragma unroll
        for (int s = 0; s < SS; ++s)
            if (2 * s + g < D_S) {
                const float e = x[s] - goal_at(s);
                part = __builtin_fmaf(e, e, part);
            }
        return -(part + __shfl_xor(part, 32));
    };
    const int n_groups = (p.n_tiles + ST - 1) / ST;
    const NetPtrs P = net_ptrs(p.net.base, p.net);
    // (up to 2^31 - 1 units: the one past a block's last may not fit an int; 64
    // bits took 1 % of the kernel)
    for (uint32_t u = unit0 + blockIdx.x; u < n_units; u += gridDim.x) {
        const int k = (int)(u / (uint32_t)n_groups);
        const int grp = (int)u - k * n_groups;
        const int tile = grp * ST + (owner ? wave : 0);
        const int i = tile * 32 + col;
        const bool valid = owner && i < p.N;
        if (owner) {
            float st[SS];
#pragma unroll
            for (int s = 0; s < SS; ++s) {
                const int f = 2 * s + g;
                st[s] = (valid && f < D_S) ? p.states[(size_t)i * D_S + f] : 0.0f;
            }
#pragma unroll
            for (int s = 0; s < SS; ++s) st_lds[s * 64] = st[s];
        }
        float G = 0.0f;
        double disc = 1.0;
        for (int t = 0; t < p.H; ++t) {
            float r_cur = 0.0f;
            if (owner) {
                float slots[NT::IN_SLOTS], st[SS];
#pragma unroll
                for (int s = 0; s < SS; ++s) st[s] = st_lds[s * 64];
#pragma unroll
                for (int s = 0; s < NT::IN_SLOTS; ++s) slots[s] = 0.0f;
#pragma unroll
                for (int s = 0; s < SS; ++s) slots[s] = st[s];
                if (D_A > 0) {
                    const kconst float* a = (const kconst float*)p.cands + ((size_t)k * p.H + t) * D_A;
#pragma unroll
                    for (int s = 0; s < SA; ++s) {
                        const float a0 = 2 * s < D_A ? a[2 * s] : 0.0f;
                        const float a1 = 2 * s + 1 < D_A ? a[2 * s + 1] : 0.0f;
                        slots[SS + s] = g ? a1 : a0;
                    }
                }
                if (p.noise) {
                    const float* nsrc = p.noise + (((size_t)k * p.N + (valid ? i : 0)) * p.H + t) * D_W;
#pragma unroll
                    for (int s = 0; s < SW; ++s) {
                        const int f = noise_feature(s, g);
                        slots[SS + SA + s] = f < D_W ? nsrc[f] : 0.0f;
                    }
                } else {
                    // this step's words only: nothing of the noise lives across the network
                    float nz[SW];
                    noise_slots_philox<SW>(nz, p.key0, p.key1, (uint32_t)i, p.crn ? 0u : (uint32_t)k, (uint32_t)t,
                                           3u, g);
#pragma unroll
                    for (int s = 0; s < SW; ++s) slots[SS + SA + s] = nz[s];
                }
                if (p.reward_at) r_cur = reward(st);
                split_stage_inputs<NT>(in_lds + wave * SplitIn<NT>::BYTES, slots, lane);
            }
            const float* b0 = P.b0;
            if (N_ACT > 0) {
                int a = ((const kconst int32_t*)p.cands)[(size_t)k * p.H + t];
                if (a < 0 || a >= N_ACT) {
                    if (p.status && wave == 0 && lane == 0) p.status[0] = 1;
                    a = 0;
                }
                b0 += (size_t)a * p.net.b0_stride;
            }
            float out[NO][16];
            run_net_split_owned<NT, ST, kPlanSplitWaves, DEPTH>(P, b0, in_lds, out, lane, g, wave, smem);
            if (owner) {
                float st[SS];
#pragma unroll
                for (int s = 0; s < SS; ++s) st[s] = st_lds[s * 64] + out[s / 16][s % 16];
#pragma unroll
                for (int s = 0; s < SS; ++s) st_lds[s * 64] = st[s];
                if (p.traj && valid) {
                    float* dst = p.traj + (((size_t)k * p.N + i) * p.H + t) * D_S;
#pragma unroll
                    for (int s = 0; s < SS; ++s)
                        if (2 * s + g < D_S) dst[2 * s + g] = st[s];
                }
                const float r = p.reward_at ? r_cur : reward(st);
                G = __builtin_fmaf((float)disc, r, G);
            }
            disc *= p.gamma;
        }
        if (owner) {
            if (p.returns && g == 0 && valid) p.returns[(size_t)k * p.N + i] = G;
            const float contrib = valid ? (p.belief_w ? (float)p.belief_w[i] * G : G) : 0.0f;
            const float tot = sum32(contrib);
            if (lane == 0 && tile < p.n_tiles) p.partials[(size_t)k * p.n_tiles + tile] = tot;
        }
    }
    }
}

// ---------------------------------------------------------------------------
// small plans: one half tile per block
// ---------------------------------------------------------------------------
// A plan of few tiles is the latency of its steps: in plan_kernel one wave runs
// a tile's 104 products of 64 cycles one after the other (32 candidates x 128
// particles: 128 waves on 32 CUs, 4.2 us per step).  Here a block advances 16
// particles of one candidate: each of its four waves produces 16 rows of a
// hidden layer (16x16 products over two packed k-steps each, its weights in
// registers for the whole rollout), every wave sums the four outputs of its
// particles itself (lane (n, g4) feature g4 of particle n, one chain over the
// hidden units, so nothing waits for a third barrier) and holds the states.
// Noise, actions and first-layer bias rows are prepared kHalfSteps steps at a
// time, one (particle, step) per thread.  All sums run in plan_kernel's order,
// so the returns are the same bits.  The block takes every second particle of a
// tile: the tile's sum adds the even and the odd particles' sums last, so a half
// tile's is one value and q_reduce_kernel adds the two (with the contributions
// left per particle for it, one candidate of 24,576 took 63 us at 5 steps, 27 in
// plan_kernel).
constexpr int kHalfSteps = 16;

template <int DT, int D_S, int D_A, int D_W, int WIDTH, int NHID>
constexpr bool plan_half() {
    return DT == DT_F32 && WIDTH == 64 && NHID == 2 && state_slots(D_S) == 2 && noise_slots(D_W) == 2 &&
           (D_A == 0 || action_slots(D_A) == 2);
}

template <int DT, int D_S, int N_ACT, int D_A, int D_W, int WIDTH, int NHID>
__global__ __launch_bounds__(256, 2) void plan_half_kernel(PlanParams p) {
    if constexpr (!plan_half<DT, D_S, D_A, D_W, WIDTH, NHID>()) {
        return;  // not chosen for the other networks
    } else {
    typedef Net<DT, WIDTH, NHID, in_slots(DT, D_S, D_A, D_W)> NT;
    typedef FragIdx<NT> FI;
    constexpr int IN_S = NT::IN_KS / 2, HID_S = NT::HID_KS / 2;  // k-step pairs
    __shared__ __attribute__((aligned(16))) float act[2][WIDTH * 16];  // [k / 16][k % 4][particle][k / 4 % 4]
    __shared__ float nz[kHalfSteps][64], av[kHalfSteps][4];
    __shared__ __attribute__((aligned(16))) float bias[kHalfSteps][WIDTH];
    const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, g4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), tile = wave >> 1, rows = 16 * (wave & 1);
    const NetPtrs P = net_ptrs(p.net.base, p.net);
    const float* const W = reinterpret_cast<const float*>(P.f0);
    const int f_lane = (g4 & 1) * 32 + rows + n, c_lane = g4 >> 1;
    float w0[IN_S], w1[HID_S], wo[WIDTH];
#pragma unroll
    for (int s = 0; s < IN_S; ++s) w0[s] = W[FI::first(2 * s + c_lane, tile) * 64 + f_lane];
#pragma unroll
    for (int s = 0; s < HID_S; ++s) w1[s] = W[FI::hidden(1, 2 * s + c_lane, tile) * 64 + f_lane];
#pragma unroll
    for (int q = 0; q < WIDTH; ++q) wo[q] = W[FI::out(q / 2) * 64 + q % 2 * 32 + out_row(g4 / 2, g4 % 2)];
    const f32x4 b1 = *reinterpret_cast<const f32x4*>(P.bh + 32 * tile + rows + 4 * g4);
    const float bo = P.bo[out_row(g4 / 2, g4 % 2)];
    const float goal = g4 < D_S ? p.goal[g4] : 0.0f;
    // -|s - goal|^2, features f and f + 2 first, then both pairs (reward_to's order)
    auto reward = [&](float x) {
        const float e = x - goal, o = __uint_as_float(swap_halves(__float_as_uint(e)));
        const float first = g4 < 2 ? e : o, second = g4 < 2 ? o : e;
        const float part = __builtin_fmaf(second, second, first * first);
        return -(part + __shfl_xor(part, 16));
    };
    auto store = [&](float* dst, const f32x4& a) {
        float* at = dst + ((wave * 4 + g4 % 2) * 16 + n) * 4 + 2 * (g4 / 2);
        *reinterpret_cast<f32x2*>(at) = (f32x2){relu_f32(a[0]), relu_f32(a[2])};
        *reinterpret_cast<f32x2*>(at + 128) = (f32x2){relu_f32(a[1]), relu_f32(a[3])};
    };
    const int n_half = 2 * p.n_tiles;
    const int u = blockIdx.x;
    const int k = u / n_half, i0 = (u - k * n_half) / 2 * 32 + (u & 1), i = i0 + 2 * n;
    const bool valid = i < p.N;
    float st = valid && g4 < D_S ? p.states[(size_t)i * D_S + g4] : 0.0f;
    float G = 0.0f;
    double disc = 1.0;
    for (int t0 = 0; t0 < p.H; t0 += kHalfSteps) {
        const int tn = min(kHalfSteps, p.H - t0);
        // every wave is past the second barrier of the previous step, after
        // which it reads none of these
        if (const int j = tid / 16, m = tid % 16, t = t0 + j; j < tn) {
            const int im = i0 + 2 * m;
            float z[4];
            if (p.noise) {
                const float* src = p.noise + (((size_t)k * p.N + (im < p.N ? im : 0)) * p.H + t) * D_W;
#pragma unroll
                for (int f = 0; f < 4; ++f) z[f] = f < D_W ? src[f] : 0.0f;
            } else {
                const uint4 w = philox4x32_10(make_uint4((uint32_t)im, p.crn ? 0u : (uint32_t)k, (uint32_t)t, 3u << 16),
                                              p.key0, p.key1);
                box_muller(w.x, w.y, z[0], z[1]);
                box_muller(w.z, w.w, z[2], z[3]);
            }
            // slot s of lane group g is feature 2 g + s, k = 2 s + g
#pragma unroll
            for (int f = 0; f < 4; ++f) nz[j][(2 * (f % 2) + f / 2) * 16 + m] = z[f];
            const float* b0 = P.b0;
            if (N_ACT > 0) {
                int a = reinterpret_cast<const int32_t*>(p.cands)[(size_t)k * p.H + t];
                if (a < 0 || a >= N_ACT) {
                    if (p.status && m == 0) p.status[0] = 1;
                    a = 0;
                }
                b0 += (size_t)a * p.net.b0_stride;
            }
            *reinterpret_cast<f32x4*>(&bias[j][4 * m]) = *reinterpret_cast<const f32x4*>(b0 + 4 * m);
            if (D_A > 0 && m < 4)
                av[j][m] = m < D_A ? reinterpret_cast<const float*>(p.cands)[((size_t)k * p.H + t) * D_A + m] : 0.0f;
        }
        __syncthreads();
        f32x4 acc;
        float z, a = 0.0f;
        auto inputs = [&](int j) {
            acc = *reinterpret_cast<const f32x4*>(&bias[j][32 * tile + rows + 4 * g4]);
            z = nz[j][lane];
            if (D_A > 0) a = av[j][g4];
        };
        inputs(0);
        for (int j = 0; j < tn; ++j) {
            float r = 0.0f;
            if (p.reward_at) r = reward(st);
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w0[0], st, acc, 0, 0, 0);
            if (D_A > 0) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w0[1], a, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w0[IN_S - 1], z, acc, 0, 0, 0);
            store(act[0], acc);
            __syncthreads();
            f32x4 h = b1;
#pragma unroll
            for (int q = 0; q < HID_S / 4; ++q) {
                const f32x4 b = *reinterpret_cast<const f32x4*>(&act[0][(q * 64 + lane) * 4]);
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    h = __builtin_amdgcn_mfma_f32_16x16x4f32(w1[4 * q + s], b[s], h, 0, 0, 0);
            }
            store(act[1], h);
            __syncthreads();
            if (j + 1 < tn) inputs(j + 1);
            float o = bo;
#pragma unroll
            for (int q = 0; q < WIDTH / 16; ++q) {
                f32x4 v[4];
#pragma unroll
                for (int g = 0; g < 4; ++g) v[g] = *reinterpret_cast<const f32x4*>(&act[1][((q * 4 + g) * 16 + n) * 4]);
#pragma unroll
                for (int s = 0; s < 16; ++s) o = __builtin_fmaf(wo[16 * q + s], v[s % 4][s / 4], o);
            }
            st += o;
            if (p.traj && valid && wave == 0 && g4 < D_S)
                p.traj[(((size_t)k * p.N + i) * p.H + t0 + j) * D_S + g4] = st;
            if (!p.reward_at) r = reward(st);
            G = __builtin_fmaf((float)disc, r, G);
            disc *= p.gamma;
        }
    }
    if (wave == 0) {
        if (p.returns && valid && g4 == 0) p.returns[(size_t)k * p.N + i] = G;
        float v = valid ? (p.belief_w ? (float)p.belief_w[i] * G : G) : 0.0f;
#pragma unroll
        for (int m = 8; m >= 1; m >>= 1) v += __shfl_xor(v, m);  // sum32's order without its last step
        if (lane == 0) p.partials[u] = v;
    }
    }
}

// Many planning instances of one network shape in one persistent launch.
// The work list holds block items (instance, first tile unit, number of
// units): a block takes items from a queue (atomic counter, list sorted by
// decreasing cost) or in a static stride, restages the instance's network in
// LDS when the instance changes, and runs one unit per wave.  At most 128
// registers per lane (four waves per SIMD): a small network's step
// alternates between matrix products and the vector work that feeds them
// (noise, ReLU, conversions), and the other waves fill each wave's gaps.
template <int DT, int D_S, int N_ACT, int D_A, int D_W, int WIDTH, int NHID>
__global__ __launch_bounds__(512, 4) void plan_batch_kernel(BatchPlanParams bp) {
    if constexpr (WIDTH > 64) {
        return;  // batches need networks that fit in LDS (the launcher refuses wider ones)
    } else {
    typedef Net<DT, WIDTH, NHID, in_slots(DT, D_S, D_A, D_W)> NT;
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
        const int4 it = bp.items[item];  // (instance, first unit, units, cost)
        PlanParams p = bp.insts[it.x];
        p.status = bp.status;
        if (it.x != loaded) {
            __syncthreads();
            stage_blob(smem, p.net.base, p.net.bytes);
            __syncthreads();
            loaded = it.x;
        }
        const NetPtrs P = net_ptrs(smem, p.net);
        DirectSrc<DT, 8 * NT::HT> src(P.f0);
        const long u = (long)it.y + wave;
        // the goal is read from the instance table (a lane-indexed read of the
        // copy above would place the whole copy in scratch memory)
        plan_unit<DT, D_S, N_ACT, D_A, D_W, WIDTH, NHID>(src, P, p, bp.insts[it.x].goal, u, wave < it.z, lane, g,
                                                         col);
    }
    }
}

__global__ __launch_bounds__(64) void reset_counter_kernel(int* counter) { if (threadIdx.x == 0) *counter = 0; }

template <bool HALVES>
__global__ __launch_bounds__(256) void q_reduce_kernel(QReduceParams p) {
    const int lane = threadIdx.x & 63;
    const int k = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (k >= p.K) return;
    float s = 0.0f;
    for (int j = lane; j < p.n_tiles; j += 64) {
        const size_t at = (size_t)k * p.n_tiles + j;
        s += HALVES ? p.partials[2 * at] + p.partials[2 * at + 1] : p.partials[at];
    }
    s += __shfl_xor(s, 32);
    s = sum32(s);
    if (lane == 0) p.q[k] = s * p.scale;
}

__global__ __launch_bounds__(256) void q_reduce_batch_kernel(const QReduceParams* qs) {
    const QReduceParams p = qs[blockIdx.y];
    const int lane = threadIdx.x & 63;
    const int k = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (k >= p.K) return;
    float s = 0.0f;
    for (int j = lane; j < p.n_tiles; j += 64) s += p.partials[(size_t)k * p.n_tiles + j];
    s += __shfl_xor(s, 32);
    s = sum32(s);
    if (lane == 0) p.q[k] = s * p.scale;
}

// launchers
#define PLAN_K(id, ds, na, da, dw, dox, dwz, w, nh, DT) plan_kernel<DT, ds, na, da, dw, w, nh, plan_mode<w>()>
// The bfloat16 instances of plan_kernel (built in k_plan_bf16.hip).
const void* plan_kernel_bf16(int shape);

size_t plan_stream_lds(int shape, int dt) {
    switch (shape * 2 + dt) {
#define X(id, ds, na, da, dw, dox, dwz, w, nh)                                      \
    case id * 2 + 0:                                                               \
        return stream_lds_of<DT_F32, ds, na, (na > 0 ? 0 : da), dw, w, nh, VOILA_PLAN_STREAM_CHB>(); \
    case id * 2 + 1:                                                               \
        return stream_lds_of<DT_BF16, ds, na, (na > 0 ? 0 : da), dw, w, nh, VOILA_PLAN_STREAM_CHB>();
        VOILA_SHAPES(X)
#undef X
    }
    return kStreamLds;
}

#define PLAN_SK(id, ds, na, da, dw, dox, dwz, w, nh, DT) plan_split_kernel<DT, ds, na, da, dw, w, nh, kPlanSplitTiles>
#define PLAN_S1(id, ds, na, da, dw, dox, dwz, w, nh, DT) plan_split_kernel<DT, ds, na, da, dw, w, nh, 1>

template <int DT, int D_S, int D_A, int D_W, int W, int NH, int ST = kPlanSplitTiles>
constexpr size_t plan_split_lds() {
    if constexpr (!plan_split<DT, W, NH>()) {
        return 0;
    } else {
        typedef Net<DT, W, NH, in_slots(DT, D_S, D_A, D_W), W / 32, cdiv(D_S, 32)> NT;
        return (size_t)PlanSplitLds<NT, D_S, ST>::BYTES;
    }
}

bool plan_split_shape(int shape, int dt) {
    switch (shape * 2 + dt) {
#define X(id, ds, na, da, dw, dox, dwz, w, nh) \
    case id * 2 + 0:                           \
        return plan_split<DT_F32, w, nh>();    \
    case id * 2 + 1:                           \
        return plan_split<DT_BF16, w, nh>();
        VOILA_SHAPES(X)
#undef X
    }
    return false;
}

template <class K>
void launch_plan_split_one(K k, size_t lds, long blocks, const PlanParams& p, long unit0, long n_units, hipStream_t s) {
    if (n_units <= unit0) return;
    if (lds > 65536) (void)hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    const long want = n_units - unit0;
    hipLaunchKernelGGL(k, (int)(want < blocks ? want : blocks), 64 * kPlanSplitWaves, lds, s, p, (uint32_t)unit0, (uint32_t)n_units);
}

// Rounds of tile groups over the chip's `cap` blocks, then the tiles of the
// remaining groups, singly if they are then one round.
template <class KS, class K1>
void launch_plan_split(KS ks, K1 k1, size_t lds, size_t lds1, long cap, int cus, const PlanParams& p, hipStream_t s) {
    constexpr int ST = kPlanSplitTiles;
    const long n_groups = (p.n_tiles + ST - 1) / ST, units = p.K * n_groups, tiles = (long)p.K * p.n_tiles;
    const long whole = units / cap * cap, tile0 = whole / n_groups * p.n_tiles + whole % n_groups * ST;
    const bool singly = tiles - tile0 <= cus;
    launch_plan_split_one(ks, lds, cap, p, 0, singly ? whole : units, s);
    if (singly) launch_plan_split_one(k1, lds1, cus, p, tile0, tiles, s);
}

hipError_t launch_plan(int shape, int dt, const PlanParams& p, int blocks, long cap, int cus, hipStream_t s) {
    if (plan_split_shape(shape, dt)) {
        switch (shape * 2 + dt) {
#define X(id, ds, na, da, dw, dox, dwz, w, nh)                                                                      \
    case id * 2 + 0:                                                                                               \
        launch_plan_split(PLAN_SK(id, ds, na, da, dw, dox, dwz, w, nh, DT_F32), PLAN_S1(id, ds, na, da, dw, dox, dwz, w, nh, DT_F32), \
                          plan_split_lds<DT_F32, ds, (na > 0 ? 0 : da), dw, w, nh>(),                             \
                          plan_split_lds<DT_F32, ds, (na > 0 ? 0 : da), dw, w, nh, 1>(), cap, cus, p, s);         \
        break;                                                                                                     \
    case id * 2 + 1:                                                                                               \
        launch_plan_split(PLAN_SK(id, ds, na, da, dw, dox, dwz, w, nh, DT_BF16), PLAN_S1(id, ds, na, da, dw, dox, dwz, w, nh, DT_BF16), \
                          plan_split_lds<DT_BF16, ds, (na > 0 ? 0 : da), dw, w, nh>(),                             \
                          plan_split_lds<DT_BF16, ds, (na > 0 ? 0 : da), dw, w, nh, 1>(), cap, cus, p, s);         \
        break;
            VOILA_SHAPES(X)
#undef X
            default:
                return hipErrorInvalidValue;
        }
        return hipGetLastError();
    }
    size_t lds = weights_in_lds(shape) ? p.net.bytes : plan_stream_lds(shape, dt) + (p.net.bytes - p.net.off_b0);
    switch (shape * 2 + dt) {
#define X(id, ds, na, da, dw, dox, dwz, w, nh)                                                              \
    case id * 2 + 0:                                                                                       \
        if (lds > 65536)                                                                                   \
            (void)hipFuncSetAttribute((const void*)PLAN_K(id, ds, na, da, dw, dox, dwz, w, nh, DT_F32),     \
                                      hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);               \
        hipLaunchKernelGGL((PLAN_K(id, ds, na, da, dw, dox, dwz, w, nh, DT_F32)), blocks, 256, lds, s, p);  \
        break;                                                                                             \
    case id * 2 + 1: {                                                                                     \
        const void* k = plan_kernel_bf16(id);                                                              \
        if (lds > 65536) (void)hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds); \
        void* args[] = {(void*)&p};                                                                        \
        (void)hipLaunchKernel(k, dim3(blocks), dim3(256), args, lds, s);                                   \
        break;                                                                                             \
    }
        VOILA_SHAPES(X)
#undef X
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

int plan_pass_tiles(int shape, int dt) {
    switch (shape * 2 + dt) {
#define X(id, ds, na, da, dw, dox, dwz, w, nh)              \
    case id * 2 + 0:                                       \
        return plan_pairs<DT_F32, w, nh>() ? kPlanPassTiles : 0; \
    case id * 2 + 1:                                       \
        return plan_pairs<DT_BF16, w, nh>() ? kPlanPassTiles : 0;
        VOILA_SHAPES(X)
#undef X
    }
    return 0;
}

int plan_tiles_per_unit(int shape, int dt) {
    return plan_split_shape(shape, dt) ? kPlanSplitTiles : plan_pass_tiles(shape, dt) ? 2 : 1;
}
int plan_units_per_block(int shape, int dt) { return plan_split_shape(shape, dt) ? 1 : kWavesPerBlock; }

int plan_blocks_per_cu(int shape, int dt) {
    if (plan_split_shape(shape, dt)) {
        switch (shape * 2 + dt) {
#define X(id, ds, na, da, dw, dox, dwz, w, nh)                                                                 \
    case id * 2 + 0:                                                                                          \
        return occupancy_t(PLAN_SK(id, ds, na, da, dw, dox, dwz, w, nh, DT_F32), 64 * kPlanSplitWaves,          \
                           plan_split_lds<DT_F32, ds, (na > 0 ? 0 : da), dw, w, nh>());                        \
    case id * 2 + 1:                                                                                          \
        return occupancy_t(PLAN_SK(id, ds, na, da, dw, dox, dwz, w, nh, DT_BF16), 64 * kPlanSplitWaves,         \
                           plan_split_lds<DT_BF16, ds, (na > 0 ? 0 : da), dw, w, nh>());
            VOILA_SHAPES(X)
#undef X
        }
        return 1;
    }
    switch (shape * 2 + dt) {
#define X(id, ds, na, da, dw, dox, dwz, w, nh)                                                               \
    case id * 2 + 0:                                                                                        \
        return occupancy(PLAN_K(id, ds, na, da, dw, dox, dwz, w, nh, DT_F32), lds_for_width<w>() ? kLdsGuess : kPlanStreamLds); \
    case id * 2 + 1:                                                                                        \
        return occupancy(plan_kernel_bf16(id), lds_for_width<w>() ? kLdsGuess : kPlanStreamLds);
        VOILA_SHAPES(X)
#undef X
    }
    return 1;
}

#define PLANB_K(id, ds, na, da, dw, dox, dwz, w, nh, DT) plan_batch_kernel<DT, ds, na, da, dw, w, nh>

hipError_t launch_plan_batch(int shape, int dt, const BatchPlanParams& p, int blocks, int wpb, size_t lds,
                             hipStream_t s) {
    if (!weights_in_lds(shape)) return hipErrorInvalidValue;
    switch (shape * 2 + dt) {
#define X(id, ds, na, da, dw, dox, dwz, w, nh)                                                                     \
    case id * 2 + 0:                                                                                              \
        hipLaunchKernelGGL((PLANB_K(id, ds, na, da, dw, dox, dwz, w, nh, DT_F32)), blocks, 64 * wpb, lds, s, p);   \
        break;                                                                                                    \
    case id * 2 + 1:                                                                                              \
        hipLaunchKernelGGL((PLANB_K(id, ds, na, da, dw, dox, dwz, w, nh, DT_BF16)), blocks, 64 * wpb, lds, s, p);  \
        break;
        VOILA_SHAPES(X)
#undef X
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

int plan_batch_blocks_per_cu(int shape, int dt, int wpb, size_t lds) {
    switch (shape * 2 + dt) {
#define X(id, ds, na, da, dw, dox, dwz, w, nh)                                                        \
    case id * 2 + 0:                                                                                 \
        return occupancy_t(PLANB_K(id, ds, na, da, dw, dox, dwz, w, nh, DT_F32), 64 * wpb, lds);      \
    case id * 2 + 1:                                                                                 \
        return occupancy_t(PLANB_K(id, ds, na, da, dw, dox, dwz, w, nh, DT_BF16), 64 * wpb, lds);
        VOILA_SHAPES(X)
#undef X
    }
    return 1;
}


hipError_t launch_q_reduce_batch(const QReduceParams* d_qs, int n_inst, int max_k, hipStream_t s) {
    if (n_inst == 0 || max_k == 0) return hipSuccess;
    hipLaunchKernelGGL(q_reduce_batch_kernel, dim3((max_k + 3) / 4, n_inst), 256, 0, s, d_qs);
    return hipGetLastError();
}

#define PLANH_K(id, ds, na, da, dw, dox, dwz, w, nh) plan_half_kernel<DT_F32, ds, na, da, dw, w, nh>

bool plan_half_shape(int shape, int dt) {
    if (dt != DT_F32) return false;
    switch (shape) {
#define X(id, ds, na, da, dw, dox, dwz, w, nh) \
    case id:                                   \
        return plan_half<DT_F32, ds, (na > 0 ? 0 : da), dw, w, nh>();
        VOILA_SHAPES(X)
#undef X
    }
    return false;
}

hipError_t launch_plan_half(int shape, const PlanParams& p, const QReduceParams& q, hipStream_t s) {
    const int blocks = 2 * p.K * p.n_tiles;
    if (!plan_half_shape(shape, DT_F32)) return hipErrorInvalidValue;
    switch (shape) {
#define X(id, ds, na, da, dw, dox, dwz, w, nh)                                                                \
    case id:                                                                                                 \
        hipLaunchKernelGGL((PLANH_K(id, ds, na, (na > 0 ? 0 : da), dw, dox, dwz, w, nh)), blocks, 256, 0, s, p); \
        break;
        VOILA_SHAPES(X)
#undef X
        default:
            return hipErrorInvalidValue;
    }
    if (const hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    hipLaunchKernelGGL(q_reduce_kernel<true>, (p.K + 3) / 4, 256, 0, s, q);
    return hipGetLastError();
}

hipError_t launch_reset_counter(int* d_counter, hipStream_t s) {
    hipLaunchKernelGGL(reset_counter_kernel, 1, 64, 0, s, d_counter);
    return hipGetLastError();
}

hipError_t launch_q_reduce(const QReduceParams& p, hipStream_t s) {
    const int blocks = (p.K + 3) / 4;
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(q_reduce_kernel<false>, blocks, 256, 0, s, p);
    return hipGetLastError();
}

}  // namespace voila
