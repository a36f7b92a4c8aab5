// grad.hip -- adjoint (reverse-mode) rollout kernel with step checkpointing.
//
// Differentiates free-running rollouts s_{t+1} = s_t + f_T([s_t, a_t, w_t]) of
// a transition network with two hidden layers of width 64 (binary32):
//   distillation objective  L = 1/(B H) sum_b sum_{t=1..H} ||s_{b,t} - T_{b,t}||^2
//   (the distillation loss of Eq. 3 along rollouts, T = teacher states), and
//   return objective        J = 1/B sum_b sum_{t<H} gamma^t (-||s_{b,t+1} - g||^2),
// giving d/d(network parameters) and, for continuous actions, d/dA.
//
// One wave owns a tile of 32 rollouts.  The forward pass keeps the states in
// registers and writes every step's to the workspace (16 bytes per rollout and
// step, in the lanes' own layout), or every C-th where the workspace is smaller;
// the reverse sweep reads them back, last step first (a segment of C steps runs
// again from its first state), recomputes the step's hidden activations, and back-propagates the
// state adjoint through the layers with MFMAs whose A operands are the
// *transposed* weights packed so that every adjoint comes out in exactly the
// register layout of the matching forward activation (ReLU masks are
// register-wise).  Weight gradients dW += dh h^T are products over the 32
// rollouts of the tile: the wave writes (dh, h) as [rollout][feature] rows into
// its own LDS scratch (row stride 97 floats) and accumulates them on MFMA with
// rollouts as the reduction dimension.  A block's waves add their partial
// gradients in wave order, each block writes one partial, and a second kernel
// sums the blocks' in a fixed order (deterministic).
#include "kernels.hpp"

#include <math.h>

namespace voila {

namespace {

constexpr int kRow = 129;    // floats per pair row of the contrastive kernel's transpose scratch
constexpr int kRowR = 97;    // floats per rollout row of the rollout kernel's (two rows of waves per SIMD fit in LDS)

// Fragment indices of the transposed pack: [T3: KS3 x HT][T2: 16HT x HT][T1: 16HT x 1]
template <int D_S, int HT> struct BwdIdx {
    static constexpr int KS3 = cdiv(D_S, 2);
    __device__ static constexpr int t3(int c, int mt) { return c * HT + mt; }
    __device__ static constexpr int t2(int c, int mt) { return KS3 * HT + c * HT + mt; }
    __device__ static constexpr int t1(int c) { return KS3 * HT + 16 * HT * HT + c; }
};

__device__ __forceinline__ float lds_frag(const char* base, int f, int lane) {
    return reinterpret_cast<const float*>(base)[f * 64 + lane];
}

}  // namespace

// Products whose result has four rows: v_mfma_f32_4x4x1 takes one k per
// instruction and lane group for all 64 lanes in 8 cycles, where a 32-row tile
// would compute 28 rows of padding in 64.
__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma16(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
// Fragment row of value m (of four, from feature f0 on) in a 32-row output
// tile: feature f sits at row out_row(f / 2, f % 2).
__device__ __forceinline__ int row_of(int f) { return out_row(f >> 1, f & 1); }
// The two lane groups hold partial sums over their own k of the same four
// values: lanes of group g get value 2 s + g in out[s].
__device__ __forceinline__ void join_halves(const f32x4& d, float (&out)[2]) {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(d[2 * s]), __float_as_uint(d[2 * s + 1]), false,
                                                        false);
        out[s] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
}

// Adjoint of a tile per wave.  Bound by the matrix cores: per tile and step
// 78 32x32x2 products to run the hidden layers, twice (forward, and again in
// the reverse sweep: reading the activations back would cost 16 KB per tile and
// step), 64 each for dW2 and dh1, and the equivalent of 40 for the rest.
// The layers with four outputs (the network's own output, dW3, the state and
// action adjoints) take 4-row products and dW1 (at most 16 columns) 16 x 16
// ones; with 32-row tiles, and with the states recomputed from checkpoints
// every five steps, the same step took 526.  Two waves per SIMD (256 registers
// each, 124 bytes per lane spilled: 105 MB written per launch of which the states are
// 21) overlap one's LDS transposes with the other's products.  65,536
// rollouts x 20 steps: the whole call 855 -> 557 us (about 340 us at the
// matrix cores' rate, which are 53 % busy).
// SEG: the workspace holds every p.C-th state only.  The reverse sweep then runs
// each segment of p.C steps forward again from its first state into the wave's
// own segment buffer (the same products, so the same states).
template <int D_S, int N_ACT, int D_A, int D_W, bool SEG>
__global__ __launch_bounds__(kGradMaxWaves * 64) void grad_kernel(GradParams p) {
    constexpr int WIDTH = 64, NHID = 2, HT = 2;
    constexpr int D_AIN = N_ACT > 0 ? N_ACT : D_A;
    constexpr int SS = state_slots(D_S), SA = action_slots(D_AIN), SW = noise_slots(D_W);
    constexpr int D_IN = D_S + D_AIN + D_W;
    static_assert(D_S == 4, "output and state adjoint are one four-row product");
    static_assert(D_IN <= 15, "inputs must fit one 16-column tile (column 15 carries the bias)");
    static_assert(N_ACT > 0 || D_A == 4, "action adjoints are one four-row product");
    typedef Net<DT_F32, WIDTH, NHID, in_slots(DT_F32, D_S, D_AIN, D_W)> NT;
    typedef BwdIdx<D_S, HT> BI;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    stage_blob(smem, p.fwd.base, p.fwd.bytes);
    stage_blob(smem + p.fwd.bytes, p.bwd.base, p.bwd.bytes);
    __syncthreads();
    const NetPtrs P = net_ptrs(smem, p.fwd);
    const char* bw = smem + p.fwd.bytes;
    const int lane = threadIdx.x & 63, g = lane >> 5, col = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wpb = p.waves;  // waves that take tiles (the others only stage)
    float* scr = reinterpret_cast<float*>(smem + p.fwd.bytes + p.bwd.bytes) + wave * 32 * kRowR;

    // weight-gradient accumulators (MFMA layouts) and per-lane bias sums
    f32x4 gW1[4], gW3[2];
    f32x16 gW2[HT][HT], gb2[HT];
#pragma unroll
    for (int a = 0; a < 4; ++a) gW1[a] = f32x4{};
#pragma unroll
    for (int a = 0; a < HT; ++a) {
        gW3[a] = f32x4{};
        gb2[a] = f32x16{};
#pragma unroll
        for (int b = 0; b < HT; ++b) gW2[a][b] = f32x16{};
    }
    float gb3[SS];
#pragma unroll
    for (int s = 0; s < SS; ++s) gb3[s] = 0.0f;
    float loss_acc = 0.0f;

    // input slots of step t for rollout b from state slots st
    auto make_slots = [&](float (&slots)[NT::IN_SLOTS], const float* st, int b, bool valid, int t) {
#pragma unroll
        for (int s = 0; s < NT::IN_SLOTS; ++s) slots[s] = 0.0f;
#pragma unroll
        for (int s = 0; s < SS; ++s) slots[s] = st[s];
        if (N_ACT > 0) {
            const int a = valid ? reinterpret_cast<const int32_t*>(p.actions)[(size_t)b * p.H + t] : -1;
#pragma unroll
            for (int s = 0; s < SA; ++s) slots[SS + s] = (2 * s + g == a) ? 1.0f : 0.0f;
        } else {
            const float* av =
                reinterpret_cast<const float*>(p.actions) + ((size_t)(valid ? b / p.particles : 0) * p.H + t) * D_A;
#pragma unroll
            for (int s = 0; s < SA; ++s) {
                int f = 2 * s + g;
                slots[SS + s] = f < D_A ? av[f] : 0.0f;
            }
        }
        if (p.noise) {
            const float* nz = p.noise + ((size_t)(valid ? b : 0) * p.H + t) * D_W;
#pragma unroll
            for (int s = 0; s < SW; ++s) {
                int f = noise_feature(s, g);
                slots[SS + SA + s] = f < D_W ? nz[f] : 0.0f;
            }
        } else {
            float nz[SW];
            noise_slots_philox<SW>(nz, p.key0, p.key1, (uint32_t)b, 0u, (uint32_t)t, 3u, g);
#pragma unroll
            for (int s = 0; s < SW; ++s) slots[SS + SA + s] = nz[s];
        }
    };
    // input column of slot s of this lane group (-1: padding)
    auto slot_col = [&](int s) -> int {
        if (s < SS) return 2 * s + g < D_S ? 2 * s + g : -1;
        if (s < SS + SA) return 2 * (s - SS) + g < D_AIN ? D_S + 2 * (s - SS) + g : -1;
        if (s < SS + SA + SW) {
            int f = noise_feature(s - SS - SA, g);
            return f < D_W ? D_S + D_AIN + f : -1;
        }
        return -1;
    };
    // the two hidden layers' activations
    auto hidden = [&](const float (&slots)[NT::IN_SLOTS], Act<DT_F32, HT>& h1, Act<DT_F32, HT>& h2) {
        DirectSrc<DT_F32, 8 * HT> src(P.f0);
        f32x16 acc[HT];
        init_bias<HT>(acc, P.b0 + opaque_zero(), g);
#pragma unroll
        for (int c = 0; c < NT::IN_KS; ++c)
#pragma unroll
            for (int mt = 0; mt < HT; ++mt)
                acc[mt] = mfma(src.load(FragIdx<NT>::first(c, mt), lane), slots[c], acc[mt]);
        h1.set_relu(acc);
        init_bias<HT>(acc, P.bh + opaque_zero(), g);
#pragma unroll
        for (int c = 0; c < NT::HID_KS; ++c)
#pragma unroll
            for (int mt = 0; mt < HT; ++mt)
                acc[mt] = mfma(src.load(FragIdx<NT>::hidden(1, c, mt), lane), h1.b(c), acc[mt]);
        h2.set_relu(acc);
    };
    // four values sum_k w[m][k] h[k] of the lane's column (m = 0..3): `frag0`
    // holds the 32-row fragments of k-steps 0 .. 31, whose rows of the four
    // features from f0 on are the A operand of every block of four lanes
    auto four = [&](const char* frag0, int f0, const f32x16 (&h)[HT]) {
        const float* a = reinterpret_cast<const float*>(frag0) + 32 * g + row_of(f0 + (lane & 3)) + opaque_zero();
        f32x4 d[2] = {f32x4{}, f32x4{}};
#pragma unroll
        for (int c = 0; c < 16 * HT; ++c) d[c & 1] = mfma4(a[c * 64], h[c >> 4][c & 15], d[c & 1]);
        return d[0] + d[1];
    };

    // the network's output: the same four values in every lane, summed over k in
    // ascending order from the bias as a 32-row tile sums them (the matrix
    // cores add one k at a time, whatever the shape), so that the rollouts are
    // the plan kernel's bit for bit
    auto output = [&](const f32x16 (&h)[HT]) {
        const int row = row_of(lane & 3);
        const float* a = reinterpret_cast<const float*>(P.fo) + row + opaque_zero();
        f32x4 d;
#pragma unroll
        for (int m = 0; m < 4; ++m) d[m] = P.bo[row_of(m)];
#pragma unroll
        for (int c = 0; c < 16 * HT; ++c) {
            const uint32_t v = __float_as_uint(h[c >> 4][c & 15]);
            const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);  // both groups' k
            d = mfma4(a[c * 64], __uint_as_float(r[0]), d);
            d = mfma4(a[c * 64 + 32], __uint_as_float(r[1]), d);
        }
        return d;
    };

    const int n_tiles = (p.B + 31) / 32;
    const int first_tile = (int)blockIdx.x * wpb + wave;
    for (long tl = wave < wpb ? first_tile : n_tiles; tl < n_tiles; tl += (long)gridDim.x * wpb) {
        const int tile = (int)tl;
        const int b = tile * 32 + col;
        const bool valid = b < p.B;
        // s_t slots of this lane, t < H; or rollouts' states (features 2 s + g of
        // this lane's) at every C-th step and, of one segment, at the steps between
        float* keep = p.states + (size_t)tile * p.H * (SS * 64) + lane;
        const int cols = 4 * min(32, p.B - 32 * tile);  // floats of one step
        float* ckpt = p.states + (size_t)128 * tile * p.NC + 4 * col + g;
        float* between = p.seg + (size_t)128 * first_tile * (p.C - 1) + 4 * col + g;
        auto put_state = [&](float* at, const float (&st)[SS]) {
            if (valid)
#pragma unroll
                for (int s = 0; s < SS; ++s) at[2 * s] = st[s];
        };
        auto get_state = [&](const float* at, float (&st)[SS]) {
#pragma unroll
            for (int s = 0; s < SS; ++s) st[s] = valid ? at[2 * s] : 0.0f;
        };
        float st[SS];
#pragma unroll
        for (int s = 0; s < SS; ++s) {
            int f = 2 * s + g;
            st[s] = (valid && f < D_S) ? p.s0[(size_t)b * D_S + f] : 0.0f;
        }
        // ---- forward (rollouts past B stay at the origin: finite, no weight in any sum)
        for (int t = 0; t < p.H; ++t) {
            if constexpr (SEG) {
                if (t % p.C == 0) put_state(ckpt + (size_t)(t / p.C) * cols, st);
            } else {
#pragma unroll
                for (int s = 0; s < SS; ++s) keep[(size_t)(t * SS + s) * 64] = st[s];
            }
            float slots[NT::IN_SLOTS];
            make_slots(slots, st, b, valid, t);
            Act<DT_F32, HT> h1, h2;
            hidden(slots, h1, h2);
            const f32x4 d = output(h2.v);
            float part = 0.0f;
#pragma unroll
            for (int s = 0; s < SS; ++s) {
                int f = 2 * s + g;
                if (f < D_S && valid) {
                    st[s] += g ? d[2 * s + 1] : d[2 * s];
                    float e = p.objective == 0 ? st[s] - p.targets[((size_t)b * p.H + t) * D_S + f] : st[s] - p.goal[f];
                    part += e * e;
                }
            }
            loss_acc += p.objective == 0 ? part : -p.disc[t] * part;
        }
        // ---- reverse sweep
        float lam[SS];
#pragma unroll
        for (int s = 0; s < SS; ++s) lam[s] = 0.0f;
        for (int t = p.H - 1; t >= 0; --t) {
            // objective gradient at s_{t+1}
#pragma unroll
            for (int s = 0; s < SS; ++s) {
                int f = 2 * s + g;
                if (f < D_S && valid) {
                    float e = p.objective == 0 ? st[s] - p.targets[((size_t)b * p.H + t) * D_S + f] : st[s] - p.goal[f];
                    lam[s] += (p.objective == 0 ? 2.0f * (float)p.scale : -2.0f * p.disc[t] * (float)p.scale) * e;
                }
            }
            if constexpr (SEG) {
                const int r = t % p.C, t0 = t - r;
                if (r == 0 || r == p.C - 1 || t == p.H - 1) get_state(ckpt + (size_t)(t0 / p.C) * cols, st);
                else get_state(between + (size_t)(r - 1) * cols, st);
                if (r == p.C - 1 || t == p.H - 1)
                    for (int q = 0; q < r; ++q) {
                        float in[NT::IN_SLOTS];
                        make_slots(in, st, b, valid, t0 + q);
                        Act<DT_F32, HT> a1, a2;
                        hidden(in, a1, a2);
                        const f32x4 d = output(a2.v);
#pragma unroll
                        for (int s = 0; s < SS; ++s)
                            if (2 * s + g < D_S && valid) st[s] += g ? d[2 * s + 1] : d[2 * s];
                        put_state(between + (size_t)q * cols, st);
                    }
            } else {
#pragma unroll
                for (int s = 0; s < SS; ++s) st[s] = keep[(size_t)(t * SS + s) * 64];
            }
            // the activations of step t again
            float slots[NT::IN_SLOTS];
            make_slots(slots, st, b, valid, t);
            Act<DT_F32, HT> h1, h2;
            hidden(slots, h1, h2);
            const bool wp = p.want_params != 0;
            // (1) dW3 += lam h2^T: rows lam (0..3), h2 (4..67)
            if (wp) {
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int s = 0; s < SS; ++s) scr[col * kRowR + 2 * s + g] = lam[s];
#pragma unroll
                for (int mt = 0; mt < HT; ++mt)
#pragma unroll
                    for (int i = 0; i < 16; ++i) scr[col * kRowR + 4 + 32 * mt + out_row(i, g)] = h2.v[mt][i];
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int r = 0; r < 32; ++r)
                    gW3[r & 1] = mfma4(scr[r * kRowR + (lane & 3)], scr[r * kRowR + 4 + lane], gW3[r & 1]);
#pragma unroll
                for (int s = 0; s < SS; ++s) gb3[s] += lam[s];
            }
            // (2) dh2 = (W3^T lam) * [h2 > 0]
            f32x16 dh2[HT];
#pragma unroll
            for (int mt = 0; mt < HT; ++mt) {
                const char* bwz = bw + opaque_zero();
                dh2[mt] = f32x16{};
#pragma unroll
                for (int c = 0; c < BI::KS3; ++c) dh2[mt] = mfma(lds_frag(bwz, BI::t3(c, mt), lane), lam[c], dh2[mt]);
#pragma unroll
                for (int i = 0; i < 16; ++i) dh2[mt][i] = h2.v[mt][i] > 0.0f ? dh2[mt][i] : 0.0f;
            }
            // (3) dW2 += dh2 h1^T, one 32-row tile of dh2 (0..31) at a time beside h1 (32..95); b2 += dh2
            if (wp) {
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int mt = 0; mt < HT; ++mt)
#pragma unroll
                    for (int i = 0; i < 16; ++i) scr[col * kRowR + 32 + 32 * mt + out_row(i, g)] = h1.v[mt][i];
#pragma unroll
                for (int mt = 0; mt < HT; ++mt) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) scr[col * kRowR + out_row(i, g)] = dh2[mt][i];
                    __builtin_amdgcn_wave_barrier();
#pragma unroll
                    for (int c = 0; c < 16; ++c) {
                        const float* r = scr + (2 * c + g) * kRowR + col;
                        const float ax = r[0];
#pragma unroll
                        for (int nt = 0; nt < HT; ++nt) gW2[mt][nt] = mfma(ax, r[32 + 32 * nt], gW2[mt][nt]);
                    }
                    __builtin_amdgcn_wave_barrier();
                    gb2[mt] += dh2[mt];
                }
            }
            // (4) dh1 = (W2^T dh2) * [h1 > 0]
            f32x16 dh1[HT];
#pragma unroll
            for (int mt = 0; mt < HT; ++mt) dh1[mt] = f32x16{};
#pragma unroll
            for (int c0 = 0; c0 < 16 * HT; c0 += 8) {
                const char* bwz = bw + opaque_zero();
#pragma unroll
                for (int c = c0; c < c0 + 8; ++c)
#pragma unroll
                    for (int mt = 0; mt < HT; ++mt)
                        dh1[mt] = mfma(lds_frag(bwz, BI::t2(c, mt), lane), dh2[c >> 4][c & 15], dh1[mt]);
            }
#pragma unroll
            for (int mt = 0; mt < HT; ++mt)
#pragma unroll
                for (int i = 0; i < 16; ++i) dh1[mt][i] = h1.v[mt][i] > 0.0f ? dh1[mt][i] : 0.0f;
            // (5) dW1 (+ b1 through the ones column 15) += dh1 x^T: rows dh1 (0..63), x (64..79)
            if (wp) {
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int mt = 0; mt < HT; ++mt)
#pragma unroll
                    for (int i = 0; i < 16; ++i) scr[col * kRowR + 32 * mt + out_row(i, g)] = dh1[mt][i];
                if (g)
#pragma unroll
                    for (int j = D_IN; j < 16; ++j) scr[col * kRowR + 64 + j] = j == 15 ? 1.0f : 0.0f;
#pragma unroll
                for (int s = 0; s < NT::IN_SLOTS; ++s) {
                    int cc = slot_col(s);
                    if (cc >= 0) scr[col * kRowR + 64 + cc] = slots[s];
                }
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    const float* r = scr + (4 * c + (lane >> 4)) * kRowR + (lane & 15);
                    const float bx = r[64];
#pragma unroll
                    for (int mt = 0; mt < 4; ++mt) gW1[mt] = mfma16(r[16 * mt], bx, gW1[mt]);
                }
                __builtin_amdgcn_wave_barrier();
            }
            // (6) dx = W1^T dh1: the state adjoint, and with continuous actions the action's
            const char* t1 = bw + (size_t)BI::t1(0) * 256;
            // action gradient of this step (continuous actions), summed over the tile
            if (N_ACT == 0 && p.apart) {
                const f32x4 da = four(t1, D_S, dh1);
#pragma unroll
                for (int j = 0; j < D_AIN; ++j) {
                    float v = valid ? da[j] : 0.0f;
                    v = sum32(v);
                    v += __shfl_xor(v, 32);
                    if (lane == 0) p.apart[((size_t)tile * p.H + t) * D_AIN + j] = v;
                }
            }
            // state adjoint: lam_t = lam_{t+1} + d(f_T)/ds_t^T lam_{t+1}
            float dx[SS];
            join_halves(four(t1, 0, dh1), dx);
#pragma unroll
            for (int s = 0; s < SS; ++s)
                if (2 * s + g < D_S) lam[s] += dx[s];
        }
    }
    // ---- the wave's objective (the waves are added up in binary64 later)
    float lsum = sum32(loss_acc);
    lsum += __shfl_xor(lsum, 32);
    if (lane == 0 && wave < wpb) p.lpart[(size_t)blockIdx.x * wpb + wave] = lsum;
    if (!p.want_params) return;
    // ---- the block's partial gradient: its waves' in wave order, gathered in LDS
    // layout: W1 [64][D_IN], b1 [64], W2 [64][64], b2 [64], W3 [D_S][64], b3 [D_S]
    float* sum = reinterpret_cast<float*>(smem);
    constexpr int oW1 = 0, ob1 = 64 * D_IN, oW2 = ob1 + 64, ob2 = oW2 + 64 * 64, oW3 = ob2 + 64, ob3 = oW3 + D_S * 64;
    for (int k = 0; k < wpb; ++k) {
        __syncthreads();
        if (wave != k) continue;
        auto put = [&](int at, float v) { sum[at] = k ? sum[at] + v : v; };
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int m = 16 * mt + 4 * (lane >> 4) + i, n = lane & 15;
                if (n < D_IN) put(oW1 + m * D_IN + n, gW1[mt][i]);
                if (n == 15) put(ob1 + m, gW1[mt][i]);
            }
#pragma unroll
        for (int mt = 0; mt < HT; ++mt)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int m = 32 * mt + out_row(i, g);
#pragma unroll
                for (int nt = 0; nt < HT; ++nt) put(oW2 + m * 64 + 32 * nt + col, gW2[mt][nt][i]);
                const float v = sum32(gb2[mt][i]);
                if (col == 0) put(ob2 + m, v);
            }
#pragma unroll
        for (int m = 0; m < D_S; ++m) put(oW3 + m * 64 + lane, gW3[0][m] + gW3[1][m]);
#pragma unroll
        for (int s = 0; s < SS; ++s) {
            const float v = sum32(gb3[s]);
            if (col == 0 && 2 * s + g < D_S) put(ob3 + 2 * s + g, v);
        }
    }
    __syncthreads();
    float* out = p.wpart + (size_t)blockIdx.x * p.n_params;
    for (int q = threadIdx.x; q < p.n_params; q += blockDim.x) out[q] = sum[q];
}

// Fixed-order sums of the partials: parameters, objective, actions.
// The partials are read once and nothing else is done, so the kernel is bound
// by the loads in flight: a block takes 64 consecutive parameters (one 256-byte
// segment of each row) with 16 waves, wave w summing rows w, w + 16, ... in
// four accumulators, and wave 0 adds the 16 wave sums in wave order.  (One
// thread per parameter walking every row took 286 us for 1,024 rows of 5,316
// parameters: the distillation gradient of 65,536 x 20 steps 1,154 -> 855 us,
// the contrastive one of B = 1,000, 256 rows of 145,409, 10.95 -> 10.84 ms.)
constexpr int kRedCols = 64, kRedWaves = 16;
__global__ __launch_bounds__(kRedCols * kRedWaves) void grad_reduce_kernel(GradReduceParams p, int param_blocks) {
    __shared__ double part[kRedWaves][kRedCols];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if ((int)blockIdx.x < param_blocks) {
        const int q = blockIdx.x * kRedCols + lane;
        const bool ok = q < p.n_params;
        const float* col = p.wpart + (ok ? q : 0);
        float s[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        int w = wave;
        for (; w + 3 * kRedWaves < p.n_rows; w += 4 * kRedWaves)
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] += col[(size_t)(w + e * kRedWaves) * p.n_params];
        for (; w < p.n_rows; w += kRedWaves) s[0] += col[(size_t)w * p.n_params];
        float(*fp)[kRedCols] = reinterpret_cast<float(*)[kRedCols]>(part);
        fp[wave][lane] = (s[0] + s[1]) + (s[2] + s[3]);
        __syncthreads();
        if (wave == 0 && ok) {
            float t = 0.0f;
#pragma unroll
            for (int k = 0; k < kRedWaves; ++k) t += fp[k][lane];
            p.grad_params[q] = t;
        }
        return;
    }
    // the blocks after the parameters': action gradients, one value per thread
    const int q = ((int)blockIdx.x - param_blocks) * (kRedCols * kRedWaves) + (int)threadIdx.x;
    if (p.grad_actions && q < p.n_action_values) {
        // q = (sequence k, step t, component j); tiles of sequence k are consecutive
        const int per_step = p.H * p.d_a;
        const int k = q / per_step, rem = q % per_step;
        float s = 0.0f;
        for (int tl = 0; tl < p.tiles_per_seq; ++tl)
            s += p.apart[(size_t)(k * p.tiles_per_seq + tl) * per_step + rem];
        p.grad_actions[q] = s;
    }
    if (p.loss && (int)blockIdx.x == param_blocks) {
        double s = 0.0;
        for (int w = threadIdx.x; w < p.n_loss; w += kRedCols * kRedWaves) s += (double)p.lpart[w];
        part[wave][lane] = s;
        __syncthreads();
        if (wave == 0) {
            s = 0.0;
#pragma unroll
            for (int k = 0; k < kRedWaves; ++k) s += part[k][lane];
#pragma unroll
            for (int m = 1; m < 64; m <<= 1) s += __shfl_xor(s, m);
            if (lane == 0) p.loss[0] = (float)(s * p.scale);
        }
    }
}

// Parameter derivative of the contrastive objective (Eq. 6): for every pair
// (i, j) the likelihood network is re-run on [s'_i, a_i, o_j] (row i's state
// and action folded into its first-layer bias row, the observation in the
// input slots) and its parameters' derivative is accumulated with weight
// G_ij = d loss / d l_ij.  One wave owns a (row i, 32 observations) tile; the
// output layer is a dot product, so its adjoint is w3 * G_ij on the active
// units; the hidden adjoints use the transposed pack; the weight gradients
// are products over the tile's 32 pairs through the wave's LDS scratch, the
// first layer's over the full input [s'_i, a_i, o_j, 1] (column 31 carries
// the bias).  Each wave writes its partial once; grad_reduce_kernel sums them
// in a fixed order.
template <int D_S, int N_ACT, int D_A, int D_O>
__global__ __launch_bounds__(256) void nce_grad_kernel(NceGradParams p) {
    constexpr int WIDTH = 64, NHID = 2, HT = 2;
    constexpr int D_AIN = N_ACT > 0 ? N_ACT : D_A;
    constexpr int D_IN = D_S + D_AIN + D_O;
    static_assert(D_IN <= 31, "inputs must fit one 32-row tile (column 31 carries the bias)");
    typedef Net<DT_F32, WIDTH, NHID, in_slots(DT_F32, D_O, 0, 0)> NT;
    typedef BwdIdx<1, HT> BI;
    constexpr int SO = state_slots(D_O);
    extern __shared__ __attribute__((aligned(16))) char smem[];
    stage_blob(smem, p.fwd.base, p.fwd.bytes);
    stage_blob(smem + p.fwd.bytes, p.bwd.base, p.bwd.bytes);
    __syncthreads();
    const NetPtrs P = net_ptrs(smem, p.fwd);
    const char* bw = smem + p.fwd.bytes;
    const int lane = threadIdx.x & 63, g = lane >> 5, col = lane & 31;
    const int wpb = blockDim.x >> 6, wave = threadIdx.x >> 6;
    float* scr = reinterpret_cast<float*>(smem + p.fwd.bytes + p.bwd.bytes) + wave * 32 * kRow;

    f32x16 gW1[HT], gW2[HT][HT], gb2[HT], gw3[HT];
#pragma unroll
    for (int a = 0; a < HT; ++a) {
        gW1[a] = f32x16{};
        gb2[a] = f32x16{};
        gw3[a] = f32x16{};
#pragma unroll
        for (int b = 0; b < HT; ++b) gW2[a][b] = f32x16{};
    }
    float gb3 = 0.0f;

    const int B = p.B, jtiles = (B + 31) / 32;
    const long n_units = (long)B * jtiles;
    for (long u = (long)blockIdx.x * wpb + wave; u < n_units; u += (long)gridDim.x * wpb) {
        const int i = (int)(u / jtiles);
        const int j = (int)(u - (long)i * jtiles) * 32 + col;
        const bool valid = j < B;
        float slots[NT::IN_SLOTS];
#pragma unroll
        for (int s = 0; s < NT::IN_SLOTS; ++s) slots[s] = 0.0f;
#pragma unroll
        for (int s = 0; s < SO; ++s) {
            const int f = 2 * s + g;
            slots[s] = (valid && f < D_O) ? p.obs[(size_t)j * D_O + f] : 0.0f;
        }
        // forward: the two hidden layers' activations of the tile
        f32x16 acc[HT];
        Act<DT_F32, HT> h1, h2;
        {
            DirectSrc<DT_F32, 8 * HT> src(P.f0);
            init_bias<HT>(acc, p.b0 + (size_t)i * WIDTH, g);
#pragma unroll
            for (int c = 0; c < NT::IN_KS; ++c)
#pragma unroll
                for (int mt = 0; mt < HT; ++mt)
                    acc[mt] = mfma(src.load(FragIdx<NT>::first(c, mt), lane), slots[c], acc[mt]);
            h1.set_relu(acc);
            init_bias<HT>(acc, P.bh + opaque_zero(), g);
#pragma unroll
            for (int c = 0; c < NT::HID_KS; ++c)
#pragma unroll
                for (int mt = 0; mt < HT; ++mt)
                    acc[mt] = mfma(src.load(FragIdx<NT>::hidden(1, c, mt), lane), h1.b(c), acc[mt]);
            h2.set_relu(acc);
        }
        const float gc = valid ? p.grad[(size_t)i * B + j] : 0.0f;
        // output layer: dw3 += G h2, db3 += G; adjoint of h2 = w3 G on active units
        f32x16 d2[HT];
#pragma unroll
        for (int mt = 0; mt < HT; ++mt)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float hv = h2.v[mt][r];
                gw3[mt][r] = __builtin_fmaf(gc, hv, gw3[mt][r]);
                d2[mt][r] = hv > 0.0f ? p.w3[32 * mt + out_row(r, g)] * gc : 0.0f;
            }
        if (g == 0) gb3 += gc;
        // dW2 += d2 h1^T over the tile's pairs (rows d2 at 0..63, h1 at 64..127); b2 += d2
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int mt = 0; mt < HT; ++mt)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                scr[col * kRow + 32 * mt + out_row(r, g)] = d2[mt][r];
                scr[col * kRow + 64 + 32 * mt + out_row(r, g)] = valid ? h1.v[mt][r] : 0.0f;
            }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int c = 0; c < 16; ++c) {
            const float* rw = scr + (2 * c + g) * kRow;
#pragma unroll
            for (int nt = 0; nt < HT; ++nt) {
                const float bx = rw[64 + 32 * nt + col];
#pragma unroll
                for (int mt = 0; mt < HT; ++mt) gW2[mt][nt] = mfma(rw[32 * mt + col], bx, gW2[mt][nt]);
            }
        }
#pragma unroll
        for (int mt = 0; mt < HT; ++mt) gb2[mt] += d2[mt];
        // adjoint of h1 = (W2^T d2) on active units
        f32x16 d1[HT];
#pragma unroll
        for (int mt = 0; mt < HT; ++mt) d1[mt] = f32x16{};
#pragma unroll
        for (int c0 = 0; c0 < 16 * HT; c0 += 8) {
            const char* bwz = bw + opaque_zero();
#pragma unroll
            for (int c = c0; c < c0 + 8; ++c)
#pragma unroll
                for (int mt = 0; mt < HT; ++mt)
                    d1[mt] = mfma(lds_frag(bwz, BI::t2(c, mt), lane), d2[c >> 4][c & 15], d1[mt]);
        }
#pragma unroll
        for (int mt = 0; mt < HT; ++mt)
#pragma unroll
            for (int r = 0; r < 16; ++r) d1[mt][r] = h1.v[mt][r] > 0.0f ? d1[mt][r] : 0.0f;
        // dW1 (+ b1 through column 31) += d1 x^T, x = [s'_i, a_i, o_j, 0, ..., 1]
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int mt = 0; mt < HT; ++mt)
#pragma unroll
            for (int r = 0; r < 16; ++r) scr[col * kRow + 32 * mt + out_row(r, g)] = d1[mt][r];
        int a_i = 0;
        if (N_ACT > 0) {
            a_i = reinterpret_cast<const int32_t*>(p.actions)[i];
            if (a_i < 0 || a_i >= N_ACT) a_i = 0;  // flagged by the fold, which uses action 0 as well
        }
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int c = 16 * g + q;
            float v = 0.0f;
            if (c < D_S) {
                v = p.states[(size_t)i * D_S + c];
            } else if (c < D_S + D_AIN) {
                if (N_ACT > 0) v = (c - D_S == a_i) ? 1.0f : 0.0f;
                else v = reinterpret_cast<const float*>(p.actions)[(size_t)i * D_AIN + (c - D_S)];
            } else if (c < D_IN) {
                v = p.obs[(size_t)(valid ? j : 0) * D_O + (c - D_S - D_AIN)];
            } else if (c == 31) {
                v = 1.0f;
            }
            scr[col * kRow + 64 + c] = valid ? v : 0.0f;
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int c = 0; c < 16; ++c) {
            const float* rw = scr + (2 * c + g) * kRow;
            const float bx = rw[64 + col];
#pragma unroll
            for (int mt = 0; mt < HT; ++mt) gW1[mt] = mfma(rw[32 * mt + col], bx, gW1[mt]);
        }
        __builtin_amdgcn_wave_barrier();
    }
    // per-wave partials: W1 [64][D_IN], b1 [64], W2 [64][64], b2 [64], W3 [1][64], b3 [1]
    const int wid = blockIdx.x * wpb + wave;
    float* out = p.wpart + (size_t)wid * p.n_params;
    constexpr int oW1 = 0, ob1 = 64 * D_IN, oW2 = ob1 + 64, ob2 = oW2 + 64 * 64, oW3 = ob2 + 64, ob3 = oW3 + 64;
#pragma unroll
    for (int mt = 0; mt < HT; ++mt)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int m = 32 * mt + out_row(r, g);
            if (col < D_IN) out[oW1 + m * D_IN + col] = gW1[mt][r];
            if (col == 31) out[ob1 + m] = gW1[mt][r];
#pragma unroll
            for (int nt = 0; nt < HT; ++nt) out[oW2 + m * 64 + 32 * nt + col] = gW2[mt][nt][r];
            const float vb = sum32(gb2[mt][r]);
            const float vw = sum32(gw3[mt][r]);
            if (col == 0) {
                out[ob2 + m] = vb;
                out[oW3 + m] = vw;
            }
        }
    const float v3 = sum32(gb3);
    if (lane == 0) out[ob3] = v3;
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
#define GRAD_SHAPES(X) X(0, 4, 5, 0, 4) X(2, 4, 0, 4, 4)

bool grad_supported(int shape) {
#define X(id, ds, na, da, dw) if (shape == id) return true;
    GRAD_SHAPES(X)
#undef X
    return false;
}

hipError_t launch_grad(int shape, const GradParams& p, int blocks, size_t lds, hipStream_t s) {
    // at least four waves stage the networks, whatever number takes tiles
    const int threads = 64 * (p.waves < 4 ? 4 : p.waves);
    auto launch = [&](void (*k)(GradParams)) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        hipLaunchKernelGGL(k, blocks, threads, lds, s, p);
    };
    switch (shape) {
#define X(id, ds, na, da, dw)                                                                          \
    case id:                                                                                          \
        launch(p.C > 1 ? grad_kernel<ds, na, da, dw, true> : grad_kernel<ds, na, da, dw, false>);      \
        break;
        GRAD_SHAPES(X)
#undef X
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

size_t grad_scratch_bytes(int waves) { return (size_t)waves * 32 * kRowR * sizeof(float); }

// (shape id, d_s, discrete actions, continuous action width, d_o)
#define NCE_GRAD_SHAPES(X) X(0, 4, 5, 0, 2) X(2, 4, 0, 4, 2)

bool nce_grad_supported(int shape) {
#define X(id, ds, na, da, dox) if (shape == id) return true;
    NCE_GRAD_SHAPES(X)
#undef X
    return false;
}

hipError_t launch_nce_grad(int shape, const NceGradParams& p, int blocks, size_t lds, hipStream_t s) {
    switch (shape) {
#define X(id, ds, na, da, dox)                                                                                \
    case id:                                                                                                 \
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(nce_grad_kernel<ds, na, da, dox>),            \
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);                      \
        hipLaunchKernelGGL((nce_grad_kernel<ds, na, da, dox>), blocks, 256, lds, s, p);                       \
        break;
        NCE_GRAD_SHAPES(X)
#undef X
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

int nce_grad_blocks_per_cu(int shape, size_t lds) {
    int n = 0;
    switch (shape) {
#define X(id, ds, na, da, dox)                                                                                 \
    case id:                                                                                                  \
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, nce_grad_kernel<ds, na, da, dox>, 256, lds) != hipSuccess) \
            n = 1;                                                                                            \
        break;
        NCE_GRAD_SHAPES(X)
#undef X
    }
    return n < 1 ? 1 : n;
}

hipError_t launch_grad_reduce(const GradReduceParams& p, hipStream_t s) {
    constexpr int threads = kRedCols * kRedWaves;
    const int param_blocks = p.grad_params ? (p.n_params + kRedCols - 1) / kRedCols : 0;
    const int acts = p.grad_actions ? (p.n_action_values + threads - 1) / threads : 0;
    const int more = acts > 0 ? acts : (p.loss ? 1 : 0);
    if (param_blocks + more == 0) return hipSuccess;
    hipLaunchKernelGGL(grad_reduce_kernel, param_blocks + more, threads, 0, s, p, param_blocks);
    return hipGetLastError();
}

}  // namespace voila
