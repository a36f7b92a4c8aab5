// k_search.hip -- planner steps above the rollout core: soft value and action
// selection, the one-level closed-loop tree, grouped progressive widening.
#include "kcommon.hpp"

namespace voila {

// ---------------------------------------------------------------------------
// soft value: V = (1/eta) log sum_k exp(eta Q_k + log pi0_k), per node
// ---------------------------------------------------------------------------
constexpr int kSoftThreads = 256;

__global__ __launch_bounds__(kSoftThreads) void soft_value_kernel(SoftValueParams p) {
    __shared__ double redd[kSoftThreads / 64];
    __shared__ int redi[kSoftThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const double lp_uniform = p.no_prior ? 0.0 : -log((double)p.K);
    for (int m = blockIdx.x; m < p.M; m += gridDim.x) {
        const float* qf = p.Q ? p.Q + (size_t)m * p.K : nullptr;
        const double* qd = p.Qd ? p.Qd + (size_t)m * p.K : nullptr;
        auto q = [&](int k) { return qd ? qd[k] : (double)qf[k]; };
        const double* lp = p.log_pi0 ? p.log_pi0 + (size_t)m * p.K : nullptr;
        // x_k = eta Q_k + log pi0_k; maximum and its first index
        double mx = -INFINITY;
        int arg = p.K;
        int bad = 0;
        for (int k = tid; k < p.K; k += kSoftThreads) {
            const double x = p.eta * q(k) + (lp ? lp[k] : lp_uniform);
            if (isnan(x) || x == INFINITY) bad = 1;
            if (x > mx) {
                mx = x;
                arg = k;
            }
        }
        // (max, lowest index) over the block, in a fixed order
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) {
            const double om = __shfl_xor(mx, d);
            const int oa = __shfl_xor(arg, d);
            if (om > mx || (om == mx && oa < arg)) {
                mx = om;
                arg = oa;
            }
            bad |= __shfl_xor(bad, d);
        }
        __syncthreads();
        if (lane == 0) {
            redd[wave] = mx;
            redi[wave] = bad ? -1 : arg;
        }
        __syncthreads();
        mx = redd[0];
        arg = redi[0];
        bad = redi[0] < 0;
        for (int w = 1; w < kSoftThreads / 64; ++w) {
            bad |= redi[w] < 0;
            if (redd[w] > mx || (redd[w] == mx && redi[w] < arg)) {
                mx = redd[w];
                arg = redi[w];
            }
        }
        if (bad || !isfinite(mx)) {
            if (tid == 0 && p.status) p.status[0] = 5;
            __syncthreads();
            continue;
        }
        double s = 0.0;
        for (int k = tid; k < p.K; k += kSoftThreads)
            s += exp(p.eta * q(k) + (lp ? lp[k] : lp_uniform) - mx);
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) s += __shfl_xor(s, d);
        __syncthreads();
        if (lane == 0) redd[wave] = s;
        __syncthreads();
        double S = 0.0;
        for (int w = 0; w < kSoftThreads / 64; ++w) S += redd[w];
        if (tid == 0) {
            p.V[m] = (mx + log(S)) / p.eta;
            if (p.best) p.best[m] = arg;
        }
        if (p.pi)
            for (int k = tid; k < p.K; k += kSoftThreads)
                p.pi[(size_t)m * p.K + k] = exp(p.eta * q(k) + (lp ? lp[k] : lp_uniform) - mx) / S;
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// one-level closed-loop tree (preference backup over observation branches)
// ---------------------------------------------------------------------------
// Successor set of branch group (a, j): the successors of first action a
// starting at successor j; the group's offsets, action and empty branch table.
__global__ __launch_bounds__(256) void tree_groups_kernel(TreeParams p) {
    const int M = p.A * p.n_obs;
    const long n_el = (long)M * p.N * p.d_s;
    for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < n_el; e += (long)gridDim.x * blockDim.x) {
        const long row = e / p.d_s;
        const int c = (int)(e - row * p.d_s);
        const int m = (int)(row / p.N), i = (int)(row - (long)m * p.N);
        const int a = m / p.n_obs, j = m - a * p.n_obs;
        int src = i + j % p.N;
        if (src >= p.N) src -= p.N;
        p.succ[e] = p.succ0[((size_t)a * p.N + src) * p.d_s + c];
    }
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    if (m <= M) p.seg[m] = m * p.N;
    if (m < M) {
        const int a = m / p.n_obs;
        p.zeros[m] = 0;
        p.zeros[M + m] = 0;
        if (p.n_actions > 0) {
            reinterpret_cast<int32_t*>(p.acts)[m] = reinterpret_cast<const int32_t*>(p.first)[a];
        } else {
            for (int c = 0; c < p.d_a; ++c)
                reinterpret_cast<float*>(p.acts)[(size_t)m * p.d_a + c] =
                    reinterpret_cast<const float*>(p.first)[(size_t)a * p.d_a + c];
        }
    }
}

// Child preferences: the mean continuation return of candidate k over the
// particles of child m, one wave per (m, k), fixed summation order.
__global__ __launch_bounds__(256) void tree_child_q_kernel(TreeParams p) {
    const int M = p.A * p.n_obs;
    const int lane = threadIdx.x & 63;
    const long item = (long)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (item >= (long)M * p.K) return;
    const int m = (int)(item / p.K), k = (int)(item - (long)m * p.K);
    const float* g = p.G2 + (size_t)k * ((size_t)M * p.N) + (size_t)m * p.N;
    double s = 0.0;
    for (int i = lane; i < p.N; i += 64) s += (double)g[i];
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) s += __shfl_xor(s, d);
    if (lane == 0) p.Qc[(size_t)m * p.K + k] = s / p.N;
}

// Psi(b, a) = (1/eta) log pi0(a) + R(b, a) + gamma mean_j V_child(a, j).
__global__ __launch_bounds__(64) void tree_backup_kernel(TreeParams p) {
    const int a = blockIdx.x * blockDim.x + threadIdx.x;
    if (a >= p.A) return;
    double v = 0.0;
    for (int j = 0; j < p.n_obs; ++j) v += p.Vc[(size_t)a * p.n_obs + j];
    const double lp = p.log_pi0 ? p.log_pi0[a] : -log((double)p.A);
    p.psi[a] = lp / p.eta + (double)p.R[a] + p.gamma * (v / p.n_obs);
    if (p.R_out) p.R_out[a] = (double)p.R[a];
}

// ---------------------------------------------------------------------------
// grouped progressive widening (simulations grouped by parent action node)
// ---------------------------------------------------------------------------
namespace {
// Group m's successors [lo, lo + n) if the offsets are consistent and the
// group fits one workgroup; otherwise the group is skipped and *status set.
__device__ __forceinline__ void pw_group(const PwParams& p, int m, int& lo, int& n) {
    if (!pw_rows(p.seg, m, p.T, lo, n) && p.status) p.status[0] = 1;
}
}  // namespace

// Widening test, branch choice and table update, 32 lanes per action node (each
// takes the test; they share the copies), and the records of the node's
// likelihood work units.
__global__ __launch_bounds__(256) void pw_branch_kernel(PwParams p) {
    const int m = blockIdx.x * (blockDim.x / 32) + threadIdx.x / 32, l = threadIdx.x & 31;
    if (m >= p.M) return;
    int lo, n;
    pw_group(p, m, lo, n);
    const int listed = p.tiles[p.M], at = p.tiles[m];
    if (listed >= 0)  // at most as many units as there are records
        for (int q = l, nu = pw_unit_count(n, 32 * p.unit_tiles); q < nu; q += 32) {
            const PwUnit w = pw_unit(m, lo, n, q, 32 * p.unit_tiles);
            p.units[at + q] = make_int4(w.group, w.first, w.end, 0);
        }
    int wid = 0, br = -1;
    const int C = p.children[m];
    if (C < 0 || C > p.B) {
        if (p.status) p.status[0] = 1;
        n = 0;
    }
    if (n > 0) {
        wid = C < p.B && (C == 0 || (double)C < p.k_o * pow((double)p.visits[m], p.alpha_o));
        float* row = p.table + (size_t)m * p.B * p.d_o;
        if (wid) {
            br = C;
        } else {
            const uint4 w = philox4x32_10(make_uint4((uint32_t)m, 1u, 0u, 6u << 16), p.key0, p.key1);
            br = (int)floor((double)word_to_uniform(w.x) * (double)C);
        }
        for (int c = l; c < p.d_o; c += 32) {
            const float v = wid ? p.o_new[(size_t)m * p.d_o + c] : row[(size_t)br * p.d_o + c];
            if (wid) row[(size_t)br * p.d_o + c] = v;
            p.o_sel[(size_t)m * p.d_o + c] = v;
        }
    } else {
        for (int c = l; c < p.d_o; c += 32) p.o_sel[(size_t)m * p.d_o + c] = 0.0f;
    }
    if (l == 0) {
        // (after every lane's read of the count: a wave's lanes step together)
        if (wid) p.children[m] = C + 1;
        if (p.widen) p.widen[m] = wid;
        if (p.branch) p.branch[m] = br;
    }
}

// Block 0: exclusive prefix of the groups' likelihood work units, or -1 as its
// last entry where they are not listed (pw_units.hpp).  The next
// blocks: first successor of each group (the state a new branch's observation
// is drawn at); the last ones: the observation network's bias rows (few groups;
// many take fold_rows_kernel).  One launch, since none needs another's result.
__global__ __launch_bounds__(1024) void pw_prepare_kernel(PwParams p, FoldStepsParams fold, int first_blocks) {
    if ((int)blockIdx.x > first_blocks) {
        const long e = (long)((int)blockIdx.x - 1 - first_blocks) * blockDim.x + threadIdx.x;
        const int j = (int)(e / fold.width), r = (int)(e - (long)j * fold.width);
        if (j < fold.rows) fold_element(fold, j, r);
        return;
    }
    if (blockIdx.x > 0) {
        const int e = (blockIdx.x - 1) * blockDim.x + threadIdx.x;
        if (e >= p.M * p.d_s) return;
        const int m = e / p.d_s, c = e - m * p.d_s;
        int lo, n;
        pw_group(p, m, lo, n);
        p.first[e] = n > 0 ? p.succ[(size_t)lo * p.d_s + c] : 0.0f;
        return;
    }
    __shared__ long wtot[16];
    const int tid = threadIdx.x, lane = tid & 63;
    const int per = (p.M + 1023) / 1024, rows = 32 * p.unit_tiles;
    const int a = tid * per, b = min(p.M, a + per);
    long run = 0;  // (groups that overlap may have more units than an int holds)
    for (int m = a; m < b; ++m) {
        int lo, n;
        pw_group(p, m, lo, n);
        run += pw_unit_count(n, rows);
    }
    long incl = run;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const long o = __shfl_up(incl, d);
        if (lane >= d) incl += o;
    }
    if (lane == 63) wtot[tid >> 6] = incl;
    __syncthreads();
    long off = incl - run;
    for (int w = 0; w < (tid >> 6); ++w) off += wtot[w];
    for (int m = a; m < b; ++m) {
        int lo, n;
        pw_group(p, m, lo, n);
        p.tiles[m] = (int)off;
        off += pw_unit_count(n, rows);
    }
    if (tid == 1023) p.tiles[p.M] = pw_listed(off, p.T, p.M);
}

// Likelihood of every successor against its group's chosen observation:
// x_j = l([s'_j, a_m, o_m]) / lambda, one work unit of one group per wave: a
// 32-row tile, or two through the paired evaluation of the rollout kernel.  A
// unit's record, states and bias row are read one unit ahead (a wave's
// consecutive units lie in different groups, and finding the group by bisection
// alone took as long as the network).  2.1 M successors of 4,096 groups,
// bfloat16 realistic network: 800 -> 600 us.
template <int DT, int D_S, int WIDTH, int NHID, int MODE>
__global__ __launch_bounds__(256) void pw_lik_kernel(PwParams p) {
    if constexpr (!generic_compiled(DT, WIDTH, NHID)) {
        return;  // refused at model creation (binary32 wider than 256) or run by the split rollout kernel
    } else {
    typedef Net<DT, WIDTH, NHID, in_slots(DT, D_S, 0, 0)> NTL;
    constexpr int SS = state_slots(D_S);
    constexpr bool PAIRS = MODE == kStream && plan_pairs<DT, WIDTH, NHID>();
    constexpr int TPU = PAIRS ? 2 : 1;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int lane = threadIdx.x & 63, g = lane >> 5, col = lane & 31;
    const int wpb = blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const kconst int32_t* units = (const kconst int32_t*)p.units;
    const int listed = ((const kconst int32_t*)p.tiles)[p.M];
    float* rowb = reinterpret_cast<float*>(smem + p.row_bias_lds) + wave * NTL::WIDTH;
    constexpr int RB = NTL::WIDTH / 64;  // bias floats per lane
    static_assert(NTL::WIDTH % 64 == 0 && RB <= 16, "bias row copy: whole lanes");
    with_weights<NTL, MODE, 1, PAIRS ? VOILA_PLAN_STREAM_CHB : VOILA_STREAM_CHB>(smem, p.lik, [&](auto& src,
                                                                                            const NetPtrs& P) {
        // the units 0 .. n_units - 1 that unit_at gives
        auto sweep = [&](long n_units, auto unit_at) {
            if (n_units == 0) return;
            int nj[TPU];
            bool nv[TPU];
            float nst[TPU][SS], nbv[RB];
            auto next_inputs = [&](long u) {
                const bool ok = u < n_units;  // wave-uniform
                const PwUnit w = unit_at(ok ? u : 0);
                const int left = ok ? w.end - w.first : 0;
#pragma unroll
                for (int q = 0; q < TPU; ++q) {
                    nj[q] = w.first + 32 * q + col;
                    nv[q] = 32 * q + col < left;
#pragma unroll
                    for (int s = 0; s < SS; ++s) {
                        const int f = 2 * s + g;
                        nst[q][s] = (nv[q] && f < D_S) ? p.succ[(size_t)nj[q] * D_S + f] : 0.0f;
                    }
                }
                const float* brow = p.b0_lik + (size_t)w.group * NTL::WIDTH;
#pragma unroll
                for (int q = 0; q < RB; ++q) nbv[q] = brow[q * 64 + lane];
            };
            next_inputs((long)blockIdx.x * wpb + wave);
            // block-uniform loop (a streamed network's chunk barriers need every wave)
            for (long ub = blockIdx.x; ub * wpb < n_units; ub += gridDim.x) {
                float slots[TPU][NTL::IN_SLOTS];
                int j[TPU];
                bool valid[TPU];
#pragma unroll
                for (int q = 0; q < TPU; ++q) {
                    j[q] = nj[q];
                    valid[q] = nv[q];
#pragma unroll
                    for (int s = 0; s < NTL::IN_SLOTS; ++s) slots[q][s] = 0.0f;
#pragma unroll
                    for (int s = 0; s < SS; ++s) slots[q][s] = nst[q][s];
                }
#pragma unroll
                for (int q = 0; q < RB; ++q) rowb[q * 64 + lane] = nbv[q];
                next_inputs((ub + gridDim.x) * wpb + wave);
                f32x16 o[TPU];
                if constexpr (PAIRS) {
                    run_net_flat<NTL, 2, kPlanPassTiles>(src, P, rowb, slots, o, lane, g);
                } else {
                    o[0] = run_net<NTL>(src, P, rowb, slots[0], lane, g);
                }
#pragma unroll
                for (int q = 0; q < TPU; ++q)
                    if (g == 0 && valid[q]) {
                        const float l = o[q][0];
                        if (p.loglik) p.loglik[j[q]] = l;
                        if (!isfinite(l) && p.status) p.status[0] = 5;
                        p.x[j[q]] = (double)l / p.lambda;
                    }
            }
        };
        // (two loops: choosing between the forms in one took 0.8 % of the whole step)
        if (listed >= 0)
            sweep(listed, [&](long u) { return PwUnit{units[4 * u], units[4 * u + 1], units[4 * u + 2]}; });
        else
            sweep(pw_unlisted_units(p.M, 32 * TPU),
                  [&](long u) { return pw_unlisted_unit(p.seg, p.T, u, 32 * TPU); });
    });
    }
}

// Weights, statistics and systematic resampling of every group of at most
// kPwSmall successors, a workgroup of 256 threads each (a group is a chain of
// reductions: many small workgroups per CU overlap their latencies, where one
// of 1,024 threads with LDS for 8,192 fills a CU alone: 159 -> 89 us for 4,096
// groups).  Element tid + 256 v plays thread tid + 256 v of the single-belief
// procedure and the sums keep its order (lanes by butterfly, then the 16
// wave sums), so the weights are its bits.
constexpr int kPwSmall = 1024, kPwThreads = 256, kPwPer = kPwSmall / kPwThreads, kPwWaves = kPwSmall / 64;
__global__ __launch_bounds__(kPwThreads) void pw_norm_res_small_kernel(PwParams pw) {
    __shared__ double buf[kPwSmall];
    __shared__ int ids[kPwSmall];
    __shared__ double redd[kPwWaves];
    __shared__ int redi[kPwThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // (waves past the group's end have nothing to compute in slot k: zeros)
    auto sum = [&](const double (&v)[kPwPer], int n) {
        double t[kPwPer];
#pragma unroll
        for (int k = 0; k < kPwPer; ++k) t[k] = kPwThreads * k + 64 * wave < n ? wave_sum_d(v[k]) : 0.0;
        __syncthreads();
        if (lane == 0)
#pragma unroll
            for (int k = 0; k < kPwPer; ++k) redd[4 * k + wave] = t[k];
        __syncthreads();
        double r = 0.0;
#pragma unroll
        for (int w = 0; w < kPwWaves; ++w) r += redd[w];
        return r;
    };
    auto max_i = [&](int v) {
        v = wave_max_i(v);
        __syncthreads();
        if (lane == 0) redi[wave] = v;
        __syncthreads();
        int r = redi[0];
#pragma unroll
        for (int w = 1; w < kPwThreads / 64; ++w) r = max(r, redi[w]);
        return r;
    };
    for (int m = blockIdx.x; m < pw.M; m += gridDim.x) {
        int lo, n;
        pw_group(pw, m, lo, n);
        if (n == 0 || n > kPwSmall) continue;
        int c = 0;
        while ((1 << c) < n) ++c;
        const int bits = 52 - c < 32 ? 52 - c : 32;
        double x[kPwPer], v[kPwPer], mx = -INFINITY;
        int bad = 0;
#pragma unroll
        for (int k = 0; k < kPwPer; ++k) {
            const int i = tid + kPwThreads * k;
            x[k] = i < n ? pw.x[(size_t)lo + i] : -INFINITY;
            if (isnan(x[k]) || x[k] == INFINITY) bad = 1;
            mx = fmax(mx, x[k]);
        }
        mx = wave_max_d(mx);
        __syncthreads();
        if (lane == 0) redd[wave] = mx;
        __syncthreads();
        mx = fmax(fmax(redd[0], redd[1]), fmax(redd[2], redd[3]));
        if (max_i(bad) || !isfinite(mx)) {
            if (tid == 0 && pw.status) pw.status[0] = 5;
            __syncthreads();
            continue;
        }
#pragma unroll
        for (int k = 0; k < kPwPer; ++k) {
            v[k] = 0.0;
            if (kPwThreads * k + 64 * wave < n) v[k] = tid + kPwThreads * k < n ? exp(x[k] - mx) : 0.0;
        }
        const double S = sum(v, n);
        double w[kPwPer];
#pragma unroll
        for (int k = 0; k < kPwPer; ++k) {
            const int i = tid + kPwThreads * k;
            w[k] = 0.0;
            if (i < n) {
                w[k] = v[k] / S;
                if (pw.w) pw.w[(size_t)lo + i] = w[k];
            }
            v[k] = w[k] * w[k];
        }
        const double SQ = sum(v, n);
        if (tid == 0 && pw.stats) {
            pw.stats[2 * (size_t)m] = mx + log(S) - log((double)n);
            pw.stats[2 * (size_t)m + 1] = 1.0 / SQ;
        }
        const double scale = ldexp((double)n, bits);
        int last = -1;
#pragma unroll
        for (int k = 0; k < kPwPer; ++k) {
            w[k] = rint(w[k] * scale);
            if (w[k] > 0.0) last = tid + kPwThreads * k;
        }
        last = max_i(last);
        if (last < 0) {
            if (tid == 0 && pw.status) pw.status[0] = 5;
            __syncthreads();
            continue;
        }
        // inclusive prefix (exact integers: any order gives the same bits)
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kPwPer; ++k) {
            v[k] = w[k];
            if (kPwThreads * k + 64 * wave < n)
#pragma unroll
                for (int d = 1; d < 64; d <<= 1) {
                    const double o = __shfl_up(v[k], d);
                    if (lane >= d) v[k] += o;
                }
            if (lane == 63) redd[4 * k + wave] = v[k];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kPwPer; ++k) {
            double off = 0.0;
            for (int q = 0; q < 4 * k + wave; ++q) off += redd[q];
            buf[tid + kPwThreads * k] = v[k] + off;
        }
        __syncthreads();
        const double step = ldexp(1.0, bits), u = (double)(pw.U[m] >> (32 - bits));
        // first i with C_i > P_j (the count of C_i <= P_j), a thread's outputs side by side
        int at[kPwPer];
#pragma unroll
        for (int k = 0; k < kPwPer; ++k) at[k] = 0;
#pragma unroll
        for (int d = kPwSmall; d >= 1; d >>= 1) {
            if (d > n) continue;
#pragma unroll
            for (int k = 0; k < kPwPer; ++k) {
                const double P = (double)(tid + kPwThreads * k) * step + u;
                const int e = at[k] + d;
                if (e <= n && !(buf[e - 1] > P)) at[k] = e;
            }
        }
#pragma unroll
        for (int k = 0; k < kPwPer; ++k) {
            const int j = tid + kPwThreads * k;
            if (j < n) {
                const int idx = at[k] < n ? at[k] : last;
                if (pw.idx) pw.idx[(size_t)lo + j] = idx;
                ids[j] = idx;
            }
        }
        __syncthreads();
        if (pw.succ_out) {
            const int rf = pw.d_s;
            const float* src = pw.succ + (size_t)lo * rf;
            float* dst = pw.succ_out + (size_t)lo * rf;
            if (rf % 4 == 0 && ((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) & 15) == 0)
                block_gather(reinterpret_cast<float4*>(dst), reinterpret_cast<const float4*>(src), ids, n, rf / 4);
            else
                block_gather(dst, src, ids, n, rf);
        }
        __syncthreads();
    }
}

// The same for groups of more than `above` successors, one workgroup of 1,024
// threads per group (the single-belief procedure on the group's rows).
__global__ __launch_bounds__(kNormResThreads) void pw_norm_res_kernel(PwParams pw, int above) {
    __shared__ double buf[kNormResMaxN];
    __shared__ int ids[kNormResMaxN];
    __shared__ double redd[kNRWaves];
    __shared__ int redi[kNRWaves];
    for (int m = blockIdx.x; m < pw.M; m += gridDim.x) {
        int lo, n;
        pw_group(pw, m, lo, n);
        if (n <= above) continue;
        int c = 0;
        while ((1 << c) < n) ++c;
        NormResParams p{};
        p.x = pw.x + lo;
        p.lambda = pw.lambda;
        p.N = n;
        p.bits = 52 - c < 32 ? 52 - c : 32;
        p.uniform_prior = 1;
        p.do_resample = 1;
        p.U = pw.U[m];
        p.w_out = pw.w ? pw.w + lo : nullptr;
        p.stats = pw.stats ? pw.stats + 2 * (size_t)m : nullptr;
        p.idx_out = pw.idx ? pw.idx + lo : nullptr;
        p.src = pw.succ_out ? pw.succ + (size_t)lo * pw.d_s : nullptr;
        p.dst = pw.succ_out ? pw.succ_out + (size_t)lo * pw.d_s : nullptr;
        p.row_floats = pw.d_s;
        p.status = pw.status;
        norm_res_body(p, buf, redd, redi, ids);
        __syncthreads();
    }
}

// launchers
#define PWL_K(id, ds, na, da, dw, dox, dwz, w, nh, DT) pw_lik_kernel<DT, ds, w, nh, plan_mode<w>()>

template <int DT, int D_S, int W, int NH>
constexpr size_t pw_stream_lds() {
    return plan_pairs<DT, W, NH>() ? stream_lds_of<DT, D_S, 0, 0, 0, W, NH, VOILA_PLAN_STREAM_CHB>()
                                   : stream_lds_of<DT, D_S, 0, 0, 0, W, NH>();
}

hipError_t launch_pw_lik(int shape, int dt, const PwParams& p0, int blocks, hipStream_t s) {
    PwParams p = p0;
    size_t lds = p.lik.bytes;
    if (!weights_in_lds(shape)) {
        switch (shape * 2 + dt) {
#define X(id, ds, na, da, dw, dox, dwz, w, nh)                           \
    case id * 2 + 0:                                                    \
        lds = pw_stream_lds<DT_F32, ds, w, nh>();                       \
        break;                                                          \
    case id * 2 + 1:                                                    \
        lds = pw_stream_lds<DT_BF16, ds, w, nh>();                      \
        break;
            VOILA_SHAPES(X)
#undef X
        }
        lds += p.lik.bytes - p.lik.off_b0;
    }
    // one first-layer bias row per wave after the staged weights and biases
    lds = (lds + 15) / 16 * 16;
    p.row_bias_lds = (uint32_t)lds;
    lds += (size_t)kWavesPerBlock * shape_info(shape).width * 4;
    switch (shape * 2 + dt) {
#define X(id, ds, na, da, dw, dox, dwz, w, nh)                                                                \
    case id * 2 + 0:                                                                                         \
        if (lds > 65536)                                                                                     \
            (void)hipFuncSetAttribute((const void*)PWL_K(id, ds, na, da, dw, dox, dwz, w, nh, DT_F32),        \
                                      hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);                 \
        hipLaunchKernelGGL((PWL_K(id, ds, na, da, dw, dox, dwz, w, nh, DT_F32)), blocks, 256, lds, s, p);     \
        break;                                                                                               \
    case id * 2 + 1:                                                                                         \
        if (lds > 65536)                                                                                     \
            (void)hipFuncSetAttribute((const void*)PWL_K(id, ds, na, da, dw, dox, dwz, w, nh, DT_BF16),       \
                                      hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);                 \
        hipLaunchKernelGGL((PWL_K(id, ds, na, da, dw, dox, dwz, w, nh, DT_BF16)), blocks, 256, lds, s, p);    \
        break;
        VOILA_SHAPES(X)
#undef X
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

int pw_lik_blocks_per_cu(int shape, int dt) {
    switch (shape * 2 + dt) {
#define X(id, ds, na, da, dw, dox, dwz, w, nh)                                                               \
    case id * 2 + 0:                                                                                        \
        return occupancy(PWL_K(id, ds, na, da, dw, dox, dwz, w, nh, DT_F32),                                \
                         lds_for_width<w>() ? kLdsGuess : pw_stream_lds<DT_F32, ds, w, nh>());               \
    case id * 2 + 1:                                                                                        \
        return occupancy(PWL_K(id, ds, na, da, dw, dox, dwz, w, nh, DT_BF16),                               \
                         lds_for_width<w>() ? kLdsGuess : pw_stream_lds<DT_BF16, ds, w, nh>());
        VOILA_SHAPES(X)
#undef X
    }
    return 1;
}

hipError_t launch_tree_groups(const TreeParams& p, hipStream_t s) {
    const int M = p.A * p.n_obs;
    const long n_el = (long)M * p.N * p.d_s;
    long blocks = (n_el + 255) / 256;
    if (blocks < (M + 1 + 255) / 256) blocks = (M + 1 + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(tree_groups_kernel, (int)blocks, 256, 0, s, p);
    return hipGetLastError();
}

hipError_t launch_tree_child_q(const TreeParams& p, hipStream_t s) {
    const long items = (long)p.A * p.n_obs * p.K;
    hipLaunchKernelGGL(tree_child_q_kernel, (int)((items + 3) / 4), 256, 0, s, p);
    return hipGetLastError();
}

hipError_t launch_tree_backup(const TreeParams& p, hipStream_t s) {
    hipLaunchKernelGGL(tree_backup_kernel, (p.A + 63) / 64, 64, 0, s, p);
    return hipGetLastError();
}

hipError_t launch_soft_value(const SoftValueParams& p, int blocks, hipStream_t s) {
    if (p.M == 0 || blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(soft_value_kernel, blocks, kSoftThreads, 0, s, p);
    return hipGetLastError();
}

hipError_t launch_pw_branch(const PwParams& p, hipStream_t s) {
    if (p.M == 0) return hipSuccess;
    hipLaunchKernelGGL(pw_branch_kernel, (p.M + 7) / 8, 256, 0, s, p);
    return hipGetLastError();
}

hipError_t launch_pw_prepare(const PwParams& p, const FoldStepsParams& fold, hipStream_t s) {
    const int first_blocks = (p.M * p.d_s + 1023) / 1024;
    const bool here = !fold_takes_rows(fold);
    const int fold_blocks = here ? (int)(((long)fold.rows * fold.width + 1023) / 1024) : 0;
    hipLaunchKernelGGL(pw_prepare_kernel, 1 + first_blocks + fold_blocks, 1024, 0, s, p, fold, first_blocks);
    const hipError_t e = hipGetLastError();
    return e != hipSuccess || here ? e : launch_fold_steps(fold, s);
}

hipError_t launch_pw_norm_res(const PwParams& p, int cus, hipStream_t s) {
    if (p.M == 0 || cus == 0) return hipSuccess;
    // a group can only be larger when there are that many successors
    const bool large = p.T > kPwSmall;
    // The kernel for large groups takes all of them where a CU has one (16 groups of
    // up to 2,048 successors of the realistic network, whole step in bfloat16: 58 us,
    // 74 with the small ones in a launch before), and where the average says that
    // some are large, as those then are a second, hardly filled launch: from 512 on
    // for two rounds of groups over the CUs (512 of up to 1,100, small networks: 79 us
    // against 94, of up to 1,000 77 either way, of up to 300 realistic 89 / 85), later
    // for more (700 of up to 1,100 101 / 109, of up to 1,000 95 / 88; 1,000 of up to
    // 1,270 134 / 145, of up to 1,100 131 / 128).
    const int rounds = (p.M + cus - 1) / cus, mean = p.T / p.M;
    if (large && (rounds == 1 || mean >= 448 + 32 * (rounds < 4 ? rounds : 4))) {
        hipLaunchKernelGGL(pw_norm_res_kernel, p.M < cus ? p.M : cus, kNormResThreads, 0, s, p, 0);
        return hipGetLastError();
    }
    const int cap = 8 * cus;
    hipLaunchKernelGGL(pw_norm_res_small_kernel, p.M < cap ? p.M : cap, kPwThreads, 0, s, p);
    if (large) hipLaunchKernelGGL(pw_norm_res_kernel, p.M < cus ? p.M : cus, kNormResThreads, 0, s, p, kPwSmall);
    return hipGetLastError();
}

}  // namespace voila
