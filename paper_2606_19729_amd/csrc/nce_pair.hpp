// nce_pair.hpp -- what the two kernels of k_nce_pair.hip and k_nce_pair_products.hip
// share: the parameter derivative of the contrastive (InfoNCE)
// objective for the bfloat16 likelihood network of three hidden layers of
// 256, in two stages per chunk of pairs:
//   1. nce_pair_bwd_kernel: every pair (i, j) runs the network forward on
//      [s'_i, a_i, o_j] and the reverse sweep with weight G_ij (Eq. 6).  A wave
//      takes two units (row i, 32 consecutive columns j each), so that every
//      weight fragment feeds two products, and stores h_2, delta_2, delta_1
//      and the sign pattern of h_3 with pairs along the registers: the operand
//      the products of stage 2 read straight from memory.
//   2. nce_pair_wgrad_kernel: the weight derivatives as products over the
//      chunk's pairs, dW_l = sum_p delta_l,p h_{l-1},p^T, on the matrix cores;
//      each block takes one layer and its own range of units into its own
//      partial sums, which are added in a fixed order at the end.
// The network is evaluated transposed (features along the registers, pairs
// along the lanes), so a result has to change places to become an operand of
// a product over pairs: the matrix cores do that exactly, as a product of the
// activation with a 0/1 matrix (two products per 32 x 32 tile).
#pragma once
#include "kcommon.hpp"

namespace voila {

namespace {

constexpr int kW = 256, kHT = kW / 32;  // hidden width, 32-row tiles of a hidden layer
constexpr int kArr = 16384;             // bytes of one stored array per unit (256 features x 32 pairs)
constexpr int kSgn = 1024;              // bytes of the sign pattern of h_3 per unit

// The sequence of fragments of a pair-unit: forward layers 0..2, then the
// reverse layers 3 (W_3^T) and 4 (W_2^T), each produced one 32-row output
// tile (PT = 1, one pass) at a time: layer, pass, k-step, tile of the pass.
template <int IN_KS>
struct PairSeq {
    static constexpr int HT = kHT, PT = 1, NP = HT / PT, HKS = 16, NL = 5, NQ = NL * NP;
    static constexpr int NF0 = IN_KS * HT, NFH = HKS * HT, NFR = NF0 + (NL - 1) * NFH;
    __host__ __device__ static constexpr int layer(int f) { return f < NF0 ? 0 : 1 + (f - NF0) / NFH; }
    __host__ __device__ static constexpr int ks(int f) { return f < NF0 ? IN_KS : HKS; }
    __host__ __device__ static constexpr int rel(int f) { return f < NF0 ? f : (f - NF0) % NFH; }
    __host__ __device__ static constexpr int pass(int f) { return rel(f) / (ks(f) * PT); }
    __host__ __device__ static constexpr int kstep(int f) { return (rel(f) / PT) % ks(f); }
    __host__ __device__ static constexpr int tile(int f) { return rel(f) % PT; }
    __host__ __device__ static constexpr int gpass(int f) { return layer(f) * NP + pass(f); }
    __host__ __device__ static constexpr int pass_len(int q) { return (q < NP ? IN_KS : HKS) * PT; }
    __host__ __device__ static constexpr int pass_start(int q) {
        return q < NP ? q * IN_KS * PT : NF0 + (q / NP - 1) * NFH + (q % NP) * HKS * PT;
    }
};
// The fragment stream: chunks of 64 KB in two LDS buffers shared by the four
// waves, as the rollout kernel's (StreamSrc).  This kernel also stores as it
// goes, and a wave's vector-memory operations complete in order, so the loads
// of the next chunk are issued over the first half of a chunk and its boundary
// waits for them alone: the stores issued after the last of them (counted at
// compile time by Stores::in_step over the later steps, whose order scheduling
// barriers fix) may still be on their way.
template <class S, int PF, class Stores>
struct PairStream {
    static constexpr int CHB = 65536, FPC = CHB / 1024, NCH = cdiv(S::NFR, FPC), kWaves = 4;
    static constexpr int ROUNDS = FPC / kWaves, LDS_BYTES = 2 * CHB;
    char* lds;
    const char* lsrc;  // this lane's 16-byte slot of this wave's first 1 KB round
    int cur = 1;
    const char* win;
    __device__ __forceinline__ PairStream(char* l, const char* s)
        : lds(l),
          lsrc(s + (size_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * 1024 + (threadIdx.x & 63) * 16), win(l) {}
    __device__ __forceinline__ void round(int ch, int buf, int r) const {
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        __builtin_amdgcn_global_load_lds(
            (const void*)(lsrc + opaque_u32((uint32_t)(ch * CHB + r * kWaves * 1024))),
            (__attribute__((address_space(3))) void*)(lds + buf * CHB + (r * kWaves + wave) * 1024), 16, 0, 0);
    }
    __device__ __forceinline__ void start() const {
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) round(0, 0, r);
    }
    static constexpr int served(int ch) { return ch == NCH - 1 ? S::NFR - ch * FPC : FPC; }
    // position within chunk ch of round r of the next chunk's loads
    static constexpr int round_at(int ch, int r) { return r * (served(ch) / 2) / ROUNDS; }
    // stores that are certainly issued between the last load of chunk ch and
    // its first fragment (read PF steps before it is multiplied)
    static constexpr int stores_after(int ch) {
        if (ch == 0) return 0;  // another pair-unit's end lies between
        int n = 0;
        for (int f = (ch - 1) * FPC + round_at(ch - 1, ROUNDS - 1) - PF + 1; f < ch * FPC - PF; ++f)
            if (f >= 0) n += Stores::in_step(f);
        return n < 63 ? n : 63;
    }
    template <int F>
    __device__ __forceinline__ bf16x8 load(int lane) {
        constexpr int ch = F / FPC, within = F % FPC;
        if constexpr (within == 0) {
            __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(stores_after(ch)));
            __builtin_amdgcn_s_barrier();
            cur ^= 1;
        }
        static_for<ROUNDS>([&](auto ri) {
            constexpr int r = decltype(ri)::value;
            if constexpr (round_at(ch, r) == within) round((ch + 1) % NCH, cur ^ 1, r);
        });
        if constexpr (within % 32 == 0) win = lds + cur * CHB + opaque_zero();
        return reinterpret_cast<const bf16x8*>(win)[within * 64 + lane];
    }
    __device__ __forceinline__ void finish() { __builtin_amdgcn_s_waitcnt(0); }
};

// 1 KB (16 bytes per lane) or 256 bytes (4 per lane, from the lane's own
// address) straight into LDS.
__device__ __forceinline__ void load16(const void* src, char* dst, int lane) {
    __builtin_amdgcn_global_load_lds((const void*)((const char*)src + (uint32_t)lane * 16),
                                     (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
}
__device__ __forceinline__ void load4(const float* lane_src, char* dst) {
    __builtin_amdgcn_global_load_lds((const void*)lane_src, (__attribute__((address_space(3))) void*)dst, 4, 0, 0);
}

__device__ __forceinline__ uint32_t bf16x2_of(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){a, b}, bf16x2));
}
// 1 in each 16-bit half whose (non-negative) bfloat16 value is not zero, and
// all ones in each half that holds 1 (one packed instruction each, spelled out:
// the compiler turns the same arithmetic into compares and selects per half).
__device__ __forceinline__ uint32_t ones16(uint32_t v) {
    uint32_t r;
    asm("v_pk_min_u16 %0, %1, %2" : "=v"(r) : "v"(v), "s"(0x00010001u));
    return r;
}
__device__ __forceinline__ uint32_t spread16(uint32_t ones) {
    uint32_t r;
    asm("v_pk_sub_i16 %0, 0, %1" : "=v"(r) : "v"(ones));
    return r;
}
__device__ __forceinline__ float bf_lo(uint32_t v) { return __uint_as_float(v << 16); }
__device__ __forceinline__ float bf_hi(uint32_t v) { return __uint_as_float(v & 0xffff0000u); }
__device__ __forceinline__ bf16x8 frag_of(const uint32_t (&w)[4]) {
    return __builtin_bit_cast(bf16x8, (u32x4){w[0], w[1], w[2], w[3]});
}
__device__ __forceinline__ uint32_t word_of(const bf16x8& v, int j) { return __builtin_bit_cast(u32x4, v)[j]; }
__device__ __forceinline__ void set_word(bf16x8& v, int j, uint32_t w) {
    u32x4 u = __builtin_bit_cast(u32x4, v);
    u[j] = w;
    v = __builtin_bit_cast(bf16x8, u);
}

}  // namespace

}  // namespace voila
