// Device-side building blocks: counter-based Philox4x32-10 and wavefront/block scans.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace spv {
namespace dev {

// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, "Parallel random numbers: as easy
// as 1, 2, 3", SC'11): ten rounds of the Philox S-box -- two 32x32->64
// multiplications by the published multipliers, the high halves xored with
// the other two counter words and the round key -- with a Weyl key schedule.
// The key and the high counter words are usually wavefront-uniform, so the
// key schedule stays in scalar registers.
struct Words4 {
    uint32_t w[4];
};

// Rounds [first, first + N) on the counter words in place, keys (k0, k1) of round 0.
template <int N>
__device__ __forceinline__ void philox_rounds(uint32_t (&c)[4], int first, uint32_t k0, uint32_t k1) {
    constexpr uint32_t kMulA = 0xD2511F53u, kMulB = 0xCD9E8D57u;
    constexpr uint32_t kWeylA = 0x9E3779B9u, kWeylB = 0xBB67AE85u;
    k0 += kWeylA * (uint32_t)first;
    k1 += kWeylB * (uint32_t)first;
#pragma unroll
    for (int round = 0; round < N; ++round) {
        const uint64_t pa = (uint64_t)kMulA * c[0];
        const uint64_t pb = (uint64_t)kMulB * c[2];
        // three-input xor in one gfx950 v_bitop3_b32 (truth table 0x96)
        const uint32_t n0 = __builtin_amdgcn_bitop3_b32((uint32_t)(pb >> 32), c[1], k0, 0x96);
        const uint32_t n2 = __builtin_amdgcn_bitop3_b32((uint32_t)(pa >> 32), c[3], k1, 0x96);
        c[1] = (uint32_t)pb;
        c[3] = (uint32_t)pa;
        c[0] = n0;
        c[2] = n2;
        k0 += kWeylA;
        k1 += kWeylB;
    }
}

__device__ __forceinline__ Words4 philox(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                         uint32_t k0, uint32_t k1) {
    uint32_t c[4] = {c0, c1, c2, c3};
    philox_rounds<10>(c, 0, k0, k1);
    Words4 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) r.w[i] = c[i];
    return r;
}

// Signed byte b (0..3) of a packed word of four int8 spins.
__device__ __forceinline__ int32_t spin_of(uint32_t w, int b) {
    return ((int32_t)(w << (24 - 8 * b))) >> 24;
}

typedef short i16x2 __attribute__((ext_vector_type(2)));

// Two records' couplings (low halves) as one pair of int16 lanes.
__device__ __forceinline__ uint32_t j_pair(uint32_t rec0, uint32_t rec1) {
    return __builtin_amdgcn_perm(rec1, rec0, 0x05040100u);
}

// acc[i] += 256 (J0 s0 + J1 s1) for NB replicas (bytes b0 .. of two neighbour words,
// signed bytes): v_perm_b32 puts the two spin bytes of a replica into the high bytes of
// two int16 lanes (+-256, no sign extension needed) and v_dot2_i32_i16 multiplies them
// with the coupling pair, so a neighbour costs one instruction per replica instead of a
// byte extraction and a multiply-add.  |acc| <= 256 * 64 * 32767 < 2^30.
// The general bodies are bound by VALU issue (and latency where few workgroups run);
// with this, straight-line records and acceptance rows loaded a sweep ahead, measured
// before -> after: SA on the Gaussian L = 10 cube, 1000 reads x 1000 sweeps, 2.90 -> 2.14
// ms; L = 20, 498 reads x 200 sweeps from global memory, 3.30 -> 2.60 ms; SQA on Chimera
// 8 x 8, 16 slices x 1000 reads x 500 sweeps, 5.52 -> 4.78 ms.
template <int NB>
__device__ __forceinline__ void pair_dot(uint32_t w0, uint32_t w1, uint32_t jj, int32_t (&acc)[NB], int b0 = 0) {
    const i16x2 j = __builtin_bit_cast(i16x2, jj);
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const uint32_t s = __builtin_amdgcn_perm(w1, w0, 0x040C000Cu + 0x01000100u * (uint32_t)(b0 + i));
        acc[i] = __builtin_amdgcn_sdot2(__builtin_bit_cast(i16x2, s), j, acc[i], false);
    }
}

// base + (rec >> 16) * mul for 16-bit factors, in one instruction (the high half of
// the record is selected by op_sel).
__device__ __forceinline__ uint32_t hi16_mad(uint32_t rec, uint32_t mul, uint32_t base) {
    uint32_t r;
    asm("v_mad_u32_u16 %0, %1, %2, %3 op_sel:[1,0,0,0]" : "=v"(r) : "v"(rec), "v"(mul), "v"(base));
    return r;
}

// Lane index inside the 64-wide wavefront.
__device__ __forceinline__ int lane_id() { return __lane_id(); }

// Exclusive prefix count of `flag` over the lanes below this one.
__device__ __forceinline__ int wave_prefix(bool flag, unsigned long long *total) {
    const unsigned long long m = __ballot(flag);
    *total = m;
    const int l = lane_id();
    const unsigned long long below = (l == 0) ? 0ull : (m & ((~0ull) >> (64 - l)));
    return __popcll(below);
}

// Block-wide exclusive scan of small non-negative integers.  `tmp` holds
// blockDim/64 + 1 ints of LDS.  Returns the prefix; *sum receives the total.
__device__ __forceinline__ int block_exclusive_scan(int v, int *tmp, int *sum) {
    const int lane = lane_id();
    const int wid = threadIdx.x >> 6;
    const int nw = (blockDim.x + 63) >> 6;
    int x = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        int y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    if (lane == 63 || threadIdx.x == blockDim.x - 1) tmp[wid] = x;
    __syncthreads();
    if (threadIdx.x == 0) {
        int acc = 0;
        for (int w = 0; w < nw; ++w) {
            int t = tmp[w];
            tmp[w] = acc;
            acc += t;
        }
        tmp[nw] = acc;
    }
    __syncthreads();
    int r = tmp[wid] + x - v;
    *sum = tmp[nw];
    __syncthreads();
    return r;
}

}  // namespace dev
}  // namespace spv
