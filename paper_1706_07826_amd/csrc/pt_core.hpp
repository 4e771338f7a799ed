// Device helpers shared by the tempering kernels: lane masks, wavefront sums
// and the replica-exchange acceptance test.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "device.hpp"
#include "internal.hpp"
#include "sa_core.hpp"

namespace spv {
namespace ptc {

__device__ __forceinline__ unsigned long long lanemask_lt() {
    const int l = dev::lane_id();
    return l == 0 ? 0ull : ((~0ull) >> (64 - l));
}

__device__ __forceinline__ long long wave_sum(long long v) {
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    return v;
}

// Xor mask (0xFE per accepted byte) of the Metropolis decisions for x[b] = -s f of
// four replicas at their own temperatures (acceptance rows tb[b]), x scaled by
// 2^field_shift<ND>: a byte is accepted
// iff every nonzero digit of x passes (x <= 0 has none).  The first digit's block is
// drawn without a branch (some byte of a word almost always has a nonzero first
// digit), so the decisions stay lane masks; a later digit's block is drawn where
// some byte has that digit nonzero (a byte already rejected stays rejected).
template <int ND>
__device__ __forceinline__ uint32_t metropolis_mask4(const int32_t x[4], const uint32_t *const tb[4], uint32_t i,
                                                     uint32_t t, uint32_t quad, uint32_t k0, uint32_t k1) {
    constexpr int SH = core::field_shift<ND>;
    uint32_t xp[4], d[4], th[4], mask = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        xp[b] = (uint32_t)max(x[b], 0);
        d[b] = (xp[b] >> SH) & (kDigitSize - 1);
        th[b] = tb[b][d[b]];  // a zero digit reads a valid entry it ignores
    }
    {
        const dev::Words4 w = dev::philox(i, t, quad, 2u << 24, k0, k1);
#pragma unroll
        for (int b = 0; b < 4; ++b)
            if ((d[b] == 0) | (w.w[b] < th[b])) mask |= 0xFEu << (8 * b);
    }
#pragma unroll
    for (int j = 1; j < ND; ++j) {
        bool need = false;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            d[b] = (xp[b] >> (SH + kDigitBits * j)) & (kDigitSize - 1);
            need |= d[b] != 0;
            th[b] = tb[b][j * kDigitSize + d[b]];
        }
        if (need) {
            const dev::Words4 w = dev::philox(i, t, quad, (2u << 24) | (uint32_t)j, k0, k1);
#pragma unroll
            for (int b = 0; b < 4; ++b)
                if ((d[b] != 0) & (w.w[b] >= th[b])) mask &= ~(0xFEu << (8 * b));
        }
    }
    return mask;
}

// Replica-exchange decision (digit test of D with the tables of dbeta_k), in three
// steps: the thresholds of every nonzero digit are fetched together, the random words
// drawn, then compared.
struct SwapTest {
    uint32_t d[7], th[7];
    bool never;  // D beyond the tables
};

__device__ __forceinline__ SwapTest swap_load(long long D, const uint32_t *__restrict__ T, int nd) {
    SwapTest s;
    s.never = D > 0 && nd < 7 && (D >> (kDigitBits * nd)) != 0;
    const bool draw = D > 0 && !s.never;
#pragma unroll
    for (int j = 0; j < 7; ++j) {
        s.d[j] = draw && j < nd ? (uint32_t)((D >> (kDigitBits * j)) & (kDigitSize - 1)) : 0u;
        s.th[j] = s.d[j] ? T[j * kDigitSize + s.d[j]] : 0u;
    }
    return s;
}

__device__ __forceinline__ void swap_draw(int nd, uint32_t k, uint32_t t, uint32_t c, uint32_t k0, uint32_t k1,
                                          dev::Words4 &w0, dev::Words4 &w1) {
    w0 = dev::philox(k, t, c, 3u << 24, k0, k1);
    w1 = w0;
    if (nd > 4) w1 = dev::philox(k, t, c, (3u << 24) | 1u, k0, k1);
}

__device__ __forceinline__ bool swap_accept(const SwapTest &s, const dev::Words4 &w0, const dev::Words4 &w1) {
    bool ok = !s.never;
#pragma unroll
    for (int j = 0; j < 7; ++j) {
        const uint32_t w = j < 4 ? w0.w[j] : w1.w[j - 4];
        if (s.d[j]) ok = ok && (w < s.th[j]);
    }
    return ok;
}

__device__ inline bool swap_test(long long D, const uint32_t *__restrict__ T, int nd, uint32_t k, uint32_t t,
                                 uint32_t c, uint32_t k0, uint32_t k1) {
    if (D <= 0) return true;
    if (nd < 7 && (D >> (kDigitBits * nd)) != 0) return false;
    const SwapTest s = swap_load(D, T, nd);
    dev::Words4 w0, w1;
    swap_draw(nd, k, t, c, k0, k1, w0, w1);
    return swap_accept(s, w0, w1);
}

// Neighbour records are fetched this many at a time when their count is only known at
// run time, so their loads (LDS or global) are in flight together; even, so they pair up.
constexpr int kRecBatch = 4;

// 256 times the neighbour sums of NB replicas, bytes b0 .. b0 + NB - 1 of word q of
// position p (spins S[pos][nq], records rec(k, p) = pos << 16 | uint16 J), added to acc.
// DK > 0: exactly DK records per site (straight-line code); DK = 0: D at run time.
template <int DK, int NB = 4, typename Rec>
__device__ __forceinline__ void quad_sums(Rec rec, int D, int p, const uint32_t *__restrict__ S, int nq, int q,
                                          int32_t (&acc)[NB], int b0 = 0) {
    const uint32_t sa = core::swar_lds_addr(S) + 4u * (uint32_t)q, row = 4u * (uint32_t)nq;
    if constexpr (DK > 0) {
        uint32_t rr[DK];
#pragma unroll
        for (int u = 0; u < DK; ++u) rr[u] = rec(u, p);
        core::neighbour_sum<DK, NB>(rr, sa, row, acc, b0);
        return;
    }
    int k0 = 0;
    for (; k0 + kRecBatch <= D; k0 += kRecBatch) {
        uint32_t rr[kRecBatch];
#pragma unroll
        for (int u = 0; u < kRecBatch; ++u) rr[u] = rec(k0 + u, p);
        core::neighbour_sum<kRecBatch, NB>(rr, sa, row, acc, b0);
    }
    if (k0 + 2 <= D) {
        const uint32_t rr[2] = {rec(k0, p), rec(k0 + 1, p)};
        core::neighbour_sum<2, NB>(rr, sa, row, acc, b0);
        k0 += 2;
    }
    if (k0 < D) {
        const uint32_t rr[1] = {rec(k0, p)};
        core::neighbour_sum<1, NB>(rr, sa, row, acc, b0);
    }
}

// Local fields f[b] = h + sum_k J_k s_k[b] of the 4 replicas in word q of position p.
template <int DK = 0, typename Rec>
__device__ __forceinline__ void quad_fields(Rec rec, int D, int p, const uint32_t *__restrict__ S, int nq, int q,
                                            int32_t h, int32_t f[4]) {
    int32_t acc[4] = {0, 0, 0, 0};
    quad_sums<DK>(rec, D, p, S, nq, q, acc);
#pragma unroll
    for (int b = 0; b < 4; ++b) f[b] = h + (acc[b] >> 8);
}

// Flip costs x[i] = -s f of NB replicas, bytes b0 .. of the word `self`, scaled by
// 2^field_shift<ND>.
template <int ND, int DK, int NB = 4, typename Rec>
__device__ __forceinline__ void quad_costs(Rec rec, int D, int p, const uint32_t *__restrict__ S, int nq, int q,
                                           int32_t h, uint32_t self, int32_t (&x)[NB], int b0 = 0) {
    constexpr int SH = core::field_shift<ND>;
    int32_t f[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) f[i] = SH ? h << SH : 0;
    quad_sums<DK, NB>(rec, D, p, S, nq, q, f, b0);
#pragma unroll
    for (int i = 0; i < NB; ++i) x[i] = core::flip_cost(self, b0 + i, SH ? f[i] : h + (f[i] >> 8));
}

// Energy change of an accepted flip added to `sum`, which is kept scaled like x.
__device__ __forceinline__ void add_flip(long long &sum, int32_t x, uint32_t taken) {
    sum += (long long)x * (long long)(int32_t)taken;
}

// Lock-free union-find in LDS over 16-bit parents.  parent[x] < x for every x that is no
// root, so a chain strictly decreases, every find terminates and a root is the smallest
// member of its tree.  A root is only ever hooked under a smaller node, which therefore lies
// in another tree (uf_union hooks it under that tree's root, the join scan's first hook under
// any member).  Path splitting writes only ancestors, so concurrent finds stay valid.
__device__ __forceinline__ uint32_t uf_find(uint16_t *parent, uint32_t x) {
    uint32_t p = parent[x];
    while (p != x) {
        const uint32_t gp = parent[p];
        if (gp != p) parent[x] = (uint16_t)gp;
        x = p;
        p = gp;
    }
    return x;
}

// Compare-and-swap of one 16-bit half through a 32-bit CAS on its word; fails
// only when the half no longer holds `expect`.
__device__ __forceinline__ bool cas16(uint16_t *addr, uint32_t expect, uint32_t desired) {
    uint32_t *word = reinterpret_cast<uint32_t *>(reinterpret_cast<uintptr_t>(addr) & ~(uintptr_t)3);
    const int sh = (reinterpret_cast<uintptr_t>(addr) & 2) ? 16 : 0;
    uint32_t old = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    for (;;) {
        if (((old >> sh) & 0xffffu) != expect) return false;
        const uint32_t want = (old & ~(0xffffu << sh)) | (desired << sh);
        const uint32_t prev = atomicCAS(word, old, want);
        if (prev == old) return true;
        old = prev;
    }
}

__device__ __forceinline__ void uf_union(uint16_t *parent, uint32_t a, uint32_t b) {
    for (;;) {
        a = uf_find(parent, a);
        b = uf_find(parent, b);
        if (a == b) return;
        if (a > b) {
            const uint32_t t = a;
            a = b;
            b = t;
        }
        if (cas16(&parent[b], b, a)) return;
    }
}

}  // namespace ptc
}  // namespace spv
