// Device body of the simulated-annealing sweep, shared by the one-instance
// launch (sa.hip) and the batched persistent launch (batch.hip).
//
// Sampler (Sec. III.A, "SA"): every read starts from its own Philox state (or
// a caller state) and performs one Metropolis sweep per entry of the beta
// schedule; the sample is the final state of every read.  A sweep visits the
// colour classes in order; a class is an independent set, so all of its spins
// are updated in parallel with the same result as any sequential order.
//
// LDS holds the position-ordered instance (ELL records: neighbour position <<
// 16 | int16 coupling), two threshold rows (current sweep and next sweep) and
// the spins as S[p][q]: one 32-bit word per (position, quad of 4 replicas), a
// signed byte per replica.  A thread keeps one quad q for the whole schedule;
// for each position it forms the four local fields, draws one Philox block
// that serves the four replicas and applies the integer threshold test.
#pragma once

#include <hip/hip_runtime.h>

#include "device.hpp"
#include "lds_shadow.hpp"
#include "internal.hpp"

namespace spv {
namespace core {

typedef unsigned int swar_v2u __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) const uint32_t swar_lds_u32;
typedef __attribute__((address_space(3))) const swar_v2u swar_lds_v2u;

// The 32-bit LDS address of a shared-memory object.
__device__ __forceinline__ uint32_t swar_lds_addr(const void *p) {
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void *)p;
}
__device__ __forceinline__ uint32_t swar_ld32(uint32_t a) { return *(swar_lds_u32 *)(uintptr_t)a; }
__device__ __forceinline__ void swar_st32(uint32_t a, uint32_t v) {
    *(__attribute__((address_space(3))) uint32_t *)(uintptr_t)a = v;
}
__device__ __forceinline__ uint2 swar_ld64(uint32_t a) {
    const swar_v2u v = *(swar_lds_v2u *)(uintptr_t)a;
    return make_uint2(v.x, v.y);
}

struct SaLds {
    uint32_t *nbr;
    int32_t *hpos;
    int32_t *ord;
    uint32_t *tab;  // [2][row_len]
    uint32_t *S;    // [n][qw]
    unsigned long long *E2;  // [4*qw]
};

// LDS layout for n positions, D records each, quads `qw` (spin capacity n*qw
// words) and energy accumulators for e2q quads (0: qw).
__host__ __device__ inline size_t sa_layout(int n, int D, int row_len, int qw, SaLds *L,
                                            unsigned char *base, int e2q = 0) {
    if (e2q < qw) e2q = qw;
    size_t o_nbr = 0;
    size_t o_h = o_nbr + (size_t)n * D * 4;
    size_t o_ord = o_h + (size_t)n * 4;
    size_t o_tab = o_ord + (size_t)n * 4;
    size_t o_S = o_tab + (size_t)2 * row_len * 4;
    size_t o_E = (o_S + (size_t)n * qw * 4 + 7) & ~(size_t)7;
    size_t end = o_E + (size_t)4 * e2q * 8;
    if (L) {
        L->nbr = reinterpret_cast<uint32_t *>(base + o_nbr);
        L->hpos = reinterpret_cast<int32_t *>(base + o_h);
        L->ord = reinterpret_cast<int32_t *>(base + o_ord);
        L->tab = reinterpret_cast<uint32_t *>(base + o_tab);
        L->S = reinterpret_cast<uint32_t *>(base + o_S);
        L->E2 = reinterpret_cast<unsigned long long *>(base + o_E);
    }
    return end;
}

// Layout when the instance stays in global memory (too large for the LDS beside
// the spins): LDS holds the two threshold rows, the spins and the accumulators.
__host__ __device__ inline size_t sa_big_layout(int n, int row_len, int qw, SaLds *L,
                                                unsigned char *base) {
    size_t o_tab = 0;
    size_t o_S = o_tab + (size_t)2 * row_len * 4;
    size_t o_E = (o_S + (size_t)n * qw * 4 + 7) & ~(size_t)7;
    size_t end = o_E + (size_t)4 * qw * 8;
    if (L) {
        L->nbr = nullptr;
        L->hpos = nullptr;
        L->ord = nullptr;
        L->tab = reinterpret_cast<uint32_t *>(base + o_tab);
        L->S = reinterpret_cast<uint32_t *>(base + o_S);
        L->E2 = reinterpret_cast<unsigned long long *>(base + o_E);
    }
    return end;
}

// One schedule over quads [q0, q0 + qw) of one instance.
struct SaItem {
    const int32_t *image;
    const uint32_t *tables;  // [sweeps][row_len]
    const int8_t *init;      // [reads][n] or null
    int8_t *out;             // [reads][n]
    int64_t *energies;       // [reads]
    int n, D, C, row_len, sweeps, reads, q0, qw;
    uint32_t sweep_offset, k0, k1;
    int wpl = 1;  // byte-parallel body: quad words per lane (1, or 2 when qw = 2)
    unsigned char *big = nullptr;  // byte-parallel body: instance in global memory (too large for LDS)
};

// Neighbour records of a site are read this many at a time when their count is only known
// at run time (loads issued together); even, so records pair up.
constexpr int kFieldBatch = 4;

// acc[i] += 256 sum_k J_k s_k for NB replicas (bytes b0 .. of a word): DK records in
// registers, `sa` the LDS byte address of the word of position 0, `row` the bytes between
// positions.  All word loads are in flight together.
template <int DK, int NB>
__device__ __forceinline__ void neighbour_sum(const uint32_t (&r)[DK], uint32_t sa, uint32_t row, int32_t (&acc)[NB],
                                              int b0 = 0) {
    uint32_t w[DK];
#pragma unroll
    for (int k = 0; k < DK; ++k) w[k] = swar_ld32(dev::hi16_mad(r[k], row, sa));
#pragma unroll
    for (int k = 0; k + 1 < DK; k += 2) dev::pair_dot(w[k], w[k + 1], dev::j_pair(r[k], r[k + 1]), acc, b0);
    if constexpr (DK & 1) dev::pair_dot(w[DK - 1], 0u, r[DK - 1] & 0xffffu, acc, b0);
}

// The same with D known at run time; record k is nb[k * stride].
__device__ __forceinline__ void neighbour_sum_any(const uint32_t *__restrict__ nb, size_t stride, int D, uint32_t sa,
                                                  uint32_t row, int32_t (&acc)[4]) {
    int k0 = 0;
    for (; k0 + kFieldBatch <= D; k0 += kFieldBatch) {
        uint32_t r[kFieldBatch];
#pragma unroll
        for (int u = 0; u < kFieldBatch; ++u) r[u] = nb[(k0 + u) * stride];
        neighbour_sum(r, sa, row, acc);
    }
    // (a pair left over stays a pair: with two records a site, SQA over 32 slices lost 9 % by it)
    if (k0 + 2 <= D) {
        const uint32_t r[2] = {nb[k0 * stride], nb[(k0 + 1) * stride]};
        neighbour_sum(r, sa, row, acc);
        k0 += 2;
    }
    if (k0 < D) {
        const uint32_t r[1] = {nb[k0 * stride]};
        neighbour_sum(r, sa, row, acc);
    }
}

struct Fields {
    int32_t f[4];
};

// f_b = h_p + sum_k J_k s_kb, records at run-time count (nb as above, word q of S[n][qw]).
__device__ __forceinline__ Fields local_fields(const uint32_t *__restrict__ nb, const uint32_t *__restrict__ S, int D,
                                               int qw, int q, int32_t hv, size_t stride) {
    int32_t acc[4] = {0, 0, 0, 0};
    neighbour_sum_any(nb, stride, D, swar_lds_addr(S) + 4u * (uint32_t)q, 4u * (uint32_t)qw, acc);
    Fields F;
#pragma unroll
    for (int b = 0; b < 4; ++b) F.f[b] = hv + (acc[b] >> 8);
    return F;
}

// Fields of the update loop are scaled by 2^field_shift(ND): up to two digits |256 f|
// fits 26 bits, so the sums keep pair_dot's factor 256 and the digits are cut out 8
// bits higher, which saves the shift; three digits need the plain value.
template <int ND>
constexpr int field_shift = ND <= 2 ? 8 : 0;

// Records, bias and variable index of one site.
template <int DK>
struct Site {
    uint32_t r[DK];
    int32_t h;
    uint32_t ord;
};

// A site block of the LDS instance with six records per site (cubes and Chimera graphs):
// {6 records, bias, index}, 32 bytes, two 16-byte reads from one address.
__device__ __forceinline__ Site<kSiteRecs> load_site(const uint32_t *__restrict__ blocks, int p) {
    const uint4 *b = reinterpret_cast<const uint4 *>(blocks) + 2 * (uint32_t)p;
    const uint4 u = b[0], v = b[1];
    Site<kSiteRecs> s;
    s.r[0] = u.x;
    s.r[1] = u.y;
    s.r[2] = u.z;
    s.r[3] = u.w;
    s.r[4] = v.x;
    s.r[5] = v.y;
    s.h = (int32_t)v.z;
    s.ord = v.w;
    return s;
}

// x = -s f of byte b of `self` (s = +-1).
__device__ __forceinline__ int32_t flip_cost(uint32_t self, int b, int32_t f) {
    const int32_t m = __builtin_amdgcn_sbfe((int32_t)~self, 8u * (uint32_t)b + 7u, 1u);  // -1 where s = +1
    return (f ^ m) - m;
}

// Xor mask (0xFE per accepted byte) of the Metropolis decisions for x[b] = -s f, given
// scaled by 2^field_shift<ND>; digits from ndt on are zero for every x of this sweep
// (ndt is wave-uniform).  A byte is accepted iff every nonzero digit of x passes its
// threshold (x <= 0 has none).  The first digit's block is drawn without a branch (some
// byte of a word almost always has a nonzero first digit), so the decisions stay lane
// masks; a later digit's block is drawn where some byte has that digit nonzero (a byte
// already rejected stays rejected, so testing it again changes nothing).  Thresholds
// are loaded for every byte (a zero digit reads a valid entry it ignores), so the four
// LDS reads overlap the Philox block.  `tag`: the draws' fourth counter word.
template <int ND>
__device__ __forceinline__ uint32_t metropolis_mask(const int32_t x[4], const uint32_t *tab, uint32_t i, uint32_t t,
                                                    uint32_t quad, uint32_t k0, uint32_t k1, uint32_t tag = 2u << 24,
                                                    int ndt = ND) {
    constexpr int SH = field_shift<ND>;
    uint32_t xp[4], d[4], th[4], mask = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        xp[b] = (uint32_t)max(x[b], 0);
        d[b] = (xp[b] >> SH) & (kDigitSize - 1);
        th[b] = tab[d[b]];
    }
    {
        const dev::Words4 w = dev::philox(i, t, quad, tag, k0, k1);
#pragma unroll
        for (int b = 0; b < 4; ++b)
            if ((d[b] == 0) | (w.w[b] < th[b])) mask |= 0xFEu << (8 * b);
    }
#pragma unroll
    for (int j = 1; j < ND; ++j) {
        if (j >= ndt) break;
        bool need = false;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            d[b] = (xp[b] >> (SH + kDigitBits * j)) & (kDigitSize - 1);
            need |= d[b] != 0;
            th[b] = tab[j * kDigitSize + d[b]];
        }
        if (need) {
            const dev::Words4 w = dev::philox(i, t, quad, tag | (uint32_t)j, k0, k1);
#pragma unroll
            for (int b = 0; b < 4; ++b)
                if ((d[b] != 0) & (w.w[b] >= th[b])) mask &= ~(0xFEu << (8 * b));
        }
    }
    return mask;
}

// The next sweep's acceptance row is loaded at the start of a sweep into N registers a
// thread and stored to its LDS buffer before the sweep's last barrier, so that no sweep
// waits for the load (what a narrow workgroup cannot hold goes straight to LDS).
// len = 0: no next sweep.
constexpr int kRowRegs = 2;
template <int N>
__device__ __forceinline__ void row_load(const uint32_t *__restrict__ src, uint32_t *dst, int len, uint32_t (&reg)[N]) {
    const int T = blockDim.x, tid = threadIdx.x;
#pragma unroll
    for (int u = 0; u < N; ++u) reg[u] = tid + u * T < len ? src[tid + u * T] : 0u;
    for (int k = tid + N * T; k < len; k += T) dst[k] = src[k];
}
template <int N>
__device__ __forceinline__ void row_store(uint32_t *dst, int len, const uint32_t (&reg)[N]) {
    const int T = blockDim.x, tid = threadIdx.x;
#pragma unroll
    for (int u = 0; u < N; ++u)
        if (tid + u * T < len) dst[tid + u * T] = reg[u];
}

// Points the instance fields at the image in global memory (records position-major:
// record k of position p at nbr[p * D + k]) and loads the colour-class starts.
// Ends with a barrier.
__device__ inline void sa_bind_image(SaLds *L, const SaItem &a, int *cs) {
    const int32_t *img = a.image;
    const int n = a.n;
    if ((int)threadIdx.x <= a.C) cs[threadIdx.x] = img[3 + threadIdx.x];
    L->ord = const_cast<int32_t *>(img + kImgHeader);
    L->hpos = const_cast<int32_t *>(img + kImgHeader + 2 * n);
    L->nbr = reinterpret_cast<uint32_t *>(const_cast<int32_t *>(img + kImgHeader + 3 * n));
    __syncthreads();
}

// Copies the instance image into LDS: site blocks when DK = kSiteRecs, else ELL records
// neighbour-major, biases and order.  Ends with a barrier.
template <int DK = 0>
__device__ inline void sa_load_instance(const SaLds &L, const SaItem &a, int *cs) {
    const int n = a.n, D = a.D, T = blockDim.x, tid = threadIdx.x;
    const int32_t *img = a.image;
    if (tid <= a.C) cs[tid] = img[3 + tid];
    const uint32_t *recs = reinterpret_cast<const uint32_t *>(img + kImgHeader + 3 * n);
    if constexpr (DK == kSiteRecs) {
        constexpr int W = kSiteRecs + 2;  // the block takes what the records, bias and index of a site take apart
        for (int idx = tid; idx < n * kSiteRecs; idx += T) {
            const int p = idx / kSiteRecs, k = idx - p * kSiteRecs;
            L.nbr[p * W + k] = recs[idx];
        }
        for (int k = tid; k < n; k += T) {
            L.nbr[k * W + kSiteRecs] = (uint32_t)img[kImgHeader + 2 * n + k];
            L.nbr[k * W + kSiteRecs + 1] = (uint32_t)img[kImgHeader + k];
        }
        __syncthreads();
        return;
    }
    for (int idx = tid; idx < n * D; idx += T) {  // neighbour-major in LDS: nbr[k][p]
        const int p = idx / D, k = idx - p * D;
        L.nbr[(size_t)k * n + p] = recs[idx];
    }
    for (int k = tid; k < n; k += T) {
        L.hpos[k] = img[kImgHeader + 2 * n + k];
        L.ord[k] = img[kImgHeader + k];
    }
    __syncthreads();
}

// The whole schedule for quads [q0, q0+qw) of an instance resident in LDS (loaded by
// sa_load_instance<DK>), or in global memory when BIG (the image's position-major
// records).  DK: records per site fixed at compile time (0: D at run time).
// Starts and ends with a barrier, so LDS can be reused by the caller.
template <int ND, bool BIG = false, int DK = 0>
__device__ void sa_run(const SaLds &L, const SaItem &a, const int *cs) {
    constexpr bool SITE = !BIG && DK == kSiteRecs;
    static_assert(BIG || DK == 0 || SITE, "the LDS instance has site blocks for kSiteRecs records only");
    constexpr int SH = field_shift<ND>;
    const int n = a.n, D = a.D, qw = a.qw, T = blockDim.x, tid = threadIdx.x;
    const int q0 = a.q0;
    const size_t rec_p = SITE ? (size_t)(DK + 2) : BIG ? (size_t)D : 1, rec_k = (BIG || SITE) ? 1 : (size_t)n;
    const int q = tid % qw, slot = tid / qw, nslots = T / qw;
    const bool active = slot < nslots;
    const uint32_t s_addr = swar_lds_addr(L.S) + 4u * (uint32_t)q, s_row = 4u * (uint32_t)qw;
    auto bias = [&](int p) __attribute__((always_inline)) -> int32_t {
        return SITE ? (int32_t)L.nbr[p * (DK + 2) + DK] : L.hpos[p];
    };
    auto index = [&](int p) __attribute__((always_inline)) -> uint32_t {
        return SITE ? L.nbr[p * (DK + 2) + DK + 1] : (uint32_t)L.ord[p];
    };
    // (no sweeps: no table was uploaded, so none is read)
    for (int k = tid; a.sweeps > 0 && k < a.row_len; k += T) L.tab[k] = a.tables[k];
    for (int k = tid; k < 4 * qw; k += T) L.E2[k] = 0ull;
    // Initial state.
    if (a.init == nullptr) {
        for (int p = slot; active && p < n; p += nslots) {
            const dev::Words4 w =
                dev::philox(index(p), 0u, (uint32_t)(q0 + q), 1u << 24, a.k0, a.k1);
            uint32_t word = 0;
#pragma unroll
            for (int b = 0; b < 4; ++b) word |= ((w.w[b] >> 31) ? 0x01u : 0xFFu) << (8 * b);
            L.S[(size_t)p * qw + q] = word;
        }
    } else {
        const int32_t *pos_of = a.image + kImgHeader + n;
        unsigned char *Sb = reinterpret_cast<unsigned char *>(L.S);
        for (int idx = tid; idx < 4 * qw * n; idx += T) {
            const int rl = idx / n, i = idx - rl * n;
            const int r = 4 * q0 + rl;
            int8_t v = 1;
            if (r < a.reads) v = a.init[(size_t)r * n + i] > 0 ? 1 : -1;
            const int p = pos_of[i];
            Sb[((size_t)p * qw + (rl >> 2)) * 4 + (rl & 3)] = (unsigned char)v;
        }
    }
    __syncthreads();
    const shadow::Pass sh = shadow::begin((uint32_t)n * (uint32_t)qw);
    // Debug build: the class pass's writes, then its neighbour reads, against the bitmap.
    auto shadow_pass = [&](int c, bool before) {
        const int pe = cs[c + 1];
        if (before) {
            for (int p = cs[c] + slot; active && p < pe; p += nslots) shadow::mark(sh, (uint32_t)(p * qw + q));
            shadow::barrier();
            for (int p = cs[c] + slot; active && p < pe; p += nslots)
                for (int k = 0; k < D; ++k) {
                    const uint32_t r = L.nbr[(size_t)p * rec_p + (size_t)k * rec_k];
                    if ((r & 0xffffu) == 0u) continue;  // padding or J = 0: the value read is unused
                    shadow::check(sh, (r >> 16) * (uint32_t)qw + (uint32_t)q);
                }
            shadow::count_pass(sh);
        } else {
            for (int p = cs[c] + slot; active && p < pe; p += nslots) shadow::unmark(sh, (uint32_t)(p * qw + q));
            shadow::barrier();
        }
    };

    for (int ls = 0; ls < a.sweeps; ++ls) {
        const uint32_t t = a.sweep_offset + (uint32_t)ls;
        const uint32_t *tcur = L.tab + (ls & 1) * a.row_len;
        uint32_t *tnext = L.tab + ((ls + 1) & 1) * a.row_len;
        const int next_len = ls + 1 < a.sweeps ? a.row_len : 0;
        uint32_t row[kRowRegs];
        row_load(a.tables + (size_t)(ls + 1) * a.row_len, tnext, next_len, row);
        // One word: its fields, four costs scaled by 2^SH, the digit tests.
        auto decide = [&](int p, uint32_t self, const int32_t f[4], uint32_t ord) __attribute__((always_inline)) {
            int32_t x[4];
#pragma unroll
            for (int b = 0; b < 4; ++b) x[b] = flip_cost(self, b, f[b]);
            const uint32_t mask = metropolis_mask<ND>(x, tcur, ord, t, (uint32_t)(q0 + q), a.k0, a.k1);
            if (mask) L.S[(size_t)p * qw + q] = self ^ mask;
        };
        auto update = [&](int p, const auto &site) __attribute__((always_inline)) {
            const uint32_t self = L.S[(size_t)p * qw + q];
            int32_t f[4];
#pragma unroll
            for (int b = 0; b < 4; ++b) f[b] = SH ? site.h << SH : 0;
            neighbour_sum(site.r, s_addr, s_row, f);
            if constexpr (SH == 0)
#pragma unroll
                for (int b = 0; b < 4; ++b) f[b] = site.h + (f[b] >> 8);
            decide(p, self, f, site.ord);
        };
        for (int c = 0; c < a.C; ++c) {
            if constexpr (shadow::kOn) shadow_pass(c, true);
            const int pe = cs[c + 1];
            if constexpr (SITE) {
                for (int p = cs[c] + slot; active && p < pe; p += nslots) update(p, load_site(L.nbr, p));
            } else if constexpr (BIG && DK > 0) {
                // The next site's records, bias and index are in flight while one is updated.
                auto fetch = [&](int p) __attribute__((always_inline)) {
                    Site<DK> s;
#pragma unroll
                    for (int k = 0; k < DK; ++k) s.r[k] = L.nbr[(size_t)p * DK + k];
                    s.h = L.hpos[p];
                    s.ord = (uint32_t)L.ord[p];
                    return s;
                };
                int p = cs[c] + slot;
                if (active && p < pe) {
                    Site<DK> next = fetch(p);
                    for (; p < pe; p += nslots) {
                        const Site<DK> cur = next;
                        if (p + nslots < pe) next = fetch(p + nslots);
                        update(p, cur);
                    }
                }
            } else {
                for (int p = cs[c] + slot; active && p < pe; p += nslots) {
                    const uint32_t self = L.S[(size_t)p * qw + q];
                    int32_t f[4];
                    const int32_t hv = L.hpos[p];
#pragma unroll
                    for (int b = 0; b < 4; ++b) f[b] = SH ? hv << SH : 0;
                    neighbour_sum_any(L.nbr + p * rec_p, rec_k, D, s_addr, s_row, f);
                    if constexpr (SH == 0)
#pragma unroll
                        for (int b = 0; b < 4; ++b) f[b] = hv + (f[b] >> 8);
                    decide(p, self, f, (uint32_t)L.ord[p]);
                }
            }
            if (c + 1 == a.C) row_store(tnext, next_len, row);
            __syncthreads();
            if constexpr (shadow::kOn) shadow_pass(c, false);
        }
    }

    // Energies: 2E = sum_p s_p (h_p + f_p) per replica.
    {
        long long e2[4] = {0, 0, 0, 0};
        for (int p = slot; active && p < n; p += nslots) {
            const uint32_t self = L.S[(size_t)p * qw + q];
            const int32_t hv = bias(p);
            const Fields F = local_fields(L.nbr + p * rec_p, L.S, D, qw, q, hv, rec_k);
#pragma unroll
            for (int b = 0; b < 4; ++b) e2[b] += (long long)dev::spin_of(self, b) * ((long long)hv + F.f[b]);
        }
        if (active)
#pragma unroll
            for (int b = 0; b < 4; ++b) atomicAdd(&L.E2[q * 4 + b], (unsigned long long)e2[b]);
    }
    __syncthreads();
    for (int rl = tid; rl < 4 * qw; rl += T) {
        const int r = 4 * q0 + rl;
        if (r < a.reads) a.energies[r] = ((long long)L.E2[rl]) / 2;
    }
    // Spins, transposed back to [read][variable] in original variable order.
    const int32_t *pos_of = a.image + kImgHeader + n;
    const unsigned char *Sb = reinterpret_cast<const unsigned char *>(L.S);
    for (int idx = tid; idx < 4 * qw * n; idx += T) {
        const int rl = idx / n, i = idx - rl * n;
        const int r = 4 * q0 + rl;
        if (r < a.reads) {
            const int p = pos_of[i];
            a.out[(size_t)r * n + i] = (int8_t)Sb[((size_t)p * qw + (rl >> 2)) * 4 + (rl & 3)];
        }
    }
    __syncthreads();
}

}  // namespace core
}  // namespace spv
