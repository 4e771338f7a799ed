// Simulated quantum annealing (Sec. III, "SQA": discrete-time path-integral
// Monte Carlo of the transverse-field Ising model over P Trotter slices, the
// Suzuki-Trotter mapping of Martonak, Santoro and Tosatti, PRB 66, 094203).
//
// One workgroup per read.  LDS holds the position-ordered instance (as the
// general SA body does; read from global memory instead when it
// does not fit beside the slices), the acceptance rows of this sweep and the
// next (beta_t / P) and the read's P slices as P/4 words per site: slice
// k = 2m + parity lives in word parity * P/8 + m/4, byte m % 4, so a word holds
// four slices of one parity.  A sweep visits the colour classes in order and,
// inside a class, the even-slice words and then the odd-slice words: every
// update in such a pass reads only words the pass does not write (the
// neighbouring sites of the class are in other classes, the neighbouring slices
// have the other parity), and one Philox block serves the four slices of a word.
//
// Update of slice k at site i: g = f_i(s^k) - Jp_t (s^{k-1}_i + s^{k+1}_i) over
// the slice ring, x = -s g, accepted iff x <= 0 or every nonzero base-512 digit
// of x passes its threshold; the random words are Philox(i, t, quad, 6 << 24 |
// digit)[byte], quad = read * P/4 + word.  After the last sweep the read's
// sample is its lowest-energy slice (ties: lowest k).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device.hpp"
#include "internal.hpp"
#include "lds_shadow.hpp"
#include "sa_core.hpp"
#include "swar_core.hpp"

namespace spv {

namespace {

constexpr uint32_t kTagSqa = 6u;

struct SqaArgs {
    const int32_t *image;
    const uint32_t *tables;  // [sweeps][row_len], thresholds for beta_t / P
    const int32_t *jp;       // [sweeps] inter-slice coupling, integer units
    int8_t *out;             // [reads][n]
    int64_t *energies;       // [reads]
    int n, D, C, row_len, sweeps, reads, P, x_bound;
    uint32_t k0, k1;
};

// Bound by VALU issue: about 170 instructions a word of four slices on one-digit sweeps.
// Capping the registers at 64 (a fourth workgroup a CU) spilled and was slower, 5.20
// against 4.82 ms on Chimera 8 x 8, 1000 reads x 500 sweeps.
// BIG: the instance stays in the global image (position-major records), LDS holds
// the acceptance rows and the slices only.  DK: records per site fixed at compile time
// (LDS instance in site blocks; 0: D at run time).
template <int ND, bool BIG = false, int DK = 0>
__global__ __launch_bounds__(1024) void sqa_kernel(SqaArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int cs[kMaxColours + 1];
    __shared__ int best_s;
    __shared__ long long bestE_s;
    constexpr bool SITE = DK == kSiteRecs;
    static_assert(DK == 0 || !BIG, "compile-time record counts are of the LDS instance");
    constexpr bool FEW = DK > 0 && !SITE;  // records neighbour-major, as when D is known at run time only
    constexpr int SH = core::field_shift<ND>;
    const int n = a.n, D = a.D, P = a.P, qw = P / 4, G8 = P / 8, T = blockDim.x, tid = threadIdx.x;
    const int read = blockIdx.x;
    core::SaItem it;
    it.image = a.image;
    it.n = n;
    it.D = D;
    it.C = a.C;
    core::SaLds L;
    if constexpr (BIG) {
        core::sa_big_layout(n, a.row_len, qw, &L, smem);
        core::sa_bind_image(&L, it, cs);  // ends with a barrier
    } else {
        core::sa_layout(n, D, a.row_len, qw, &L, smem);
        core::sa_load_instance<SITE ? DK : 0>(L, it, cs);  // ends with a barrier
    }
    // record k of position p: nbr[p * rec_p + k * rec_k]
    const size_t rec_p = SITE ? (size_t)(DK + 2) : BIG ? (size_t)D : 1, rec_k = (BIG || SITE) ? 1 : (size_t)n;
    auto bias = [&](int p) __attribute__((always_inline)) -> int32_t {
        return SITE ? (int32_t)L.nbr[p * (DK + 2) + DK] : L.hpos[p];
    };
    auto index = [&](int p) __attribute__((always_inline)) -> uint32_t {
        return SITE ? L.nbr[p * (DK + 2) + DK + 1] : (uint32_t)L.ord[p];
    };
    const uint32_t quad0 = (uint32_t)read * (uint32_t)qw;
    for (int k = tid; a.sweeps > 0 && k < a.row_len; k += T) L.tab[k] = a.tables[k];  // none uploaded without sweeps
    for (int k = tid; k < 4 * qw; k += T) L.E2[k] = 0ull;
    // Initial slices: replica r = read * P + parity * P/2 + m, i.e. quad quad0 + word.
    for (int idx = tid; idx < n * qw; idx += T) {
        const int p = idx / qw, w = idx - p * qw;
        const dev::Words4 r = dev::philox(index(p), 0u, quad0 + (uint32_t)w, 1u << 24, a.k0, a.k1);
        uint32_t word = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b) word |= ((r.w[b] >> 31) ? 0x01u : 0xFFu) << (8 * b);
        L.S[idx] = word;
    }
    __syncthreads();

    const int q = tid % G8, slot = tid / G8, nslots = T / G8;
    const bool active = slot < nslots;
    uint32_t s_addr = core::swar_lds_addr(L.S);
    const uint32_t s_row = 4u * (uint32_t)qw;
    // (few records: their loop is short enough for an address stepped per read to show, so a
    // site's addresses are taken from one opaque base instead)
#ifdef __OPTIMIZE__
    if constexpr (FEW) asm volatile("" : "+s"(s_addr));
#endif
    // Race-detection build: each (class, parity) pass's slice-word writes, then its
    // reads (the ring neighbours' words of the other parity and the classical
    // neighbours' words), against the LDS bitmap.
    const shadow::Pass sh = shadow::begin((uint32_t)n * (uint32_t)qw);
    auto shadow_pass = [&](int c, int par, bool before) {
        const int pe = cs[c + 1], w = par * G8 + q;
        const int wa = par ? q : G8 + q;
        const int wb = par ? (q + 1 == G8 ? 0 : q + 1) : G8 + (q == 0 ? G8 - 1 : q - 1);
        if (before) {
            for (int p = cs[c] + slot; active && p < pe; p += nslots) shadow::mark(sh, (uint32_t)(p * qw + w));
            shadow::barrier();
            for (int p = cs[c] + slot; active && p < pe; p += nslots) {
                shadow::check(sh, (uint32_t)(p * qw + wa));
                shadow::check(sh, (uint32_t)(p * qw + wb));
                for (int k = 0; k < D; ++k) {
                    const uint32_t rec = L.nbr[(size_t)p * rec_p + (size_t)k * rec_k];
                    if ((rec & 0xffffu) != 0u) shadow::check(sh, (rec >> 16) * (uint32_t)qw + (uint32_t)w);
                }
            }
            shadow::count_pass(sh);
        } else {
            for (int p = cs[c] + slot; active && p < pe; p += nslots) shadow::unmark(sh, (uint32_t)(p * qw + w));
            shadow::barrier();
        }
    };
    int32_t jp_next = a.sweeps > 0 ? a.jp[0] : 0;  // loaded a sweep ahead, like the acceptance row
    for (int ls = 0; ls < a.sweeps; ++ls) {
        const uint32_t t = (uint32_t)ls;
        const int32_t jp = __builtin_amdgcn_readfirstlane(jp_next);
        if (ls + 1 < a.sweeps) jp_next = a.jp[ls + 1];
        // digits that |x| <= x_bound + 2 Jp can have in this sweep
        const int64_t xmax = (int64_t)a.x_bound + 2 * (int64_t)jp;
        int ndt = 1;
        while (ndt < ND && (xmax >> (kDigitBits * ndt)) != 0) ++ndt;
        const uint32_t *tcur = L.tab + (ls & 1) * a.row_len;
        uint32_t *tnext = L.tab + ((ls + 1) & 1) * a.row_len;
        const int next_len = ls + 1 < a.sweeps ? a.row_len : 0;
        uint32_t nrow[core::kRowRegs];
        core::row_load(a.tables + (size_t)(ls + 1) * a.row_len, tnext, next_len, nrow);
        // The ring neighbours are two more neighbours with coupling -Jp, as one pair of
        // int16 lanes while Jp fits (else a multiplication apart).
        const bool jp16 = jp <= 32767;
        const uint32_t jpp = ((uint32_t)(-jp) & 0xffffu) * 0x10001u;
        for (int c = 0; c < a.C; ++c) {
            const int pe = cs[c + 1];
#pragma unroll 1
            for (int par = 0; par < 2; ++par) {
                if constexpr (shadow::kOn) shadow_pass(c, par, true);
                const int w = par * G8 + q;
                // words of the other parity holding slices k - 1 and k + 1
                const int wa = par ? q : G8 + q;
                const int wb = par ? (q + 1 == G8 ? 0 : q + 1) : G8 + (q == 0 ? G8 - 1 : q - 1);
                for (int p = cs[c] + slot; active && p < pe; p += nslots) {
                    const uint32_t row = s_addr + __umul24((uint32_t)p, s_row);
                    auto word = [&](int v) __attribute__((always_inline)) -> uint32_t {
                        return FEW ? core::swar_ld32(row + 4u * (uint32_t)v) : L.S[(size_t)p * qw + v];
                    };
                    const uint32_t self = word(w), A = word(wa), B = word(wb);
                    // even word: k-1 = odd slice m-1 (A byte b-1, or B byte 3), k+1 = odd slice m (A byte b);
                    // odd word: k-1 = even slice m (A byte b), k+1 = even slice m+1 (A byte b+1, or B byte 0)
                    const uint32_t up = par ? A : __builtin_amdgcn_alignbyte(A, B, 3);
                    const uint32_t dn = par ? __builtin_amdgcn_alignbyte(B, A, 1) : A;
                    int32_t f[4], hv;
                    uint32_t ord;
                    auto start = [&]() __attribute__((always_inline)) {
#pragma unroll
                        for (int b = 0; b < 4; ++b) f[b] = SH ? hv << SH : 0;
                        if (jp16) dev::pair_dot(up, dn, jpp, f);
                    };
                    if constexpr (SITE) {
                        const core::Site<DK> site = core::load_site(L.nbr, p);
                        hv = site.h;
                        ord = site.ord;
                        start();
                        core::neighbour_sum(site.r, s_addr + 4u * (uint32_t)w, s_row, f);
                    } else {
                        hv = L.hpos[p];
                        ord = (uint32_t)L.ord[p];
                        start();
                        if constexpr (FEW) {
                            uint32_t r[DK];
#pragma unroll
                            for (int k = 0; k < DK; ++k) r[k] = L.nbr[(uint32_t)p + (uint32_t)k * (uint32_t)n];
                            core::neighbour_sum(r, s_addr + 4u * (uint32_t)w, s_row, f);
                        } else {
                            core::neighbour_sum_any(L.nbr + p * rec_p, rec_k, D, s_addr + 4u * (uint32_t)w, s_row, f);
                        }
                    }
                    if constexpr (SH == 0)
#pragma unroll
                        for (int b = 0; b < 4; ++b) f[b] = hv + (f[b] >> 8);
                    if (!jp16)  // full 32-bit products: Jp <= 2^24 (below 2^17 where the shift is 8)
#pragma unroll
                        for (int b = 0; b < 4; ++b)
                            f[b] -= (jp * (dev::spin_of(up, b) + dev::spin_of(dn, b))) << SH;
                    int32_t x[4];
#pragma unroll
                    for (int b = 0; b < 4; ++b) x[b] = core::flip_cost(self, b, f[b]);
                    const uint32_t mask = core::metropolis_mask<ND>(x, tcur, ord, t, quad0 + (uint32_t)w, a.k0, a.k1,
                                                                    kTagSqa << 24, ndt);
                    if constexpr (FEW) {
                        if (mask) core::swar_st32(row + 4u * (uint32_t)w, self ^ mask);
                    } else {
                        if (mask) L.S[(size_t)p * qw + w] = self ^ mask;
                    }
                }
                if (c + 1 == a.C && par == 1) core::row_store(tnext, next_len, nrow);
                __syncthreads();
                if constexpr (shadow::kOn) shadow_pass(c, par, false);
            }
        }
    }

    // Classical energy of every slice: 2E = sum_p s_p (h_p + f_p).
    {
        for (int idx = tid; idx < n * qw; idx += T) {
            const int p = idx / qw, w = idx - p * qw;
            const uint32_t self = L.S[idx];
            const int32_t hv = bias(p);
            const core::Fields F = core::local_fields(L.nbr + p * rec_p, L.S, D, qw, w, hv, rec_k);
#pragma unroll
            for (int b = 0; b < 4; ++b)
                atomicAdd(&L.E2[w * 4 + b],
                          (unsigned long long)((long long)dev::spin_of(self, b) * ((long long)hv + F.f[b])));
        }
    }
    __syncthreads();
    if (tid == 0) {
        int best = 0;
        long long bestE = 0;
        for (int k = 0; k < P; ++k) {
            const int m = k >> 1, w = (k & 1) * G8 + (m >> 2), b = m & 3;
            const long long E = ((long long)L.E2[w * 4 + b]) / 2;
            if (k == 0 || E < bestE) {
                bestE = E;
                best = k;
            }
        }
        best_s = best;
        bestE_s = bestE;
    }
    __syncthreads();
    const int best = best_s, m = best >> 1, bw = (best & 1) * G8 + (m >> 2), bb = m & 3;
    if (tid == 0) a.energies[read] = bestE_s;
    const int32_t *pos_of = a.image + kImgHeader + n;
    const unsigned char *Sb = reinterpret_cast<const unsigned char *>(L.S);
    for (int i = tid; i < n; i += T)
        a.out[(size_t)read * n + i] = (int8_t)Sb[((size_t)pos_of[i] * qw + bw) * 4 + bb];
}

}  // namespace

size_t sqa_lds_bytes(int n, int D, int row_len, int P, bool big) {
    return big ? core::sa_big_layout(n, row_len, P / 4, nullptr, nullptr)
               : core::sa_layout(n, D, row_len, P / 4, nullptr, nullptr);
}

hipError_t launch_sqa(const SqaLaunch &L, hipStream_t s) {
    SqaArgs a;
    a.image = L.image;
    a.tables = L.tables;
    a.jp = L.jp;
    a.out = L.out;
    a.energies = L.energies;
    a.n = L.n;
    a.D = L.D;
    a.C = L.C;
    a.row_len = L.row_len;
    a.sweeps = L.sweeps;
    a.reads = L.reads;
    a.P = L.P;
    a.x_bound = L.x_bound;
    a.k0 = (uint32_t)L.seed;
    a.k1 = (uint32_t)(L.seed >> 32);
    const size_t lds = sqa_lds_bytes(L.n, L.D, L.row_len, L.P, L.global_instance);
    if (L.P % 8 != 0 || L.P < 8 || L.threads % (L.P / 8) != 0 || L.reads < 1) return hipErrorInvalidValue;
#define SPV_SQA_GO(...) hipLaunchKernelGGL((sqa_kernel<__VA_ARGS__>), dim3(L.reads), dim3(L.threads), lds, s, a)
    // The record counts with straight-line loops: six (cubes, Chimera graphs; 500 sweeps of 1000
    // reads on Chimera 8 x 8 4.8 ms, D at run time 5.5), and one to three, where the run-time loop
    // costs as much as the records (n = 200, two records, 64 slices x 300 reads x 100 sweeps: 1.06
    // ms, D at run time 1.15).
#define SPV_SQA(ND_)                                                                                  \
    do {                                                                                              \
        if (L.global_instance)                                                                        \
            SPV_SQA_GO(ND_, true);                                                                    \
        else if (L.D == kSiteRecs)                                                                    \
            SPV_SQA_GO(ND_, false, kSiteRecs);                                                        \
        else if (L.D == 1)                                                                            \
            SPV_SQA_GO(ND_, false, 1);                                                                \
        else if (L.D == 2)                                                                            \
            SPV_SQA_GO(ND_, false, 2);                                                                \
        else if (L.D == 3)                                                                            \
            SPV_SQA_GO(ND_, false, 3);                                                                \
        else                                                                                          \
            SPV_SQA_GO(ND_);                                                                          \
    } while (0)
    switch (L.nd) {
        case 1:
            SPV_SQA(1);
            break;
        case 2:
            SPV_SQA(2);
            break;
        case 3:
            SPV_SQA(3);
            break;
        default:
            return hipErrorInvalidValue;
    }
#undef SPV_SQA
#undef SPV_SQA_GO
    return hipGetLastError();
}

hipError_t shadow_stats_sqa(unsigned long long *out, bool reset) { return shadow::read_stats(out, reset); }

}  // namespace spv
