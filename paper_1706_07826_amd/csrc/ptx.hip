// Parallel tempering with each run's ladder split over several workgroups
// (Sec. III.D.1 "PTICM" at sizes where one run does not fit one workgroup, or
// where there are too few runs to fill the device).
//
// A run's K slots are cut into G groups of m consecutive slots, m a multiple
// of 4 (every quad of 4 replicas of the replica index r = (run * chains +
// chain) * K + slot lies inside one group), or m = 2 or 1 (a group owns half
// or a quarter of its quad: it draws the quad's whole random block and updates
// its own bytes; the other bytes of its LDS copy are never changed or read out).
// When K is no multiple of 4 the quads of a chain start at another slot in every
// (run, chain), so a group holds every quad its slots of a chain touch and owns
// some of their bytes, at an offset of the chain's own (26 slots x 2 chains x 8 runs of
// the L = 6 cube with cluster moves, 300 sweeps: 54.3 ms in one workgroup a run, 5.2 ms
// as 26 groups of one slot).
// A group of one slot reading its instance from the global image keeps both
// chains' bytes of that slot in one word per site (byte c: chain c), each byte
// drawing from its own chain's quad block.
// Workgroup (run, g) holds the group's slots of EVERY chain, so the Houdayer
// partners (chain 0 and chain 1 at one slot) share its LDS.  A sweep is
//   1. Metropolis on the group's replicas (colour classes in order),
//   2. replica exchange of pairs (k, k+1), k = t mod 2.  Pairs inside the
//      group are decided from LDS energies and swapped within a site's words; a pair that
//      straddles a group boundary (on odd sweeps when m is even; the lower and
//      the upper boundary on alternate sweeps when m = 1) is decided by both
//      neighbours from the energies each publishes (with the edge
//      configuration) as sweep-tagged atomic words; an accepted pair copies
//      the partner's published configuration in,
//   3. Houdayer moves at the group's slots, up to four slot pairs at a time
//      with the whole workgroup (lock-free union-find over the disagreeing
//      sites; with one pair, the join scan also gathers each disagreeing
//      site's energy term, so the energy pass needs no neighbour reads),
//   4. the top-10 offers of the group's colder slots.
// The instance lives in LDS when it fits beside the replicas; otherwise the
// neighbour records, biases and orderings are read from the global image
// (shared by every workgroup, L2-resident).
//
// Waits for a neighbour's words are bounded: a workgroup whose neighbour does
// not publish within the spin limit stops and marks its lists with
// top_count = -1, or, when K is no multiple of 4, its run, which the one-workgroup
// kernel then runs again.  The host only launches grids that fit on the device at once.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "device.hpp"
#include "internal.hpp"
#include "lds_shadow.hpp"
#include "pt_core.hpp"

namespace spv {

namespace {

using ptc::lanemask_lt;
using ptc::swap_test;
using ptc::wave_sum;

struct PtxArgs {
    const int32_t *image;
    const uint32_t *mtab;  // [K][row_len]
    const uint32_t *stab;  // [K-1][7*512]
    const int32_t *snd;    // [K-1]
    int8_t *final_spins;
    long long *final_E;
    int8_t *top_spins;
    long long *top_E;
    int32_t *top_count;
    int8_t *tops;          // [runs][Ls][10][n], position order
    uint32_t *xw;          // [runs][G][side 2][buf 2][chains][xmsg] tagged boundary messages; before
                           // them, from xw[-1] down, a mark per run with an abandoned wait (K % 4 != 0)
    PtResume rs;           // checkpoint to start from
    int n, D, C, K, chains, sweeps, row_len, icm_lo, icm_hi, nw_icm, G, m, xmsg, esum;
    uint32_t sweep_offset, k0, k1;
    unsigned spin_limit;
};

struct PtxLds {
    uint32_t *nbr;      // [D][n]   (LDS-resident instance)
    int32_t *hpos;      // [n]      (LDS-resident instance)
    int32_t *ord;       // [n]      (LDS-resident instance)
    int32_t *pos;       // [n]      (LDS-resident instance)
    uint32_t *tab;      // [m][row_len]
    uint32_t *S;        // [n][nq]
    unsigned char *Sb;
    long long *E;       // [chains*m]
    long long *LE;      // [chains*m][10]
    int32_t *Lwhen;     // [chains*m][10]
    int32_t *Lcnt;      // [chains*m]
    int32_t *Lbad;      // [chains*m] checkpoint count was outside 0..10
    int32_t *Lord;      // [chains*m][10]
    int32_t *Lins;      // [chains*m] entry a list's offer replaces this sweep (-1: none)
    long long *Lmax;    // [chains*m] a full list's largest energy (LLONG_MAX: not known)
    int32_t *snd;       // [m + 1] digit counts of the swap tables of pairs s0-1 .. s0+m-1
    int32_t *acc;       // [nq <= chains*m] per word: bytes that take their successor (bits 0-3), predecessor (4-7)
    int32_t *cin;       // [2*chains] accepted boundary pairs (side, chain)
    uint16_t *parent;          // [pairs][n rounded to even] union-find forests over positions
    unsigned long long *dmask; // [pairs][ceil(n / 64)] disagreement masks in variable order
    int32_t *misc;             // [4] broadcast scalars
    uint32_t *ubuf;            // [16 waves][kJoinBuf] pending joins: site | neighbour << 16
    unsigned char *ubj;        // [16 waves][kJoinBuf] their slot pair
    int32_t *esite;            // [n] one slot pair's cluster energy terms (esum)
};

// Pending-join buffer per wavefront (64 appended at most on top of < 64 pending).
constexpr int kJoinBuf = 128;

// Quad words a group of m slots holds per chain.  With K a multiple of 4 its slots start on a
// quad's boundary (or lie inside one quad), with K and m even at byte 0 or 2 of a quad, else at
// any byte; a group has no more slots than the ladder.
__host__ __device__ inline int ptx_chain_words(int K, int m) {
    const int last = K % 4 == 0 ? 3 : K % 2 == 0 && m % 2 == 0 ? 5 : 6;  // bytes before the slots, and 3
    return ((m < K ? m : K) + last) / 4;
}
__host__ __device__ inline bool ptx_packed(bool big, int m, int chains) { return big && m == 1 && chains == 2; }

__host__ __device__ inline size_t ptx_layout(int n, int D, int K, int m, int chains, int row_len, int nw_icm, bool big,
                                             bool esum, PtxLds *L, unsigned char *base) {
    const int nq = ptx_packed(big, m, chains) ? 1 : chains * ptx_chain_words(K, m), nl = chains * m,
              vstride = 2 * ((n + 63) / 64);
    size_t o = 0;
    auto take = [&](size_t bytes) {
        size_t at = o;
        o = (o + bytes + 15) & ~(size_t)15;
        return at;
    };
    const size_t in_lds = big ? 0 : 1;
    const size_t o_nbr = take(in_lds * n * D * 4), o_h = take(in_lds * n * 4), o_ord = take(in_lds * n * 4),
                 o_pos = take(in_lds * n * 4), o_tab = take((size_t)m * row_len * 4), o_S = take((size_t)n * nq * 4),
                 o_E = take((size_t)nl * 8), o_LE = take((size_t)nl * 80), o_Lw = take((size_t)nl * 40),
                 o_Lc = take((size_t)nl * 4), o_Lb = take((size_t)nl * 4), o_Lo = take((size_t)nl * 40),
                 o_Li = take((size_t)nl * 4), o_Lm = take((size_t)nl * 8), o_snd = take((size_t)(m + 1) * 4),
                 o_acc = take((size_t)nl * 4),
                 o_cin = take((size_t)2 * chains * 4), o_par = take((size_t)nw_icm * ((n + 1) & ~1) * 2),
                 o_dm = take((size_t)nw_icm * vstride * 4), o_misc = take(16),
                 o_ub = take(nw_icm ? (size_t)16 * kJoinBuf * 4 : 0), o_uj = take(nw_icm ? (size_t)16 * kJoinBuf : 0),
                 o_es = take(esum ? (size_t)n * 4 : 0);
    if (L) {
        L->nbr = reinterpret_cast<uint32_t *>(base + o_nbr);
        L->hpos = reinterpret_cast<int32_t *>(base + o_h);
        L->ord = reinterpret_cast<int32_t *>(base + o_ord);
        L->pos = reinterpret_cast<int32_t *>(base + o_pos);
        L->tab = reinterpret_cast<uint32_t *>(base + o_tab);
        L->S = reinterpret_cast<uint32_t *>(base + o_S);
        L->Sb = base + o_S;
        L->E = reinterpret_cast<long long *>(base + o_E);
        L->LE = reinterpret_cast<long long *>(base + o_LE);
        L->Lwhen = reinterpret_cast<int32_t *>(base + o_Lw);
        L->Lcnt = reinterpret_cast<int32_t *>(base + o_Lc);
        L->Lbad = reinterpret_cast<int32_t *>(base + o_Lb);
        L->Lord = reinterpret_cast<int32_t *>(base + o_Lo);
        L->Lins = reinterpret_cast<int32_t *>(base + o_Li);
        L->Lmax = reinterpret_cast<long long *>(base + o_Lm);
        L->snd = reinterpret_cast<int32_t *>(base + o_snd);
        L->acc = reinterpret_cast<int32_t *>(base + o_acc);
        L->cin = reinterpret_cast<int32_t *>(base + o_cin);
        L->parent = reinterpret_cast<uint16_t *>(base + o_par);
        L->dmask = reinterpret_cast<unsigned long long *>(base + o_dm);
        L->misc = reinterpret_cast<int32_t *>(base + o_misc);
        L->ubuf = reinterpret_cast<uint32_t *>(base + o_ub);
        L->ubj = base + o_uj;
        L->esite = reinterpret_cast<int32_t *>(base + o_es);
    }
    return o;
}

// Slot pairs whose cluster moves run together (one forest and mask set each).
constexpr int kIcmBatch = 4;

__global__ void xw_zero_kernel(uint32_t *w, size_t count) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < count; i += (size_t)gridDim.x * blockDim.x)
        w[i] = 0u;
}

// a byte in LDS, addressed with 32-bit offsets
typedef __attribute__((address_space(3))) const unsigned char lds_u8;
typedef __attribute__((address_space(3))) uint32_t lds_mu32;
typedef __attribute__((address_space(1))) uint32_t glb_u32;
typedef __attribute__((address_space(1))) int32_t glb_i32;

// What a launch's groups do between exchanges, fixed at compile time for the common
// shapes: one kernel with every body in it held 128 registers and spilled 132 bytes (216
// with the instance in global memory), whichever body ran; alone they spill 0 to 76.
// With the 16-bit dot-product fields, before -> after: L = 10 Gaussian cube, 32 slots x
// 64 runs, no moves, 11.8 -> 11.1 ms per 1000 sweeps; L = 20, 40 slots x 2 chains, packed
// single pairs, 18.0 -> 15.5 ms per 300.
enum PtxMove {
    kMoveNone,    // no cluster moves
    kMoveSingle,  // one slot pair at a time, its energy terms gathered in the join scan
    kMovePacked,  // the same, both chains' bytes of the group's slot in one word per site
    kMoveAny      // up to kIcmBatch pairs at a time (or none, or one), decided at run time
};

template <int CTRL>
__device__ __forceinline__ int32_t row_move(int32_t v) {
    return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xF, 0xF, false);
}

// v summed over the rows 0 and 1, 2 and 3 (lane by lane), and over the two halves: a swap
// of a register with its copy leaves one operand of the sum in each.
__device__ __forceinline__ int32_t add_row_pairs(int32_t v) {
    const auto r = __builtin_amdgcn_permlane16_swap((uint32_t)v, (uint32_t)v, false, false);
    return (int32_t)(r[0] + r[1]);
}
__device__ __forceinline__ int32_t add_halves(int32_t v) {
    const auto r = __builtin_amdgcn_permlane32_swap((uint32_t)v, (uint32_t)v, false, false);
    return (int32_t)(r[0] + r[1]);
}

// Every lane of a row of 16 gets the row's entry ordered last by (energy, stamp): a
// butterfly of DPP moves (quads by two permutations, then the two mirrors).
__device__ __forceinline__ void last_of_16(long long &e, int32_t &w, int32_t &i) {
    auto step = [&](auto move) __attribute__((always_inline)) {
        const long long oe = (long long)(((unsigned long long)(uint32_t)move((int32_t)(e >> 32)) << 32) |
                                         (uint32_t)move((int32_t)e));
        const int32_t ow = move(w), oi = move(i);
        if (oe > e || (oe == e && ow > w)) {
            e = oe;
            w = ow;
            i = oi;
        }
    };
    step([](int32_t v) { return row_move<0xB1>(v); });
    step([](int32_t v) { return row_move<0x4E>(v); });
    step([](int32_t v) { return row_move<0x141>(v); });
    step([](int32_t v) { return row_move<0x140>(v); });
}

__device__ __forceinline__ unsigned long long read_first(unsigned long long v) {
    return ((unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32) |
           (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}

// ND threshold digits; BIG: instance read from the global image; DK: records per
// site fixed at compile time (0: D at run time).
template <int ND, bool BIG, int DK, int MV>
__global__ __launch_bounds__(1024) void ptx_kernel(PtxArgs a) {
    constexpr int kBatch = MV == kMoveAny ? kIcmBatch : 1;  // slot pairs of a pass
    // The boundary copy's message words a thread loads together, so that their latencies
    // overlap: an instance in LDS gives a thread one or two sites, one in global memory about
    // eight (L = 10 cube, 32 slots: 10.1 ms per 1000 sweeps, with four 10.2).  kCopySites: a
    // thread takes one site of a message word, or, in a group of one slot, which swaps no
    // pair of its own, both (L = 20, 40 slots x 2 chains, 300 sweeps: 14.7 ms, one 14.9).
    constexpr int kCopySites = MV == kMovePacked ? 2 : 1;
    constexpr int kCopyBatch = (BIG ? 8 : 2) / kCopySites;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int cs[kMaxColours + 1];
    __shared__ int nacc;
    __shared__ int stop;
    const int n = a.n, D = a.D, K = a.K, chains = a.chains, G = a.G, row_len = a.row_len, xmsg = a.xmsg;
    PtxLds Lay;
    ptx_layout(n, D, K, a.m, chains, row_len, a.nw_icm, BIG, a.esum != 0, &Lay, smem);
    // LDS regions as plain locals (keeps the layout record out of scratch memory)
    auto *const L_nbr = Lay.nbr;
    auto *const L_hpos = Lay.hpos;
    auto *const L_ord = Lay.ord;
    auto *const L_pos = Lay.pos;
    auto *const L_tab = Lay.tab;
    auto *const L_S = Lay.S;
    auto *const L_Sb = Lay.Sb;
    auto *const L_E = Lay.E;
    auto *const L_LE = Lay.LE;
    auto *const L_Lwhen = Lay.Lwhen;
    auto *const L_Lcnt = Lay.Lcnt;
    auto *const L_Lbad = Lay.Lbad;
    auto *const L_Lord = Lay.Lord;
    auto *const L_Lins = Lay.Lins;
    auto *const L_Lmax = Lay.Lmax;
    auto *const L_snd = Lay.snd;
    auto *const L_acc = Lay.acc;
    auto *const L_cin = Lay.cin;
    auto *const L_parent = Lay.parent;
    auto *const L_dmask = Lay.dmask;
    auto *const L_misc = Lay.misc;
    auto *const L_ubuf = Lay.ubuf;
    auto *const L_ubj = Lay.ubj;
    auto *const L_es = Lay.esite;
    int tid = threadIdx.x, lane = dev::lane_id(), wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int T = blockDim.x, nw = T >> 6;
    // Thread, lane and wavefront as new values for each phase of a sweep: what a phase
    // derives from them (addresses above all) is not kept in registers, and spilled,
    // across the others.
    auto phase = [&]() __attribute__((always_inline)) {
#ifdef __OPTIMIZE__
        asm volatile("" : "+v"(tid), "+v"(lane));
#endif
        wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    };
    const int run = blockIdx.x / G, g = blockIdx.x - run * G;
    const int s0 = g * a.m, mg = min(a.m, K - s0);
    // byte of its quad word that holds the group's first slot of a chain; with K a
    // multiple of 4 the same in every chain and run, and 0 when m is one too
    const uint32_t r00 = (uint32_t)run * (uint32_t)(chains * K) + (uint32_t)s0;
    auto boff_of = [=](int ch) __attribute__((always_inline)) -> int {
        return (int)((r00 + (uint32_t)(ch * K)) & 3u);
    };
    const int boff = boff_of(0), boff1 = chains > 1 ? boff_of(1) : boff;
    const bool k4 = (K & 3) == 0;
    const int qpc = k4 ? (boff + mg + 3) >> 2 : ptx_chain_words(K, a.m);
    // pk: a group of one slot (cluster moves on, two chains) reading its instance from
    // the global image keeps both chains' bytes of its slot in one word per site,
    // chain c in byte c (with the instance in LDS the layout stays one word per chain)
    const bool pk = MV == kMoveAny ? ptx_packed(BIG, a.m, chains) : MV == kMovePacked;
    const int nq = pk ? 1 : chains * qpc, nl = chains * mg;
    const int32_t *img = a.image;
    // (global address space spelled out: past the opaque copies below the compiler no longer
    // knows it, and a flat load counts as an LDS operation too, so that every wait for an LDS
    // read would wait for the records fetched ahead)
    using ImgI = std::conditional_t<BIG, const glb_i32, const int32_t>;
    using ImgU = std::conditional_t<BIG, const glb_u32, const uint32_t>;
    ImgI *gpos = (ImgI *)(img + kImgHeader + n), *gord = (ImgI *)(img + kImgHeader),
         *ghpos = (ImgI *)(img + kImgHeader + 2 * n);
    ImgU *gnbr = (ImgU *)(img + kImgHeader + 3 * n);
#ifdef __OPTIMIZE__
    // Kept as values of their own: otherwise each use rebuilds them from the whole
    // argument block, which comes back from spill lanes sixteen registers at a time.
    asm volatile("" : "+s"(gnbr), "+s"(gord), "+s"(ghpos));
#endif
    const uint32_t *const lnbr = L_nbr;
    const int32_t *const lhpos = L_hpos, *const lord = L_ord, *const lpos = L_pos;
    unsigned char *const Sb = L_Sb;
    auto NBR = [=](int k, int p) __attribute__((always_inline)) -> uint32_t {
        return BIG ? gnbr[(size_t)p * D + k] : lnbr[(size_t)k * n + p];
    };
    auto HPOS = [=](int p) __attribute__((always_inline)) -> int32_t { return BIG ? ghpos[p] : lhpos[p]; };
    auto ORD = [=](int p) __attribute__((always_inline)) -> int32_t { return BIG ? gord[p] : lord[p]; };
    auto POS = [=](int i) __attribute__((always_inline)) -> int32_t { return BIG ? gpos[i] : lpos[i]; };
    // byte of local replica l = chain * mg + (slot - s0) at position p
    auto sbyte = [=](int l, int p) __attribute__((always_inline)) -> unsigned char * {
        if (pk) return Sb + (size_t)p * 4 + l;
        const int ch = l / mg, o = l - ch * mg + boff_of(ch);
        return Sb + ((size_t)p * nq + ch * qpc + (o >> 2)) * 4 + (o & 3);
    };
    // its byte at position 0 (chain ch, slot s0 + o); a replica's bytes lie pst apart
    auto sbase = [=](int ch, int o) __attribute__((always_inline)) -> unsigned char * {
        if (pk) return Sb + ch;
        const int b = o + boff_of(ch);
        return Sb + (ch * qpc + (b >> 2)) * 4 + (b & 3);
    };
    // x = chain * per + rest, by subtraction (few chains; a division by a run-time value
    // costs some forty instructions, in phases where every instruction is waited for)
    auto chain_of = [](int &x, int per) __attribute__((always_inline)) -> int {
        int ch = 0;
        for (; x >= per; x -= per) ++ch;
        return ch;
    };
    const uint32_t pst = (uint32_t)nq * 4u;

    if (tid <= a.C) cs[tid] = img[3 + tid];
    if (tid == 0) stop = 0;
    if (!BIG) {
        for (int idx = tid; idx < n * D; idx += T) {
            const int p = idx / D, k = idx - p * D;
            L_nbr[(size_t)k * n + p] = gnbr[idx];
        }
        for (int k = tid; k < n; k += T) {
            L_ord[k] = gord[k];
            L_pos[k] = gpos[k];
            L_hpos[k] = ghpos[k];
        }
    }
    for (int k = tid; k < mg * row_len; k += T) L_tab[k] = a.mtab[(size_t)s0 * row_len + k];
    // the swap tables' digit counts of the pairs this group decides, k = s0 - 1 .. s0 + mg - 1
    for (int i = tid; i <= mg; i += T) {
        const int k = s0 - 1 + i;
        L_snd[i] = k >= 0 && k < K - 1 ? a.snd[k] : 0;
    }
    const int half = K / 2, Ls = chains * half;
    // Local slot l = chain * mg + (slot - s0); slots k >= K - half hold list gl.
    auto list_of = [=](int l) __attribute__((always_inline)) -> int {
        const int ch = l / mg, k = s0 + (l - ch * mg);
        return k >= K - half ? ch * half + (k - (K - half)) : -1;
    };
    for (int k = tid; k < nl; k += T) {
        L_E[k] = 0;
        L_Lmax[k] = 0x7FFFFFFFFFFFFFFFll;
        const int gl = list_of(k);
        const int c = (gl >= 0 && a.rs.top_count) ? a.rs.top_count[(size_t)run * Ls + gl] : 0;
        const bool bad = c < 0 || c > 10;
        L_Lcnt[k] = bad ? 0 : c;
        L_Lbad[k] = bad ? 1 : 0;
    }
    __syncthreads();
    if (a.rs.top_count) {
        // Checkpoint entries, inserted before this launch's offers in list order.
        for (int le = tid; le < nl * 10; le += T) {
            const int l = le / 10, e = le - l * 10, gl = list_of(l);
            if (gl >= 0 && e < L_Lcnt[l]) {
                L_LE[le] = a.rs.top_E[((size_t)run * Ls + gl) * 10 + e];
                L_Lwhen[le] = e - 10;
            }
        }
        for (size_t idx = tid; idx < (size_t)nl * 10 * n; idx += T) {
            const int lr = (int)(idx / n), i = (int)(idx - (size_t)lr * n);
            const int l = lr / 10, e = lr - l * 10, gl = list_of(l);
            if (gl >= 0 && e < L_Lcnt[l]) {
                const size_t row = ((size_t)run * Ls + gl) * 10 + e;
                a.tops[row * n + POS(i)] = a.rs.top_spins[row * n + i] > 0 ? (int8_t)1 : (int8_t)-1;
            }
        }
    }

    const int q = tid % nq, pt = tid / nq, nstr = T / nq;
    const bool active = pt < nstr;
    const int chq = q / qpc, jq = q - chq * qpc, boffq = boff_of(chq);
    const uint32_t quad = (uint32_t)((((size_t)run * chains + chq) * K + s0) / 4 + jq);
    // pk: chain 1's quad (byte 1 of the word draws its word boff1 from that quad's block)
    const uint32_t quad1 = (uint32_t)((((size_t)run * chains + 1) * K + s0) / 4);
    auto wsel = [](const dev::Words4 &w, int i) __attribute__((always_inline)) -> uint32_t {
        return i == 0 ? w.w[0] : i == 1 ? w.w[1] : i == 2 ? w.w[2] : w.w[3];
    };
    // byte b of the thread's word is the group's local slot 4 jq + b - boffq; own marks
    // (0xFE) the bytes that are the group's
    int loc[4];
    const uint32_t *tb[4];
    uint32_t own = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const int o = 4 * jq + b - boffq;
        const bool mine = o >= 0 && o < mg;
        own |= mine ? 0xFEu << (8 * b) : 0u;
        loc[b] = chq * mg + (mine ? o : 0);
        tb[b] = L_tab + (size_t)(mine ? o : 0) * row_len;
        if (pk) {
            // byte b < 2: chain b of the group's slot (local replica b), table row 0
            loc[b] = b < 2 ? b : 0;
            tb[b] = L_tab;
        }
    }
    if (pk) own = 0xFEFEu;
    const bool pow2 = (nq & (nq - 1)) == 0 && nq <= 64;
    // the group owns 1 or 2 bytes of each of its words (the same bytes in every word)
    const bool part = !pk && k4 && qpc == 1 && mg < 4;
    const bool owner = active && own != 0;  // (a quad the group's slots of a chain do not reach has nothing to update)

    // Initial state and energies.
    for (int p = pt; active && p < n; p += nstr) {
        const dev::Words4 w = dev::philox((uint32_t)ORD(p), 0u, quad, 1u << 24, a.k0, a.k1);
        uint32_t word = 0;
        if (pk) {
            const dev::Words4 w1 = dev::philox((uint32_t)ORD(p), 0u, quad1, 1u << 24, a.k0, a.k1);
            word = ((wsel(w, boff) >> 31) ? 0x01u : 0xFFu) | (((wsel(w1, boff1) >> 31) ? 0x01u : 0xFFu) << 8) |
                   0x01010000u;
        } else {
#pragma unroll
            for (int b = 0; b < 4; ++b) word |= ((w.w[b] >> 31) ? 0x01u : 0xFFu) << (8 * b);
        }
        L_S[(size_t)p * nq + q] = word;
    }
    __syncthreads();
    if (a.rs.spins) {
        // The group's replicas start from the checkpoint.
        for (int idx = tid; idx < nl * n; idx += T) {
            const int l = idx / n, i = idx - l * n;
            const int ch = l / mg, slot = s0 + (l - ch * mg);
            *sbyte(l, POS(i)) =
                a.rs.spins[(((size_t)run * chains + ch) * K + slot) * n + i] > 0 ? (unsigned char)0x01 : (unsigned char)0xFF;
        }
        __syncthreads();
    }
    {
        long long e2[4] = {0, 0, 0, 0};
        for (int p = pt; active && p < n; p += nstr) {
            const uint32_t self = L_S[(size_t)p * nq + q];
            const int32_t hp = HPOS(p);
            int32_t f[4];
            ptc::quad_fields<DK>(NBR, D, p, L_S, nq, q, hp, f);
#pragma unroll
            for (int b = 0; b < 4; ++b) e2[b] += (long long)dev::spin_of(self, b) * ((long long)hp + f[b]);
        }
        if (active)
#pragma unroll
            for (int b = 0; b < 4; ++b)
                if (own & (0xFEu << (8 * b)))
                    atomicAdd(reinterpret_cast<unsigned long long *>(&L_E[loc[b]]), (unsigned long long)e2[b]);
    }
    __syncthreads();
    for (int l = tid; l < nl; l += T) L_E[l] /= 2;  // sum of s(h + f) counts every coupler twice
    __syncthreads();

    // Race-detection build: each class pass's spin-word writes, then its neighbour
    // reads, against the LDS bitmap (a word is (position, quad)).
    const shadow::Pass sh = shadow::begin((uint32_t)n * (uint32_t)nq);
    auto shadow_pass = [&](int c, bool before) {
        const int pe = cs[c + 1];
        if (before) {
            for (int p = cs[c] + pt; active && p < pe; p += nstr) shadow::mark(sh, (uint32_t)(p * nq + q));
            shadow::barrier();
            for (int p = cs[c] + pt; active && p < pe; p += nstr)
                for (int k = 0; k < D; ++k) {
                    const uint32_t rec = NBR(k, p);
                    if ((rec & 0xffffu) != 0u) shadow::check(sh, (rec >> 16) * (uint32_t)nq + (uint32_t)q);
                }
            shadow::count_pass(sh);
        } else {
            for (int p = cs[c] + pt; active && p < pe; p += nstr) shadow::unmark(sh, (uint32_t)(p * nq + q));
            shadow::barrier();
        }
    };

    // Race-detection build: the words a thread's in-group swaps store, marked for the
    // exchange; a byte stored by another thread into one is a conflict.
    auto shadow_swaps = [&](bool before) {
        for (int p = tid; p < n; p += T)
            for (int w = 0; w < nq; ++w)
                if (L_acc[w]) before ? shadow::mark(sh, (uint32_t)(p * nq + w)) : shadow::unmark(sh, (uint32_t)(p * nq + w));
        if (before) shadow::count_pass(sh);
        shadow::barrier();
    };

    for (int ls = 0; ls < a.sweeps; ++ls) {
        phase();
        const uint32_t t = a.sweep_offset + (uint32_t)ls;
        // 1. Metropolis on the group's replicas (costs and their sums scaled by 2^SH).
        constexpr int SH = core::field_shift<ND>;
        long long dE[4] = {0, 0, 0, 0}, dEp[2] = {0, 0};
        for (int c = 0; c < a.C; ++c) {
            if constexpr (shadow::kOn) shadow_pass(c, true);
            const int pe = cs[c + 1];
            auto update = [&](int p, auto rec, int32_t hp, uint32_t ord) __attribute__((always_inline)) {
                const uint32_t self = L_S[(size_t)p * nq + q];
                int32_t x[4];
                ptc::quad_costs<ND, DK>(rec, D, p, L_S, nq, q, hp, self, x);
                // The key enters each site's draws opaquely: otherwise the twenty round
                // keys are hoisted out of the loop, outgrow the scalar registers and
                // come back one vector-lane read at a time.  (Unoptimised device builds
                // keep it in vector registers, where a scalar operand cannot bind.)
                uint32_t k0 = a.k0, k1 = a.k1;
#ifdef __OPTIMIZE__
                asm volatile("" : "+s"(k0), "+s"(k1));
#endif
                const uint32_t mask = own & ptc::metropolis_mask4<ND>(x, tb, ord, t, quad, k0, k1);
#pragma unroll
                for (int b = 0; b < 4; ++b) ptc::add_flip(dE[b], x[b], (mask >> (8 * b + 1)) & 1u);
                if (mask) L_S[(size_t)p * nq + q] = self ^ mask;
            };
            // A group of 1 or 2 slots owns bytes boff.. of its words: those bytes alone are
            // updated (the quad's random blocks drawn whole, so the draws are the same).
            auto update_part = [&](int p, const uint32_t *rr, int32_t hp, uint32_t ord) __attribute__((always_inline)) {
                const uint32_t self = L_S[(size_t)p * nq + q];
                // bytes b0 and b0 + 1 hold the owned ones (a 1-slot group's other is unused)
                const int b0 = min(boff, 2), o0 = boff - b0;
                int32_t xx[2];
                ptc::quad_costs<ND, DK, 2>([&](int u, int) __attribute__((always_inline)) { return rr[u]; }, D, p, L_S,
                                           nq, q, hp, self, xx, b0);
                uint32_t k0 = a.k0, k1 = a.k1;
#ifdef __OPTIMIZE__
                asm volatile("" : "+s"(k0), "+s"(k1));
#endif
                int32_t x[2];
                uint32_t d[2], th[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    x[i] = xx[min(o0 + i, 1)];
                    d[i] = ((uint32_t)max(x[i], 0) >> SH) & (kDigitSize - 1);
                    th[i] = L_tab[(size_t)min(i, mg - 1) * row_len + d[i]];
                }
                auto pick = [&](const dev::Words4 &w, int i) __attribute__((always_inline)) -> uint32_t {
                    const int bb = min(boff + i, 3);
                    return bb == 0 ? w.w[0] : bb == 1 ? w.w[1] : bb == 2 ? w.w[2] : w.w[3];
                };
                bool acc[2];
                {
                    const dev::Words4 w = dev::philox(ord, t, quad, 2u << 24, k0, k1);
#pragma unroll
                    for (int i = 0; i < 2; ++i) acc[i] = (d[i] == 0) | (pick(w, i) < th[i]);
                }
#pragma unroll
                for (int j = 1; j < ND; ++j) {
                    bool need = false;
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        d[i] = ((uint32_t)max(x[i], 0) >> (SH + kDigitBits * j)) & (kDigitSize - 1);
                        need |= i < mg && d[i] != 0;
                        th[i] = L_tab[(size_t)min(i, mg - 1) * row_len + j * kDigitSize + d[i]];
                    }
                    if (need) {
                        const dev::Words4 w = dev::philox(ord, t, quad, (2u << 24) | (uint32_t)j, k0, k1);
#pragma unroll
                        for (int i = 0; i < 2; ++i)
                            if ((d[i] != 0) & (pick(w, i) >= th[i])) acc[i] = false;
                    }
                }
                uint32_t mask = 0;
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    if (i < mg && acc[i]) {
                        mask |= 0xFEu << (8 * (boff + i));
                        dEp[i] += x[i];
                    }
                if (mask) L_S[(size_t)p * nq + q] = self ^ mask;
            };
            // pk: bytes 0 and 1 of the site's word are chains 0 and 1 of the group's slot;
            // each draws word boff of its own chain's quad block, digit by digit.
            auto update_pk = [&](int p, auto rec, int32_t hp, uint32_t ord) __attribute__((always_inline)) {
                const uint32_t self = L_S[p];
                int32_t x[2];
                ptc::quad_costs<ND, DK, 2>(rec, D, p, L_S, 1, 0, hp, self, x);
                uint32_t k0 = a.k0, k1 = a.k1;
#ifdef __OPTIMIZE__
                asm volatile("" : "+s"(k0), "+s"(k1));
#endif
                uint32_t d[2], th[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    d[i] = ((uint32_t)max(x[i], 0) >> SH) & (kDigitSize - 1);
                    th[i] = L_tab[d[i]];
                }
                bool acc[2];
                {
                    const dev::Words4 w0 = dev::philox(ord, t, quad, 2u << 24, k0, k1);
                    const dev::Words4 w1 = dev::philox(ord, t, quad1, 2u << 24, k0, k1);
                    acc[0] = (d[0] == 0) | (wsel(w0, boff) < th[0]);
                    acc[1] = (d[1] == 0) | (wsel(w1, boff1) < th[1]);
                }
#pragma unroll
                for (int j = 1; j < ND; ++j) {
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        d[i] = ((uint32_t)max(x[i], 0) >> (SH + kDigitBits * j)) & (kDigitSize - 1);
                        th[i] = L_tab[j * kDigitSize + d[i]];
                    }
                    if (d[0] != 0) {
                        const dev::Words4 w = dev::philox(ord, t, quad, (2u << 24) | (uint32_t)j, k0, k1);
                        if (wsel(w, boff) >= th[0]) acc[0] = false;
                    }
                    if (d[1] != 0) {
                        const dev::Words4 w = dev::philox(ord, t, quad1, (2u << 24) | (uint32_t)j, k0, k1);
                        if (wsel(w, boff1) >= th[1]) acc[1] = false;
                    }
                }
                uint32_t mask = 0;
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    if (acc[i]) {
                        mask |= 0xFEu << (8 * i);
                        dEp[i] += x[i];
                    }
                if (mask) L_S[p] = self ^ mask;
            };
            if constexpr (BIG && DK > 0) {
                // Records, h and index of a site come from global memory: those of the
                // thread's next site are in flight while the current one is updated.
                uint32_t rn[DK];
                int32_t hn = 0, on = 0;
                auto fetch = [&](int pp) __attribute__((always_inline)) {
#pragma unroll
                    for (int u = 0; u < DK; ++u) rn[u] = gnbr[(size_t)pp * DK + u];
                    hn = ghpos[pp];
                    on = gord[pp];
                };
                auto sites = [&](auto body) __attribute__((always_inline)) {
                    int p = cs[c] + pt;
                    if (owner && p < pe) fetch(p);
                    for (; owner && p < pe; p += nstr) {
                        uint32_t rr[DK];
#pragma unroll
                        for (int u = 0; u < DK; ++u) rr[u] = rn[u];
                        const int32_t hp = hn, od = on;
                        if (p + nstr < pe) fetch(p + nstr);
                        body(p, rr, hp, (uint32_t)od);
                    }
                };
                if (pk)
                    sites([&](int p, const uint32_t *rr, int32_t hp, uint32_t od) __attribute__((always_inline)) {
                        update_pk(p, [&](int u, int) __attribute__((always_inline)) { return rr[u]; }, hp, od);
                    });
                else if (part)
                    sites([&](int p, const uint32_t *rr, int32_t hp, uint32_t od)
                              __attribute__((always_inline)) { update_part(p, rr, hp, od); });
                else
                    sites([&](int p, const uint32_t *rr, int32_t hp, uint32_t od) __attribute__((always_inline)) {
                        update(p, [&](int u, int) __attribute__((always_inline)) { return rr[u]; }, hp, od);
                    });
            } else if (pk) {
                for (int p = cs[c] + pt; owner && p < pe; p += nstr) update_pk(p, NBR, HPOS(p), (uint32_t)ORD(p));
            } else {
                for (int p = cs[c] + pt; owner && p < pe; p += nstr) update(p, NBR, HPOS(p), (uint32_t)ORD(p));
            }
            __syncthreads();
            if constexpr (shadow::kOn) shadow_pass(c, false);
        }
        if (part)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    if (i < mg && boff + i == b) dE[b] += dEp[i];
        if (pk) {
            dE[0] += dEp[0];
            dE[1] += dEp[1];
        }
#pragma unroll
        for (int b = 0; b < 4; ++b) dE[b] = 2 * (dE[b] >> SH);  // a flip changes E by 2 x
        if (pow2 && (ND == 1 || (ND == 2 && n < 8192))) {
            // |sum over the sites| < n 512^ND < 2^31: summed over the wavefront in 32 bits by
            // DPP moves and lane swaps.  (The 64-bit shuffles below are 40 LDS operations a
            // wavefront: 5000 of 28000 clocks of a sweep of the L = 10 cube, 8 slots a group.)
            int32_t s4[4];
#pragma unroll
            for (int b = 0; b < 4; ++b) s4[b] = (int32_t)(dE[b] >> 1);
            if (nq <= 1)
#pragma unroll
                for (int b = 0; b < 4; ++b) s4[b] += row_move<0xB1>(s4[b]);
            if (nq <= 2)
#pragma unroll
                for (int b = 0; b < 4; ++b) s4[b] += row_move<0x4E>(s4[b]);
            if (nq <= 4)
#pragma unroll
                for (int b = 0; b < 4; ++b) s4[b] += row_move<0x124>(s4[b]);
            if (nq <= 8)
#pragma unroll
                for (int b = 0; b < 4; ++b) s4[b] += row_move<0x128>(s4[b]);
            if (nq <= 16)
#pragma unroll
                for (int b = 0; b < 4; ++b) s4[b] = add_row_pairs(s4[b]);
            if (nq <= 32)
#pragma unroll
                for (int b = 0; b < 4; ++b) s4[b] = add_halves(s4[b]);
            if (active && lane < nq)
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    if (s4[b])
                        atomicAdd(reinterpret_cast<unsigned long long *>(&L_E[loc[b]]),
                                  (unsigned long long)(2ll * s4[b]));
        } else if (pow2) {
#pragma unroll
            for (int b = 0; b < 4; ++b)
                for (int off = nq; off < 64; off <<= 1) dE[b] += __shfl_xor(dE[b], off, 64);
            if (active && lane < nq)
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    if (dE[b]) atomicAdd(reinterpret_cast<unsigned long long *>(&L_E[loc[b]]), (unsigned long long)dE[b]);
        } else if (active) {
#pragma unroll
            for (int b = 0; b < 4; ++b)
                if (dE[b]) atomicAdd(reinterpret_cast<unsigned long long *>(&L_E[loc[b]]), (unsigned long long)dE[b]);
        }
        if (tid == 0) nacc = 0;
        if (tid < 2 * chains) L_cin[tid] = 0;
        for (int w = tid; w < nq; w += T) L_acc[w] = 0;
        __syncthreads();

        // 2. Replica exchange.
        phase();
        // This sweep's pairs (k, k+1) have k of parity par: nin of them lie inside the
        // group from slot kin on; lo_act / hi_act: the pair across the lower / upper
        // boundary is one of them.  Each boundary pair comes every other sweep, so
        // a side publishes every other sweep and its two buffers alternate.
        const int par = (int)(t & 1u);
        const int kin = s0 + ((s0 ^ par) & 1), nin = max(0, (s0 + mg - kin) / 2);
        const bool lo_act = g > 0 && ((s0 - 1) & 1) == par, hi_act = g < G - 1 && ((s0 + mg - 1) & 1) == par;
        const bool edge = lo_act || hi_act;
        const int buf = (int)((t >> 1) & 1u);
        // Boundary messages: relaxed agent-scope atomic words, each 16 payload bits
        // under a 16-bit sweep tag (never 0; the area is cleared before the launch).
        // Per-word coherence of atomics makes a word with the expected tag carry
        // that sweep's payload, so no fence (and no L2 write-back) is needed.
        const uint32_t tag = ((((uint32_t)ls + 1u) & 0x7FFFu) | 0x8000u) << 16;
        auto msg = [=](int grp, int side, int ch) __attribute__((always_inline)) -> uint32_t * {
            return a.xw + ((((size_t)run * G + grp) * 2 + side) * 2 + buf) * chains * xmsg + (size_t)ch * xmsg;
        };
        auto recv = [=](const uint32_t *w) __attribute__((always_inline)) -> int {
            unsigned it = 0;
            for (;;) {
                const uint32_t v = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if ((v & 0xFFFF0000u) == tag) return (int)(v & 0xFFFFu);
                if (++it > a.spin_limit) return -1;
                __builtin_amdgcn_s_sleep(1);
            }
        };
        if (edge) {
            // publish the first / last slot of every chain for an active lower / upper
            // boundary pair (pre-exchange states, energies)
            for (int side = 0; side < 2; ++side) {
                if (side == 0 ? !lo_act : !hi_act) continue;
                for (int ch = 0; ch < chains; ++ch) {
                    const int l = ch * mg + (side ? mg - 1 : 0);
                    const unsigned char *rb = sbase(ch, side ? mg - 1 : 0);
                    uint32_t *dst = msg(g, side, ch);
                    const unsigned long long El = (unsigned long long)L_E[l];
                    for (int w = tid; w < xmsg; w += T) {
                        uint32_t pay;
                        if (w < 4) {
                            pay = (uint32_t)((El >> (16 * w)) & 0xFFFFu);
                        } else {
                            const uint32_t p = 2u * (uint32_t)(w - 4);
                            pay = (uint32_t)rb[p * pst] | ((int)p + 1 < n ? (uint32_t)rb[(p + 1u) * pst] << 8 : 0u);
                        }
                        __hip_atomic_store(dst + w, tag | pay, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
                }
            }
        }
        // The pairs' decisions, a thread each.  What does not need a neighbour's energy (an
        // in-group pair's thresholds, every pair's random words) is done before the wait.
        const int per = nin + (edge ? 2 : 0);      // + the straddling pairs
        int pe = tid;
        const int pch = tid < chains * per ? chain_of(pe, per) : 0;
        const bool inner = pe < nin, lower = pe == nin;
        const bool decides = tid < chains * per && (inner || (lower ? lo_act : hi_act));
        const int pk0 = inner ? kin + 2 * pe : lower ? s0 - 1 : s0 + mg - 1;  // the pair (k, k + 1)
        const int pl = pch * mg + (inner ? pk0 - s0 : lower ? 0 : mg - 1);     // its own (lower) replica
        ptc::SwapTest test;
        dev::Words4 w0, w1;
        const uint32_t *stab = a.stab + (size_t)(decides ? pk0 : 0) * 7 * kDigitSize;
        int pnd = 0;
        if (decides) {
            pnd = L_snd[pk0 - s0 + 1];
            if (inner) test = ptc::swap_load(L_E[pl] - L_E[pl + 1], stab, pnd);
            ptc::swap_draw(pnd, (uint32_t)pk0, t, (uint32_t)(run * chains + pch), a.k0, a.k1, w0, w1);
        }
        if (edge) __syncthreads();
        if (decides && inner) {
            if (ptc::swap_accept(test, w0, w1)) {
                const long long x = L_E[pl];
                L_E[pl] = L_E[pl + 1];
                L_E[pl + 1] = x;
                // the pair's replicas are neighbouring bytes of a site's words: the lower one
                // takes its successor (bit 0..3), the upper its predecessor (bit 4..7)
                const int o = (int)(sbase(pch, pk0 - s0) - Sb);
                nacc = 1;
                atomicOr(&L_acc[o >> 2], 1 << (o & 3));
                atomicOr(&L_acc[(o + 1) >> 2], 16 << ((o + 1) & 3));
            }
        } else if (decides) {
            // the pair straddling a group boundary: (s0 - 1, s0) against the lower
            // neighbour's last slot, (s0 + mg - 1, s0 + mg) against the upper one's first
            const uint32_t *m = msg(lower ? g - 1 : g + 1, lower ? 1 : 0, pch);
            // the four energy words are loaded together (one round trip when the
            // message is there); a word without the expected tag is waited for
            uint32_t ew[4];
#pragma unroll
            for (int w = 0; w < 4; ++w) ew[w] = __hip_atomic_load(m + w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            unsigned long long eu = 0;
            bool ok = true;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const int v = (ew[w] & 0xFFFF0000u) == tag ? (int)(ew[w] & 0xFFFFu) : recv(m + w);
                ok = ok && v >= 0;
                eu |= (unsigned long long)(v < 0 ? 0 : v) << (16 * w);
            }
            if (!ok) {
                stop = 1;
            } else {
                const long long En = (long long)eu;
                test = ptc::swap_load(lower ? En - L_E[pl] : L_E[pl] - En, stab, pnd);
                if (ptc::swap_accept(test, w0, w1)) {
                    L_E[pl] = En;
                    L_cin[(lower ? 0 : chains) + pch] = 1;
                }
            }
        }
        __syncthreads();
        if (stop) break;
        {
            // accepted pairs swap their bytes word by word, a site's words by one thread
            // (a byte moves by one place, within its word or to the next one)
            if constexpr (shadow::kOn)
                if (nacc) shadow_swaps(true);
            if (nacc) {
                lds_mu32 *const S3 = (lds_mu32 *)L_S;
                for (int p = tid; p < n; p += T) {
                    const uint32_t o = (uint32_t)p * (uint32_t)nq;
                    uint32_t prev = 0, cur = S3[o];
                    for (int w = 0; w < nq; ++w) {
                        const uint32_t next = w + 1 < nq ? S3[o + w + 1] : 0u;
                        const uint32_t m = (uint32_t)L_acc[w];
                        if (m) {
                            const uint32_t up = (((m & 15u) * 0x00204081u) & 0x01010101u) * 255u;
                            const uint32_t dn = ((((m >> 4) & 15u) * 0x00204081u) & 0x01010101u) * 255u;
                            S3[o + w] = (cur & ~(up | dn)) | (((cur >> 8) | (next << 24)) & up) |
                                        (((cur << 8) | (prev >> 24)) & dn);
                        }
                        prev = cur;
                        cur = next;
                    }
                }
            }
            if (edge) {
                // an accepted straddling pair takes the neighbour's published configuration
                // (kCopyBatch sites per thread loaded together; a word whose tag is not
                // yet the expected one is waited for).  A swap stores words whole and this
                // bytes of the same words (groups of 4 slots: the pair (1, 2) lies between
                // the two boundary bytes), so a site is the same thread's in both, and no
                // barrier lies between; two threads read a message word.  (A barrier between
                // the two instead: 10.55 ms per 1000 sweeps of the L = 10 cube, 32 slots x 64
                // runs, against 10.1.)
                for (int sc = 0; sc < 2 * chains; ++sc) {
                    if (!L_cin[sc]) continue;
                    const int side = sc >= chains ? 1 : 0, ch = sc - side * chains;
                    const uint32_t *src = msg(side == 0 ? g - 1 : g + 1, side == 0 ? 1 : 0, ch) + 4;
                    unsigned char *rb = sbase(ch, side ? mg - 1 : 0);
                    constexpr int NS = kCopySites;
                    for (int p0 = NS * tid; p0 < n; p0 += kCopyBatch * NS * T) {
                        uint32_t v[kCopyBatch];
#pragma unroll
                        for (int u = 0; u < kCopyBatch; ++u) {
                            const int p = p0 + u * NS * T;
                            v[u] = p < n ? __hip_atomic_load(src + (p >> 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
                        }
#pragma unroll
                        for (int u = 0; u < kCopyBatch; ++u) {
                            const int p = p0 + u * NS * T;
                            if (p >= n) continue;
                            const int pay = (v[u] & 0xFFFF0000u) == tag ? (int)(v[u] & 0xFFFFu) : recv(src + (p >> 1));
                            if (pay < 0) {
                                stop = 1;
                                continue;
                            }
#pragma unroll
                            for (int s = 0; s < NS; ++s) {
                                if (p + s >= n) continue;
                                if constexpr (shadow::kOn)  // (its own thread's swap of the site is in order)
                                    if ((p + s) % T != tid)
                                        shadow::check(sh, (uint32_t)((p + s) * nq) + (uint32_t)(rb - Sb) / 4u);
                                rb[(uint32_t)(p + s) * pst] = (unsigned char)(pay >> (8 * ((p + s) & 1)));
                            }
                        }
                    }
                }
            }
            __syncthreads();
            if constexpr (shadow::kOn)
                if (nacc) shadow_swaps(false);
            if (stop) break;
        }

        phase();
        // 3. Houdayer cluster moves between chains 0 and 1 at the group's slots, up to
        // kIcmBatch slot pairs at a time with the whole workgroup: each cluster is the
        // connected component of its seed in the graph of J != 0 edges between sites
        // where the pair's replicas disagree, found with a lock-free union-find in LDS
        // (the pairs share every neighbour-record fetch).
        const int kb = max(a.icm_lo, s0), ke = min(a.icm_hi, s0 + mg);
        const int nchunks = (n + 63) / 64, vstr = 2 * nchunks, n16 = (n + 1) & ~1;
        // records per site (compile-time when DK > 0, so record batches stay in registers)
        const int Dn = DK > 0 ? DK : D;
        // One slot pair per pass (esum): the join scan also gathers, for every
        // disagreeing site v, E_v = sum of J s_v s_u over its agreeing neighbours u in
        // replica A, so the energy pass needs no neighbour reads (a cluster's change is
        // -2 sum over its sites of s_v h_v + E_v, as in the general pass below).
        const bool esum = MV == kMoveAny ? a.esum != 0 : true;
        constexpr int KB = DK > 0 ? DK : ptc::kRecBatch;
        const size_t pstride = (size_t)nq * 4;
        if constexpr (MV != kMoveNone)
        for (int kq = kb; a.nw_icm > 0 && kq < ke; kq += kBatch == 1 ? 1 : a.nw_icm) {
            const int nb = kBatch == 1 ? 1 : min(a.nw_icm, ke - kq);
            unsigned char *pa[kBatch], *pb[kBatch];
#pragma unroll
            for (int j = 0; j < kBatch; ++j) {
                const int o = min(kq + j, ke - 1) - s0;
                pa[j] = pk ? Sb : Sb + o + boff;
                pb[j] = pk ? Sb + 1 : Sb + 4 * qpc + o + boff1;
            }
            auto dis = [=](int j, int p) __attribute__((always_inline)) -> bool {
                return pa[j][(size_t)p * pstride] != pb[j][(size_t)p * pstride];
            };
            // The batch's disagreements at position p as bits (bit j: pair j).  When its
            // pairs lie in one quad word per chain, one XOR of the two words gives them all
            // (a byte is 0xFE where the replicas differ and 0 where they agree).
            const int o0 = kq - s0 + boff, qa0 = o0 >> 2, off0 = o0 & 3;
            const bool word_dis = off0 + nb <= 4 && boff1 == boff;
            const uint32_t pmask = (1u << nb) - 1u;
            // Chain 0's spin bytes of the batch's pairs at position p (byte j: pair j) and
            // their disagreement bits.
            auto pair_bytes = [=](int p, uint32_t &wa, uint32_t &db) __attribute__((always_inline)) {
                if (pk) {
                    // one word: chain 0's byte, then chain 1's
                    const uint32_t w = L_S[p];
                    wa = w & 0xFFu;
                    db = ((w ^ (w >> 8)) >> 1) & 1u;
                    return;
                }
                if (word_dis) {
                    const uint32_t w0 = L_S[(size_t)p * nq + qa0], w1 = L_S[(size_t)p * nq + qpc + qa0];
                    wa = w0 >> (8 * off0);
                    uint32_t m = (((w0 ^ w1) >> (8 * off0)) >> 1) & 0x01010101u;
                    m |= m >> 7;
                    m |= m >> 14;
                    db = m & pmask;
                    return;
                }
                wa = 0;
                db = 0;
#pragma unroll
                for (int j = 0; j < kBatch; ++j) {
                    const unsigned char x = pa[j][(size_t)p * pstride], y = pb[j][(size_t)p * pstride];
                    wa |= (uint32_t)x << (8 * j);
                    if (j < nb && x != y) db |= 1u << j;
                }
            };
            auto dis_bits = [=](int p) __attribute__((always_inline)) -> uint32_t {
                if (pk) {
                    const uint32_t w = L_S[p];
                    return ((w ^ (w >> 8)) >> 1) & 1u;
                }
                if (word_dis) {
                    const uint32_t x =
                        (L_S[(size_t)p * nq + qa0] ^ L_S[(size_t)p * nq + qpc + qa0]) >> (8 * off0);
                    uint32_t m = (x >> 1) & 0x01010101u;
                    m |= m >> 7;
                    m |= m >> 14;
                    return m & pmask;
                }
                uint32_t m = 0;
#pragma unroll
                for (int j = 0; j < kBatch; ++j)
                    if (j < nb && dis(j, p)) m |= 1u << j;
                return m;
            };
            // disagreement masks in variable-index order, 64 variables per chunk
            for (int c0 = wid; c0 < nchunks; c0 += 4 * nw) {
                int pp[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int i = (c0 + u * nw) * 64 + lane;
                    pp[u] = (c0 + u * nw < nchunks && i < n) ? POS(i) : -1;
                }
                uint32_t db[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) db[u] = pp[u] >= 0 ? dis_bits(pp[u]) : 0u;
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int j = 0; j < kBatch; ++j) {
                        if (j >= nb) break;
                        const unsigned long long m = __ballot((db[u] >> j) & 1u);
                        if (lane == 0 && c0 + u * nw < nchunks) L_dmask[(size_t)j * nchunks + c0 + u * nw] = m;
                    }
            }
            __syncthreads();
            if (wid < nb) {
                // seed of pair wid = the target-th disagreeing variable
                const int j = wid, k = kq + j;
                const unsigned long long *dm = L_dmask + (size_t)j * nchunks;
                int n_neg = 0;
                for (int c = lane; c < nchunks; c += 64) n_neg += __popcll(dm[c]);
                for (int d = 32; d >= 1; d >>= 1) n_neg += __shfl_xor(n_neg, d, 64);
                int seed_p = -1;
                if (n_neg > 0) {
                    const uint32_t w = dev::philox((uint32_t)k, t, (uint32_t)run, 4u << 24, a.k0, a.k1).w[0];
                    const int target = (int)(((unsigned long long)w * (unsigned long long)n_neg) >> 32);
                    int seen = 0;
                    for (int c0 = 0; c0 < nchunks && seed_p < 0; c0 += 64) {
                        const int c = c0 + lane;
                        const unsigned long long m = c < nchunks ? dm[c] : 0ull;
                        const int cnt = __popcll(m);
                        int incl = cnt;
                        for (int d = 1; d < 64; d <<= 1) {
                            const int y = __shfl_up(incl, d, 64);
                            if (lane >= d) incl += y;
                        }
                        const int excl = seen + incl - cnt;
                        const unsigned long long who = __ballot(target >= excl && target < excl + cnt);
                        if (who) {
                            const int src = __ffsll((long long)who) - 1;
                            const unsigned long long ms = __shfl(m, src, 64);
                            const int rest = target - __shfl(excl, src, 64);
                            const bool mine = ((ms >> lane) & 1ull) && __popcll(ms & lanemask_lt()) == rest;
                            const int bitl = __ffsll((long long)__ballot(mine)) - 1;
                            seed_p = POS((c0 + src) * 64 + bitl);
                        }
                        seen += __shfl(incl, 63, 64);
                    }
                }
                if (lane == 0) L_misc[j] = seed_p;
            }
            // fresh forests and energy terms, written by the other wavefronts while the
            // seeds are searched (by all of them when every wavefront searches a seed)
            const int iw = T > 64 * nb ? nb : 0;
            if (wid >= iw) {
                const int t0 = tid - 64 * iw, ts = T - 64 * iw;
                for (int j = 0; j < nb; ++j)
                    for (int p = t0; p < n16; p += ts) L_parent[(size_t)j * n16 + p] = (uint16_t)p;
                if (esum)
                    for (int p = t0; p < n; p += ts) L_es[p] = 0;
            }
            __syncthreads();
            // The masks are consumed: their words now collect cluster membership.
            uint32_t *const memb = reinterpret_cast<uint32_t *>(L_dmask);
            if (!esum)
                for (int wd = tid; wd < nb * vstr; wd += T) memb[wd] = 0u;
            // join the endpoints of every J != 0 edge between disagreeing sites.  Each
            // wavefront scans 64 sites at a time and appends the qualifying
            // (pair, site, neighbour) joins to its own LDS buffer; whenever 64 are
            // pending, every lane performs one (full lanes instead of the ~1 in 4 that
            // a per-site loop would keep busy).  Join order does not change the sets.
            {
                uint32_t *const wb = L_ubuf + wid * kJoinBuf;
                unsigned char *const wj = L_ubj + wid * kJoinBuf;
                int cnt = 0;
                auto run_joins = [&](int m) __attribute__((always_inline)) {
                    __builtin_amdgcn_wave_barrier();
                    if (lane < m) {
                        const uint32_t it = wb[cnt - m + lane];
                        ptc::uf_union(L_parent + (size_t)wj[cnt - m + lane] * n16, it & 0xFFFFu, it >> 16);
                    }
                    cnt -= m;
                    __builtin_amdgcn_wave_barrier();
                };
                // Every edge is taken from its larger end, and the first colour class (the
                // lowest positions; no edge joins two sites of one class) has none: the
                // scan starts where that class ends.
                const int scan_begin = a.C > 0 ? cs[1] : n;
                auto scan_site = [&](int p, auto rec) __attribute__((always_inline)) {
                    uint32_t dp = 0, ap = 0;
                    if (esum) {
                        if (p < n) pair_bytes(p, ap, dp);
                    } else {
                        dp = p < n ? dis_bits(p) : 0u;
                    }
                    // with esum every site's edges are read (an agreeing site may border a
                    // disagreeing one)
                    const bool need = esum ? p < n : dp != 0u;
                    for (int k0 = 0; k0 < Dn; k0 += KB) {
                        uint32_t rr[KB];
#pragma unroll
                        for (int uu = 0; uu < KB; ++uu) rr[uu] = (need && k0 + uu < Dn) ? rec(k0 + uu, p) : 0u;
                        // the pairs each edge joins, every neighbour's words read before the
                        // joins (an absent edge reads the site's own)
                        uint32_t fb[KB];
                        if (esum) {
                            uint32_t au[KB], du[KB];
#pragma unroll
                            for (int uu = 0; uu < KB; ++uu)
                                pair_bytes(min((int)(rr[uu] >> 16), n - 1), au[uu], du[uu]);
#pragma unroll
                            for (int uu = 0; uu < KB; ++uu) {
                                const int u = (int)(rr[uu] >> 16);
                                const bool edge_ok = k0 + uu < Dn && (rr[uu] & 0xffffu) != 0u && u < p;
                                fb[uu] = edge_ok ? dp & du[uu] : 0u;
                                if (edge_ok && ((dp ^ du[uu]) & 1u)) {
                                    // an edge with one disagreeing end: its term goes to that end
                                    const int32_t Jv = (int32_t)(int16_t)(rr[uu] & 0xffffu);
                                    const int32_t prod =
                                        Jv * (int32_t)(int8_t)(ap & 0xFFu) * (int32_t)(int8_t)(au[uu] & 0xFFu);
                                    atomicAdd(&L_es[(dp & 1u) ? p : u], prod);
                                }
                            }
                        } else {
#pragma unroll
                            for (int uu = 0; uu < KB; ++uu) {
                                const int u = (int)(rr[uu] >> 16);
                                const bool edge_ok = k0 + uu < Dn && (rr[uu] & 0xffffu) != 0u && u < p;
                                fb[uu] = edge_ok ? (dp & dis_bits(u)) : 0u;
                            }
                        }
                        // a site that is still its own root is hooked under its first
                        // disagreeing neighbour at once (a smaller one; whatever tree that is
                        // in): one join in three of a site of six neighbours goes, and the
                        // others find shallow trees
#pragma unroll
                        for (int j = 0; j < kBatch; ++j) {
                            if (j >= nb) break;
                            uint32_t first = KB, to = 0;
#pragma unroll
                            for (int uu = KB - 1; uu >= 0; --uu)
                                if ((fb[uu] >> j) & 1u) {
                                    first = uu;
                                    to = rr[uu] >> 16;
                                }
                            if (first < KB && ptc::cas16(L_parent + (size_t)j * n16 + p, (uint32_t)p, to))
#pragma unroll
                                for (int uu = 0; uu < KB; ++uu)
                                    if (first == (uint32_t)uu) fb[uu] &= ~(1u << j);
                        }
#pragma unroll
                        for (int uu = 0; uu < KB; ++uu) {
                            if (k0 + uu >= Dn) break;
                            const int u = (int)(rr[uu] >> 16);
#pragma unroll
                            for (int j = 0; j < kBatch; ++j) {
                                if (j >= nb) break;
                                const bool f = (fb[uu] >> j) & 1u;
                                const unsigned long long msk = __ballot(f);
                                if (f) {
                                    const int at = cnt + __popcll(msk & lanemask_lt());
                                    wb[at] = (uint32_t)p | ((uint32_t)u << 16);
                                    wj[at] = (unsigned char)j;
                                }
                                cnt += __popcll(msk);
                                if (cnt >= 64) run_joins(64);
                            }
                        }
                    }
                };
                if constexpr (BIG && DK > 0) {
                    // the records of the wavefront's next 64 sites are in flight while
                    // the current ones are scanned
                    uint32_t rn[DK];
                    auto fetch = [&](int pp) __attribute__((always_inline)) {
#pragma unroll
                        for (int u = 0; u < DK; ++u) rn[u] = pp < n ? gnbr[(size_t)pp * DK + u] : 0u;
                    };
                    int p0 = scan_begin + wid * 64;
                    if (p0 < n) fetch(p0 + lane);
                    for (; p0 < n; p0 += nw * 64) {
                        uint32_t rr[DK];
#pragma unroll
                        for (int u = 0; u < DK; ++u) rr[u] = rn[u];
                        if (p0 + nw * 64 < n) fetch(p0 + nw * 64 + lane);
                        scan_site(p0 + lane, [&](int k, int) __attribute__((always_inline)) { return rr[k]; });
                    }
                } else {
                    for (int p0 = scan_begin + wid * 64; p0 < n; p0 += nw * 64) scan_site(p0 + lane, NBR);
                }
                if (cnt > 0) run_joins(cnt);
            }
            __syncthreads();
            // energy change of flipping each seed's component: -2 s_v (h_v + sum over
            // agreeing neighbours J s_u) per site (a neighbour across a J != 0 edge is in
            // the cluster exactly when it disagrees); the replicas are only written after
            // every site has been read
            uint32_t root[kBatch];
#pragma unroll
            for (int j = 0; j < kBatch; ++j) {
                const int sp = j < nb ? L_misc[j] : -1;
                root[j] = sp >= 0 ? ptc::uf_find(L_parent + (size_t)j * n16, (uint32_t)sp) : 0xffffffffu;
            }
            long long dA[kBatch];
#pragma unroll
            for (int j = 0; j < kBatch; ++j) dA[j] = 0;
            auto energy_site = [&](int p, auto rec, int32_t hp) __attribute__((always_inline)) {
                unsigned in = 0;
                const uint32_t dpb = dis_bits(p);
#pragma unroll
                for (int j = 0; j < kBatch; ++j)
                    if (root[j] != 0xffffffffu && ((dpb >> j) & 1u) &&
                        ptc::uf_find(L_parent + (size_t)j * n16, (uint32_t)p) == root[j])
                        in |= 1u << j;
                if (!in) return;
                // f = h + sum of J s over the neighbours that agree (those outside the
                // cluster); replica B's field is the same (it agrees with A there) and its
                // spin at p is -s_A, so its energy change is -dA: the pair energy is
                // conserved exactly
                int32_t fA[kBatch];
#pragma unroll
                for (int j = 0; j < kBatch; ++j) fA[j] = hp;
                for (int k0 = 0; k0 < Dn; k0 += KB) {
                    uint32_t rr[KB];
#pragma unroll
                    for (int uu = 0; uu < KB; ++uu) rr[uu] = k0 + uu < Dn ? rec(k0 + uu, p) : 0u;
                    uint32_t wa[KB], db[KB];
#pragma unroll
                    for (int uu = 0; uu < KB; ++uu) pair_bytes((int)(rr[uu] >> 16), wa[uu], db[uu]);
#pragma unroll
                    for (int uu = 0; uu < KB; ++uu) {
                        const int32_t Jv = (int32_t)(int16_t)(rr[uu] & 0xffffu);
                        if (k0 + uu >= Dn || Jv == 0) continue;
#pragma unroll
                        for (int j = 0; j < kBatch; ++j)
                            if (((in >> j) & 1u) && !((db[uu] >> j) & 1u))
                                fA[j] += Jv * (int32_t)(int8_t)(wa[uu] >> (8 * j));
                    }
                }
                uint32_t wp, dbp;
                pair_bytes(p, wp, dbp);
#pragma unroll
                for (int j = 0; j < kBatch; ++j)
                    if ((in >> j) & 1u) {
                        atomicOr(&memb[(size_t)j * vstr + (p >> 5)], 1u << (p & 31));
                        dA[j] += -2ll * (int32_t)(int8_t)(wp >> (8 * j)) * (long long)fA[j];
                    }
            };
            if (esum) {
                // the seed's cluster: its disagreeing sites whose root is the seed's
                auto esite = [&](int p, int32_t hp) __attribute__((always_inline)) {
                    uint32_t wp, dbp;
                    pair_bytes(p, wp, dbp);
                    if (root[0] == 0xffffffffu || !(dbp & 1u)) return;
                    if (ptc::uf_find(L_parent, (uint32_t)p) != root[0]) return;
                    dA[0] += -2ll * ((long long)(int8_t)(wp & 0xFFu) * hp + (long long)L_es[p]);
                    // no other thread reads this site's bytes in this pass: flip it here
                    pa[0][(size_t)p * pstride] = (unsigned char)(-(int)(int8_t)pa[0][(size_t)p * pstride]);
                    pb[0][(size_t)p * pstride] = (unsigned char)(-(int)(int8_t)pb[0][(size_t)p * pstride]);
                };
                if constexpr (BIG) {
                    // the next site's bias is in flight while the current one is tested
                    int p = tid;
                    int32_t hn = p < n ? ghpos[p] : 0;
                    for (; p < n; p += T) {
                        const int32_t hp = hn;
                        if (p + T < n) hn = ghpos[p + T];
                        esite(p, hp);
                    }
                } else {
                    for (int p = tid; p < n; p += T) esite(p, HPOS(p));
                }
            } else {
                if constexpr (BIG && DK > 0) {
                    // the records and h of the thread's next site are in flight while the
                    // current one is tested and summed
                    uint32_t rn[DK];
                    int32_t hn = 0;
                    auto fetch = [&](int pp) __attribute__((always_inline)) {
#pragma unroll
                        for (int u = 0; u < DK; ++u) rn[u] = gnbr[(size_t)pp * DK + u];
                        hn = ghpos[pp];
                    };
                    int p = tid;
                    if (p < n) fetch(p);
                    for (; p < n; p += T) {
                        uint32_t rr[DK];
#pragma unroll
                        for (int u = 0; u < DK; ++u) rr[u] = rn[u];
                        const int32_t hp = hn;
                        if (p + T < n) fetch(p + T);
                        energy_site(p, [&](int k, int) __attribute__((always_inline)) { return rr[k]; }, hp);
                    }
                } else {
                    for (int p = tid; p < n; p += T) energy_site(p, NBR, HPOS(p));
                }
            }
#pragma unroll
            for (int j = 0; j < kBatch; ++j) {
                if (j >= nb) break;
                const long long sa = wave_sum(dA[j]), sb = -sa;
                const int la = kq + j - s0, lb = mg + la;
                if (lane == 0) {
                    if (sa) atomicAdd(reinterpret_cast<unsigned long long *>(&L_E[la]), (unsigned long long)sa);
                    if (sb) atomicAdd(reinterpret_cast<unsigned long long *>(&L_E[lb]), (unsigned long long)sb);
                }
            }
            __syncthreads();
            // flip the clusters in both replicas (the gathered-terms pass flipped its own)
            for (int p = tid; !esum && p < n; p += T)
#pragma unroll
                for (int j = 0; j < kBatch; ++j)
                    if (j < nb && ((memb[(size_t)j * vstr + (p >> 5)] >> (p & 31)) & 1u)) {
                        pa[j][(size_t)p * pstride] = (unsigned char)(-(int)(int8_t)pa[j][(size_t)p * pstride]);
                        pb[j][(size_t)p * pstride] = (unsigned char)(-(int)(int8_t)pb[j][(size_t)p * pstride]);
                    }
            __syncthreads();
        }

        // 4. Top-10 lists of the group's colder slots: a wavefront per list decides the
        // offer (candidate test, duplicate check, victim entry) and updates the list;
        // the inserted state is stored by that wavefront, or for long states (where one
        // wavefront's copy outlasts a barrier) by the whole workgroup afterwards.  While a
        // run still descends every second offer is an insertion (0.56 per list and sweep in
        // the first 300 sweeps of the L = 10 cube, 0.29 over 1000).
        phase();
        const int kc = max(K - half, s0), ncold = max(0, s0 + mg - kc);
        const bool wide_copy = n >= 2048;
        // a replica's bytes at positions 4 w .. 4 w + 3 (from its byte at position 0 on)
        auto four = [=](const lds_u8 *rb, int w) __attribute__((always_inline)) -> uint32_t {
            const uint32_t o = 4u * (uint32_t)w * pst;
            return (uint32_t)rb[o] | ((uint32_t)rb[o + pst] << 8) | ((uint32_t)rb[o + 2 * pst] << 16) |
                   ((uint32_t)rb[o + 3 * pst] << 24);
        };
        // replica l's state into dst by threads first, first + step, ...
        auto store_state = [&](int ch, int k, int8_t *dst, int first, int step) __attribute__((always_inline)) {
            if (pk && (n & 3) == 0) {
                // chain l's byte of four consecutive sites' words per thread, one word store
                const int sh = 8 * ch;
                for (int w = first; w < (n >> 2); w += step) {
                    const uint4 v = *reinterpret_cast<const uint4 *>(L_S + 4 * w);
                    *reinterpret_cast<uint32_t *>(dst + 4 * w) =
                        ((v.x >> sh) & 0xFFu) | (((v.y >> sh) & 0xFFu) << 8) | (((v.z >> sh) & 0xFFu) << 16) |
                        (((v.w >> sh) & 0xFFu) << 24);
                }
            } else if ((n & 3) == 0) {
                const lds_u8 *rb = (const lds_u8 *)sbase(ch, k - s0);
#pragma unroll 4
                for (int w = first; w < (n >> 2); w += step) *reinterpret_cast<uint32_t *>(dst + 4 * w) = four(rb, w);
            } else {
                // 32-bit LDS offsets stepped by addition (no 64-bit address arithmetic)
                const lds_u8 *rb = (const lds_u8 *)sbase(ch, k - s0);
                const uint32_t ostep = (uint32_t)step * pst;
                uint32_t o = (uint32_t)first * pst;
                for (uint32_t p = (uint32_t)first; p < (uint32_t)n; p += (uint32_t)step, o += ostep)
                    dst[p] = (int8_t)rb[o];
            }
        };
        for (int li = wid; li < chains * ncold; li += nw) {
            int k = li;
            const int ch = chain_of(k, ncold);
            k += kc;
            const int l = ch * mg + (k - s0);
            const int gl = ch * half + (k - (K - half));
            const long long Ec = L_E[l];
            const int cnt = L_Lcnt[l];
            // a full list whose largest energy is known and not above the offered one
            // fails the candidate test without reading its entries
            if (cnt == 10 && Ec >= L_Lmax[l]) {
                if (wide_copy && lane == 0) L_Lins[li] = -1;
                continue;
            }
            long long *LE = L_LE + (size_t)l * 10;
            int32_t *LW = L_Lwhen + (size_t)l * 10;
            int8_t *base = a.tops + ((size_t)run * Ls + gl) * 10 * n;
            int victim = -1;
            // lane e holds entry e; a full list's victim is the entry ordered last by
            // (energy, insertion stamp) (stamps are distinct, so the order is strict), known
            // from the insertion before (L_Lmax, and its place in the rank storage)
            const bool held = lane < cnt;
            long long le = held ? LE[lane] : (long long)0x8000000000000000ll;
            int32_t lw = held ? LW[lane] : (int32_t)0x80000000;
            long long worst = L_Lmax[l];
            int32_t worst_at = L_Lord[(size_t)l * 10];
            auto rank_last = [&]() __attribute__((always_inline)) {
                worst = le;
                int32_t w = lw;
                worst_at = lane;
                last_of_16(worst, w, worst_at);
            };
            const bool known = worst != 0x7FFFFFFFFFFFFFFFll;
            if (cnt == 10 && !known) rank_last();
            const bool cand = cnt < 10 || Ec < (long long)read_first((unsigned long long)worst);
            if (cand) {
                const lds_u8 *rb = (const lds_u8 *)sbase(ch, k - s0);
                bool dup = false;
                // entries of equal energy get a full comparison of their states
                for (unsigned long long eq = __ballot(held && le == Ec); eq && !dup; eq &= eq - 1) {
                    const int8_t *ent = base + (size_t)(__ffsll((long long)eq) - 1) * n;
                    bool diff = false;
                    if ((n & 3) == 0) {
#pragma unroll 4
                        for (int w = lane; w < (n >> 2); w += 64)
                            diff |= *reinterpret_cast<const uint32_t *>(ent + 4 * w) != four(rb, w);
                    } else {
                        uint32_t o = (uint32_t)lane * pst;
                        for (uint32_t p = (uint32_t)lane; p < (uint32_t)n; p += 64u, o += 64u * pst)
                            diff |= ent[p] != (int8_t)rb[o];
                    }
                    dup = !__any(diff);
                }
                if (!dup) {
                    victim = cnt < 10 ? cnt : __builtin_amdgcn_readfirstlane(worst_at);
                    if (!wide_copy) store_state(ch, k, base + (size_t)victim * n, lane, 64);
                }
            }
            const int now = victim >= 0 && cnt < 10 ? cnt + 1 : cnt;
            if (victim >= 0 && now == 10) {
                le = lane == victim ? Ec : le;
                lw = lane == victim ? ls : lw;
                rank_last();
            }
            __builtin_amdgcn_wave_barrier();
            if (lane == 0) {
                if (wide_copy) L_Lins[li] = victim;
                if (victim >= 0) {
                    LE[victim] = Ec;
                    LW[victim] = ls;
                    L_Lcnt[l] = now;
                }
                L_Lmax[l] = now < 10 ? 0x7FFFFFFFFFFFFFFFll : worst;
                L_Lord[(size_t)l * 10] = worst_at;
            }
            __builtin_amdgcn_wave_barrier();
        }
        if (wide_copy && ncold > 0) {
            __syncthreads();
            for (int li = 0; li < chains * ncold; ++li) {
                const int victim = L_Lins[li];
                if (victim < 0) continue;
                int k = li;
                const int ch = chain_of(k, ncold);
                k += kc;
                const int gl = ch * half + (k - (K - half));
                store_state(ch, k, a.tops + (((size_t)run * Ls + gl) * 10 + victim) * n, tid, T);
            }
        }
        __syncthreads();
    }

    const int kc = max(K - half, s0), ncold = max(0, s0 + mg - kc);
    if (stop && !k4) {
        if (tid == 0) *(a.xw - 1 - run) = 1u;
        return;
    }
    if (stop) {
        // A neighbour never published: mark the group's lists as invalid.
        if (a.top_count)
            for (int li = tid; li < chains * ncold; li += T) {
                const int ch = li / ncold, k = kc + (li - ch * ncold);
                a.top_count[(size_t)run * Ls + ch * half + (k - (K - half))] = -1;
            }
        return;
    }
    // Outputs of the group's replicas.
    if (a.final_E)
        for (int l = tid; l < nl; l += T) {
            const int ch = l / mg, slot = s0 + (l - ch * mg);
            a.final_E[((size_t)run * chains + ch) * K + slot] = L_E[l];
        }
    if (a.final_spins)
        for (int idx = tid; idx < nl * n; idx += T) {
            const int l = idx / n, i = idx - l * n;
            const int ch = l / mg, slot = s0 + (l - ch * mg);
            a.final_spins[(((size_t)run * chains + ch) * K + slot) * n + i] = (int8_t)*sbyte(l, POS(i));
        }
    if (a.top_E || a.top_spins || a.top_count) {
        // Rank of entry e of a list = number of entries ordered before it by (E, insertion).
        const int nlist = chains * ncold;
        for (int le = tid; le < nlist * 10; le += T) L_Lord[le] = -1;
        __syncthreads();
        for (int le = tid; le < nlist * 10; le += T) {
            const int li = le / 10, e = le - li * 10;
            const int ch = li / ncold, k = kc + (li - ch * ncold);
            const int l = ch * mg + (k - s0);
            const long long *LE = L_LE + (size_t)l * 10;
            const int32_t *LW = L_Lwhen + (size_t)l * 10;
            const int cnt = L_Lcnt[l];
            if (e < cnt) {
                int rank = 0;
                for (int o = 0; o < cnt; ++o) rank += (LE[o] < LE[e] || (LE[o] == LE[e] && LW[o] < LW[e])) ? 1 : 0;
                L_Lord[li * 10 + rank] = e;
            }
            if (e == 0 && a.top_count)
                a.top_count[(size_t)run * Ls + ch * half + (k - (K - half))] = L_Lbad[l] ? -1 : cnt;
        }
        __syncthreads();
        if (a.top_E)
            for (int le = tid; le < nlist * 10; le += T) {
                const int li = le / 10, rank = le - li * 10;
                const int ch = li / ncold, k = kc + (li - ch * ncold);
                const int l = ch * mg + (k - s0), gl = ch * half + (k - (K - half));
                const int e = L_Lord[le];
                a.top_E[((size_t)run * Ls + gl) * 10 + rank] = e >= 0 ? L_LE[(size_t)l * 10 + e] : 0x7FFFFFFFFFFFFFFFll;
            }
        if (a.top_spins)
            for (size_t idx = tid; idx < (size_t)nlist * 10 * n; idx += T) {
                const int lr = (int)(idx / n), i = (int)(idx - (size_t)lr * n);
                const int li = lr / 10, rank = lr - li * 10;
                const int ch = li / ncold, k = kc + (li - ch * ncold);
                const int gl = ch * half + (k - (K - half));
                const int e = L_Lord[li * 10 + rank];
                a.top_spins[((size_t)run * Ls + gl) * 10 * n + (size_t)rank * n + i] =
                    e >= 0 ? a.tops[(((size_t)run * Ls + gl) * 10 + e) * n + POS(i)] : (int8_t)0;
            }
    }
}

// The kernel of a launch: instances with kSiteRecs records and up to two digits have
// their move compiled in, the others decide it at run time.
template <int ND, bool BIG, int DK>
void *ptx_entry(int move) {
    if constexpr (DK > 0 && ND <= 2) {
        if (move == kMoveNone) return reinterpret_cast<void *>(ptx_kernel<ND, BIG, DK, kMoveNone>);
        if (move == kMoveSingle) return reinterpret_cast<void *>(ptx_kernel<ND, BIG, DK, kMoveSingle>);
        if constexpr (BIG)
            if (move == kMovePacked) return reinterpret_cast<void *>(ptx_kernel<ND, BIG, DK, kMovePacked>);
    }
    return reinterpret_cast<void *>(ptx_kernel<ND, BIG, DK, kMoveAny>);
}

template <int ND>
void *ptx_pick(bool big, int D, int move) {
    if (D == kSiteRecs) return big ? ptx_entry<ND, true, kSiteRecs>(move) : ptx_entry<ND, false, kSiteRecs>(move);
    return big ? ptx_entry<ND, true, 0>(move) : ptx_entry<ND, false, 0>(move);
}

void *ptx_fn(const PtxShape &s) {
    const int move = s.nw_icm == 0                        ? kMoveNone
                     : !s.esum                            ? kMoveAny
                     : ptx_packed(s.big, s.m, s.chains) ? kMovePacked
                                                          : kMoveSingle;
    switch (s.nd) {
        case 1:
            return ptx_pick<1>(s.big, s.D, move);
        case 2:
            return ptx_pick<2>(s.big, s.D, move);
        case 3:
            return ptx_pick<3>(s.big, s.D, move);
        default:
            return nullptr;
    }
}

}  // namespace

int ptx_msg_words(int n) { return 4 + (n + 1) / 2; }

int ptx_words_per_site(int K, int m, int chains) { return chains * ptx_chain_words(K, m); }

size_t ptx_lds_bytes(const PtxShape &s) {
    return ptx_layout(s.n, s.D, s.K, s.m, s.chains, s.row_len, s.nw_icm, s.big, s.esum, nullptr, nullptr);
}

hipError_t ptx_max_groups_resident(const PtxShape &s, int threads, size_t lds, int *blocks_per_cu) {
    void *f = ptx_fn(s);
    if (!f) return hipErrorInvalidValue;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, f, threads, lds);
}

hipError_t launch_ptx(const PtxLaunch &P, hipStream_t s) {
    PtxArgs a;
    a.image = P.image;
    a.mtab = P.mtab;
    a.stab = P.stab;
    a.snd = P.snd;
    a.final_spins = P.out->final_spins;
    a.final_E = reinterpret_cast<long long *>(P.out->final_E);
    a.top_spins = P.out->top_spins;
    a.top_E = reinterpret_cast<long long *>(P.out->top_E);
    a.top_count = P.out->top_count;
    a.tops = P.tops;
    a.rs = P.resume;
    a.xw = P.xw;
    a.xmsg = ptx_msg_words(P.n);
    a.n = P.n;
    a.D = P.D;
    a.C = P.C;
    a.K = P.K;
    a.chains = P.chains;
    a.sweeps = P.sweeps;
    a.row_len = P.row_len;
    a.icm_lo = P.icm_lo;
    a.icm_hi = P.icm_hi;
    a.nw_icm = P.nw_icm;
    a.esum = P.esum ? 1 : 0;
    a.G = P.G;
    a.m = P.m;
    a.sweep_offset = P.sweep_offset;
    a.k0 = (uint32_t)P.seed;
    a.k1 = (uint32_t)(P.seed >> 32);
    a.spin_limit = P.spin_limit;
    if (P.G > 1) {
        const size_t words = (size_t)P.runs * (1 + (size_t)P.G * 4 * P.chains * ptx_msg_words(P.n));
        hipLaunchKernelGGL(xw_zero_kernel, dim3((unsigned)std::min<size_t>((words + 255) / 256, 4096)), dim3(256), 0,
                           s, P.xw - P.runs, words);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const PtxShape shape{P.n, P.D, P.K, P.m, P.chains, P.row_len, P.nd, P.nw_icm, P.big, P.esum};
    const size_t lds = ptx_lds_bytes(shape);
    void *f = ptx_fn(shape);
    if (!f) return hipErrorInvalidValue;
    void *args[] = {&a};
    return hipLaunchKernel(f, dim3(P.runs * P.G), dim3(P.threads), args, lds, s);
}

hipError_t shadow_stats_ptx(unsigned long long *out, bool reset) { return shadow::read_stats(out, reset); }

}  // namespace spv
