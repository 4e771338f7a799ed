// Instance packing, the one-instance simulated-annealing launch and the energy kernel.
//
// Sampler (Sec. III.A, "SA"): every read starts from its own Philox state (or
// a caller state) and performs one Metropolis sweep per entry of the beta
// schedule; the sample is the final state of every read.  A sweep visits the
// colour classes in order; a class is an independent set, so all of its
// spins are updated in parallel with the same result as any sequential order.
//
// Layout: the instance is renumbered by position p (colour-major, index order
// inside a class) and held in LDS as an ELL table of 32-bit records
// (neighbour position << 16 | int16 coupling).  Spins live in LDS as S[p][q]:
// one 32-bit word per (position, quad of 4 replicas), a byte per replica.  A
// lane owns one (position, quad) task: it forms the four local fields, draws
// one Philox block that serves the four replicas, and applies the integer
// threshold test, so instance data is shared by the replicas of a quad and
// every random word is used.
#include <hip/hip_runtime.h>

#include <cstdlib>

#include "device.hpp"
#include "internal.hpp"
#include "sa_core.hpp"
#include "swar_core.hpp"

namespace spv {

namespace {

__global__ __launch_bounds__(1024) void prep_order_kernel(const uint8_t *__restrict__ colour,
                                                          int n, int D, int C,
                                                          int32_t *__restrict__ image) {
    __shared__ int cnt[kMaxColours];
    __shared__ int cs[kMaxColours + 1];
    __shared__ int tmp[1024 / 64 + 1];
    int32_t *order = image + kImgHeader;
    int32_t *pos_of = order + n;
    const int tid = threadIdx.x;
    if (tid < kMaxColours) cnt[tid] = 0;
    __syncthreads();
    for (int i = tid; i < n; i += blockDim.x) {
        int c = colour[i];
        c = c < C ? c : C - 1;
        atomicAdd(&cnt[c], 1);
    }
    __syncthreads();
    if (tid == 0) {
        int acc = 0;
        for (int c = 0; c < C; ++c) {
            cs[c] = acc;
            acc += cnt[c];
        }
        cs[C] = acc;
        image[0] = n;
        image[1] = D;
        image[2] = C;
        for (int c = 0; c <= C; ++c) image[3 + c] = cs[c];
    }
    __syncthreads();
    for (int c = 0; c < C; ++c) {
        int base = cs[c];
        for (int start = 0; start < n; start += blockDim.x) {
            const int i = start + tid;
            int ci = 0;
            if (i < n) {
                ci = colour[i];
                ci = ci < C ? ci : C - 1;
            }
            const bool flag = (i < n) && ci == c;
            int tot;
            const int pre = dev::block_exclusive_scan(flag ? 1 : 0, tmp, &tot);
            if (flag) {
                order[base + pre] = i;
                pos_of[i] = base + pre;
            }
            base += tot;
        }
    }
}

__global__ __launch_bounds__(256) void prep_nbr_kernel(const int32_t *__restrict__ row_ptr,
                                                       const int32_t *__restrict__ col,
                                                       const int32_t *__restrict__ J,
                                                       const int32_t *__restrict__ h, int n,
                                                       int nnz, int D, int32_t *__restrict__ image) {
    const int32_t *order = image + kImgHeader;
    const int32_t *pos_of = order + n;
    int32_t *hpos = image + kImgHeader + 2 * n;
    uint32_t *nbr = reinterpret_cast<uint32_t *>(image + kImgHeader + 3 * n);
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    int i = order[p];
    i = i < 0 ? 0 : (i >= n ? n - 1 : i);
    int rb = row_ptr[i], re = row_ptr[i + 1];
    rb = rb < 0 ? 0 : (rb > nnz ? nnz : rb);
    re = re < rb ? rb : (re > nnz ? nnz : re);
    const int deg = (re - rb) < D ? (re - rb) : D;
    for (int k = 0; k < D; ++k) {
        uint32_t rec = (uint32_t)p << 16;
        if (k < deg) {
            int j = col[rb + k];
            j = j < 0 ? 0 : (j >= n ? n - 1 : j);
            int v = J[rb + k];
            v = v > 32767 ? 32767 : (v < -32767 ? -32767 : v);
            rec = ((uint32_t)pos_of[j] << 16) | (uint32_t)(uint16_t)(int16_t)v;
        }
        nbr[(size_t)p * D + k] = rec;
    }
    hpos[p] = h[i];
}

// ND = number of threshold digits; ND = 0 selects the byte-parallel path.  The
// neighbour loop is straight-line code for a record count DK (0: any).
// BIG: the instance lives in global memory, LDS holds the tables and the spins.
// The byte-parallel body reads its own records from a.big (built beforehand by
// big_prep_kernel); the general body reads the prepared image itself.
template <int ND, int DK = 0, bool BIG = false>
__global__ __launch_bounds__(1024) void sa_kernel(core::SaItem a) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int cs[kMaxColours + 1];
    a.q0 = blockIdx.x * a.qw;
    if constexpr (ND == 0) {
        core::SwarLds L;
        if constexpr (BIG) {
            core::swar_big_layout(a.n, a.qw, &L, smem);
            core::swar_bind_big(&L, a.big, a.n, a.D);
            core::swar_load_colours(a, cs);
        } else {
            core::swar_layout(a.n, a.D, a.row_len, a.qw, &L, smem);
            core::swar_load_instance(L, a, cs);
        }
        if (a.wpl == 2 && a.qw == 2)
            core::swar_run<DK, 2, BIG>(L, a, cs);
        else
            core::swar_run<DK, 1, BIG>(L, a, cs);
    } else if constexpr (BIG) {
        core::SaLds L;
        core::sa_big_layout(a.n, a.row_len, a.qw, &L, smem);
        core::sa_bind_image(&L, a, cs);
        core::sa_run<ND, true, DK>(L, a, cs);
    } else {
        core::SaLds L;
        core::sa_layout(a.n, a.D, a.row_len, a.qw, &L, smem);
        core::sa_load_instance<DK>(L, a, cs);
        core::sa_run<ND, false, DK>(L, a, cs);
    }
}

// Byte-parallel SA with every lane's sites held in registers (see SwarHeld).
template <int DK, int NC>
__global__ __launch_bounds__(1024, NC > 2 ? 4 : 8) void sa_held_kernel(core::SaItem a) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int cs[kMaxColours + 1];
    a.q0 = blockIdx.x * a.qw;
    core::SwarLds L;
    core::swar_big_layout(a.n, a.qw, &L, smem);
    core::swar_load_colours(a, cs);
    core::SwarHeld<DK, NC> held;
    held.load(L, a, cs);
    held.run(L, a, cs, core::SwarChunk());
}

// Streamed byte-parallel SA: resident workgroups take (group of qw quads, chunk of
// sweeps) tasks from a counter in chunk-major order, so that the replicas are
// spread over the whole device however their count divides into workgroups.  A
// group's spin words pass from one chunk to the next through global memory as
// self-validating 32-bit words {tag, spins}, stored and polled with relaxed
// device-scope atomics (tag = chunks done, plus an abandoned-wait bit; the
// words are cleared before every launch), so no cache-wide fence is needed.  A
// spin byte of the byte-parallel body is a mask (0xFF or 0), so a word carries 4
// spin words as 4-bit nibbles under a 16-bit tag.  A task polls (bounded) until
// every word of its group carries the previous chunk's tag.  Every task uses the
// same counters as the one-launch schedule, so the sample is bit-identical.
struct StreamArgs {
    core::SaItem a;
    int G, K, Lc;    // groups, chunks per group, sweeps per chunk
    int *counter;
    uint32_t *state;  // [G][ceil(n qw / 4)] {tag << 16, 4 spin words as nibbles}
    int spin_limit;
};

constexpr uint32_t kTagPoison = 1u << 8;  // tags are chunk counts <= 255 plus this bit

// Spin word (4 mask bytes) <-> nibble (bit b = byte b).
__device__ __forceinline__ uint32_t spin_nibble(uint32_t w) {
    uint32_t m = w & 0x01010101u;
    m |= m >> 7;
    m |= m >> 14;
    return m & 0xFu;
}
__device__ __forceinline__ uint32_t spin_word(uint32_t nib) { return ((nib * 0x00204081u) & 0x01010101u) * 0xFFu; }

// Every branch of a task loop depends on wave-uniform values only (the task
// index is read back with readfirstlane), so that no lane can be split from its
// wave across loop iterations and barriers.
struct StreamShared {
    int task, late, poison;
};

// The next task's index, into LDS.  Ends with a barrier.
__device__ __forceinline__ int stream_pop(const StreamArgs &s, StreamShared *sh) {
    if (__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) == 0) {
        // one increment per workgroup: lane 0 adds 1, the others 0
        const int v = __hip_atomic_fetch_add(s.counter, threadIdx.x == 0 ? 1 : 0, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
        if (threadIdx.x == 0) {
            sh->task = v;
            sh->late = 0;
            sh->poison = 0;
        }
    }
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(sh->task);
}

// Spin words of group g after k chunks into S and ~S, waiting (bounded) for each.
__device__ __forceinline__ void stream_resume(const StreamArgs &s, const core::SwarLds &L, int g, int k,
                                              StreamShared *sh) {
    const int words = s.a.n * s.a.qw, hw = (words + 3) / 4, T = blockDim.x;
    const uint32_t *st = s.state + (size_t)g * (size_t)hw;
    // every word must carry this launch's tag for k chunks done
    const uint32_t want = (uint32_t)k;
    bool late = false, poison = false;
    for (int h = threadIdx.x; h < hw; h += T) {
        uint32_t v = 0;
        for (int spins = 0;; ++spins) {
            v = __hip_atomic_load(st + h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (((v >> 16) & ~kTagPoison) == want) break;
            if (spins >= s.spin_limit) {
                late = true;
                break;
            }
            __builtin_amdgcn_s_sleep(2);
        }
        poison |= ((v >> 16) & kTagPoison) != 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int w = 4 * h + q;
            if (w < words) {
                const uint32_t word = spin_word((v >> (4 * q)) & 0xFu);
                L.S[w] = word;
                L.S[w + words] = ~word;
            }
        }
    }
    if (late) sh->late = 1;
    if (poison) sh->poison = 1;
}

// Task tau's share of the schedule, after its resume and a barrier.
__device__ __forceinline__ core::SwarChunk stream_chunk(const StreamArgs &s, int k, const StreamShared *sh) {
    const bool late = __builtin_amdgcn_readfirstlane(sh->late) != 0;
    core::SwarChunk ch;
    ch.ls0 = k * s.Lc;
    ch.count = min(s.Lc, s.a.sweeps - ch.ls0);
    // An abandoned wait restarts the group from its initial state: words that may
    // still be in flight are not used.
    ch.resume = k > 0 && !late;
    ch.keep = k + 1 < s.K;
    ch.poisoned = late || __builtin_amdgcn_readfirstlane(sh->poison) != 0;
    return ch;
}

// Spin words of group g after chunk k to its next task.
__device__ __forceinline__ void stream_handoff(const StreamArgs &s, const core::SwarLds &L, int g, int k,
                                               bool poisoned) {
    const int words = s.a.n * s.a.qw, hw = (words + 3) / 4, T = blockDim.x;
    uint32_t *st = s.state + (size_t)g * (size_t)hw;
    const uint32_t tag = (poisoned ? kTagPoison : 0u) | (uint32_t)(k + 1);
    for (int h = threadIdx.x; h < hw; h += T) {
        uint32_t pay = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (4 * h + q < words) pay |= spin_nibble(L.S[4 * h + q]) << (4 * q);
        __hip_atomic_store(st + h, (tag << 16) | pay, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

template <int DK, int W, bool BIG = false>
__global__ __launch_bounds__(1024) void sa_stream_kernel(StreamArgs s) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int cs[kMaxColours + 1];
    __shared__ StreamShared sh;
    core::SwarLds L;
    if constexpr (BIG) {
        core::swar_big_layout(s.a.n, s.a.qw, &L, smem);
        core::swar_bind_big(&L, s.a.big, s.a.n, s.a.D);
        core::swar_load_colours(s.a, cs);
    } else {
        core::swar_layout(s.a.n, s.a.D, s.a.row_len, s.a.qw, &L, smem);
        core::swar_load_instance(L, s.a, cs);
    }
    for (;;) {
        const int tau = stream_pop(s, &sh);
        if (tau >= s.G * s.K) break;
        const int g = tau % s.G, k = tau / s.G;
        if (k > 0) stream_resume(s, L, g, k, &sh);
        __syncthreads();
        const core::SwarChunk ch = stream_chunk(s, k, &sh);
        core::SaItem it = s.a;
        it.q0 = g * s.a.qw;
        core::swar_run<DK, W, BIG>(L, it, cs, ch);  // ends with a barrier
        if (ch.keep) stream_handoff(s, L, g, k, ch.poisoned);
    }
}

// The launch's arguments read again from where the kernel received them: a phase that
// takes them from here does not keep them in scalar registers through the phases before.
__device__ __forceinline__ StreamArgs stream_args() {
#ifdef __HIP_DEVICE_COMPILE__
    auto p = (const __attribute__((address_space(4))) StreamArgs *)__builtin_amdgcn_kernarg_segment_ptr();
#ifdef __OPTIMIZE__
    asm volatile("" : "+s"(p));
#endif
    return *p;
#else
    return StreamArgs();
#endif
}

// The same with every lane's sites in registers (see SwarHeld).  Registers for eight
// waves per SIMD at two classes: the sites are read again
// for every task and each phase takes the arguments anew, so that little else is live in
// the sweeps (spilled scalars cost them twelve more vector instructions a word).
template <int DK, int NC>
__global__ __launch_bounds__(1024, NC > 2 ? 4 : 8) void sa_held_stream_kernel(StreamArgs) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int cs[kMaxColours + 1];
    __shared__ StreamShared sh;
    auto layout = [&](const StreamArgs &s) __attribute__((always_inline)) {
        core::SwarLds L;
        core::swar_big_layout(s.a.n, s.a.qw, &L, smem);
        return L;
    };
    core::swar_load_colours(stream_args().a, cs);
    for (;;) {
        {
            const StreamArgs s = stream_args();
            const int tau = stream_pop(s, &sh);
            if (tau >= s.G * s.K) break;
            if (tau >= s.G) stream_resume(s, layout(s), tau % s.G, tau / s.G, &sh);
            __syncthreads();
        }
        core::SwarHeld<DK, NC> held;
        {
            const StreamArgs s = stream_args();
            const int tau = __builtin_amdgcn_readfirstlane(sh.task);
            core::SaItem it = s.a;
            it.q0 = (tau % s.G) * s.a.qw;
            const core::SwarLds L = layout(s);
            held.load(L, it, cs);
            held.sweeps(L, it, stream_chunk(s, tau / s.G, &sh));
        }
        {
            const StreamArgs s = stream_args();
            const int tau = __builtin_amdgcn_readfirstlane(sh.task), g = tau % s.G, k = tau / s.G;
            const core::SwarChunk ch = stream_chunk(s, k, &sh);
            const core::SwarLds L = layout(s);
            core::SaItem it = s.a;
            it.q0 = g * s.a.qw;
            if (ch.keep)
                stream_handoff(s, L, g, k, ch.poisoned);
            else
                held.finish(L, it, ch.poisoned);
            __syncthreads();  // the flags are read before the next task resets them
        }
    }
}

// Task counter and tags back to zero (no word then matches a chunk tag >= 1).
__global__ void stream_reset_kernel(int *counter, uint32_t *state, size_t words) {
    const size_t i0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i0 == 0) *counter = 0;
    for (size_t i = i0; i < words; i += (size_t)gridDim.x * blockDim.x) state[i] = 0u;
}

// The global-memory instance of the byte-parallel body (record addresses relative
// to the spin words).
__global__ __launch_bounds__(256) void big_prep_kernel(core::SaItem a) {
    core::SwarLds L;
    core::swar_bind_big(&L, a.big, a.n, a.D);
    core::swar_build(L.rec, L.co, L.hpos, a, 0u, blockIdx.x * blockDim.x + threadIdx.x, gridDim.x * blockDim.x);
}

// Energies of arbitrary states: one workgroup per 64 rows... one thread per (row, variable).
// Energies of given rows.  2E = sum_i s_i (2 h_i + sum_j J_ij s_j).
// A workgroup stages NR rows in LDS by position, one int16 lane per row (any int8 value
// is exact there), so a neighbour is one LDS read of all its rows and two neighbours
// cost a row one v_perm_b32 and one v_dot2_i32_i16 (|sum| <= 64 * 2^15 * 2^7 < 2^29).
// What it replaces gathered every neighbour's byte from global memory through the
// position map, a row per workgroup: L = 10 cube, 10^4 rows, 96 -> 16 us; L = 20, 5000
// rows, 444 -> 135 us a call.  Bound by each workgroup's reading of the n D records
// through the vector cache.  8 rows a workgroup halve those reads, but leave half the
// workgroups, and measured the same at n = 512 and 1000 and slower at 8000 (158 us).
constexpr int kEnergyRows = 4;

__global__ __launch_bounds__(1024) void energy_rows_kernel(const int32_t *__restrict__ image, int n, int D,
                                                           const int8_t *__restrict__ spins, int R,
                                                           long long *__restrict__ E) {
    constexpr int NR = kEnergyRows;
    extern __shared__ __align__(16) uint32_t row_lds[];
    __shared__ long long part[1024 / 64][NR];
    struct alignas(2 * NR) Rows {
        uint32_t w[NR / 2];
    };
    Rows *sp = reinterpret_cast<Rows *>(row_lds);
    const int tid = threadIdx.x, T = blockDim.x;
    const int r0 = blockIdx.x * NR, nr = min(NR, R - r0);
    const int32_t *pos_of = image + kImgHeader + n;
    const int32_t *hpos = pos_of + n;
    const uint32_t *nbr = reinterpret_cast<const uint32_t *>(hpos + n);
    const int8_t *s = spins + (size_t)r0 * n;
    for (int i = tid; i < n; i += T) {
        int v[NR];
#pragma unroll
        for (int u = 0; u < NR; ++u) v[u] = u < nr ? s[(size_t)u * n + i] : 0;
        Rows x;
#pragma unroll
        for (int u = 0; u < NR / 2; ++u) x.w[u] = ((uint32_t)v[2 * u] & 0xFFFFu) | ((uint32_t)v[2 * u + 1] << 16);
        sp[pos_of[i]] = x;
    }
    __syncthreads();
    long long acc_h[NR] = {}, acc_f[NR] = {};
    for (int p = tid; p < n; p += T) {
        const uint32_t *rec = nbr + (size_t)p * D;
        int32_t F[NR] = {};
        auto pair = [&](uint32_t a, uint32_t b) {
            const dev::i16x2 j = __builtin_bit_cast(dev::i16x2, dev::j_pair(a, b));
            const Rows x = sp[a >> 16], y = sp[b >> 16];
#pragma unroll
            for (int u = 0; u < NR; ++u) {
                const uint32_t w = __builtin_amdgcn_perm(y.w[u / 2], x.w[u / 2], u & 1 ? 0x07060302u : 0x05040100u);
                F[u] = __builtin_amdgcn_sdot2(__builtin_bit_cast(dev::i16x2, w), j, F[u], false);
            }
        };
        int k = 0;
        for (; k + 2 <= D; k += 2) pair(rec[k], rec[k + 1]);
        if (k < D) pair(rec[k], 0u);
        const int h = hpos[p];
        const Rows own = sp[p];
#pragma unroll
        for (int u = 0; u < NR; ++u) {
            const int su = (int)(int16_t)(u & 1 ? own.w[u / 2] >> 16 : own.w[u / 2]);
            acc_h[u] += (long long)su * h;
            acc_f[u] += (long long)su * F[u];
        }
    }
#pragma unroll
    for (int u = 0; u < NR; ++u) {
        long long a = 2 * acc_h[u] + acc_f[u];
        for (int d = 32; d >= 1; d >>= 1) a += __shfl_down(a, d, 64);
        if ((tid & 63) == 0) part[tid >> 6][u] = a;
    }
    __syncthreads();
    if (tid < nr) {
        long long tot = 0;
        for (int w = 0; w < (T >> 6); ++w) tot += part[w][tid];
        E[r0 + tid] = tot / 2;
    }
}

// The same for few rows of few sites, and for problems whose rows do not fit the LDS: a
// row per workgroup, every neighbour gathered from global memory.
__global__ __launch_bounds__(256) void energy_kernel(const int32_t *__restrict__ image, int n,
                                                     int D, const int8_t *__restrict__ spins,
                                                     int R, long long *__restrict__ E) {
    const int r = blockIdx.x;
    if (r >= R) return;
    const int32_t *order = image + kImgHeader;
    const int32_t *hpos = order + 2 * n;
    const uint32_t *nbr = reinterpret_cast<const uint32_t *>(order + 3 * n);
    const int8_t *s = spins + (size_t)r * n;
    long long acc = 0;
    for (int p = threadIdx.x; p < n; p += blockDim.x) {
        const int i = order[p];
        long long f = 2ll * hpos[p];
        for (int k = 0; k < D; ++k) {
            const uint32_t rec = nbr[(size_t)p * D + k];
            const int jp = (int)(rec >> 16);
            f += (long long)(int16_t)(rec & 0xffffu) * s[order[jp]];
        }
        acc += (long long)s[i] * f;
    }
    __shared__ long long part[256 / 64];
    for (int d = 32; d >= 1; d >>= 1) acc += __shfl_down(acc, d, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        long long tot = 0;
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) tot += part[w];
        E[r] = tot / 2;
    }
}

}  // namespace

hipError_t launch_prep(const Inst *P, int32_t *image, hipStream_t s) {
    hipLaunchKernelGGL(prep_order_kernel, dim3(1), dim3(1024), 0, s, P->colour, P->n,
                       P->max_degree, P->n_colours, image);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (P->n > 0) {
        hipLaunchKernelGGL(prep_nbr_kernel, dim3((P->n + 255) / 256), dim3(256), 0, s,
                           P->row_ptr, P->col, P->J, P->h, P->n, P->nnz, P->max_degree, image);
        e = hipGetLastError();
    }
    return e;
}

// The byte-parallel path serves single-digit tables of at most 256 entries
// (x_bound <= 255); SPVAR_NO_SWAR=1 forces the general path (for comparisons).
bool sa_use_swar(int nd, int row_len) {
    static const bool off = [] {
        const char *v = getenv("SPVAR_NO_SWAR");
        return v && v[0] == '1';
    }();
    return nd == 1 && row_len <= 256 && !off;
}

size_t sa_lds_bytes(int n, int D, int row_len, int qw, bool big) {
    if (sa_use_swar(1 + (row_len > kDigitSize ? 1 : 0), row_len))
        return big ? core::swar_big_lds_bytes(n, qw) : core::swar_layout(n, D, row_len, qw, nullptr, nullptr);
    return big ? core::sa_big_layout(n, row_len, qw, nullptr, nullptr)
               : core::sa_layout(n, D, row_len, qw, nullptr, nullptr);
}

size_t sa_held_lds_bytes(int n, int qw) { return core::swar_big_lds_bytes(n, qw); }

static size_t launch_lds(const SaLaunch &L) {
    return L.held ? sa_held_lds_bytes(L.n, L.qw) : sa_lds_bytes(L.n, L.D, L.row_len, L.qw, L.global_instance);
}

size_t sa_big_bytes(int n, int D) { return core::swar_big_bytes(n, D); }

static hipError_t launch_big_prep(const core::SaItem &a, hipStream_t s) {
    const size_t work = (size_t)a.n * (size_t)core::swar_rec_stride(a.D);
    const int grid = (int)std::min<size_t>(4096, std::max<size_t>(1, (work + 255) / 256));
    hipLaunchKernelGGL(big_prep_kernel, dim3(grid), dim3(256), 0, s, a);
    return hipGetLastError();
}

// The kernels of the held-sites body for a launch's record count (4, 6 or 8) and classes.
using HeldFn = void (*)(core::SaItem);
using HeldStreamFn = void (*)(StreamArgs);
template <int DK>
static HeldFn held_fn_of(int C) {
    return C == 2 ? sa_held_kernel<DK, 2> : C == 3 ? sa_held_kernel<DK, 3> : C == 4 ? sa_held_kernel<DK, 4> : nullptr;
}
template <int DK>
static HeldStreamFn held_stream_fn_of(int C) {
    return C == 2   ? sa_held_stream_kernel<DK, 2>
           : C == 3 ? sa_held_stream_kernel<DK, 3>
           : C == 4 ? sa_held_stream_kernel<DK, 4>
                    : nullptr;
}
static HeldFn held_fn(const SaLaunch &L) {
    return L.D == 4 ? held_fn_of<4>(L.C) : L.D == 6 ? held_fn_of<6>(L.C) : L.D == 8 ? held_fn_of<8>(L.C) : nullptr;
}
static HeldStreamFn held_stream_fn(const SaLaunch &L) {
    return L.D == 4   ? held_stream_fn_of<4>(L.C)
           : L.D == 6 ? held_stream_fn_of<6>(L.C)
           : L.D == 8 ? held_stream_fn_of<8>(L.C)
                      : nullptr;
}
hipError_t launch_sa(const SaLaunch &L, hipStream_t s, size_t lds_limit) {
    core::SaItem a;
    a.image = L.image;
    a.tables = L.tables;
    a.init = L.init;
    a.out = L.out;
    a.energies = L.energies;
    a.n = L.n;
    a.D = L.D;
    a.C = L.C;
    a.row_len = L.row_len;
    a.sweeps = L.sweeps;
    a.reads = L.reads;
    a.q0 = 0;
    a.qw = L.qw;
    a.sweep_offset = L.sweep_offset;
    a.wpl = (L.wpl == 2 && L.qw == 2) ? 2 : 1;
    a.k0 = (uint32_t)L.seed;
    a.k1 = (uint32_t)(L.seed >> 32);
    a.big = L.big;
    const bool swar = sa_use_swar(L.nd, L.row_len);
    const bool big = L.global_instance;
    const size_t lds = launch_lds(L);
    if (lds > lds_limit || (big && swar && L.big == nullptr)) return hipErrorInvalidValue;
    const int quads = (L.reads + 3) / 4;
    const int grid = (quads + L.qw - 1) / L.qw;
#define SPV_GEN(ND_, BIG_)                                                                                    \
    do {                                                                                                      \
        if (L.D == 6)                                                                                         \
            hipLaunchKernelGGL((sa_kernel<ND_, 6, BIG_>), dim3(grid), dim3(L.threads), lds, s, a);            \
        else                                                                                                  \
            hipLaunchKernelGGL((sa_kernel<ND_, 0, BIG_>), dim3(grid), dim3(L.threads), lds, s, a);            \
    } while (0)
    if (big && !swar) {
        switch (L.nd) {
            case 1:
                SPV_GEN(1, true);
                break;
            case 2:
                SPV_GEN(2, true);
                break;
            case 3:
                SPV_GEN(3, true);
                break;
            default:
                return hipErrorInvalidValue;
        }
        return hipGetLastError();
    }
    if (big) {
        hipError_t e = launch_big_prep(a, s);
        if (e != hipSuccess) return e;
        if (L.D == 6)
            hipLaunchKernelGGL((sa_kernel<0, 6, true>), dim3(grid), dim3(L.threads), lds, s, a);
        else
            hipLaunchKernelGGL((sa_kernel<0, 0, true>), dim3(grid), dim3(L.threads), lds, s, a);
        return hipGetLastError();
    }
    if (swar && L.held) {
        const HeldFn f = held_fn(L);
        if (!f) return hipErrorInvalidValue;
        hipLaunchKernelGGL(f, dim3(grid), dim3(L.threads), lds, s, a);
        return hipGetLastError();
    }
    switch (sa_use_swar(L.nd, L.row_len) ? 0 : L.nd) {
        case 0:
            if (L.D == 6)
                hipLaunchKernelGGL((sa_kernel<0, 6>), dim3(grid), dim3(L.threads), lds, s, a);
            else if (L.D == 4)
                hipLaunchKernelGGL((sa_kernel<0, 4>), dim3(grid), dim3(L.threads), lds, s, a);
            else if (L.D == 8)
                hipLaunchKernelGGL((sa_kernel<0, 8>), dim3(grid), dim3(L.threads), lds, s, a);
            else
                hipLaunchKernelGGL(sa_kernel<0>, dim3(grid), dim3(L.threads), lds, s, a);
            break;
        case 1:
            SPV_GEN(1, false);
            break;
        case 2:
            SPV_GEN(2, false);
            break;
        case 3:
            SPV_GEN(3, false);
            break;
        default:
            return hipErrorInvalidValue;
    }
#undef SPV_GEN
    return hipGetLastError();
}

template <int DK, int W, bool BIG>
static hipError_t stream_occupancy(int threads, size_t lds, int *per_cu) {
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, sa_stream_kernel<DK, W, BIG>, threads, lds);
}
// Chunks per group: the fewest (sweeps per chunk >= kStreamMinSweeps) whose tasks
// fill the resident workgroups to kStreamFill, else the best filling count.  Every
// chunk boundary moves a group's spin words through global memory once each way.
static int stream_chunks(int G, int sweeps, int resident) {
    constexpr int kStreamMinSweeps = 64, kStreamMaxChunks = 32;
    constexpr double kStreamFill = 0.985;
    int best = 1;
    double best_eff = 0.0;
    for (int K = 1; K <= kStreamMaxChunks && (K == 1 || sweeps / K >= kStreamMinSweeps); ++K) {
        const long long tasks = (long long)G * K;
        const long long rounds = (tasks + resident - 1) / resident;
        const double eff = (double)tasks / (double)(rounds * resident);
        if (eff >= kStreamFill) return K;
        if (eff > best_eff + 1e-3) {
            best_eff = eff;
            best = K;
        }
    }
    return best;
}

size_t sa_stream_bytes(int n, int reads, int qw) {
    const size_t G = (size_t)((reads + 3) / 4 + qw - 1) / (size_t)qw;
    return 256 + G * (((size_t)n * (size_t)qw + 3) / 4) * 4;
}

// Chunks per group for a streamed launch of L, or 1 when the plain launch is used
// (not the byte-parallel body, one wave of workgroups covers the replicas, or a
// short schedule).
int sa_stream_plan(const SaLaunch &L, int num_cus, int force_grid) {
    if (!sa_use_swar(L.nd, L.row_len)) return 1;
    if (force_grid > 0) {  // tests: a given grid, chunk dependencies whatever the shape
        const int K = std::max(2, std::min(32, L.sweeps / 16));
        return L.sweeps >= 2 ? (K | (force_grid << 8)) : 1;
    }
    if (L.sweeps < 128) return 1;
    const int quads = (L.reads + 3) / 4;
    const int G = (quads + L.qw - 1) / L.qw;
    const int W = (L.wpl == 2 && L.qw == 2) ? 2 : 1;
    const bool big = L.global_instance;
    const size_t lds = launch_lds(L);
    const int dk = (L.D == 6 || L.D == 4 || L.D == 8) ? L.D : 0;
    int per_cu = 0;
    hipError_t e;
#define SPV_OCC(D_, W_) e = stream_occupancy<D_, W_, false>(L.threads, lds, &per_cu)
    if (L.held) {
        const HeldStreamFn f = held_stream_fn(L);
        e = f ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, f, L.threads, lds) : hipErrorInvalidValue;
    } else if (big) {
        if (dk == 6) {
            if (W == 2) e = stream_occupancy<6, 2, true>(L.threads, lds, &per_cu);
            else e = stream_occupancy<6, 1, true>(L.threads, lds, &per_cu);
        } else {
            if (W == 2) e = stream_occupancy<0, 2, true>(L.threads, lds, &per_cu);
            else e = stream_occupancy<0, 1, true>(L.threads, lds, &per_cu);
        }
    } else if (W == 2) {
        if (dk == 6) SPV_OCC(6, 2); else if (dk == 4) SPV_OCC(4, 2); else if (dk == 8) SPV_OCC(8, 2); else SPV_OCC(0, 2);
    } else {
        if (dk == 6) SPV_OCC(6, 1); else if (dk == 4) SPV_OCC(4, 1); else if (dk == 8) SPV_OCC(8, 1); else SPV_OCC(0, 1);
    }
#undef SPV_OCC
    const int resident = per_cu * num_cus;
    if (e != hipSuccess || resident <= 0 || G <= resident) return 1;
    // Held sites: a last round that is half empty or less runs about as fast in one launch,
    // its workgroups having the CUs almost to themselves (1250 workgroups on 1024 resident,
    // N = 1000, 500 sweeps: 1.43 ms, streamed 1.58; on 512 resident, N = 1728: 3.39, streamed
    // 2.62).
    if (L.held && 2 * G < 3 * resident) return 1;
    const char *kv = getenv("SPVAR_SA_CHUNKS");  // tuning: a fixed chunk count
    const int K = kv && atoi(kv) > 0 ? std::min(255, atoi(kv)) : stream_chunks(G, L.sweeps, resident);
    return K <= 1 ? 1 : (K | (resident << 8));
}

int sa_stream_chunks_of(const SaLaunch &L, int plan) {
    const int K0 = plan & 0xff;
    const int Lc = (L.sweeps + K0 - 1) / K0;
    return (L.sweeps + Lc - 1) / Lc;
}

hipError_t launch_sa_stream(const SaLaunch &L, int plan, void *buf, hipStream_t s) {
    const int K0 = plan & 0xff, resident = plan >> 8;
    const int quads = (L.reads + 3) / 4;
    const int G = (quads + L.qw - 1) / L.qw;
    const int W = (L.wpl == 2 && L.qw == 2) ? 2 : 1;
    const bool big = L.big != nullptr;
    const size_t lds = launch_lds(L);
    const int dk = (L.D == 6 || L.D == 4 || L.D == 8) ? L.D : 0;
    StreamArgs a;
    a.a.image = L.image;
    a.a.tables = L.tables;
    a.a.init = L.init;
    a.a.out = L.out;
    a.a.energies = L.energies;
    a.a.n = L.n;
    a.a.D = L.D;
    a.a.C = L.C;
    a.a.row_len = L.row_len;
    a.a.sweeps = L.sweeps;
    a.a.reads = L.reads;
    a.a.q0 = 0;
    a.a.qw = L.qw;
    a.a.sweep_offset = L.sweep_offset;
    a.a.k0 = (uint32_t)L.seed;
    a.a.k1 = (uint32_t)(L.seed >> 32);
    a.a.wpl = W;
    a.a.big = L.big;
    a.G = G;
    a.Lc = (L.sweeps + K0 - 1) / K0;
    a.K = (L.sweeps + a.Lc - 1) / a.Lc;
    unsigned char *b = static_cast<unsigned char *>(buf);
    a.counter = reinterpret_cast<int *>(b);
    a.state = reinterpret_cast<uint32_t *>(b + 256);
    a.spin_limit = L.spin_limit;
    const size_t words = (size_t)G * (((size_t)L.n * (size_t)L.qw + 3) / 4);
    const int rgrid = (int)std::min<size_t>(1024, std::max<size_t>(1, (words + 255) / 256));
    hipLaunchKernelGGL(stream_reset_kernel, dim3(rgrid), dim3(256), 0, s, a.counter, a.state, words);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int grid = std::min(resident, G * a.K);
    if (L.held) {
        const HeldStreamFn f = held_stream_fn(L);
        if (!f) return hipErrorInvalidValue;
        hipLaunchKernelGGL(f, dim3(grid), dim3(L.threads), lds, s, a);
        return hipGetLastError();
    }
    if (big) {
        e = launch_big_prep(a.a, s);
        if (e != hipSuccess) return e;
        if (dk == 6) {
            if (W == 2) hipLaunchKernelGGL((sa_stream_kernel<6, 2, true>), dim3(grid), dim3(L.threads), lds, s, a);
            else hipLaunchKernelGGL((sa_stream_kernel<6, 1, true>), dim3(grid), dim3(L.threads), lds, s, a);
        } else {
            if (W == 2) hipLaunchKernelGGL((sa_stream_kernel<0, 2, true>), dim3(grid), dim3(L.threads), lds, s, a);
            else hipLaunchKernelGGL((sa_stream_kernel<0, 1, true>), dim3(grid), dim3(L.threads), lds, s, a);
        }
        return hipGetLastError();
    }
#define SPV_GO(D_, W_) hipLaunchKernelGGL((sa_stream_kernel<D_, W_>), dim3(grid), dim3(L.threads), lds, s, a)
    if (W == 2) {
        if (dk == 6) SPV_GO(6, 2); else if (dk == 4) SPV_GO(4, 2); else if (dk == 8) SPV_GO(8, 2); else SPV_GO(0, 2);
    } else {
        if (dk == 6) SPV_GO(6, 1); else if (dk == 4) SPV_GO(4, 1); else if (dk == 8) SPV_GO(8, 1); else SPV_GO(0, 1);
    }
#undef SPV_GO
    return hipGetLastError();
}

// LDS of the rows of one workgroup: to n = 16384.  Few sites take small workgroups (more
// of them on a CU: n = 64, 10^4 rows, 44 us a call with 256 threads, 60 with 1024), many
// sites large ones, which share the one copy of the rows (n = 8000, 5000 rows: 158 us
// with 1024, 304 with 256).
constexpr size_t kEnergyLds = 128 * 1024;

hipError_t launch_energy(const int32_t *image, int n, int D, const int8_t *spins, int R,
                         int64_t *E, hipStream_t s) {
    if (R <= 0) return hipSuccess;
    long long *e = reinterpret_cast<long long *>(E);
    const size_t lds = (size_t)n * 2 * kEnergyRows;
    // Few rows of few sites: a row per workgroup has every gather in flight at once and no
    // barrier after staging (kernel trace, median us, row / four rows a workgroup: n = 64, 137
    // rows 4.05 / 4.7; n = 125, 137 rows 4.2 / 4.7; n = 288, 1000 rows 6.0 / 6.3; n = 512, 300
    // rows 5.8 / 6.3; n = 512, 1000 rows 7.0 / 6.6; a call at n = 512, 4000 rows 51.5 / 43.8).
    if (lds > kEnergyLds || (n <= 512 && R <= 1024))
        hipLaunchKernelGGL(energy_kernel, dim3(R), dim3(256), 0, s, image, n, D, spins, R, e);
    else
        hipLaunchKernelGGL(energy_rows_kernel, dim3((unsigned)((R + kEnergyRows - 1) / kEnergyRows)),
                           dim3(n <= 1024 ? 256 : n <= 4096 ? 512 : 1024), lds, s, image, n, D, spins, R, e);
    return hipGetLastError();
}

hipError_t shadow_stats_sa(unsigned long long *out, bool reset) { return shadow::read_stats(out, reset); }

}  // namespace spv
