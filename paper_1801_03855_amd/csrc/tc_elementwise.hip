// K-way reduction and fused elastic-averaging SGD step over flat copies.
//
// Both are streams over the flat index space with no reuse: every input is
// read once and every output written once, so they are bound by HBM
// bandwidth (well under one flop per byte) and use no matrix cores.
//
// Mapping: a tile is 64 16-byte slots (4 binary32 values; 4 bfloat16
// gradients are 8 bytes), so each wave instruction moves 1 KiB (512 B) of
// contiguous memory of one buffer.  The copies are split over the waves of a
// workgroup, one copy to a wave where K is small enough (reduce_copies,
// launch_step), and the K-way sums meet in LDS.  Non-temporal loads and
// stores, since nothing is re-read; only the center, which every wave of a
// tile reads, is loaded cacheably.
//
// What bounds these kernels is how the memory takes 2K + 1 read and K + 1
// write streams at once.  A workgroup of one worker per wave reads 1 KiB of
// each and is gone; a lane that owned one or two slots of all K copies (the
// earlier mapping, 152 VGPRs and 34 loads in flight per lane at K = 8) moved 4
// to 8 KiB of each stream per workgroup at 10 waves per CU, so the workgroups
// running at one time were spread over 5 to 10 times as much of every buffer.
// Measured on MI355X over three sets of buffers in turn, 25 M elements, GB/s
// before and now: fused step K = 2 5,942 -> 6,275, K = 4 5,717 -> 6,493, K = 8
// 5,426 -> 6,525, K = 16 5,198 -> 6,400, K = 32 4,923 -> 6,060; with the
// gradients' average K = 8 5,278 -> 6,440; bfloat16 gradients K = 8 5,477 ->
// 6,354; the 138 M element group at K = 4 5,483 -> 6,130.  Two or four tiles
// per workgroup, and runs of tiles kept on one XCD, measured 3-15% slower.
//
// A ragged tail of fewer than 4 elements is taken element by element by a
// workgroup of its own.  Buffers that are not aligned to their slots (16 bytes
// of binary32, 8 of bfloat16) take the same kernels with unaligned accesses.
//
// The K terms are summed by a pairwise tree (adjacent pairs, level by level,
// an odd last term carried up) for K <= 16; larger K is summed as trees of 16
// (zero-padded) combined by a tree of the four partials (zero-padded).
#include <type_traits>

#include "tc_internal.h"

#ifndef TC_EW_THREADS
#define TC_EW_THREADS 256
#endif
#ifndef TC_NT_LOADS
#define TC_NT_LOADS 1
#endif
#ifndef TC_NT_STORES
#define TC_NT_STORES 1
#endif

namespace tc {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef unsigned int u2 __attribute__((ext_vector_type(2)));
typedef unsigned int u4 __attribute__((ext_vector_type(4)));

constexpr int kSpecialisedK = 16;

// ---------------------------------------------------------------- memory

template <typename T>
__device__ __forceinline__ T ld(const T* p) {
#if TC_NT_LOADS
    return __builtin_nontemporal_load(p);
#else
    return *p;
#endif
}

template <typename T>
__device__ __forceinline__ void st(T* p, T v) {
#if TC_NT_STORES
    __builtin_nontemporal_store(v, p);
#else
    *p = v;
#endif
}

// bfloat16 -> binary32 is exact: the bfloat16 code is the upper half of the
// binary32 code.
__device__ __forceinline__ float bf16_lo(unsigned int w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(unsigned int w) { return __uint_as_float(w & 0xffff0000u); }
__device__ __forceinline__ f4 widen(u2 w) { return f4{bf16_lo(w.x), bf16_hi(w.x), bf16_lo(w.y), bf16_hi(w.y)}; }

// How a lane reaches its item of a buffer: a slot of four elements, aligned to
// its own bytes (Slot) or to its elements only (SlotAny), or one element (Elem).
// V is its value in registers, the index counts items.  Index type I is uint32_t
// when every buffer is below 4 GiB: the address is then a uniform 64-bit base
// plus one 32-bit byte offset that all streams share, which the compiler emits
// as SGPR-base + VGPR-offset loads and stores instead of one 64-bit VGPR address
// per stream.
template <typename I>
__device__ __forceinline__ const char* at(const void* p, I byte_off) {
    return static_cast<const char*>(p) + byte_off;
}

struct Slot {
    typedef f4 V;
    static constexpr int kFloats = 4;
    template <typename I> static __device__ __forceinline__ f4 load_cached(const float* p, I i) {
        return *reinterpret_cast<const f4*>(at(p, i * I(16)));
    }
    template <typename I> static __device__ __forceinline__ f4 load(const float* p, I i) {
        return ld(reinterpret_cast<const f4*>(at(p, i * I(16))));
    }
    template <typename I> static __device__ __forceinline__ f4 load(const uint16_t* p, I i) {
        return widen(ld(reinterpret_cast<const u2*>(at(p, i * I(8)))));
    }
    template <typename I> static __device__ __forceinline__ void store(float* p, I i, f4 v) {
        st(reinterpret_cast<f4*>(const_cast<char*>(at(p, i * I(16)))), v);
    }
    // two bfloat16 slots, on a slot's boundary
    typedef u4 Two __attribute__((aligned(8)));
    template <typename I> static __device__ __forceinline__ u4 load_two(const uint16_t* p, I i) {
        return __builtin_nontemporal_load(reinterpret_cast<const Two*>(at(p, i * I(8))));
    }
};

// Global memory is accessed in unaligned mode on gfx950: a slot that starts on
// any element is one access all the same.  Cacheable, since neighbouring waves
// share lines.  Measured on MI355X, buffers one element past a boundary, 3 M
// elements, and with one element per lane: step K = 8 59.3 us (98.6),
// asynchronous exchange K = 5 27.6 (63.3), bfloat16 reduction K = 17 27.2
// (55.2).  Over K = 1 to 48 and 10 thousand to 24 million elements
// non-temporal loads and stores were 5% slower, non-temporal stores level.
struct SlotAny {
    typedef f4 V;
    typedef f4 F __attribute__((aligned(4)));
    typedef u2 H __attribute__((aligned(2)));
    typedef u4 Two __attribute__((aligned(2)));
    static constexpr int kFloats = 4;
    template <typename I> static __device__ __forceinline__ f4 load_cached(const float* p, I i) {
        return *reinterpret_cast<const F*>(at(p, i * I(16)));
    }
    template <typename I> static __device__ __forceinline__ f4 load(const float* p, I i) {
        return *reinterpret_cast<const F*>(at(p, i * I(16)));
    }
    template <typename I> static __device__ __forceinline__ f4 load(const uint16_t* p, I i) {
        return widen(*reinterpret_cast<const H*>(at(p, i * I(8))));
    }
    template <typename I> static __device__ __forceinline__ void store(float* p, I i, f4 v) {
        *reinterpret_cast<F*>(const_cast<char*>(at(p, i * I(16)))) = v;
    }
    template <typename I> static __device__ __forceinline__ u4 load_two(const uint16_t* p, I i) {
        return *reinterpret_cast<const Two*>(at(p, i * I(8)));
    }
};

struct Elem {
    typedef float V;
    static constexpr int kFloats = 1;
    template <typename I> static __device__ __forceinline__ float load_cached(const float* p, I i) {
        return *reinterpret_cast<const float*>(at(p, i * I(4)));
    }
    template <typename I> static __device__ __forceinline__ float load(const float* p, I i) {
        return ld(reinterpret_cast<const float*>(at(p, i * I(4))));
    }
    template <typename I> static __device__ __forceinline__ float load(const uint16_t* p, I i) {
        return __uint_as_float(static_cast<unsigned int>(ld(reinterpret_cast<const uint16_t*>(at(p, i * I(2))))) << 16);
    }
    template <typename I> static __device__ __forceinline__ void store(float* p, I i, float v) {
        st(reinterpret_cast<float*>(const_cast<char*>(at(p, i * I(4)))), v);
    }
};

// Output stores with explicit cache-policy bits (bit 0 sc0, bit 1 nt, bit 4
// sc1), as raw buffer stores when offsets are 32-bit; a negative policy
// keeps the plain non-temporal global store.  Measured on MI355X for the
// reduction's output, sc1 against nt, three sets of buffers in turn: K = 1
// 6,501 against 6,363 GB/s and K = 2 6,515 against 6,258, but K = 3 6,526
// against 6,842 and K = 4 6,691 against 6,879; bfloat16 inputs K = 1 5,840
// against 5,288, K = 8 6,513 against 5,975.
constexpr int kReduceStoreSc1 = 16, kStoreNt = -1;

template <int AUX, typename M, typename I>
__device__ __forceinline__ void store_pol(float* p, I i, f4 v, uint32_t bytes) {
    if constexpr (AUX >= 0 && sizeof(I) == 4 && std::is_same_v<M, Slot>) {
        const __amdgpu_buffer_rsrc_t r =
            __builtin_amdgcn_make_buffer_rsrc(p, static_cast<short>(0), static_cast<int>(bytes), 0x00020000);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, v), r, i * 16u, 0, AUX);
    } else {
        M::store(p, i, v);
    }
}

// ------------------------------------------------------------ arithmetic

__device__ __forceinline__ float fmav(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ f4 fmav(f4 a, f4 b, f4 c) {
    return f4{__builtin_fmaf(a.x, b.x, c.x), __builtin_fmaf(a.y, b.y, c.y),
              __builtin_fmaf(a.z, b.z, c.z), __builtin_fmaf(a.w, b.w, c.w)};
}
template <typename V> __device__ __forceinline__ V splat(float s) { return V(s); }

// Pairwise tree over v[0..M): adjacent pairs level by level; an odd last
// element moves up unchanged.  Overwrites v.
template <int M> struct Tree {
    template <typename V> static __device__ __forceinline__ V sum(V* v) {
#pragma unroll
        for (int p = 0; p < M / 2; ++p) v[p] = v[2 * p] + v[2 * p + 1];
        if constexpr (M & 1) v[M / 2] = v[M - 1];
        return Tree<(M + 1) / 2>::sum(v);
    }
};
template <> struct Tree<1> {
    template <typename V> static __device__ __forceinline__ V sum(V* v) { return v[0]; }
};

// ---------------------------------------------------------------- grid

// The workgroup's place in a grid that may go on along y (grid_of).  Workgroups
// past the items do nothing.
template <typename I>
__device__ __forceinline__ I block_index() {
    return static_cast<I>(blockIdx.y) * static_cast<I>(gridDim.x) + static_cast<I>(blockIdx.x);
}
// The elements after the last of `items` whole slots are a workgroup's of their
// own, the one after the last tile's, so that a small group does not wait for
// two passes: lane's element in block `b` (past n in the blocks after it).
template <typename I>
__device__ __forceinline__ I tail_element(I b, I items, int per_block, int lane) {
    const I tiles = (items + static_cast<I>(per_block - 1)) / static_cast<I>(per_block);
    return I(4) * items + (b - tiles) * static_cast<I>(per_block) + static_cast<I>(lane);
}

// --------------------------------------------------------------- waves
//
// The K copies of a tile of slots are split over the waves of a workgroup,
// B copies to a wave, and the waves' terms meet in LDS.

struct Wave {
    int w;        // the wave's place among its tile's
    int waves;    // how many those are: W, or fewer in the kernels for K > 16
    int row;      // the tile's place in the workgroup
    int lane;
    int threads;  // of the workgroup
};

// The kernels for K > 16 (K == TC_MAX_K here) are given the number of copies
// when they are launched.  Their sums are trees of 16 copies, zero-padded,
// combined as (p0 + p1) + (p2 + p3).
static_assert(TC_MAX_K == 4 * kSpecialisedK, "four groups of 16 copies");

// Whether copy b of a wave's B exists.
template <int K, int B>
__device__ __forceinline__ bool has_copy(int w, int b, int k_total) {
    if constexpr (K == TC_MAX_K) return w * B + b < k_total;
    else return K % B == 0 || w * B + b < K;
}

// Runs f(b) for the wave's copies, straight through for each number of them:
// a load under a condition of its own can compile to a branch around it and a
// wait for it.
template <int N, typename F>
__device__ __forceinline__ void each_of(int count, F f) {
    if (count == N) {
#pragma unroll
        for (int b = 0; b < N; ++b) f(b);
    } else if constexpr (N > 1) {
        each_of<N - 1>(count, f);
    }
}
template <int K, int B, typename F>
__device__ __forceinline__ void each_copy(int w, int k_total, F f) {
    const int left = (K == TC_MAX_K ? k_total : K) - w * B;
    if (left >= B) {
#pragma unroll
        for (int b = 0; b < B; ++b) f(b);
    } else if constexpr (K == TC_MAX_K) {
        if constexpr (B > 1) each_of<B - 1>(left, f);
    } else {
#pragma unroll
        for (int b = 0; b < K % B; ++b) f(b);
    }
}

// A wave's term of the K-way sum: B is a power of two, so the tree over its
// copies is a subtree of Tree<K>'s; a last wave of fewer copies takes theirs.
// For K > 16 the copies past k_total are the caller's +0.
template <int K, int W, int B, typename V>
__device__ __forceinline__ V copies_sum(V* v, int w) {
    constexpr int L = K - (W - 1) * B;
    if constexpr (K != TC_MAX_K && L < B)
        if (w == W - 1) return Tree<L>::sum(v);
    return Tree<B>::sum(v);
}

// The sum of the waves' terms, in rows of `stride` values.  For K > 16 it is
// the tree over W * B zero-padded copies, and for W * B = 32 the third and
// the fourth group's sum is the +0 added last.
template <int K, int W, int B, typename V>
__device__ __forceinline__ V waves_sum(const V* sh, int stride, int waves) {
    V p[W];
#pragma unroll
    for (int k = 0; k < W; ++k) p[k] = (K < TC_MAX_K || k < waves) ? sh[k * stride] : splat<V>(0.0f);
    V s = Tree<W>::sum(p);
    if constexpr (K == TC_MAX_K && W * B == 2 * kSpecialisedK) s = s + splat<V>(0.0f);
    return s;
}

// --------------------------------------------------------------- reduce

template <int K, typename T>
struct ReduceArgs {
    const T* in[K];
    float* out;
    uint32_t out_bytes;  // size of out when below 4 GiB
    int op;
    int k_total;  // the number of copies (== K except in the generic kernel)
};

template <int K, typename V, typename T>
__device__ __forceinline__ V quotient(const ReduceArgs<K, T>& a, V s) {
    return a.op == TC_AVG ? s / splat<V>(static_cast<float>(K == TC_MAX_K ? a.k_total : K)) : s;
}

// ---------------------------------------------------------------- easgd

template <int K, typename T>
struct EasgdArgs {
    float* x[K];
    const T* g[K];
    float* xc;
    float eta, rho, a;  // a = eta*rho rounded to binary32
    int k_total;
    static constexpr bool kReduce = false;
};

// The step fused with the K-way reduction of the gradients it reads: out =
// the SUM (or AVG) of g_0 .. g_{K-1}, by the reduction's own tree and
// quotient, so the result is bit for bit that of the reduction call.
template <int K, typename T>
struct ReduceEasgdArgs : EasgdArgs<K, T> {
    float* out;
    int op;
    static constexpr bool kReduce = true;
};

// Every wave reads the tile's center (once from HBM: the waves of a tile run
// together and those loads may stay in the caches), or, with up to four waves,
// takes it from LDS (138 M elements, K = 4: 6,231 GB/s against 6,076; K = 8
// 6,409 against 6,567).  The workers are stored before the sums are formed; wave 0 then
// stores the center and, fused with the reduction, the last wave the
// gradients' sum or average.
template <int K, int W, int B, typename M, typename I, typename A>
__device__ __forceinline__ void easgd_wave(const A& a, I i, bool active, const Wave& q, typename M::V* sh) {
    typedef typename M::V V;
    constexpr bool kStageC = W >= 2 && W <= 4;
    const int me = (q.row * W + q.w) * 64 + q.lane;
    V* const gsh = sh + q.threads;
    V* const csh = gsh + (A::kReduce ? q.threads : 0);
    V c = splat<V>(0.0f), x[B], g[B];
    if (active) {
        if constexpr (W == 1) c = M::load(a.xc, i);
        else if constexpr (!kStageC) c = M::load_cached(a.xc, i);
        each_copy<K, B>(q.w, a.k_total, [&](int b) {
            x[b] = M::load(a.x[q.w * B + b], i);
            g[b] = M::load(a.g[q.w * B + b], i);
        });
    }
    if constexpr (kStageC) {
        if (q.w == 0 && active) csh[q.row * 64 + q.lane] = M::load(a.xc, i);
        __syncthreads();
        c = csh[q.row * 64 + q.lane];
    }
    if (active) {
        V d[B];
#pragma unroll
        for (int b = 0; b < B; ++b) {
            if (has_copy<K, B>(q.w, b, a.k_total)) {
                d[b] = x[b] - c;
                M::store(a.x[q.w * B + b], i,
                              fmav(splat<V>(-a.eta), fmav(splat<V>(a.rho), d[b], g[b]), x[b]));
            } else {
                d[b] = splat<V>(0.0f);
                g[b] = splat<V>(0.0f);
            }
        }
        sh[me] = copies_sum<K, W, B>(d, q.w);
        if constexpr (A::kReduce) gsh[me] = copies_sum<K, W, B>(g, q.w);
    }
    if constexpr (W > 1) __syncthreads();
    if (!active) return;
    const int at = q.row * W * 64 + q.lane;
    if (q.w == 0) M::store(a.xc, i, fmav(splat<V>(a.a), waves_sum<K, W, B>(sh + at, 64, q.waves), c));
    if constexpr (A::kReduce) {
        if (q.w == q.waves - 1) {
            V s = waves_sum<K, W, B>(gsh + at, 64, q.waves);
            if (a.op == TC_AVG) s = s / splat<V>(static_cast<float>(K == TC_MAX_K ? a.k_total : K));
            M::store(a.out, i, s);
        }
    }
}

// ---------------------------------------------------- sgd / sync / async

// Plain SGD on every worker: x_i = fma(-eta, g_i, x_i).  No worker's update
// needs another's, so every workgroup takes TC_EW_THREADS slots of one worker
// and the grid goes through the workers one after the other.
template <int K, typename T>
struct SgdArgs {
    float* x[K];
    const T* g[K];
    float eta;
};

template <typename M, typename T, typename I>
__device__ __forceinline__ void sgd_one(float* x, const T* g, float eta, I i) {
    typedef typename M::V V;
    const V xv = M::load(x, i), gv = M::load(g, i);
    M::store(x, i, fmav(splat<V>(-eta), gv, xv));
}

// One slot per lane; items: slots of a worker.
template <int K, typename T, typename M, typename I>
__global__ __launch_bounds__(TC_EW_THREADS) void sgd_kernel(SgdArgs<K, T> a, I items, I n) {
    const I b = block_index<I>(), i = b * TC_EW_THREADS + threadIdx.x;
    float* const x = a.x[blockIdx.z];
    const T* const g = a.g[blockIdx.z];
    if (b * TC_EW_THREADS < items) {
        if (i < items) sgd_one<M>(x, g, a.eta, i);
    } else {
        const I j = tail_element(b, items, TC_EW_THREADS, threadIdx.x);
        if (j < n) sgd_one<Elem>(x, g, a.eta, j);
    }
}

// Synchronous SGD through pushpull: S = pairwise sum of the K gradients,
// x_i = fma(-eta*rescale, S, x_i) for every worker, and, when broadcast,
// g_i = S (binary32 gradients only).
template <int K, typename T>
struct SyncArgs {
    float* x[K];
    T* g[K];
    float step;  // eta * rescale, rounded once to binary32
    int broadcast;
    int k_total;
};

template <int K, int W, int B, typename T, typename M, typename I>
__device__ __forceinline__ void sync_wave(const SyncArgs<K, T>& a, I i, bool active, const Wave& q, typename M::V* sh) {
    typedef typename M::V V;
    V x[B];
    if (active) {
        V g[B];
        each_copy<K, B>(q.w, a.k_total, [&](int b) {
            g[b] = M::load(static_cast<const T*>(a.g[q.w * B + b]), i);
            x[b] = M::load(static_cast<const float*>(a.x[q.w * B + b]), i);
        });
        if constexpr (K == TC_MAX_K) {
#pragma unroll
            for (int b = 0; b < B; ++b) g[b] = has_copy<K, B>(q.w, b, a.k_total) ? g[b] : splat<V>(0.0f);
        }
        sh[(q.row * W + q.w) * 64 + q.lane] = copies_sum<K, W, B>(g, q.w);
    }
    if constexpr (W > 1) __syncthreads();
    if (!active) return;
    const V S = waves_sum<K, W, B>(sh + q.row * W * 64 + q.lane, 64, q.waves);
#pragma unroll
    for (int b = 0; b < B; ++b) {
        const int k = q.w * B + b;
        if (has_copy<K, B>(q.w, b, a.k_total)) {
            M::store(a.x[k], i, fmav(splat<V>(-a.step), S, x[b]));
            if constexpr (sizeof(T) == 4)
                if (a.broadcast) M::store(a.g[k], i, S);
        }
    }
}

// Asynchronous elastic exchanges: for r < R, with x[r] the r-th exchanged
// worker (no worker twice): d = x_r - c; c = fma(alpha, d, c);
// x_r = fma(-alpha, d, x_r).
template <int K, typename T>
struct AsyncArgs {
    float* x[K];  // the exchanged workers, in their order
    float* xc;
    int R;
    float alpha;
    int k_total;
};

// Wave w holds the workers of the exchanges w*B .. w*B + B - 1 and puts their
// values in rows of LDS.  Each of the tile's 64 * kFloats elements then has
// its recurrence over the R rows run by one lane, 16 rows at a time (read,
// exchanged, written back), and the waves store their rows.  end: the
// elements there are.
template <int K, int W, int B, typename M, typename I, typename T>
__device__ __forceinline__ void async_wave(const AsyncArgs<K, T>& a, I i, bool active, const Wave& q, typename M::V* sh,
                                           I end) {
    constexpr int E = 64 * M::kFloats;
    constexpr int kLeast = K < TC_MAX_K ? 64 * W : 64 * ((kSpecialisedK + B) / B);  // threads launched
    constexpr int C = (E + kLeast - 1) / kLeast;                                    // recurrences per lane
    constexpr int G = K < kSpecialisedK ? K : kSpecialisedK;
    const int r0 = q.w * B;
    if (active) {
#pragma unroll
        for (int b = 0; b < B; ++b)
            if (r0 + b < a.R)
                sh[(r0 + b) * 64 + q.lane] = M::load(static_cast<const float*>(a.x[r0 + b]), i);
    }
    const I e0 = (i - static_cast<I>(q.lane)) * I(M::kFloats);
    float c[C];
#pragma unroll
    for (int k = 0; k < C; ++k) {
        const int e = static_cast<int>(threadIdx.x) + k * q.threads;
        c[k] = e < E && e0 + I(e) < end ? Elem::load(static_cast<const float*>(a.xc), e0 + I(e)) : 0.0f;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < C; ++k) {
        const int e = static_cast<int>(threadIdx.x) + k * q.threads;
        if (e < E) {
            float* row = reinterpret_cast<float*>(sh) + e;
            for (int r1 = 0; r1 < a.R; r1 += G, row += G * E) {
                float x[G];
#pragma unroll
                for (int r = 0; r < G; ++r)
                    if (r1 + r < a.R) x[r] = row[r * E];
#pragma unroll
                for (int r = 0; r < G; ++r)
                    if (r1 + r < a.R) {
                        const float d = x[r] - c[k];
                        c[k] = fmav(a.alpha, d, c[k]);
                        row[r * E] = fmav(-a.alpha, d, x[r]);
                    }
            }
            if (e0 + I(e) < end) Elem::store(a.xc, e0 + I(e), c[k]);
        }
    }
    __syncthreads();
    if (active) {
#pragma unroll
        for (int b = 0; b < B; ++b)
            if (r0 + b < a.R) M::store(a.x[r0 + b], i, sh[(r0 + b) * 64 + q.lane]);
    }
}

// More than 32 workers: rows for all of them in LDS would leave two or three
// tiles per CU (K = 48: 5.1 TB/s; of half the slots, 4.1), so a lane holds one
// slot and takes the exchanges in turn.  Large groups: one at a time, each store
// done before the next load, so that the workgroups stay with the same few
// workers' buffers (K = 48, 3 M elements: 1.02 times as fast as without the wait,
// 1.11 as with eight loads ahead).  Below kAsyncAhead elements, where the
// buffers are in the caches and the chip is not full, the exchanges' latencies
// are the time, and AHEAD = 8 loads go before them (K = 48: 10,007 elements 31.6
// -> 10.1 us, 100,003 35.7 -> 12.0, 300,007 52 -> 26, 900,001 71 -> 70).
constexpr int64_t kAsyncAhead = 1000000;

template <typename M, int AHEAD, typename I, typename T>
__device__ __forceinline__ void async_lane(const AsyncArgs<TC_MAX_K, T>& a, I i) {
    typedef typename M::V V;
    V c = M::load(static_cast<const float*>(a.xc), i);
#pragma unroll 1
    for (int r = 0; r < a.R; r += AHEAD) {
        V x[AHEAD];
#pragma unroll
        for (int u = 0; u < AHEAD; ++u)  // past the last: the last again, not used
            x[u] = M::load(static_cast<const float*>(a.x[r + u < a.R ? r + u : a.R - 1]), i);
#pragma unroll
        for (int u = 0; u < AHEAD; ++u)
            if (r + u < a.R) {
                const V d = x[u] - c;
                c = fmav(splat<V>(a.alpha), d, c);
                M::store(a.x[r + u], i, fmav(splat<V>(-a.alpha), d, x[u]));
            }
        if constexpr (AHEAD == 1) __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
    }
    M::store(a.xc, i, c);
}

template <int AHEAD, typename T, typename M, typename I>
__global__ __launch_bounds__(TC_EW_THREADS) void async_lane_kernel(AsyncArgs<TC_MAX_K, T> a, I items, I n) {
    const I b = block_index<I>(), i = b * TC_EW_THREADS + threadIdx.x;
    if (b * TC_EW_THREADS < items) {
        if (i < items) async_lane<M, AHEAD, I>(a, i);
    } else {
        const I j = tail_element(b, items, TC_EW_THREADS, threadIdx.x);
        if (j < n) async_lane<Elem, AHEAD, I>(a, j);
    }
}

// -------------------------------------------------------------- kernels

// The operation is selected by the argument type.
template <int K, int W, int B, typename M, typename I, typename T>
__device__ __forceinline__ void op_wave(const EasgdArgs<K, T>& a, I i, bool active, const Wave& q, typename M::V* sh, I) {
    easgd_wave<K, W, B, M, I>(a, i, active, q, sh);
}
template <int K, int W, int B, typename M, typename I, typename T>
__device__ __forceinline__ void op_wave(const ReduceEasgdArgs<K, T>& a, I i, bool active, const Wave& q, typename M::V* sh, I) {
    easgd_wave<K, W, B, M, I>(a, i, active, q, sh);
}
template <int K, int W, int B, typename M, typename I, typename T>
__device__ __forceinline__ void op_wave(const SyncArgs<K, T>& a, I i, bool active, const Wave& q, typename M::V* sh, I) {
    sync_wave<K, W, B, T, M, I>(a, i, active, q, sh);
}
template <int K, int W, int B, typename M, typename I, typename T>
__device__ __forceinline__ void op_wave(const AsyncArgs<K, T>& a, I i, bool active, const Wave& q, typename M::V* sh, I end) {
    async_wave<K, W, B, M, I>(a, i, active, q, sh, end);
}

extern __shared__ __align__(16) char wave_rows[];

// ROWS tiles of 64 slots per workgroup, W waves to a tile; items: the slots.
template <int K, int W, int B, int ROWS, typename T, typename M, typename I, template <int, typename> class Args>
__global__ __launch_bounds__(64 * W * ROWS) void wave_kernel(Args<K, T> a, I items, I n) {
    Wave q;
    q.threads = K == TC_MAX_K ? static_cast<int>(blockDim.x) : 64 * W * ROWS;
    q.waves = q.threads / (64 * ROWS);
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
    q.w = ROWS == 1 ? wave : wave % W;
    q.row = ROWS == 1 ? 0 : wave / W;
    q.lane = static_cast<int>(threadIdx.x) & 63;
    const I b = block_index<I>(), i0 = b * (64 * ROWS);
    const int own = q.row * 64 + q.lane;
    if (i0 < items) {
        const I i = i0 + static_cast<I>(own);
        op_wave<K, W, B, M, I>(a, i, i < items, q, reinterpret_cast<f4*>(wave_rows), I(4) * items);
    } else {
        const I j = tail_element(b, items, 64 * ROWS, own);
        op_wave<K, W, B, Elem, I>(a, j, j < n, q, reinterpret_cast<float*>(wave_rows), n);
    }
}

// 16 bytes of one copy from slot s on: one slot of binary32, two of bfloat16.
template <typename M, int B, typename I>
__device__ __forceinline__ void load16(const float* p, I s, f4 (&v)[1][B], int b) {
    v[0][b] = M::load(p, s);
}
template <typename M, int B, typename I>
__device__ __forceinline__ void load16(const uint16_t* p, I s, f4 (&v)[2][B], int b) {
    const u4 q = M::load_two(p, s);
    v[0][b] = widen(u2{q.x, q.y});
    v[1][b] = widen(u2{q.z, q.w});
}

// The copies past k_total of a wave's B are +0.
template <int K, int B, typename V>
__device__ __forceinline__ void clear_absent(V* v, int w, int k_total) {
    if constexpr (K == TC_MAX_K) {
#pragma unroll
        for (int b = 0; b < B; ++b) v[b] = has_copy<K, B>(w, b, k_total) ? v[b] : splat<V>(0.0f);
    }
}

// The reduction.  A lane loads 16 bytes of each of its wave's B copies, one
// slot of binary32 or two of bfloat16 (NS), a tile is 64 * NS slots, and
// waves 0 to NS - 1 store 64 sums each.
template <int K, int W, int B, typename T, typename M, typename I>
__global__ __launch_bounds__(64 * W) void reduce_kernel(ReduceArgs<K, T> a, I nslot, I n) {
    constexpr int NS = 4 / sizeof(T);
    __shared__ f4 sh[W * 64 * NS];
    const int w = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
    const int lane = static_cast<int>(threadIdx.x) & 63;
    const int waves = K == TC_MAX_K ? static_cast<int>(blockDim.x >> 6) : W;
    const I block = block_index<I>(), s0 = block * (64 * NS);
    if (s0 >= nslot) {  // the elements after the last whole slot
        const I j = tail_element(block, nslot, 64 * NS, lane);
        float v[B];
        if (j < n) each_copy<K, B>(w, a.k_total, [&](int b) { v[b] = Elem::load(a.in[w * B + b], j); });
        clear_absent<K, B>(v, w, a.k_total);
        float* const sums = reinterpret_cast<float*>(sh);
        sums[w * 64 + lane] = copies_sum<K, W, B>(v, w);
        if constexpr (W > 1) __syncthreads();
        if (w == 0 && j < n)
            Elem::store(a.out, j, quotient<K, float>(a, waves_sum<K, W, B>(sums + lane, 64, waves)));
        return;
    }
    const I s = s0 + static_cast<I>(lane * NS);
    f4 v[NS][B];
    if (s + I(NS - 1) < nslot) {
        each_copy<K, B>(w, a.k_total, [&](int b) { load16<M>(a.in[w * B + b], s, v, b); });
    } else if (s < nslot) {  // the last one of an odd number of bfloat16 slots
        each_copy<K, B>(w, a.k_total, [&](int b) { v[0][b] = M::load(a.in[w * B + b], s); });
    }
#pragma unroll
    for (int e = 0; e < NS; ++e) clear_absent<K, B>(v[e], w, a.k_total);
#pragma unroll
    for (int e = 0; e < NS; ++e) sh[w * (64 * NS) + lane * NS + e] = copies_sum<K, W, B>(v[e], w);
    if constexpr (W > 1 || NS > 1) __syncthreads();
#pragma unroll
    for (int e = 0; e < NS; ++e) {
        const I o = s0 + static_cast<I>(e * 64 + lane);
        if ((W == 1 || w == e) && o < nslot)
            store_pol<(K <= 2 || NS == 2 ? kReduceStoreSc1 : kStoreNt), M, I>(
                a.out, o, quotient<K, f4>(a, waves_sum<K, W, B>(sh + e * 64 + lane, 64 * NS, waves)), a.out_bytes);
    }
}

// -------------------------------------------------------------- launching

// 32-bit byte offsets when the largest buffer is below 4 GiB.
bool off32(int64_t n) { return n * 4 < (int64_t(1) << 32) - 64; }

// Copies per wave of the reduction, for K <= 16.  Binary32: one load per lane
// is enough up to six waves (25 M elements, GB/s at 1 / 2 / 4 copies per wave:
// K = 4 6,801 / 6,307 / 6,143, K = 6 6,370 / 6,343 / 6,294), then two keep a
// tile at eight waves (K = 8 6,382 / 6,446 / 6,134, K = 16 4,393 / 6,612 /
// 6,313; the earlier kernel, one lane for all copies, 6,081 at K = 4, 5,812
// at 8 and 5,817 at 16).  bfloat16 (16 bytes, two slots, per load): two from
// K = 3, but four for K = 13 and 14, whose seven waves of two ran at 4,960
// against 6,180.  K > 16: four up to 32 copies, then eight (K = 32 6,587,
// against 5,846 with two; K = 48 6,606 with eight, 6,173 with four).  At K = 2
// one wave for both (4 M elements 8.5 us, one per wave 9.4; bfloat16 1.05 to
// 1.15 times as fast from 3 M elements on).
template <typename T>
constexpr int reduce_copies(int K) {
    if (sizeof(T) == 2) return K == 1 ? 1 : K == 13 || K == 14 ? 4 : 2;
    return K == 1 || (K >= 3 && K <= 6) ? 1 : 2;
}

// Elements of all copies, [from, to), between which a wave takes every copy
// (K <= 16): a pass of 5 to 15 us, a few memory latencies, on buffers that the
// caches hold, where the tiles of several waves are just more than the chip
// takes at once and the meeting in LDS is a latency of its own.  Measured on
// MI355X, us with several waves, one wave, and the kernels before the waves:
// step K = 7, 360,000 elements 7.8, 6.7, 6.4, 512,000 9.6, 9.3, 7.4; K = 10
// 256,000 7.2, 6.2, 5.8; synchronous SGD K = 11, 180,000 7.1, 5.4, 5.4; K = 3 to
// 12 3 to 30% faster between 1.5 and 6 M, level below and 2 to 10% slower above,
// K = 13 to 16, whose waves take two copies anyway, between 2.5 and 4.5 M (K = 16,
// 128,000 elements 3 to 6% slower, 256,000 10% faster, 360,000 4% slower);
// reduction K = 5, 720,000 elements 5.0, 4.5, 4.3; K = 5 to 16 up to 12% faster
// between 3.3 and 8 M.  The bfloat16 reduction is level.
struct CopyRange {
    int64_t from, to;
};
constexpr CopyRange kReduceOneWave{3300000, 8000000};
constexpr CopyRange step_one_wave(int K) {
    return K <= 12 ? CopyRange{1500000, 6000000} : CopyRange{2500000, 4500000};
}
bool one_wave(CopyRange r, int K, int64_t n) { return n * K >= r.from && n * K < r.to; }

// Launches f(M, items, n, grid) with M a slot, aligned or not (vec), items the
// whole slots, in the smallest index type, and a workgroup for the elements
// after them where there are any.
// SMALL: buffers that are always below 4 GiB.
template <bool SMALL = false, typename F>
hipError_t launch_items(int64_t n, bool vec, int per_block, int threads, F f) {
    const int64_t items = n / 4;
    const GridXY xy = grid_of((items + per_block - 1) / per_block + (n % 4 != 0), threads);
    const dim3 grid(xy.x, xy.y);
    if (SMALL || off32(n)) {
        if (vec) f(Slot{}, static_cast<uint32_t>(items), static_cast<uint32_t>(n), grid);
        else f(SlotAny{}, static_cast<uint32_t>(items), static_cast<uint32_t>(n), grid);
    } else if constexpr (!SMALL) {
        if (vec) f(Slot{}, items, n, grid);
        else f(SlotAny{}, items, n, grid);
    }
    return hipGetLastError();
}

template <int K, int B, typename T, bool SMALL = false>
hipError_t launch_reduce_k(const ReduceArgs<K, T>& a, int64_t n, bool vec, hipStream_t s) {
    constexpr int W = (K + B - 1) / B, NS = 4 / sizeof(T);
    const int threads = 64 * ((a.k_total + B - 1) / B);
    return launch_items<SMALL>(n, vec, 64 * NS, threads, [&](auto M, auto items, auto size, dim3 grid) {
        hipLaunchKernelGGL((reduce_kernel<K, W, B, T, decltype(M), decltype(items)>), grid,
                           dim3(static_cast<unsigned>(threads)), 0, s, a, items, size);
    });
}

// LDS: `per_wave` rows per wave and `extra` per tile, or (per_copy) one row
// per copy.
template <int K, int ROWS, int B, typename T, template <int, typename> class Args, bool SMALL = false>
hipError_t launch_waves(const Args<K, T>& a, int k_total, int per_wave, int extra, bool per_copy, int64_t n, bool vec,
                        hipStream_t s) {
    constexpr int W = K < TC_MAX_K ? (K + B - 1) / B : B == 2 ? kSpecialisedK : TC_MAX_K / B;
    const int waves = K < TC_MAX_K ? W * ROWS : (k_total + B - 1) / B;
    const int rows = (per_copy ? k_total : waves / ROWS * per_wave + extra) * ROWS;
    const unsigned lds = static_cast<unsigned>(rows) * 64u * 16u;
    const dim3 block(static_cast<unsigned>(64 * waves));
    return launch_items<SMALL>(n, vec, 64 * ROWS, 64 * waves, [&](auto M, auto items, auto size, dim3 grid) {
        hipLaunchKernelGGL((wave_kernel<K, W, B, ROWS, T, decltype(M), decltype(items), Args>), grid, block, lds, s, a,
                           items, size);
    });
}

// Copies per wave of the steps: one, the smallest footprint, up to K = 12; two
// from 13, so that a tile is at most 8 waves and several fit on a CU (K = 16
// 6,376 with one, 6,412 with two; K = 12 6,570 and 6,344).  K > 16: four, but
// two for binary32 gradients up to K = 24 (K = 20 6,274 with two, 5,938 with
// four; bfloat16 gradients 5,718 and 6,188; K = 32 5,788 and 5,959; eight
// from K = 33 lost up to 15%).
template <int K, typename T, template <int, typename> class Args>
hipError_t launch_step(const Args<K, T>& a, int k_total, int per_wave, int extra, int64_t n, bool vec, hipStream_t s) {
    constexpr int ROWS = K == 1 ? 4 : 1;
    if constexpr (K > 1 && K < TC_MAX_K)
        if (one_wave(step_one_wave(K), K, n))
            return launch_waves<K, 1, K, T, Args, true>(a, k_total, per_wave, extra, false, n, vec, s);
    if constexpr (K < TC_MAX_K)
        return launch_waves<K, ROWS, (K <= 12 ? 1 : 2), T, Args>(a, k_total, per_wave, extra, false, n, vec, s);
    else if (sizeof(T) == 4 && k_total <= 24)
        return launch_waves<K, ROWS, 2, T, Args>(a, k_total, per_wave, extra, false, n, vec, s);
    else
        return launch_waves<K, ROWS, 4, T, Args>(a, k_total, per_wave, extra, false, n, vec, s);
}

template <int K, typename T>
hipError_t run_reduce(const void* const* in, float* out, int op, int k_total, int64_t n, bool vec, hipStream_t s) {
    ReduceArgs<K, T> a{};
    for (int q = 0; q < k_total; ++q) a.in[q] = static_cast<const T*>(in[q]);
    a.out = out;
    a.out_bytes = n * 4 < (int64_t(1) << 32) ? static_cast<uint32_t>(n * 4) : 0;
    a.op = op;
    a.k_total = k_total;
    if constexpr (sizeof(T) == 4 && K >= 5 && K < TC_MAX_K)
        if (one_wave(kReduceOneWave, K, n)) return launch_reduce_k<K, K, T, true>(a, n, vec, s);
    if constexpr (K < TC_MAX_K) return launch_reduce_k<K, reduce_copies<T>(K), T>(a, n, vec, s);
    else if (k_total <= 2 * kSpecialisedK) return launch_reduce_k<K, 4, T>(a, n, vec, s);
    else return launch_reduce_k<K, 8, T>(a, n, vec, s);
}

template <int K, typename T>
hipError_t run_easgd(float* const* x, const void* const* g, float* xc, float* out, int op, float eta, float rho,
                     int k_total, int64_t n, bool vec, hipStream_t s) {
    ReduceEasgdArgs<K, T> a{};
    for (int q = 0; q < k_total; ++q) {
        a.x[q] = x[q];
        a.g[q] = static_cast<const T*>(g[q]);
    }
    a.xc = xc;
    a.eta = eta;
    a.rho = rho;
    a.a = eta * rho;  // one binary32 rounding, on the host
    a.k_total = k_total;
    a.out = out;
    a.op = op;
    if (out) return launch_step<K, T, ReduceEasgdArgs>(a, k_total, 2, 1, n, vec, s);
    return launch_step<K, T, EasgdArgs>(a, k_total, 1, 1, n, vec, s);
}

#define TC_FOR_K(X) X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16)

template <typename T>
hipError_t dispatch_reduce(int K, const void* const* in, float* out, int op, int64_t n, bool vec, hipStream_t s) {
    switch (K) {
#define TC_CASE(k) \
    case k: return run_reduce<k, T>(in, out, op, K, n, vec, s);
        TC_FOR_K(TC_CASE)
#undef TC_CASE
        default: return run_reduce<TC_MAX_K, T>(in, out, op, K, n, vec, s);
    }
}

template <typename T>
hipError_t dispatch_easgd(int K, float* const* x, const void* const* g, float* xc, float* out, int op, float eta,
                          float rho, int64_t n, bool vec, hipStream_t s) {
    switch (K) {
#define TC_CASE(k) \
    case k: return run_easgd<k, T>(x, g, xc, out, op, eta, rho, K, n, vec, s);
        TC_FOR_K(TC_CASE)
#undef TC_CASE
        default: return run_easgd<TC_MAX_K, T>(x, g, xc, out, op, eta, rho, K, n, vec, s);
    }
}

// Broadcast of one flat buffer to K copies, bit for bit: 16-byte slots when
// every buffer is 16-byte aligned, element by element otherwise; the last
// workgroup copies the bytes after the last whole slot.
//
// Slot path: a workgroup copies one chunk of TC_EW_THREADS slots of the
// source into C of the copies.  The grid runs window by window (window
// chunks of the source each): within a window, the chunks for copies 0..C-1
// come first, then those for copies C..2C-1, and so on, so that the
// workgroups resident at one time write about C copies rather than all K,
// and the later passes over a window find its source in the last-level
// cache.  The source is read with ordinary (cacheable) loads for that reuse.
// Measured on MI355X with calls rotating over sources that total > 768 MB,
// so no call finds its source cached by an earlier one (GB/s; ResNet-50
// group K = 8 / 16 / 4, VGG-16 group K = 8 / 4): every copy per workgroup
// with non-temporal source loads 4,458-4,490 / 4,912-4,931 / 5,094-5,145 /
// 5,155-5,200 / 5,198-5,270; C = 4 over windows of 8,192 chunks (32 MiB of
// binary32 source) 5,297-5,329 / 5,295-5,337 / 5,325-5,354 / 5,627-5,684.
#ifndef TC_BCAST_COPIES
#define TC_BCAST_COPIES 4
#endif
#ifndef TC_BCAST_WINDOW
#define TC_BCAST_WINDOW 8192
#endif
#ifndef TC_BCAST_NT_SRC
#define TC_BCAST_NT_SRC 0
#endif
struct BcastArgs {
    const char* src;
    char* dst[TC_MAX_K];
    int K, es;
    int64_t nbytes;
    int64_t nchunk, window;  // chunks of TC_EW_THREADS slots; chunks per window (>= 1)
    int C, groups;           // copies per workgroup; ceil(K / C)
};

// K = 1 with 16-byte aligned buffers, a plain copy: every workgroup copies
// one chunk of TC_EW_THREADS slots, read once (non-temporal).  Its
// arguments are only what that needs, so the load issues after one round
// of scalar loads, where the general kernel's prologue waits on a chain of
// them.  Measured on MI355X, 1 GiB: 6.17-6.24 TB/s through the general
// kernel, 6.44-6.52 through this one; at K = 2 and 4 the same shape (all
// copies per workgroup, non-temporal source) was 1.6-2.2% slower than the
// general kernel.  Lanes past the last whole slot copy that slot again
// (the same bytes to the same place), so no branch holds the loads back;
// the host takes this kernel only with at least one whole slot.  Workgroup
// 0 also copies the bytes after the last whole slot.
struct CopyArgs {
    const u4* src;
    u4* dst;
    int64_t nvec;    // whole 16-byte slots (>= 1)
    int64_t nbytes;  // all bytes (tail: nvec * 16 .. nbytes)
    int es;
};

__global__ __launch_bounds__(TC_EW_THREADS) void copy_kernel(CopyArgs a) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * TC_EW_THREADS + threadIdx.x;
    const int64_t v = i < a.nvec ? i : a.nvec - 1;
    __builtin_nontemporal_store(__builtin_nontemporal_load(a.src + v), a.dst + v);
    if (blockIdx.x == 0)
        for (int64_t b = a.nvec * 16 + threadIdx.x * a.es; b < a.nbytes; b += TC_EW_THREADS * a.es) {
            const char* sp = reinterpret_cast<const char*>(a.src) + b;
            char* dp = reinterpret_cast<char*>(a.dst) + b;
            if (a.es == 4) *reinterpret_cast<uint32_t*>(dp) = *reinterpret_cast<const uint32_t*>(sp);
            else *reinterpret_cast<uint16_t*>(dp) = *reinterpret_cast<const uint16_t*>(sp);
        }
}

template <bool VEC>
__global__ __launch_bounds__(TC_EW_THREADS) void bcast_kernel(BcastArgs a) {
    if (VEC) {
        const int64_t nvec = a.nbytes / 16;
        if (a.nchunk > 0) {
            const int64_t b = blockIdx.x;
            const int64_t per_window = a.window * a.groups;  // every window but the last is full
            const int64_t w = b / per_window;
            const int64_t rest = a.nchunk - w * a.window;
            const int64_t wlen = rest < a.window ? rest : a.window;
            const int64_t r = b - w * per_window;
            const int64_t cg = r / wlen;
            const int64_t v = (w * a.window + (r - cg * wlen)) * TC_EW_THREADS + threadIdx.x;
            const int k0 = static_cast<int>(cg) * a.C;
            const int k1 = k0 + a.C < a.K ? k0 + a.C : a.K;
            if (v < nvec) {
                const u4* sp = reinterpret_cast<const u4*>(a.src) + v;
                const u4 x = TC_BCAST_NT_SRC ? __builtin_nontemporal_load(sp) : *sp;
                for (int k = k0; k < k1; ++k) __builtin_nontemporal_store(x, reinterpret_cast<u4*>(a.dst[k]) + v);
            }
        }
        if (blockIdx.x == gridDim.x - 1)
            for (int64_t b = nvec * 16 + threadIdx.x * a.es; b < a.nbytes; b += TC_EW_THREADS * a.es)
                for (int k = 0; k < a.K; ++k) {
                    if (a.es == 4) *reinterpret_cast<uint32_t*>(a.dst[k] + b) = *reinterpret_cast<const uint32_t*>(a.src + b);
                    else *reinterpret_cast<uint16_t*>(a.dst[k] + b) = *reinterpret_cast<const uint16_t*>(a.src + b);
                }
    } else {
        const int64_t stride = static_cast<int64_t>(gridDim.x) * TC_EW_THREADS;
        const int64_t t0 = static_cast<int64_t>(blockIdx.x) * TC_EW_THREADS + threadIdx.x;
        for (int64_t e = t0; e * a.es < a.nbytes; e += stride)
            for (int k = 0; k < a.K; ++k) {
                if (a.es == 4) reinterpret_cast<uint32_t*>(a.dst[k])[e] = reinterpret_cast<const uint32_t*>(a.src)[e];
                else reinterpret_cast<uint16_t*>(a.dst[k])[e] = reinterpret_cast<const uint16_t*>(a.src)[e];
            }
    }
}

template <int K, typename T>
hipError_t run_sgd(float* const* x, const void* const* g, float eta, int k_total, int64_t n, bool vec, hipStream_t s) {
    SgdArgs<K, T> a{};
    for (int q = 0; q < k_total; ++q) {
        a.x[q] = x[q];
        a.g[q] = static_cast<const T*>(g[q]);
    }
    a.eta = eta;
    return launch_items(n, vec, TC_EW_THREADS, TC_EW_THREADS, [&](auto M, auto items, auto size, dim3 grid) {
        grid.z = static_cast<unsigned>(k_total);
        hipLaunchKernelGGL((sgd_kernel<K, T, decltype(M), decltype(items)>), grid, dim3(TC_EW_THREADS), 0, s, a, items,
                           size);
    });
}

template <int K, typename T>
hipError_t run_sync(float* const* x, void* const* g, float step, int broadcast, int k_total, int64_t n, bool vec,
                    hipStream_t s) {
    SyncArgs<K, T> a{};
    for (int q = 0; q < k_total; ++q) {
        a.x[q] = x[q];
        a.g[q] = static_cast<T*>(g[q]);
    }
    a.step = step;
    a.broadcast = broadcast;
    a.k_total = k_total;
    return launch_step<K, T, SyncArgs>(a, k_total, 1, 0, n, vec, s);
}

template <int K, typename T>
hipError_t run_async(float* const* x, float* xc, const int32_t* order, int R, float alpha, int k_total, int64_t n,
                     bool vec, hipStream_t s) {
    AsyncArgs<K, T> a{};
    for (int r = 0; r < R; ++r) a.x[r] = x[order[r]];
    a.xc = xc;
    a.R = R;
    a.alpha = alpha;
    a.k_total = k_total;
    if constexpr (K < TC_MAX_K)
        return launch_waves<K, 1, (K == 1 ? 1 : 2), T, AsyncArgs>(a, k_total, 1, 0, true, n, vec, s);
    else if (k_total <= 32)
        return launch_waves<K, 1, 4, T, AsyncArgs>(a, k_total, 1, 0, true, n, vec, s);
    else if (n < kAsyncAhead)
        return launch_items<true>(n, vec, TC_EW_THREADS, TC_EW_THREADS, [&](auto M, auto items, auto size, dim3 grid) {
            hipLaunchKernelGGL((async_lane_kernel<8, T, decltype(M), decltype(items)>), grid, dim3(TC_EW_THREADS), 0, s,
                               a, items, size);
        });
    else
        return launch_items(n, vec, TC_EW_THREADS, TC_EW_THREADS, [&](auto M, auto items, auto size, dim3 grid) {
            hipLaunchKernelGGL((async_lane_kernel<1, T, decltype(M), decltype(items)>), grid, dim3(TC_EW_THREADS), 0, s,
                               a, items, size);
        });
}

template <typename T>
hipError_t dispatch_sgd(int K, float* const* x, const void* const* g, float eta, int64_t n, bool vec, hipStream_t s) {
    // three sizes of arguments: nothing else depends on K
    if (K <= 4) return run_sgd<4, T>(x, g, eta, K, n, vec, s);
    if (K <= kSpecialisedK) return run_sgd<kSpecialisedK, T>(x, g, eta, K, n, vec, s);
    return run_sgd<TC_MAX_K, T>(x, g, eta, K, n, vec, s);
}

template <typename T>
hipError_t dispatch_sync(int K, float* const* x, void* const* g, float step, int broadcast, int64_t n, bool vec,
                         hipStream_t s) {
    switch (K) {
#define TC_CASE(k) \
    case k: return run_sync<k, T>(x, g, step, broadcast, K, n, vec, s);
        TC_FOR_K(TC_CASE)
#undef TC_CASE
        default: return run_sync<TC_MAX_K, T>(x, g, step, broadcast, K, n, vec, s);
    }
}

hipError_t dispatch_async(int K, float* const* x, float* xc, const int32_t* order, int R, float alpha, int64_t n,
                          bool vec, hipStream_t s) {
    switch (K) {
#define TC_CASE(k) \
    case k: return run_async<k, float>(x, xc, order, R, alpha, K, n, vec, s);
        TC_FOR_K(TC_CASE)
#undef TC_CASE
        default: return run_async<TC_MAX_K, float>(x, xc, order, R, alpha, K, n, vec, s);
    }
}

}  // namespace

hipError_t launch_sgd(int K, float* const* x, const void* const* g, int g_dtype, float eta, int64_t n, bool vector_ok,
                      hipStream_t stream) {
    if (g_dtype == TC_BF16) return dispatch_sgd<uint16_t>(K, x, g, eta, n, vector_ok, stream);
    return dispatch_sgd<float>(K, x, g, eta, n, vector_ok, stream);
}

hipError_t launch_sync_sgd(int K, float* const* x, void* const* g, int g_dtype, float eta, float rescale, int broadcast,
                           int64_t n, bool vector_ok, hipStream_t stream) {
    const float step = eta * rescale;  // one binary32 rounding, on the host
    if (g_dtype == TC_BF16) return dispatch_sync<uint16_t>(K, x, g, step, 0, n, vector_ok, stream);
    return dispatch_sync<float>(K, x, g, step, broadcast, n, vector_ok, stream);
}

hipError_t launch_elastic_async(int K, float* const* x, float* xc, const int32_t* order, int R, float alpha,
                                int64_t n, bool vector_ok, hipStream_t stream) {
    return dispatch_async(K, x, xc, order, R, alpha, n, vector_ok, stream);
}

hipError_t launch_broadcast(int K, const void* src, void* const* dst, int es, int64_t n, bool vector_ok,
                            hipStream_t stream) {
    BcastArgs a{};
    a.src = static_cast<const char*>(src);
    for (int k = 0; k < K; ++k) a.dst[k] = static_cast<char*>(dst[k]);
    a.K = K;
    a.es = es;
    a.nbytes = n * es;
    if (vector_ok && K == 1 && a.nbytes >= 16) {
        CopyArgs c{static_cast<const u4*>(src), static_cast<u4*>(dst[0]), a.nbytes / 16, a.nbytes, es};
        dim3 grid(static_cast<unsigned>((c.nvec + TC_EW_THREADS - 1) / TC_EW_THREADS));
        hipLaunchKernelGGL(copy_kernel, grid, dim3(TC_EW_THREADS), 0, stream, c);
    } else if (vector_ok) {
        a.nchunk = (a.nbytes / 16 + TC_EW_THREADS - 1) / TC_EW_THREADS;
        a.window = a.nchunk < TC_BCAST_WINDOW ? (a.nchunk > 0 ? a.nchunk : 1) : TC_BCAST_WINDOW;
        a.C = TC_BCAST_COPIES < K ? TC_BCAST_COPIES : K;
        a.groups = (K + a.C - 1) / a.C;
        const int64_t blocks = a.nchunk * a.groups;
        dim3 grid(static_cast<unsigned>(blocks > 0 ? blocks : 1));
        hipLaunchKernelGGL((bcast_kernel<true>), grid, dim3(TC_EW_THREADS), 0, stream, a);
    } else {
        dim3 grid(static_cast<unsigned>((n + TC_EW_THREADS - 1) / TC_EW_THREADS));
        hipLaunchKernelGGL((bcast_kernel<false>), grid, dim3(TC_EW_THREADS), 0, stream, a);
    }
    return hipGetLastError();
}

hipError_t launch_reduce(int K, const void* const* in, int in_dtype, float* out, int op, int64_t n, bool vector_ok,
                         hipStream_t stream) {
    if (in_dtype == TC_BF16) return dispatch_reduce<uint16_t>(K, in, out, op, n, vector_ok, stream);
    return dispatch_reduce<float>(K, in, out, op, n, vector_ok, stream);
}

hipError_t launch_easgd(int K, float* const* x, const void* const* g, int g_dtype, float* xc, float* out, int op,
                        float eta, float rho, int64_t n, bool vector_ok, hipStream_t stream) {
    if (g_dtype == TC_BF16) return dispatch_easgd<uint16_t>(K, x, g, xc, out, op, eta, rho, n, vector_ok, stream);
    return dispatch_easgd<float>(K, x, g, xc, out, op, eta, rho, n, vector_ok, stream);
}

}  // namespace tc
