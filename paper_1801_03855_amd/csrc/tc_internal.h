// Internal declarations shared by the library's translation units.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <vector>

#include "tc.h"
#include "tc_grid.h"

#define TC_API extern "C" __attribute__((visibility("default")))

namespace tc {

// Elements per chunk, of which the group holds the first tensor of each.  Each
// kind of kernel cuts the group its own way (measured on MI355X):
// - the staged separate-buffer pack, a workgroup to a chunk of one copy: groups
//   of large tensors (almost every chunk inside one tensor) move best in short
//   chunks that a workgroup covers in one batch per lane; groups of many small
//   tensors in longer chunks, which spread the per-chunk segment staging over
//   more data (4,096: 4% faster than with 8,192, 10% faster than with 2,048),
//   and 2-byte elements on groups of large tensors in chunks of twice the
//   elements (the bytes of a binary32 chunk);
// - the tiles of the tensor layout (pack, unpack, the one-call step), and the
//   separate unpack's and small packs' waves: one table for each size, 1,024,
//   512 and 256 elements (smaller tiles share the last).
// All are multiples of every vector width (4, 8).
#ifndef TC_PACK_CHUNK_LARGE
#define TC_PACK_CHUNK_LARGE 2048
#endif
#ifndef TC_PACK_CHUNK_SMALL
#define TC_PACK_CHUNK_SMALL 4096
#endif
#ifndef TC_TPACK_CHUNK
#define TC_TPACK_CHUNK 1024
#endif
#ifndef TC_PIPE_CHUNK
#define TC_PIPE_CHUNK 512
#endif
#ifndef TC_PIPE_CHUNK_FINE
#define TC_PIPE_CHUNK_FINE 256
#endif
#ifndef TC_PACK_LARGE_MEAN
#define TC_PACK_LARGE_MEAN 32768
#endif

// Segments (tensors overlapping one chunk) whose offsets and pointers a
// workgroup stages in LDS; chunks touching more tensors search the global
// tables instead.
constexpr int kMaxStage = 1024;

// Device access to global memory at an address held as an integer (pointers
// read from the tensor lists' tables, addresses formed by arithmetic).  The
// address space is stated so that the compiler emits global, not flat,
// instructions: a flat access also counts against the LDS wait counter, so
// every later wait for an LDS access would wait for it as well.
#define TC_GLOBAL __attribute__((address_space(1)))
template <typename V>
__device__ __forceinline__ V gld(uintptr_t a) {
    return *reinterpret_cast<const TC_GLOBAL V*>(a);
}
template <typename V>
__device__ __forceinline__ V gld_nt(uintptr_t a) {
    return __builtin_nontemporal_load(reinterpret_cast<const TC_GLOBAL V*>(a));
}
template <typename V>
__device__ __forceinline__ void gst(uintptr_t a, V v) {
    *reinterpret_cast<TC_GLOBAL V*>(a) = v;
}
template <typename V>
__device__ __forceinline__ void gst_nt(uintptr_t a, V v) {
    __builtin_nontemporal_store(v, reinterpret_cast<TC_GLOBAL V*>(a));
}

// A load or store at an address with no alignment beyond the element size:
// on gfx950 global memory is accessed in unaligned mode, so a 16-byte (or
// 8-byte) access at any byte address is one vector instruction, which the
// memory pipeline splits over the cache lines it touches.
template <typename V>
__device__ __forceinline__ V gld_u(uintptr_t a) {
    typedef V Vu __attribute__((aligned(1)));
    return *reinterpret_cast<const TC_GLOBAL Vu*>(a);
}
template <typename V>
__device__ __forceinline__ void gst_u(uintptr_t a, V v) {
    typedef V Vu __attribute__((aligned(1)));
    *reinterpret_cast<TC_GLOBAL Vu*>(a) = v;
}

// Workgroup w of a launch runs on XCD w % 8, and each of the 8 XCDs has its
// own L2 cache and address-translation caches.  tile_of<R> renumbers the
// workgroups so that, within every 8R consecutive tiles, each XCD takes R
// consecutive tiles (R = 1: no renumbering; a last partial group of 8R
// tiles keeps its order).  The tensor-layout reduction, step and broadcast
// kernels take R = 128 (runs of 128 tiles of 32 to 128 slots): measured on
// MI355X against R = 1, the fused step +2.5% (VGG-16, K = 4), +5% (ResNet-50,
// K = 8) and +3.6% (10,000 tensors, K = 16), the reduction +2 to +4%; R = 32
// to 512 gain less or the same.  The one-call step up to 32 copies and, by K
// and direction, the tensor-layout pack and unpack take runs of their own
// length, given with what they measured at kRun there.  The separate-buffer
// kernels and the staged kernels measured level or slower with any R, and keep
// their order.
#ifndef TC_XCD_RUN_STEP
#define TC_XCD_RUN_STEP 128
#endif
template <int R>
__device__ __forceinline__ uint32_t tile_of(uint32_t b, uint32_t nb) {
    if constexpr (R <= 1) {
        return b;
    } else {
        constexpr uint32_t S = 8u * R;
        if (b >= nb / S * S) return b;
        return b / S * S + (b % 8u) * R + (b / 8u) % R;
    }
}

// A tensor's start relative to a chunk's first element, clamped to the
// chunk [0, clen]: the chunk-relative segment bounds that the staged kernels
// (the separate-buffer pack, the one-call step above 32 copies) hold.
__device__ __forceinline__ int32_t clamp_rel(int64_t v, int32_t clen) {
    return static_cast<int32_t>(v < 0 ? 0 : (v > clen ? clen : v));
}

// Records a printf-style message as this thread's last error.
void set_error(const char* fmt, ...) __attribute__((format(printf, 1, 2)));
void clear_error();

// Launchers, defined next to their kernels.  Arguments are validated by the
// caller; these only pick a kernel and enqueue it on `stream`.
hipError_t launch_reduce(int K, const void* const* in, int in_dtype, float* out, int op,
                         int64_t n, bool vector_ok, hipStream_t stream);
// out == nullptr: the step alone; otherwise the step fused with the
// reduction of the gradients into out (op TC_SUM or TC_AVG).
hipError_t launch_easgd(int K, float* const* x, const void* const* g, int g_dtype, float* xc, float* out, int op,
                        float eta, float rho, int64_t n, bool vector_ok, hipStream_t stream);

hipError_t launch_sgd(int K, float* const* x, const void* const* g, int g_dtype, float eta, int64_t n, bool vector_ok,
                      hipStream_t stream);
hipError_t launch_sync_sgd(int K, float* const* x, void* const* g, int g_dtype, float eta, float rescale, int broadcast,
                           int64_t n, bool vector_ok, hipStream_t stream);
hipError_t launch_elastic_async(int K, float* const* x, float* xc, const int32_t* order, int R, float alpha,
                                int64_t n, bool vector_ok, hipStream_t stream);
hipError_t launch_broadcast(int K, const void* src, void* const* dst, int es, int64_t n, bool vector_ok,
                            hipStream_t stream);

hipError_t launch_pack(const tc_tensorlist* tl, void* const* flat, bool unpack, hipStream_t stream);

// Tensor layout (K copies interleaved in slots of 4 elements).
hipError_t launch_tensor_reduce(int K, const void* in, int in_dtype, float* out, int op, int64_t n,
                                hipStream_t stream);
hipError_t launch_tensor_easgd(int K, float* x, const void* g, int g_dtype, float* xc, float* out, int op, float eta,
                               float rho, int64_t n, hipStream_t stream);
hipError_t launch_tensor_pack(const tc_tensorlist* tl, void* tensor, bool unpack, hipStream_t stream);
hipError_t launch_tensor_sgd(int K, float* x, const void* g, int g_dtype, float eta, int64_t n, hipStream_t s);
hipError_t launch_tensor_sync_sgd(int K, float* x, void* g, int g_dtype, float eta, float rescale, int broadcast,
                                  int64_t n, hipStream_t s);
hipError_t launch_tensor_elastic_async(int K, float* x, float* xc, const int32_t* order, int R, float alpha, int64_t n,
                                       hipStream_t s);
hipError_t launch_tensor_broadcast(int K, const void* src, void* dst, int es, int64_t n, hipStream_t s);
hipError_t launch_tensor_pipeline(const tc_tensorlist* grads, const tc_tensorlist* params, void* gt, float* gbar,
                                  float* x, float* xc, float eta, float rho, hipStream_t stream);

}  // namespace tc

// One cut of the flat index space into chunks of `chunk` elements (the last
// one shorter) with, per chunk, the first tensor it touches.
struct tc_chunking {
    int64_t chunk = 0;           // elements per chunk
    int64_t nchunks = 0;         // ceil(N / chunk)
    std::vector<int32_t> first;  // nchunks + 1
    int32_t* d_first = nullptr;  // device copy
};

// Group descriptor: host copies of sizes and offsets, and device copies of
// the offset table and of each chunking's first-segment table.
struct tc_group {
    int32_t n = 0;
    int64_t N = 0;
    int device = 0;
    std::vector<int64_t> sizes;
    std::vector<int64_t> offsets;  // n + 1
    bool large = false;            // mean tensor size >= TC_PACK_LARGE_MEAN
    tc_chunking sep;               // staged separate-buffer pack
    tc_chunking tpack;             // tiles of 1,024 elements
    tc_chunking pipe;              // tiles of 512 elements, waves of 2-byte elements
    tc_chunking pipe_fine;         // tiles of up to 256 elements, waves of binary32
    tc_chunking sep2;              // staged separate-buffer pack, 2-byte elements
    bool slot_bounds = false;      // every tensor boundary before the last,
                                   // partial slot is a multiple of 4
    int64_t* d_offsets = nullptr;
};

// K copies of a group held as separate tensors: device table of K*n
// pointers, copy-major.
struct tc_tensorlist {
    const tc_group* g = nullptr;
    int32_t K = 0;
    int32_t dtype = TC_F32;
    int32_t elem = 4;
    std::vector<const void*> ptrs;
    bool slot_aligned = false;  // every non-empty tensor starts on a 4-element boundary
    void** d_ptrs = nullptr;
};
