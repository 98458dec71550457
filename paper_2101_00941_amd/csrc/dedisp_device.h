// Device-side pieces shared by the dedispersion kernels.
#pragma once

#include "aa_internal.h"
#include "xcd.h"

namespace aa {

typedef void (*DedispFn)(DedispArgs);
typedef void (*DedispBatchFn)(const DedispArgs*, const int64_t*, int, int64_t, unsigned long long*);
// The strip kernels (strip.hip).
extern const DedispFn kStripKernel;
extern const DedispBatchFn kStripBatchKernel;

namespace {

// Read-only device data that is the same in every lane, read through the constant address
// space so that its loads are scalar even where the pointer comes from memory (the persistent
// batch kernel reads it from the beam's argument block).
template <class T>
__device__ __forceinline__ T load_uniform(const T* src) {
    static_assert(sizeof(T) % 4 == 0, "whole dwords");
    typedef const __attribute__((address_space(4))) int32_t* word_ptr;
    const word_ptr p = (word_ptr)(const void*)src;
    int32_t w[sizeof(T) / 4];
#pragma unroll
    for (int i = 0; i < static_cast<int>(sizeof(T) / 4); ++i) w[i] = p[i];
    T v;
    __builtin_memcpy(&v, w, sizeof(v));
    return v;
}

// A DM block's table entry: read-only for the launch.
__device__ __forceinline__ DmBlock load_block(const DmBlock* blocks, int blk) { return load_uniform(blocks + blk); }

constexpr int kRawBufferFlags = 0x00020000;   // word 3 of a gfx9 buffer resource: raw 32-bit data

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lds_void;

typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x16 __attribute__((ext_vector_type(16)));

// Waits until the results of the matrix operations before it may be read by inline assembly.
// v_mfma_i32_32x32x32_i8 takes eight passes, and 12 wait states must pass before an LDS or
// vector instruction reads its result. The hardware does not hold the reader back: the compiler
// puts the wait in front of its own instructions, and none in front of an asm statement. Each
// tile goes through an asm statement of its own, so that no matrix operation moves past the wait.
template <int N>
__device__ __forceinline__ void wait_matrix_results(i32x16 (&acc)[N]) {
#pragma unroll
    for (int j = 1; j < N; ++j) asm volatile("" : "+v"(acc[j]));
    asm volatile("s_nop 11" : "+v"(acc[0])::"memory");
}

// The batched persistent launch: a work-group pulls item indexes from the device counter
// until they run out (every work-group reaches that exit) and runs tile(args, block, t0) of
// the item's beam, found by binary search over item_begin. Consecutive items are adjacent
// DM blocks of the same time tile of the same beam (their input rows overlap).
template <class Tile>
__device__ __forceinline__ void batch_items(const DedispArgs* __restrict__ args, const int64_t* __restrict__ item_begin,
                                            int nbeams, int64_t total, unsigned long long* counter, Tile tile) {
    __shared__ int64_t item;
    for (;;) {
        if (threadIdx.x == 0) item = static_cast<int64_t>(atomicAdd(counter, 1ull));
        __syncthreads();
        // the item index is the same in every lane: keep it in scalar registers
        const uint64_t itu = static_cast<uint64_t>(item);
        const int64_t it = static_cast<int64_t>(
            (static_cast<uint64_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(itu >> 32))) << 32) |
            static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(itu))));
        __syncthreads();
        if (it >= total) break;
        int lo = 0, hi = nbeams - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (load_uniform(item_begin + mid) <= it) lo = mid; else hi = mid - 1;
        }
        // the beam is the same in every lane; stating it keeps the beam's arguments and
        // the tile's step records in scalar registers
        lo = __builtin_amdgcn_readfirstlane(lo);
        const DedispArgs a = load_uniform(args + lo);
        const int64_t local = it - load_uniform(item_begin + lo);
        tile(a, static_cast<int>(local % a.nblk), local / a.nblk);
        __syncthreads();   // the next item restages the LDS
    }
}

}  // namespace
}  // namespace aa
