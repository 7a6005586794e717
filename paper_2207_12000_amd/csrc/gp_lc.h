// What the two kernels of the LC-version forward pass share (gp_lc.hip: fp32 products as six bf16 products;
// gp_lc_f32.hip: the fp32 matrix instruction).
#pragma once

#include <hip/hip_runtime.h>

#include "gp_internal.h"

namespace gp {

constexpr int kPanel = 256;  // widest inner dimension staged in LDS at once
constexpr int kMaxLayers = 8;
constexpr int kMaxHops = 16;

typedef float v4f __attribute__((ext_vector_type(4)));
typedef unsigned short v4u16 __attribute__((ext_vector_type(4)));

struct LcArgs {
    const void* stack;
    int64_t ld, slab;  // elements: row stride, distance between hop slabs
    int64_t n;
    int d;
    int hops;                 // branches in use: work item = tile * hops + branch
    int hop_of[kMaxHops];     // branch -> slab of the stack it reads
    int depth[kMaxHops];      // branch -> number of weight matrices it applies
    int out_off[kMaxHops];    // branch -> first output column when branches are written side by side
    int direct;               // 1: branches write the final result (side by side, or there is just one)
    const int32_t* batch;
    int64_t B;
    float gamma[kMaxHops];
    int T;
    const float* W[kMaxLayers];
    int width[kMaxLayers];
    int wvec[kMaxLayers];  // gp_lc_f32.hip: 1: rows of W_t may be read with vector loads
    const char* frags;     // gp_lc.hip: split weights (gp_lc_split_weights), or nullptr: split where they are used
    int64_t frag_off[kMaxLayers];  // layer -> its first byte there
    int xvec;              // 1: stack rows may be read four elements at a time
    float* dst;            // the result (direct), else the partial results [branch][B][ldd]
    int64_t ldd;
};

__device__ __forceinline__ float widen(float v) { return v; }
__device__ __forceinline__ float widen(unsigned short v) { return __uint_as_float((unsigned)v << 16); }

__device__ __forceinline__ v4f load4(const float* p) { return *reinterpret_cast<const v4f*>(p); }
__device__ __forceinline__ v4f load4(const unsigned short* p)
{
    const v4u16 b = *reinterpret_cast<const v4u16*>(p);
    v4f r;
    r.x = widen(b.x), r.y = widen(b.y), r.z = widen(b.z), r.w = widen(b.w);
    return r;
}

// tile_rows: 32 or 64 rows to a work item
gp_status launch_lc_f32(gp_dtype dtype, int tile_rows, const LcArgs& a, unsigned grid, hipStream_t stream);

}  // namespace gp
