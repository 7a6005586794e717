// Forward pass of an LC-version model over the hop stack (Appendix A: the LC version
// of GPRGNN; Section 3.1: the H^LC formula for the single-branch case):
//
//     H[batch] = sum_k gamma_k * MLP(X_k[batch]),   MLP(Z) = relu(..relu(Z W_1)..W_{T-1}) W_T.
//
// This is the one dense contraction on the path, so it runs on the matrix cores, all
// layers of one hop fused in one kernel.  A workgroup of four waves owns 16, 32 or 48
// batch rows of one hop; the hops' results are summed afterwards in hop order.  The rows'
// features (later: the previous layer's activations) sit in LDS, the weights come straight
// from L2 ahead of the products that use them, and the layer output stays in accumulator
// registers until every wave is done with the LDS tile, then replaces it (ReLU applied on
// the way).  Nothing but the gathered rows and the per-hop B x C results touches HBM.
//
// Arithmetic.  The fp32 matrix instruction runs at 157 TFLOP/s on this chip, the bf16 one
// at 2.5 PFLOP/s.  An fp32 number times 2^16 is a sum of three bf16 numbers (8 bits each,
// rounded to nearest: 2^16 x = x1 + x2 + x3, |x2| <= 2^-8 |x1|, |x3| <= 2^-17 |x1|), without loss
// down to the smallest subnormal: 2^-149 becomes 2^-133, bf16's own smallest, which the
// conversions and the matrix instruction keep.  (Without the factor, the parts of numbers below
// 2^-110 run out of exponents.)  A product of two bf16 numbers is exact in fp32, so
//
//     2^32 x w = x1 w1 + (x1 w2 + x2 w1) + (x1 w3 + x2 w2 + x3 w1) + (x2 w3 + x3 w2 + x3 w3),
//
// of which the last bracket, at most 2^-24 of the product, is left out: six bf16 products with fp32
// accumulation, the large ones with one accumulation per 32 terms.  Measured against fp64
// on a 128-256-256-256-40 model with normal weights and features: relative error 0.99e-7, where
// the fp32 instruction left 2.7e-7.  That is a matter of long sums, whose own roundings outweigh
// the part left out: sums of at most kShortSum terms are taken on the fp32 instruction.  (A bf16
// stack's first layer has one part, x itself: three products.  Splitting fp32 operands into bf16 parts is
// due to Henry, Tang and Heinecke, "Leveraging the bfloat16 artificial intelligence datatype for
// higher-precision computations", 2019.)  Features and activations are split once, when they enter
// LDS; weights once per call (gp_lc_split_weights) or, in calls of few work items, in each of them.
// Infinities, NaNs and numbers that the factor carries beyond the largest bf16 one do not survive the
// split, but whatever they touch comes out of it as infinite or NaN: a wave whose sums are not all
// finite takes that layer again on the fp32 instruction (lc_layer_exact) and keeps these sums for
// the rows concerned, so results with such numbers are those of plain fp32 arithmetic, and a row's
// bits do not depend on the rows beside it.
//
// What bounds it: the matrix cores, 64 % busy at about 2 GHz (counters of the call over 169,343 fp32 rows); what they
// wait for is gather, splits and barriers, which the second workgroup of a compute unit covers in part.  us per
// call, on the fp32 instruction / here: four hops of a 128-256-256-256-40 model over all rows 1991 / 1050 - 1130 (the clock
// varies with the power that is left; 225 to 209 TFLOP/s of fp32 work, 1.35 to 1.25 PFLOP/s of bf16 products), a batch of
// 4096 rows with its launches 59.3 / 42.4; 100-256-256-256 branches of growing depth side by side from a bf16 stack,
// all rows, 920 / 505.  Models of few products have a kernel of their own (small_model).
//
// Index freedom used: MFMA sums over k, and which k a lane supplies is the kernel's choice
// as long as both operands agree; lanes 16 kg .. + 16 take k = 32 kt + 8 kg .. + 8 in step kt
// (one 16-byte LDS read per part).  Weights are the instruction's first operand (its rows
// are the layer's output columns) and batch rows its second, so a lane ends up with 4 CT
// consecutive output columns of one batch row: wide stores of the next layer's operand and
// of the result.
#include <algorithm>
#include <atomic>
#include <mutex>

#include "gp_lc.h"

namespace gp {

namespace {

constexpr int kLcThreads = 256;   // reduction and softmax
constexpr int kMlpThreads = 256;
constexpr int kLd = kPanel + 16;  // LDS row stride in bf16: 544 bytes, with which the 16 lanes of an LDS pass read 16-byte pieces of different banks
constexpr int64_t kWorkspaceBytes = INT64_C(256) << 20;  // cap on the partial results of one piece

typedef float v4f_a4 __attribute__((ext_vector_type(4), aligned(4)));  // 16-byte access from a dword boundary
typedef float v2f __attribute__((ext_vector_type(2)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef unsigned v2u __attribute__((ext_vector_type(2)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));

// Two fp32 numbers (times 2^16 already) as three pairs of bf16, packed as the matrix instructions take them,
// p1 + p2 + p3 = x: exactly, for |x| < kMaxBf16 that are 2^16 times an fp32 number.
// (The dot-product instruction would form a - p1 in one step, but beside another wave's matrix instructions it
// takes 81 cycles against 10 for an ordinary one: measured.)
constexpr float kUp = 0x1p16f;
constexpr float kMaxBf16 = 3.38953139e38f;
__device__ __forceinline__ unsigned pack_bf16(float a, float b) { return __builtin_bit_cast(unsigned, __builtin_convertvector((v2f){a, b}, v2bf)); }
__device__ __forceinline__ float low_bf16(unsigned p) { return __uint_as_float(p << 16); }
__device__ __forceinline__ float high_bf16(unsigned p) { return __uint_as_float(p & 0xFFFF0000u); }
__device__ __forceinline__ void split2(float a, float b, unsigned (&p)[3])
{
    p[0] = pack_bf16(a, b);
    const float ra = a - low_bf16(p[0]), rb = b - high_bf16(p[0]);
    p[1] = pack_bf16(ra, rb);
    p[2] = pack_bf16(ra - low_bf16(p[1]), rb - high_bf16(p[1]));
}
// eight fp32 numbers: one lane's operand, part by part
__device__ __forceinline__ void split8(const float (&v)[8], v4u (&q)[3])
{
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        unsigned p[3];
        split2(v[2 * s] * kUp, v[2 * s + 1] * kUp, p);
        q[0][s] = p[0], q[1][s] = p[1], q[2][s] = p[2];
    }
}
// an activation that cannot be split has a NaN as its first part, so that its row's sums come out as NaN, and its
// own bits, high and low half, as the others (low: it is the lower number of the pair)
__device__ __forceinline__ void keep_whole(float v, bool low, unsigned (&p)[3])
{
    const unsigned u = __float_as_uint(v), mask = low ? 0xFFFFu : 0xFFFF0000u;
    p[0] = (p[0] & ~mask) | (0x7FC07FC0u & mask);
    p[1] = (p[1] & ~mask) | (low ? u >> 16 : u & 0xFFFF0000u);
    p[2] = (p[2] & ~mask) | (low ? u & 0xFFFFu : u << 16);
}
// the number again from its parts
__device__ __forceinline__ float join3(__bf16 x1, __bf16 x2, __bf16 x3)
{
    const float a = (float)x1;
    if (a != a) return __uint_as_float((unsigned)__builtin_bit_cast(unsigned short, x2) << 16 | __builtin_bit_cast(unsigned short, x3));
    return (((float)x3 + (float)x2) + a) * (1.0f / kUp);
}

// TM x kin panel of the batch rows of one slab -> LDS, split into its bf16 parts (a bf16 stack has one),
// zero beyond kin (up to the next multiple of 32), zero for rows past the batch or ids outside [0, n)
// (those rows are never stored).  Six independent requests per thread are in flight before the first is
// written to LDS.
template <typename T, int TM>
__device__ __forceinline__ void lc_gather(__bf16* __restrict__ tile, const T* __restrict__ slab, const LcArgs& a,
                                          int64_t row0, int p0, int kin, int tid)
{
    constexpr int U = 6;
    constexpr int kPlane = TM * kLd;
    const unsigned nq = (unsigned)(((kin + 31) & ~31) >> 2);  // groups of four columns per row
    const unsigned total = TM * nq;
    for (unsigned base = 0; base < total; base += U * kMlpThreads) {
        int64_t id[U];
        unsigned r[U], q[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const unsigned idx = base + u * kMlpThreads + tid;
            r[u] = idx / nq, q[u] = idx - r[u] * nq;
            const int64_t br = row0 + r[u];
            id[u] = -1;
            if (idx < total && br < a.B) id[u] = a.batch ? (int64_t)a.batch[br] : br;
        }
        v4f v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            v[u] = (v4f){0.0f, 0.0f, 0.0f, 0.0f};
            if (id[u] >= 0 && id[u] < a.n) {
                const T* src = slab + id[u] * a.ld + p0 + 4 * q[u];
                const int c0 = 4 * (int)q[u];
                if (a.xvec && c0 + 4 <= kin) {
                    v[u] = load4(src);
                } else {
                    if (c0 + 0 < kin) v[u].x = widen(src[0]);
                    if (c0 + 1 < kin) v[u].y = widen(src[1]);
                    if (c0 + 2 < kin) v[u].z = widen(src[2]);
                    if (c0 + 3 < kin) v[u].w = widen(src[3]);
                }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (base + u * kMlpThreads + tid < total) {
                v2u* dst = reinterpret_cast<v2u*>(tile + r[u] * kLd + 4 * q[u]);
                if constexpr (sizeof(T) == 2) {  // (exact: the low half of the widened value is zero)
                    *dst = (v2u){(__float_as_uint(v[u].x) >> 16) | __float_as_uint(v[u].y),
                                 (__float_as_uint(v[u].z) >> 16) | __float_as_uint(v[u].w)};
                } else {
                    unsigned lo[3], hi[3];
                    asm("" : "+v"(v[u]));  // (the multiplications are not moved to the loads, each of which would then be waited for)
                    split2(v[u].x * kUp, v[u].y * kUp, lo);
                    split2(v[u].z * kUp, v[u].w * kUp, hi);
#pragma unroll
                    for (int i = 0; i < 3; ++i) dst[i * (kPlane / 4)] = (v2u){lo[i], hi[i]};
                }
            }
    }
}

__device__ __forceinline__ void lc_fence() { __builtin_amdgcn_sched_barrier(0); }  // the instruction scheduler moves nothing across

// the same in every lane: said so, so that it stays in scalar registers
typedef const __attribute__((address_space(1))) char global_char;
__device__ __forceinline__ global_char* uniform(const char* p)
{
    const uint64_t u = (uint64_t)p;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)u), hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(u >> 32));
    return (global_char*)(((uint64_t)hi << 32) | lo);
}

// How the four waves of a workgroup share a layer with N output columns: wave w takes CT tiles of 16 columns
// of every batch row, so that a weight is fetched by one wave.  Column i of a wave's tile t is output column
// 16 CT w + CT i + t: the four accumulator elements of a lane's CT tiles are 4 CT consecutive columns.
__host__ __device__ __forceinline__ int tiles_per_wave(int N) { return N > 128 ? 4 : N > 64 ? 2 : 1; }

// Split weights, in the order the waves read them: for every step of 32 rows, wave of the workgroup and tile of 16
// columns three fragments (the parts) of 64 lanes x 16 bytes; lane (i, kg) holds rows 32 kt + 8 kg .. + 8 of
// column i of the tile.  Beyond the matrix: zeros.  Steps are padded to a multiple of 4 / CT, so that a wave
// walks whole groups of four tiles (a panel of the first layer is 8 steps, a multiple already).
constexpr int64_t kFragBytes = 1024;
constexpr int64_t kFragSlack = 64 << 10;  // requests past a layer's end reach this far at most
__host__ __device__ __forceinline__ int64_t padded_steps(int64_t kin, int ct) { return ((kin + 31) / 32 + 4 / ct - 1) / (4 / ct) * (4 / ct); }
__host__ __device__ __forceinline__ int64_t layer_tiles(int64_t kin, int N)
{
    const int ct = tiles_per_wave(N);
    return padded_steps(kin, ct) * 4 * ct;
}

struct SplitArgs {
    int T;
    const float* W[kMaxLayers];
    int kin[kMaxLayers], width[kMaxLayers];
    int first[kMaxLayers + 1];  // tiles (three fragments) before layer t
    char* out;
};

// one wave per (layer, step, wave, tile).  A few microseconds for a few hundred thousand weights; done once per
// call, where splitting them in every workgroup that uses them costs as much vector work as all of the
// activations (128-256-256-256-40 model, 4 hops side by side, 60,000 rows: 572 us that way, 390 us this way).
__global__ __launch_bounds__(256) void gp_lc_split_weights(const SplitArgs a)
{
    const int g = (int)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));  // (a slot holds a few thousand tiles)
    if (g >= a.first[a.T]) return;
    const int lane = threadIdx.x & 63, i = lane & 15, kg = lane >> 4;
    int t = 0;
    while (g >= a.first[t + 1]) ++t;
    const int N = a.width[t], kin = a.kin[t], CT = tiles_per_wave(N);
    const unsigned u = (unsigned)(g - a.first[t]), kt = u / (4 * CT);
    const int w = (int)(u / CT % 4), ct = (int)(u % CT), col = 16 * CT * w + CT * i + ct;
    // (all eight in flight: read at a clamped place and replaced beyond the matrix, not read under a condition)
    const float* at = a.W[t] + min(col, N - 1);
    float v[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) v[s] = at[(int64_t)min((int)kt * 32 + 8 * kg + s, kin - 1) * N];
#pragma unroll
    for (int s = 0; s < 8; ++s)
        if ((int)kt * 32 + 8 * kg + s >= kin || col >= N) v[s] = 0.0f;
    v4u q[3];
    split8(v, q);
#pragma unroll
    for (int p = 0; p < 3; ++p) reinterpret_cast<v4u*>(a.out + ((int64_t)g * 3 + p) * kFragBytes)[lane] = q[p];
}

// One term of a sum is off by up to 2^-23 of itself in six products (2^-24 left out, 2^-24 for the fp32 result), by half of
// that on the fp32 instruction; n terms of like size by about sqrt(n) 2^-25 in either way from their additions.
constexpr int kShortSum = 16;

// The elements that sums on the fp32 instruction are taken of: a row of the stack (an element that cannot be split is not
// in the tile), or of the tile.
template <typename T>
struct StackRows {
    const T* panel;  // row 0 of the slab, from the panel's first column on
    const int32_t* batch;
    int64_t ld, n, row0, B;
    struct Row {
        const T* p;
        bool in;
    };
    __device__ __forceinline__ Row row(int r) const
    {
        const int64_t br = row0 + r, id = br >= B ? -1 : batch ? (int64_t)batch[br] : br;
        const bool in = id >= 0 && id < n;
        return {panel + (in ? id * ld : 0), in};
    }
    __device__ __forceinline__ float at(const Row& r, int k) const { return r.in ? widen(r.p[k]) : 0.0f; }
};
template <int TM>
struct TileRows {
    const __bf16* tile;
    typedef const __bf16* Row;
    __device__ __forceinline__ Row row(int r) const { return tile + r * kLd; }
    __device__ __forceinline__ float at(Row p, int k) const { return join3(p[k], p[TM * kLd + k], p[2 * TM * kLd + k]); }
};

// acc += X(16 R rows x kin) * W(kin x the 16 CT columns from colbase on) on the fp32 instruction: plain fp32
// arithmetic, for short sums and for those that infinities, NaNs or very large numbers take part in.  (Elements are
// read at clamped places and replaced beyond the matrix, so that those of a step are in flight together.)
template <int R, int CT, typename Rows>
__device__ __forceinline__ void lc_layer_exact(const Rows& rows, int kin, const float* W, int N, int colbase, int i, int kg, v4f (&acc)[R][4])
{
    // (so that no part of this is worked out ahead of the branch to it, in registers that the other way needs)
    asm volatile("" : "+v"(i), "+v"(kg));
    typename Rows::Row row[R];
#pragma unroll
    for (int r = 0; r < R; ++r) row[r] = rows.row(r * 16 + i);
    for (int k0 = 0; k0 < kin; k0 += 4) {
        const int k = min(k0 + kg, kin - 1);
        const bool in = k0 + kg < kin;
        float x[R], w[CT];
#pragma unroll
        for (int r = 0; r < R; ++r) x[r] = rows.at(row[r], k);
#pragma unroll
        for (int c = 0; c < CT; ++c) w[c] = W[(int64_t)k * N + min(colbase + CT * i + c, N - 1)];
#pragma unroll
        for (int r = 0; r < R; ++r) x[r] = in ? x[r] : 0.0f;
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const float v = in && colbase + CT * i + c < N ? w[c] : 0.0f;
#pragma unroll
            for (int r = 0; r < R; ++r) acc[r][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(v, x[r], acc[r][c], 0, 0, 0);
        }
    }
}

// Numbers are taken up by 2^16 where they are split, sums are taken down again where they are used (CARRY: at once).
__host__ __device__ constexpr float sum_down(int parts, bool carry) { return carry ? 1.0f : 1.0f / (parts == 1 ? kUp : kUp * kUp); }

template <int R, int C>
__device__ __forceinline__ void lc_zero(v4f (&acc)[R][C])
{
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int c = 0; c < C; ++c) acc[r][c] = (v4f){0.0f, 0.0f, 0.0f, 0.0f};
}

// acc = tile(16 R rows x kin) * W(kin x the 16 CT columns from colbase on), see the head of the file, or a multiple
// of it: the sums are acc * sum_down().  Returns a bit for each row 16 r + i whose sums in this lane are not all finite (or
// cannot be split).  frags: the split weights from W's first row on.
// PARTS: bf16 parts of a row's elements in LDS, 3 (of 2^16 x) or (bf16 stack, first layer) 1 (x itself).  CARRY: acc
// comes in with sums of earlier panels, to which these are added (and which are put aside in `before`).
// RAW: no split weights, they are split here.  The products x1 w1 and
// the small ones have accumulators of their own, added at the end: the small ones then cost the large sum no
// roundings.  Four tiles' weights are in registers at any time: a tile's products done, its registers take
// the weights of the tile four further on.
template <int R, int CT, int PARTS, bool CARRY, bool RAW>
__device__ __forceinline__ unsigned lc_layer_six(const __bf16* tile, int kin, const float* W, int N, const char* frags, int wave, int colbase,
                                                 int i, int kg, v4f (&acc)[R][4], v4f (&before)[R][CT])
{
    constexpr int kPlane = 16 * R * kLd;
    const int steps = (kin + 31) >> 5, units = (int)padded_steps(kin, CT) * CT;
    const __bf16* xrow = tile + i * kLd + 8 * kg;
    // fragments of unit u = kt CT + ct: ((kt 4 + wave) CT + ct) * 3 ..
    global_char* mine = uniform(frags + wave * (CT * 3 * kFragBytes));
    const unsigned lane_off = (unsigned)(16 * kg + i) * 16;
    v4f big[R][CT], small[R][CT];
    lc_zero(big), lc_zero(small);
    if constexpr (CARRY) {
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int c = 0; c < CT; ++c) before[r][c] = acc[r][c];
    }
    v8bf part[4][3], x[R][PARTS];
    // RAW: weights of the steps ahead, as loaded: two where the accumulators leave the room.  (One load for all widths of
    // rows: with a way of its own for widths that are no multiple of CT, every load was waited for at the end of its
    // branch: 600-100 model, 60,000 rows, captured, 904 us that way, 469 this way; 128-256-256-256-40 632, 572.)
    typedef float vec __attribute__((ext_vector_type(CT), aligned(4)));
    constexpr int kAhead = CT == 4 ? 1 : 2;
    vec raw[RAW ? kAhead : 1][RAW ? 8 : 1];
    const int rawcol = min(colbase + CT * i, N - CT), shift = colbase + CT * i - rawcol;  // (columns beyond N: not used)
    auto load_raw = [&](int kt, int to) {
#pragma unroll
        for (int s = 0; s < 8; ++s)  // (rows beyond kin meet zeros)
            raw[to][s] = *reinterpret_cast<const vec*>(W + (int64_t)min(kt * 32 + 8 * kg + s, kin - 1) * N + rawcol);
    };
    auto load_w = [&](int u, int to) {  // (beyond the last unit: not used)
        global_char* at = mine + ((u / CT) * 4 * CT + u % CT) * (3 * kFragBytes);
#pragma unroll
        for (int p = 0; p < 3; ++p) part[to][p] = *reinterpret_cast<const __attribute__((address_space(1))) v8bf*>(at + p * kFragBytes + lane_off);
    };
    auto load_x = [&](int kt) {
        kt = min(kt, steps - 1);  // (padding steps have zero weights)
#pragma unroll
        for (int p = PARTS - 1; p >= 0; --p)
#pragma unroll
            for (int r = 0; r < R; ++r) x[r][p] = *reinterpret_cast<const v8bf*>(xrow + p * kPlane + r * 16 * kLd + kt * 32);
    };
    auto products = [&](int ct, int from) {
        auto mul = [&](int wi, int xi) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                v4f& to = wi + xi > 0 ? small[r][ct] : big[r][ct];
                to = __builtin_amdgcn_mfma_f32_16x16x32_bf16(part[from][wi], x[r][xi], to, 0, 0, 0);
            }
        };
        if constexpr (PARTS == 3) mul(0, 2), mul(1, 1), mul(0, 1);
        mul(2, 0), mul(1, 0), mul(0, 0);
    };
    auto split_raw = [&](int from, int first) {  // a step's raw weights into the parts of its tiles
        if (CT > 1 && N % CT != 0) {  // a lane whose last columns lie beyond N has read its first ones further right
#pragma unroll
            for (int s = 0; s < 8; ++s)
#pragma unroll
                for (int k = 0; k < CT - 1; ++k)  // one to the left, `shift` times at most
                    if (k < shift) {
#pragma unroll
                        for (int c = 0; c + 1 < CT; ++c) raw[from][s][c] = raw[from][s][c + 1];
                    }
        }
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            float v[8];
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                if constexpr (CT == 1) v[s] = raw[from][s][0];
                else v[s] = raw[from][s][c];
            }
            v4u q[3];
            split8(v, q);
#pragma unroll
            for (int p = 0; p < 3; ++p) part[first + c][p] = __builtin_bit_cast(v8bf, q[p]);
        }
    };
    if constexpr (RAW) {
#pragma unroll
        for (int k = 0; k < kAhead; ++k) load_raw(k, k);
    } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) load_w(u, u);
    }
    load_x(0);
    __builtin_amdgcn_s_setprio(0);
    for (int u = 0; u < units; u += 4) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            if constexpr (RAW) {
                if (u + v >= steps * CT) break;
                constexpr int kMask = kAhead - 1;
                if (v % CT == 0) split_raw((v / CT) & kMask, v), load_raw((u + v) / CT + kAhead, (v / CT) & kMask);
            }
            products(v % CT, v);
            if constexpr (!RAW) load_w(u + v + 4, v);
            if ((v + 1) % CT == 0) load_x((u + v + 1) / CT);
            lc_fence();
        }
    }
    __builtin_amdgcn_s_setprio(2);
    constexpr float kDown = sum_down(PARTS, false), kMost = CARRY ? kMaxBf16 / kUp : kMaxBf16;
    unsigned odd = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        bool finite = true;
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            acc[r][c] = big[r][c] + small[r][c];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if constexpr (CARRY) acc[r][c][e] = fmaf(acc[r][c][e], kDown, before[r][c][e]);
                finite &= fabsf(acc[r][c][e]) < kMost;
            }
        }
        if (!finite) odd |= 1u << r;
    }
    return odd;
}

// a layer for this wave, each row the way its sums need.  Returns a bit for each row 16 r + i whose sums come from the
// fp32 instruction: these are acc itself, the others acc * sum_down().
template <int R, int CT, int PARTS, bool CARRY, bool RAW, typename Rows>
__device__ __forceinline__ unsigned lc_layer(const __bf16* tile, const Rows& rows, int kin, const float* W, int N, const char* frags, int wave,
                                             int i, int kg, v4f (&acc)[R][4])
{
    const int colbase = wave * 16 * CT;
    if (__builtin_expect(kin <= kShortSum, 0)) {
        if constexpr (!CARRY) lc_zero(acc);
        lc_layer_exact<R, CT>(rows, kin, W, N, colbase, i, kg, acc);
        return ~0u;
    }
    v4f before[R][CT];
    const unsigned odd = lc_layer_six<R, CT, PARTS, CARRY, RAW>(tile, kin, W, N, frags, wave, colbase, i, kg, acc, before);
    if (__builtin_expect(!__any(odd), 1)) return 0;
    v4f exact[R][4];
    lc_zero(exact);
    if constexpr (CARRY) {
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int c = 0; c < CT; ++c) exact[r][c] = before[r][c];
    }
    lc_layer_exact<R, CT>(rows, kin, W, N, colbase, i, kg, exact);
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (odd >> r & 1) {
#pragma unroll
            for (int c = 0; c < CT; ++c) acc[r][c] = exact[r][c];
        }
    return odd;
}

template <int R, int PARTS, bool CARRY, bool RAW, typename Rows>
__device__ __forceinline__ unsigned lc_layer_any(const __bf16* tile, const Rows& rows, int kin, const float* W, int N, const char* frags, int wave,
                                                 int i, int kg, v4f (&acc)[R][4])
{
    const int ct = tiles_per_wave(N);
    if (wave * 16 * ct >= N) {
        lc_zero(acc);
        return 0;
    }
    if (ct == 4) return lc_layer<R, 4, PARTS, CARRY, RAW>(tile, rows, kin, W, N, frags, wave, i, kg, acc);
    if (ct == 2) return lc_layer<R, 2, PARTS, CARRY, RAW>(tile, rows, kin, W, N, frags, wave, i, kg, acc);
    return lc_layer<R, 1, PARTS, CARRY, RAW>(tile, rows, kin, W, N, frags, wave, i, kg, acc);
}

// tile <- relu(sums) for this wave's share of a layer of width Np (odd, down: how the sums stand in acc, see lc_layer);
// columns beyond Np become zeros, and every column below the next multiple of 32 is written (the next layer reads
// that far)
template <int R, int CT>
__device__ __forceinline__ void lc_store_relu(__bf16* __restrict__ tile, int Np, unsigned odd, float down, int colbase, int i, int kg,
                                              const v4f (&acc)[R][4])
{
    constexpr int kPlane = 16 * R * kLd;
    const int c0 = colbase + 4 * CT * kg;
    const bool some_odd = __any(odd), whole = !some_odd && colbase + 16 * CT <= Np;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        __bf16* row = tile + (r * 16 + i) * kLd + c0;
        unsigned q[3][2 * CT];
        if (whole) {  // every value may be split
            const float up = down * kUp;
#pragma unroll
            for (int h = 0; h < 2 * CT; ++h) {
                const int u = 2 * h;
                unsigned p[3];
                split2(fmaxf(acc[r][u % CT][u / CT], 0.0f) * up, fmaxf(acc[r][(u + 1) % CT][(u + 1) / CT], 0.0f) * up, p);
                q[0][h] = p[0], q[1][h] = p[1], q[2][h] = p[2];
            }
        } else {
            const float up = (odd >> r & 1 ? 1.0f : down) * kUp;
#pragma unroll
            for (int h = 0; h < 2 * CT; ++h) {
                float v[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int u = 2 * h + e;
                    v[e] = acc[r][u % CT][u / CT];
                    if (v[e] < 0.0f || c0 + u >= Np) v[e] = 0.0f;  // NaN stays NaN
                }
                unsigned p[3];
                split2(v[0] * up, v[1] * up, p);
                if (some_odd) {  // (where that cannot be split the row's sums are v itself)
                    if (!(v[0] * up < kMaxBf16)) keep_whole(v[0], true, p);
                    if (!(v[1] * up < kMaxBf16)) keep_whole(v[1], false, p);
                }
                q[0][h] = p[0], q[1][h] = p[1], q[2][h] = p[2];
            }
        }
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            if constexpr (CT == 1) {
                *reinterpret_cast<v2u*>(row + p * kPlane) = (v2u){q[p][0], q[p][1]};
            } else {
#pragma unroll
                for (int h = 0; h < CT / 2; ++h)
                    reinterpret_cast<v4u*>(row + p * kPlane)[h] = (v4u){q[p][4 * h], q[p][4 * h + 1], q[p][4 * h + 2], q[p][4 * h + 3]};
            }
        }
    }
}

template <int R>
__device__ __forceinline__ void lc_store_relu_any(__bf16* tile, int Np, unsigned odd, float down, int wave, int i, int kg, const v4f (&acc)[R][4])
{
    const int ct = tiles_per_wave(Np), colbase = wave * 16 * ct;
    if (colbase >= ((Np + 31) & ~31)) return;  // (its sums are zeros: it sat the layer out)
    if (ct == 4) lc_store_relu<R, 4>(tile, Np, odd, down, colbase, i, kg, acc);
    else if (ct == 2) lc_store_relu<R, 2>(tile, Np, odd, down, colbase, i, kg, acc);
    else lc_store_relu<R, 1>(tile, Np, odd, down, colbase, i, kg, acc);
}

template <int R, int CT>
__device__ __forceinline__ void lc_write(float* __restrict__ dst, const LcArgs& a, int64_t row0, int C, int colbase, float g,
                                         unsigned odd, float down, int i, int kg, const v4f (&acc)[R][4])
{
    const int c0 = colbase + 4 * CT * kg;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t row = row0 + r * 16 + i;
        if (row >= a.B) continue;
        float* out = dst + row * a.ldd + c0;
        const float f = odd >> r & 1 ? 1.0f : down;
#pragma unroll
        for (int h = 0; h < CT; ++h) {
            v4f v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = g * (f * acc[r][(4 * h + e) % CT][(4 * h + e) / CT]);
            if (c0 + 4 * h + 4 <= C) {
                *reinterpret_cast<v4f_a4*>(out + 4 * h) = v;
            } else {
#pragma unroll
                for (int e = 0; e < 3; ++e)
                    if (c0 + 4 * h + e < C) out[4 * h + e] = v[e];
            }
        }
    }
}

// One workgroup: 16 R batch rows of one branch (hop k, the first depth_k layers); writes
// gamma_k * branch_k either to its slab of the partial results or, when branches are
// concatenated, to its columns of the result.  48 rows take 78 KB of LDS: two workgroups share a compute unit,
// and while one gathers, stores or waits at a barrier the other keeps the matrix cores busy.
template <typename T, int R, bool CARRY, bool RAW>
__global__ __launch_bounds__(kMlpThreads, 2) void gp_lc_mlp(const LcArgs a)
{
    constexpr int TM = 16 * R;
    constexpr int kParts = sizeof(T) == 2 ? 1 : 3;
    extern __shared__ __align__(16) __bf16 tile[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15, kg = lane >> 4;
    const int br = (int)(blockIdx.x % (unsigned)a.hops);
    const int k = a.hop_of[br], layers = a.depth[br];
    const int64_t row0 = (int64_t)(blockIdx.x / (unsigned)a.hops) * TM;
    const int C = a.width[layers - 1];

    v4f acc[R][4];
    lc_zero(acc);

    const T* slab = static_cast<const T*>(a.stack) + (int64_t)k * a.slab;
    const int N1 = a.width[0];
    // whoever is not multiplying goes first: the other workgroup's products leave the vector units room
    __builtin_amdgcn_s_setprio(2);
    unsigned odd = 0;
    float down = sum_down(kParts, CARRY);
    for (int p0 = 0; p0 < a.d; p0 += kPanel) {  // first layer, one panel of feature columns at a time
        const int kin = min(kPanel, a.d - p0);
        if (p0 > 0) __syncthreads();  // every wave is done with the previous panel (nothing is in the tile before the first)
        lc_gather<T, TM>(tile, slab, a, row0, p0, kin, tid);
        __syncthreads();
        const char* frags = a.frags + a.frag_off[0] + (int64_t)(p0 / 32) * 4 * tiles_per_wave(N1) * (3 * kFragBytes);
        const StackRows<T> rows{slab + p0, a.batch, a.ld, a.n, row0, a.B};
        odd = lc_layer_any<R, kParts, CARRY, RAW>(tile, rows, kin, a.W[0] + (int64_t)p0 * N1, N1, frags, wave, i, kg, acc);
    }
    for (int t = 1; t < layers; ++t) {
        const int Np = a.width[t - 1], N = a.width[t];
        __syncthreads();  // every wave is done reading the tile
        lc_store_relu_any<R>(tile, Np, odd, down, wave, i, kg, acc);
        down = sum_down(3, false);
        __syncthreads();
        const TileRows<TM> rows{tile};
        odd = lc_layer_any<R, 3, false, RAW>(tile, rows, Np, a.W[t], N, a.frags + a.frag_off[t], wave, i, kg, acc);
    }

    const float g = a.gamma[k];
    float* dst = a.direct ? a.dst + a.out_off[br] : a.dst + (int64_t)br * a.B * a.ldd;
    const int ct = tiles_per_wave(C), colbase = wave * 16 * ct;
    if (ct == 4) lc_write<R, 4>(dst, a, row0, C, colbase, g, odd, down, i, kg, acc);
    else if (ct == 2) lc_write<R, 2>(dst, a, row0, C, colbase, g, odd, down, i, kg, acc);
    else lc_write<R, 1>(dst, a, row0, C, colbase, g, odd, down, i, kg, acc);
}

// out[i][c] = sum (or maximum) over the branches, in branch order, of the partial results
__global__ __launch_bounds__(kLcThreads) void gp_lc_reduce(const float* __restrict__ part, int items, int take_max, int64_t B,
                                                           int C, float* __restrict__ out, int64_t ldo)
{
    const int64_t total = B * C;
    for (int64_t i = (int64_t)blockIdx.x * kLcThreads + threadIdx.x; i < total; i += (int64_t)gridDim.x * kLcThreads) {
        float s = part[i];
        for (int it = 1; it < items; ++it) {
            const float v = part[(int64_t)it * total + i];
            s = take_max ? (v > s || v != v ? v : s) : s + v;  // a NaN branch makes the maximum NaN
        }
        out[(i / C) * ldo + i % C] = s;
    }
}

// Y = softmax(H) row by row, in place: one wave per row, row maximum subtracted first
__global__ __launch_bounds__(kLcThreads) void gp_lc_softmax_rows(float* __restrict__ H, int64_t B, int C, int64_t ld)
{
    const int lane = threadIdx.x & 63;
    const int64_t wave = ((int64_t)blockIdx.x * kLcThreads + threadIdx.x) >> 6;
    const int64_t waves = (int64_t)gridDim.x * (kLcThreads >> 6);
    for (int64_t r = wave; r < B; r += waves) {
        float* row = H + r * ld;
        float m = -INFINITY;
        for (int c = lane; c < C; c += 64) m = fmaxf(m, row[c]);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
        float sum = 0.0f;
        for (int c = lane; c < C; c += 64) sum += expf(row[c] - m);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
        const float inv = 1.0f / sum;
        for (int c = lane; c < C; c += 64) row[c] = expf(row[c] - m) * inv;
    }
}

// partial results: one grow-only buffer per device
struct Workspace {
    float* p = nullptr;
    size_t bytes = 0;
};
std::mutex g_ws_mu;
Workspace g_ws[64];

gp_status workspace(size_t bytes, float** out)
{
    int dev = 0;
    GP_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= 64) return fail(GP_ERR_UNSUPPORTED, "device ordinal %d not supported", dev);
    std::lock_guard<std::mutex> lk(g_ws_mu);
    Workspace& w = g_ws[dev];
    if (w.bytes < bytes) {
        if (w.p) GP_HIP(hipFree(w.p));  // waits for the device: no earlier launch still uses it
        w.p = nullptr, w.bytes = 0;
        GP_HIP(hipMalloc((void**)&w.p, bytes));
        w.bytes = bytes;
    }
    *out = w.p;
    return GP_OK;
}

// Room for split weights: a fixed array on every device, held from load to process end, so that no call
// allocates, frees or waits for the device on their account (another thread may be capturing a graph, which
// an allocation would break), and what is held is bounded.  Weights that do not fit their slot are split where they
// are used: 8 MiB are 1.3 million weights, one 256-wide layer on 5,400 features.
// Slot 0 is for calls with partial results, captured ones too: they do not overlap.  Direct calls (no partial
// results, so calls may overlap) share the other slots, handed out by stream handle so that calls on different
// streams do not wait for one another.  Equal handles are not taken for an order: one handle can be several
// streams (hipStreamPerThread is another one in every thread; a destroyed stream's handle comes back).  Every call
// waits for the event recorded behind the call that used its slot last, which costs nothing where both are on
// one stream.  A stream without a slot takes a new one, or, once all are taken, the one whose last call was longest
// ago.  g_slot_mu is held while a call enqueues: nobody takes the slot between the wait and the next record.
constexpr int kSlots = 8;
constexpr size_t kSlotBytes = 8 << 20;
static __device__ __align__(256) char split_room[kSlots * kSlotBytes];
struct Slot {
    hipStream_t stream = nullptr;
    bool taken = false;
    hipEvent_t done = nullptr;  // recorded behind the last call that used it
    bool used = false;          // it has been recorded
    uint64_t last = 0;
};
std::mutex g_slot_mu;
Slot g_slots[64][kSlots];
char* g_room[64];
uint64_t g_slot_calls = 0;

gp_status room_on_current_device(int* dev, char** out)  // (g_slot_mu held)
{
    GP_HIP(hipGetDevice(dev));
    if (*dev < 0 || *dev >= 64) return fail(GP_ERR_UNSUPPORTED, "device ordinal %d not supported", *dev);
    if (!g_room[*dev]) {
        void* p = nullptr;
        GP_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(split_room)));
        g_room[*dev] = (char*)p;
    }
    *out = g_room[*dev];
    return GP_OK;
}

gp_status take_slot(hipStream_t stream, Slot** out, char** where)  // (g_slot_mu held)
{
    int dev = 0;
    char* room = nullptr;
    gp_status st = room_on_current_device(&dev, &room);
    if (st != GP_OK) return st;
    Slot *const first = g_slots[dev] + 1, *const end = g_slots[dev] + kSlots;
    Slot* s = nullptr;  // the stream's own, else a free one, else the one longest unused
    for (Slot* t = first; t < end; ++t)
        if (t->taken && t->stream == stream) s = t;
    if (!s)
        for (Slot* t = first; t < end; ++t)
            if (!s || (s->taken && (!t->taken || t->last < s->last))) s = t;
    if (!s->done) GP_HIP(hipEventCreateWithFlags(&s->done, hipEventDisableTiming));
    if (s->used) GP_HIP(hipStreamWaitEvent(stream, s->done, 0));
    s->stream = stream, s->taken = true, s->last = ++g_slot_calls;
    *out = s, *where = room + (s - g_slots[dev]) * kSlotBytes;
    return GP_OK;
}

// Marks the end of a call that took a slot, however the call ends: whatever it enqueued is in front of the event.
// A call whose event cannot be recorded waits for its stream instead.
struct SlotUse {
    Slot* s = nullptr;
    ~SlotUse()
    {
        if (!s) return;
        if (hipEventRecord(s->done, s->stream) == hipSuccess)
            s->used = true;
        else
            (void)hipStreamSynchronize(s->stream);
    }
};

int compute_units()
{
    static int cus = [] {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1)
            n = 256;
        return n;
    }();
    return cus;
}

template <typename T, int R, bool CARRY, bool RAW>
gp_status launch_mlp_t(const LcArgs& a, unsigned grid, hipStream_t stream)
{
    constexpr size_t lds = (size_t)16 * R * kLd * 3 * sizeof(uint16_t);
    // the kernel's LDS tile is above the 64 KB a kernel gets by default: raise the limit
    // once per device (the attribute belongs to the device's copy of the kernel)
    static std::atomic<uint64_t> done{0};
    int dev = 0;
    GP_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= 64) return fail(GP_ERR_UNSUPPORTED, "device ordinal %d not supported", dev);
    if (!(done.load(std::memory_order_acquire) >> dev & 1)) {
        GP_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&gp_lc_mlp<T, R, CARRY, RAW>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        done.fetch_or(UINT64_C(1) << dev, std::memory_order_release);
    }
    profile_begin("gp_lc_mlp", stream);
    hipLaunchKernelGGL((gp_lc_mlp<T, R, CARRY, RAW>), dim3(grid), dim3(kMlpThreads), lds, stream, a);
    profile_end(stream);
    GP_HIP(hipGetLastError());
    return GP_OK;
}

template <typename T, bool CARRY>
gp_status launch_mlp_c(int tile_rows, const LcArgs& a, unsigned grid, hipStream_t stream)
{
    if (!a.frags) return tile_rows == 16 ? launch_mlp_t<T, 1, CARRY, true>(a, grid, stream) : launch_mlp_t<T, 2, CARRY, true>(a, grid, stream);
    if (tile_rows == 16) return launch_mlp_t<T, 1, CARRY, false>(a, grid, stream);
    if (tile_rows == 32) return launch_mlp_t<T, 2, CARRY, false>(a, grid, stream);
    return launch_mlp_t<T, 3, CARRY, false>(a, grid, stream);
}

template <typename T>
gp_status launch_mlp(int tile_rows, const LcArgs& a, unsigned grid, hipStream_t stream)
{
    return a.d > kPanel ? launch_mlp_c<T, true>(tile_rows, a, grid, stream) : launch_mlp_c<T, false>(tile_rows, a, grid, stream);
}

// Rows of a work item.  Two items share a compute unit; a round of items lasts (measured on a 128-256-256-256-40
// model, microseconds) 21 / 28 / 38 for 16 / 32 / 48 rows where every unit has two, 19 / 22 / 28 where none has
// more than one: the height with the least sum over the call's rounds.  (4 hops: 512 rows 25 us with 16-row items,
// 33 with 48; 4096 rows 41 us with 32, 54 with 16, 48 with 48; 60,000 rows 397 us with 48, 433 with 32.)  Over 17
// models (widths 16 to 256, 1 to 7 layers, 32 to 602 features, both types, sums and side by side, 1024 to 60,000 rows) the
// height chosen is 1.1 % from the best on average.  It is wrong where it gives every unit exactly two 16-row items, which
// a single round of 32-row items beats by 10 to 35 % (2048 rows x 4 hops).
int choose_tile_rows(int64_t B, int hops)
{
    const int64_t both[3] = {21, 28, 38}, alone[3] = {19, 22, 28};
    int best = 0;
    int64_t best_cost = 0;
    for (int r = 0; r < 3; ++r) {
        const int64_t items = (B + 16 * (r + 1) - 1) / (16 * (r + 1)) * hops, cus = compute_units();
        const int64_t rest = items % (2 * cus);
        const int64_t cost = items / (2 * cus) * both[r] + (rest == 0 ? 0 : rest <= cus ? alone[r] : both[r]);
        if (r == 0 || cost <= best_cost) best = r, best_cost = cost;
    }
    return 16 * (best + 1);
}

// Which models run on the fp32 instruction (gp_lc_f32.hip): those of few products per row, whatever the batch, so that a
// row's bits do not depend on it.  Products of a layer at most 64 wide on fewer than 128 inputs do not count: its steps
// are padded to 128.  us per call, fp32 instruction / six products, 4 hops side by side:
//   model               counted   1024 rows     60,000 rows     60,000 rows of a bf16 stack
//   16-16                     0   12.0 / 12.8     33 /  56        34 /  51
//   64-64-64-40               0   12.7 / 13.2    100 / 115       109 / 111
//   16-256                4,096   12.5 / 12.9    103 / 125       102 / 111
//   128-40                5,120   12.4 / 12.5     77 /  73        92 /  78
//   32-200-16             9,600   12.7 / 13.1    122 / 106       125 / 101
//   300-40               12,000   13.9 / 12.5    189 / 185       197 / 158
//   128-128-40           21,504   12.6 / 12.5    145 / 110       159 / 108
//   100-256-40           35,840   15.5 / 12.3    231 / 168       232 / 142
//   128-128-128-40       37,888   14.2 / 13.3    214 / 146       217 / 140
//   128-256-256-256-40  174,080   33.8 / 25      723 / 389       731 / 367
constexpr int64_t kSmallModel = 5000;
bool small_model(int T, int d, const int32_t* width)
{
    int64_t products = 0;
    for (int t = 0; t < T; ++t) {
        const int64_t in = t == 0 ? d : width[t - 1];
        if (width[t] > 64 || in >= 128) products += in * width[t];
    }
    return products < kSmallModel;
}

// Where a call's work items are few, splitting the weights in each of them costs less than the launch that splits them
// once: the launch takes 2 to 3 us, with the event of a direct call 4 to 5 (host time, where the queue runs dry), and a step
// of 32 weight rows takes 0.1 to 0.2 us longer in a layer wider than 64, twice that where two items share a unit.
// us, 4 hops, split beforehand / where used:
//                                       items alone (1024 rows)      two to a unit (2048)
//   steps  model                 side by side   summed          side by side   summed
//       4  100-256-40               18.0 / 12.3    17.0 / 15.0     19.0 / 15.0    18.6 / 18.7
//       8  128-128-128-40           16.3 / 13.3    15.8 / 15.4     18.2 / 15.1    17.7 / 18.7
//      12  128-128-128-128-40       18.6 / 14.5    18.0 / 18.0     21.5 / 18.9    20.9 / 22.6
//      20  128-256-256-256-40       25.8 / 24.6    25.7 / 28.3     33.6 / 35.3    34.5 / 39.3
//      24  128, six times 128, 40   24.3 / 22.5    23.4 / 26.0     28.4 / 30.9    28.3 / 35.1
// Every workgroup of the call is resident at once: a second round would pay again, except in models without a wider layer
// on one panel of features (128-40 side by side, 16,384 rows 31.5 / 26.0 in four rounds of 32-row items, 60,000 rows
// 73 / 81; 602-64-40, 16,384 rows 120 / 129).
bool split_where_used(int wide_steps, int d, bool direct, int64_t items)
{
    const int cus = compute_units();
    if (wide_steps == 0 && d <= kPanel) return items <= 8 * cus;
    if (items > 2 * cus) return false;
    const bool alone = items <= cus;
    return wide_steps <= (direct ? (alone ? 30 : 15) : (alone ? 12 : 4));
}

}  // namespace

gp_status lc_forward(const void* stack, int64_t ld, gp_dtype dtype, int64_t n, int32_t d, int32_t K, const int32_t* batch,
                     int64_t B, const float* gamma, const int32_t* depth, gp_comb comb, int32_t T, const float* const* W,
                     const int32_t* width, float* out, int64_t ldo, hipStream_t stream)
{
    if (!stack || !gamma || !W || !width || !out) return fail(GP_ERR_INVALID_ARG, "NULL argument");
    if (dtype != GP_F32 && dtype != GP_BF16) return fail(GP_ERR_INVALID_ARG, "unknown dtype %d", (int)dtype);
    if (comb != GP_COMB_SUM && comb != GP_COMB_CONCAT && comb != GP_COMB_MAX)
        return fail(GP_ERR_INVALID_ARG, "unknown combination %d", (int)comb);
    if (n < 1 || d < 1 || ld < d) return fail(GP_ERR_INVALID_ARG, "need n >= 1, d >= 1, ld >= d");
    if (K < 0 || K + 1 > kMaxHops) return fail(GP_ERR_UNSUPPORTED, "K = %d: 0 .. %d hops supported", K, kMaxHops - 1);
    if (T < 1 || T > kMaxLayers) return fail(GP_ERR_UNSUPPORTED, "T = %d: 1 .. %d layers supported", T, kMaxLayers);
    if (B < 0 || (!batch && B > n)) return fail(GP_ERR_INVALID_ARG, "B = %lld out of range", (long long)B);
    for (int t = 0; t < T; ++t) {
        if (!W[t]) return fail(GP_ERR_INVALID_ARG, "W[%d] is NULL", t);
        if (width[t] < 1 || width[t] > kPanel)
            return fail(GP_ERR_UNSUPPORTED, "layer %d is %d wide: 1 .. %d supported", t + 1, width[t], kPanel);
    }

    LcArgs a{};
    a.stack = stack, a.ld = ld, a.slab = n * ld, a.n = n, a.d = d;
    a.batch = batch, a.B = B, a.T = T;
    // branches in use, their depths and where their columns go
    int C = 0, total_width = 0;
    for (int k = 0; k <= K; ++k) {
        const int dk = depth ? depth[k] : T;
        if (dk < 0 || dk > T) return fail(GP_ERR_INVALID_ARG, "depth[%d] = %d outside 0 .. T", k, dk);
        a.gamma[k] = gamma[k];
        if (dk == 0) continue;
        const int wk = width[dk - 1];
        if (comb != GP_COMB_CONCAT && a.hops > 0 && wk != C)
            return fail(GP_ERR_INVALID_ARG, "branches of widths %d and %d cannot be summed or maximised", C, wk);
        C = std::max(C, wk);
        a.hop_of[a.hops] = k, a.depth[a.hops] = dk, a.out_off[a.hops] = comb == GP_COMB_CONCAT ? total_width : 0;
        total_width += wk;
        ++a.hops;
    }
    if (a.hops == 0) return fail(GP_ERR_INVALID_ARG, "every hop is left out (all depths are 0)");
    const int out_width = comb == GP_COMB_CONCAT ? total_width : C;
    if (ldo < out_width) return fail(GP_ERR_INVALID_ARG, "ldo < output width %d", out_width);
    if (B == 0) return GP_OK;
    a.direct = comb == GP_COMB_CONCAT || a.hops == 1;
    for (int t = 0; t < T; ++t) a.W[t] = W[t], a.width[t] = width[t];
    const size_t esz = dtype == GP_F32 ? 4 : 2;
    a.xvec = ld % 4 == 0 && (uintptr_t)stack % (4 * esz) == 0;

    // One workgroup per (row tile, branch), so that a mini-batch of a few thousand rows still fills the chip; the
    // branches' results are then combined in hop order.  Large batches go through in pieces that keep the
    // partial results within a fixed size.
    for (int t = 0; t < T; ++t) a.wvec[t] = width[t] > 128 && width[t] % 2 == 0 && (uintptr_t)W[t] % 8 == 0;  // two tiles per wave, pairs aligned
    const bool small = small_model(T, d, width);
    const int asked = (int)options().lc_tile_rows;
    int tm, wide_steps = 0;  // (wide_steps: of 32 weight rows, in layers wider than 64)
    for (int t = 0; t < T; ++t)
        if (width[t] > 64) wide_steps += ((t == 0 ? d : width[t - 1]) + 31) / 32;
    if (small)  // 32 rows where even these give no more than one workgroup per CU: the call lasts as long as one item
        tm = asked != 0 ? asked : (B + 31) / 32 * a.hops <= compute_units() ? 32 : 64;
    else
        tm = asked == 0 ? choose_tile_rows(B, a.hops) : asked >= 48 ? 48 : 32;
    if (!small && asked == 0 && tm > 32 && wide_steps == 0 && split_where_used(0, d, a.direct, (B + 31) / 32 * a.hops)) tm = 32;
    const int64_t piece = a.direct ? B : std::max<int64_t>(64, kWorkspaceBytes / ((int64_t)a.hops * C * 4) / 64 * 64);
    SplitArgs sp{};
    sp.T = T;
    for (int t = 0; t < T; ++t) {
        const int in = t == 0 ? d : width[t - 1];
        sp.W[t] = W[t], sp.kin[t] = in, sp.width[t] = width[t];
        a.frag_off[t] = (int64_t)sp.first[t] * 3 * kFragBytes;
        sp.first[t + 1] = sp.first[t] + (int)layer_tiles(in, width[t]);  // (at most 2^30, of the widest first layer)
    }
    const int64_t frag_bytes = (int64_t)sp.first[T] * 3 * kFragBytes + kFragSlack;
    // Where the split weights go: into slot 0 where there are partial results (such calls do not overlap), else into
    // a slot of the stream's.  A direct call under graph capture goes without and splits weights where it uses them: its
    // replays may run beside other calls, which a shared slot would not survive.
    float* part = nullptr;
    std::unique_lock<std::mutex> slot_lock(g_slot_mu, std::defer_lock);
    SlotUse slot;  // (after the lock: it ends before the lock does)
    const bool split = !small && (size_t)frag_bytes <= kSlotBytes &&
                       !(tm <= 32 && split_where_used(wide_steps, d, a.direct, (B + tm - 1) / tm * a.hops));
    if (!a.direct) {
        gp_status st = workspace((size_t)a.hops * std::min(piece, B) * C * sizeof(float), &part);
        if (st != GP_OK) return st;
        if (split) {
            int dev = 0;
            std::lock_guard<std::mutex> lk(g_slot_mu);
            if ((st = room_on_current_device(&dev, &sp.out)) != GP_OK) return st;
        }
    } else if (split) {
        hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
        GP_HIP(hipStreamIsCapturing(stream, &capture));
        if (capture == hipStreamCaptureStatusNone) {
            slot_lock.lock();
            gp_status st = take_slot(stream, &slot.s, &sp.out);
            if (st != GP_OK) return st;
        }
    }
    a.frags = sp.out;
    if (a.frags) {
        profile_begin("gp_lc_split_weights", stream);
        hipLaunchKernelGGL(gp_lc_split_weights, dim3((unsigned)(sp.first[T] + 3) / 4), dim3(256), 0, stream, sp);
        profile_end(stream);
        GP_HIP(hipGetLastError());
    } else if (!small) {
        tm = std::min(tm, 32);  // (raw weights take registers: 32 rows at most)
    }
    for (int64_t b0 = 0; b0 < B; b0 += piece) {
        LcArgs p = a;
        p.B = std::min(piece, B - b0);
        p.batch = batch ? batch + b0 : nullptr;
        if (!batch) p.stack = static_cast<const char*>(stack) + (size_t)b0 * ld * esz, p.n = n - b0;
        if (a.direct)
            p.dst = out + b0 * ldo, p.ldd = ldo;
        else
            p.dst = part, p.ldd = C;
        const int64_t grid = (p.B + tm - 1) / tm * a.hops;
        if (grid > 0x7fffffffLL) return fail(GP_ERR_UNSUPPORTED, "batch too large for one launch");
        gp_status st = small             ? launch_lc_f32(dtype, tm, p, (unsigned)grid, stream)
                       : dtype == GP_F32 ? launch_mlp<float>(tm, p, (unsigned)grid, stream)
                                         : launch_mlp<unsigned short>(tm, p, (unsigned)grid, stream);
        if (st != GP_OK) return st;
        if (!a.direct) {
            const unsigned rgrid = (unsigned)std::min<int64_t>((p.B * C + kLcThreads - 1) / kLcThreads, 256 * 8);
            profile_begin("gp_lc_reduce", stream);
            hipLaunchKernelGGL(gp_lc_reduce, dim3(rgrid), dim3(kLcThreads), 0, stream, part, a.hops, comb == GP_COMB_MAX ? 1 : 0,
                               p.B, C, out + b0 * ldo, ldo);
            profile_end(stream);
            GP_HIP(hipGetLastError());
        }
    }
    return GP_OK;
}

}  // namespace gp

extern "C" gp_status gp_lc_forward(const void* stack, int64_t ld, gp_dtype dtype, int64_t n, int32_t d, int32_t K,
                                   const int32_t* batch, int64_t B, const float* gamma, int32_t T, const float* const* W,
                                   const int32_t* width, float* out, int64_t ldo, void* hip_stream)
{
    try {
        return gp::lc_forward(stack, ld, dtype, n, d, K, batch, B, gamma, nullptr, GP_COMB_SUM, T, W, width, out, ldo,
                              (hipStream_t)hip_stream);
    } catch (const std::exception& e) {
        return gp::fail(GP_ERR_OOM_HOST, "gp_lc_forward: %s", e.what());
    }
}

extern "C" gp_status gp_lc_softmax(float* H, int64_t B, int32_t C, int64_t ld, void* hip_stream)
{
    using namespace gp;
    if (!H) return fail(GP_ERR_INVALID_ARG, "NULL argument");
    if (B < 0 || C < 1 || ld < C) return fail(GP_ERR_INVALID_ARG, "need B >= 0, C >= 1, ld >= C");
    if (B == 0) return GP_OK;
    hipStream_t stream = (hipStream_t)hip_stream;
    const unsigned grid = (unsigned)std::min<int64_t>((B + 3) / 4, 256 * 16);
    profile_begin("gp_lc_softmax_rows", stream);
    hipLaunchKernelGGL(gp_lc_softmax_rows, dim3(grid), dim3(kLcThreads), 0, stream, H, B, (int)C, ld);
    profile_end(stream);
    GP_HIP(hipGetLastError());
    return GP_OK;
}

extern "C" gp_status gp_lc_forward_branches(const void* stack, int64_t ld, gp_dtype dtype, int64_t n, int32_t d, int32_t K,
                                            const int32_t* batch, int64_t B, const float* gamma, const int32_t* depth,
                                            gp_comb comb, int32_t T, const float* const* W, const int32_t* width, float* out,
                                            int64_t ldo, void* hip_stream)
{
    try {
        if (!depth) return gp::fail(GP_ERR_INVALID_ARG, "NULL argument");
        return gp::lc_forward(stack, ld, dtype, n, d, K, batch, B, gamma, depth, comb, T, W, width, out, ldo,
                              (hipStream_t)hip_stream);
    } catch (const std::exception& e) {
        return gp::fail(GP_ERR_OOM_HOST, "gp_lc_forward_branches: %s", e.what());
    }
}
