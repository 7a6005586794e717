// Row clusters on the GPU: the label propagation of gp_cluster.cpp (synchronous; a row takes the most frequent label
// among its sources, ties to the smallest; at most kClusterRounds rounds, until fewer than one row in 2000 changes),
// the renumbering, and the figures the cache schedule is chosen by.  Counts are exact integers, so labels and figures
// are the host's whatever the order in which the GPU counts.
//
// What bounds it: the label of every source, a random 4-byte read per non-zero and round, and what a row's counting takes
// beside them.  490,000 rows and 12.5 million non-zeros of a power law: 1.3 ms in all kernels, 5 rounds (16 host threads:
// 24 ms); 233,000 rows and 114 million non-zeros in 50 communities: 4.8 ms (100 ms).  A row is taken by one workgroup at
// most, in time proportional to its sources: 1,200,000 rows, one of them of a million sources, 33 ms, 23 of them that row's
// (874 with a table in LDS that goes over such a row 123 times a round).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <vector>

#include "gp_block_scan.h"
#include "gp_internal.h"

namespace gp {

namespace {

constexpr int kThreads = 256;
constexpr int kTileRows = 16;          // consecutive rows a wavefront takes at a time
constexpr int kShortRow = 64;          // rows of up to as many sources: one per lane
constexpr int kMidRow = 512;           // rows of up to as many: a workgroup of one wavefront and a table of twice as many places
constexpr int kMidTable = 1024;
constexpr int kBigRow = 12288;         // rows of up to as many: a workgroup of 1024 and a table that they fill to three quarters at
constexpr int kBigTable = 16384;       // most; longer rows ("huge"): a workgroup of 1024 and a counter in memory per label
constexpr int kMaxRounds = kClusterRounds;

// Words the rounds share.  changed[r]: rows that round r gave another label.
struct Tally {
    uint32_t changed[kMaxRounds];
    uint32_t mid_rows, big_rows, huge_rows;
    unsigned long long inside;      // non-zeros whose source has the row's label
    unsigned long long weight_size; // sum over the rows of (their non-zeros x rows of their cluster)
};

__device__ inline uint32_t mix(uint32_t x)
{
    x ^= x >> 16;
    x *= 0x7feb352dU;
    x ^= x >> 15;
    x *= 0x846ca68bU;
    x ^= x >> 16;
    return x;
}

// Rounds that count among the first `before`: the host enqueues all of them, and those after one that changed few rows
// return at once.
__device__ __host__ inline int rounds_that_count(const uint32_t* changed, int before, int64_t n)
{
    for (int r = 0; r < before; ++r)
        if ((int64_t)changed[r] * 2000 < n) return r + 1;
    return before;
}
__device__ inline bool over_before(const Tally* t, int round, int64_t n)
{
    return round > 0 && (rounds_that_count(t->changed, round, n) < round || (int64_t)t->changed[round - 1] * 2000 < n);
}

__device__ inline int64_t lane_value(int64_t v, int lane)  // the same for the whole wavefront, in scalar registers
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(uint64_t)v, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), lane);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// (count, smallest label first) as one number that is larger for the better candidate
__device__ inline unsigned long long candidate(uint32_t count, int32_t label) { return ((unsigned long long)count << 32) | (uint32_t)~(uint32_t)label; }

__global__ __launch_bounds__(kThreads) void gp_first_labels(int32_t* __restrict__ lab, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kThreads) lab[i] = (int32_t)i;
}

// The rows of more than kShortRow sources, listed once: a workgroup takes kListRows rows and asks for its places on the lists
// of mid and big rows with one atomic each (one per row queues at the counters: 490,000 rows, 407 us; 233,000 rows, all long, 2.7 ms).
constexpr int kListItems = 8;
constexpr int64_t kListRows = (int64_t)kThreads * kListItems;
__global__ __launch_bounds__(kThreads) void gp_list_long_rows(const int64_t* __restrict__ rowptr, int64_t n, Tally* __restrict__ tally,
                                                              int32_t* __restrict__ mid, int32_t* __restrict__ big, int32_t* __restrict__ huge)
{
    __shared__ uint32_t ws[kScanWaves + 1];
    __shared__ uint32_t first[2];
    const int64_t r0 = (int64_t)blockIdx.x * kListRows + (int64_t)threadIdx.x * kListItems;
    uint32_t is_mid = 0, is_big = 0;
    for (int j = 0; j < kListItems; ++j) {
        if (r0 + j >= n) break;
        const int64_t len = rowptr[r0 + j + 1] - rowptr[r0 + j];
        if (len > kBigRow)
            huge[atomicAdd(&tally->huge_rows, 1u)] = (int32_t)(r0 + j);  // (few: one in kBigRow non-zeros at most)
        else if (len > kMidRow)
            is_big |= 1u << j;
        else if (len > kShortRow)
            is_mid |= 1u << j;
    }
    uint32_t mids, bigs;
    uint32_t at_mid = block_exclusive((uint32_t)__popc(is_mid), ws, &mids);
    uint32_t at_big = block_exclusive((uint32_t)__popc(is_big), ws, &bigs);
    if (threadIdx.x == 0) {
        first[0] = mids ? atomicAdd(&tally->mid_rows, mids) : 0;
        first[1] = bigs ? atomicAdd(&tally->big_rows, bigs) : 0;
    }
    __syncthreads();
    at_mid += first[0];
    at_big += first[1];
    for (int j = 0; j < kListItems; ++j) {
        if (is_mid >> j & 1) mid[at_mid++] = (int32_t)(r0 + j);
        if (is_big >> j & 1) big[at_big++] = (int32_t)(r0 + j);
    }
}

// Rows of at most kShortRow sources, a wavefront per row: the labels lie one to a lane, and every distinct one is counted
// by a ballot, until those left are fewer than the best has.  In the first round labels are row numbers and a row's
// sources are distinct, so the first (smallest) source is the answer for rows of any length.
__global__ __launch_bounds__(kThreads) void gp_label_short_rows(const int64_t* __restrict__ rowptr, const int32_t* __restrict__ col, int64_t n,
                                                                const int32_t* __restrict__ even, const int32_t* __restrict__ odd, int round,
                                                                Tally* __restrict__ tally)
{
    if (over_before(tally, round, n)) return;
    const int32_t* lab = round & 1 ? odd : even;
    int32_t* nxt = const_cast<int32_t*>(round & 1 ? even : odd);
    const int lane = threadIdx.x & 63;
    const int64_t waves = (int64_t)gridDim.x * (kThreads / 64);
    uint32_t changed = 0;
    for (int64_t tile = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6); tile * kTileRows < n; tile += waves) {
        const int64_t r0 = tile * kTileRows;
        const int rows = (int)min((int64_t)kTileRows, n - r0);
        // all ends, sources and labels of the tile are asked for before the first is looked at
        const int64_t at = rowptr[r0 + min(lane, rows)];
        const int32_t own = lab[r0 + min(lane, rows - 1)];
        int32_t l[kTileRows];
        int len[kTileRows];
#pragma unroll
        for (int r = 0; r < kTileRows; ++r) {
            const int64_t s = lane_value(at, r), e = lane_value(at, r + 1);  // (rows past the last: empty)
            len[r] = (int)min(e - s, (int64_t)INT32_MAX);
            l[r] = -1;
            if (lane < len[r] && (len[r] <= kShortRow || round == 0)) l[r] = col[s + lane];
        }
        if (round > 0) {
#pragma unroll
            for (int r = 0; r < kTileRows; ++r)
                if (l[r] >= 0) l[r] = lab[l[r]];
        }
        int32_t found = own;  // lane r: row r's label
        bool here = lane < rows;
#pragma unroll
        for (int r = 0; r < kTileRows; ++r) {  // (conditions that are the same for the whole wavefront)
            if (len[r] == 0) continue;
            int32_t best = -1;
            if (round == 0) {
                best = __builtin_amdgcn_readfirstlane(l[r]);
            } else if (len[r] > kShortRow) {
                if (lane == r) here = false;
                continue;
            } else {
                unsigned long long left = __ballot(lane < len[r]);
                int most = 0;
                while (left && __popcll(left) >= most) {
                    const int32_t one = __builtin_amdgcn_readlane(l[r], __builtin_ctzll(left));
                    const unsigned long long same = __ballot(l[r] == one) & left;
                    const int count = __popcll(same);
                    if (count > most || (count == most && one < best)) {
                        best = one;
                        most = count;
                    }
                    left &= ~same;
                }
            }
            if (lane == r) found = best;
        }
        if (here) nxt[r0 + lane] = found;
        changed += (uint32_t)__popcll(__ballot(here && found != own));
    }
    __shared__ uint32_t part[kThreads / 64];
    if (lane == 0) part[threadIdx.x >> 6] = changed;
    __syncthreads();
    if (threadIdx.x == 0) {  // (one atomic per workgroup, not per wavefront: they queue)
        for (int w = 1; w < kThreads / 64; ++w) changed += part[w];
        if (changed) atomicAdd(&tally->changed[round], changed);
    }
}

// The lanes whose label is the first lane's count it once together: most rows have one label for most sources.  True for
// lanes that then have `votes` to add to the count of l (l < 0: no label).
__device__ inline bool counts_label(int32_t l, int lane, uint32_t& votes)
{
    votes = 1;
    const unsigned long long on = __ballot(l >= 0);
    if (!on) return false;
    const int first = __builtin_ctzll(on);
    const int32_t one = __builtin_amdgcn_readlane(l, first);
    const int together = __popcll(__ballot(l == one));
    if (lane == first) votes = (uint32_t)together;
    return l >= 0 && (l != one || lane == first);
}

// The workgroup's best candidate; thread 0 gives it to the row.  wave_best: a word per wavefront, in LDS
template <int NT>
__device__ inline void label_row(unsigned long long best, unsigned long long* wave_best, int32_t row, const int32_t* lab, int32_t* nxt,
                                 uint32_t& changed)
{
#pragma unroll
    for (int o = 32; o; o >>= 1) best = max(best, (unsigned long long)__shfl_xor(best, o, 64));
    if ((threadIdx.x & 63) == 0) wave_best[threadIdx.x >> 6] = best;
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 1; w < NT / 64; ++w) best = max(best, wave_best[w]);
        const int32_t label = (int32_t)~(uint32_t)best, before = lab[row];
        nxt[row] = label;
        changed += label != before;
    }
}

// Longer rows, a workgroup per row: labels counted in a table in LDS (open addressing), which has more places than the row
// sources.
template <int NT, int TABLE>
__global__ __launch_bounds__(NT) void gp_label_long_rows(const int64_t* __restrict__ rowptr, const int32_t* __restrict__ col, int64_t n,
                                                         const int32_t* __restrict__ even, const int32_t* __restrict__ odd, int round,
                                                         Tally* __restrict__ tally, const int32_t* __restrict__ list)
{
    extern __shared__ uint32_t places[];  // TABLE keys, TABLE counts
    uint32_t* key = places;
    uint32_t* cnt = places + TABLE;
    __shared__ unsigned long long wave_best[NT / 64];
    if (over_before(tally, round, n)) return;
    const int32_t* lab = round & 1 ? odd : even;
    int32_t* nxt = const_cast<int32_t*>(round & 1 ? even : odd);
    const uint32_t rows = TABLE == kMidTable ? tally->mid_rows : tally->big_rows;
    const int lane = threadIdx.x & 63;
    uint32_t changed = 0;
    for (uint32_t k = blockIdx.x; k < rows; k += gridDim.x) {
        const int32_t row = list[k];
        const int64_t s = rowptr[row];
        const int len = (int)(rowptr[row + 1] - s);
        uint32_t table = TABLE;  // no more of it than the row needs is cleared and looked through
        while (table / 4 >= (uint32_t)len && table > 256) table /= 2;
        unsigned long long best = 0;
        __syncthreads();  // (the row before is done with table and wave_best)
        for (uint32_t j = threadIdx.x; j < table; j += NT) {
            key[j] = 0xFFFFFFFFu;
            cnt[j] = 0;
        }
        __syncthreads();
        for (int j0 = 0; j0 < len; j0 += NT) {
            const int j = j0 + (int)threadIdx.x;
            const int32_t l = j < len ? lab[col[s + j]] : -1;
            uint32_t votes;
            if (counts_label(l, lane, votes)) {
                uint32_t at = mix((uint32_t)l) & (table - 1);
                for (;;) {
                    const uint32_t was = atomicCAS(&key[at], 0xFFFFFFFFu, (uint32_t)l);
                    if (was == 0xFFFFFFFFu || was == (uint32_t)l) break;
                    at = (at + 1) & (table - 1);
                }
                atomicAdd(&cnt[at], votes);
            }
        }
        __syncthreads();
        for (uint32_t j = threadIdx.x; j < table; j += NT)
            if (cnt[j]) best = max(best, candidate(cnt[j], (int32_t)key[j]));
        label_row<NT>(best, wave_best, row, lab, nxt, changed);
    }
    if (threadIdx.x == 0 && changed) atomicAdd(&tally->changed[round], changed);
}

// Rows longer than that table serves, a workgroup per row and a counter in memory for every label there may be: n words per
// workgroup, zero before and after.  The last to add to a label's counter sees its whole count, so the counters are not
// looked through; they are put back by going over the row once more.  What bounds it: two random reads and an atomic per
// source, four of each in flight per lane.
constexpr int kHugeThreads = 1024;
__global__ __launch_bounds__(kHugeThreads) void gp_label_huge_rows(const int64_t* __restrict__ rowptr, const int32_t* __restrict__ col, int64_t n,
                                                                   const int32_t* __restrict__ even, const int32_t* __restrict__ odd, int round,
                                                                   Tally* __restrict__ tally, const int32_t* __restrict__ list,
                                                                   uint32_t* counters)
{
    constexpr int U = 4;
    __shared__ unsigned long long wave_best[kHugeThreads / 64];
    if (over_before(tally, round, n)) return;
    const int32_t* lab = round & 1 ? odd : even;
    int32_t* nxt = const_cast<int32_t*>(round & 1 ? even : odd);
    uint32_t* cnt = counters + (int64_t)blockIdx.x * n;
    const uint32_t rows = tally->huge_rows;
    const int lane = threadIdx.x & 63;
    uint32_t changed = 0;
    for (uint32_t k = blockIdx.x; k < rows; k += gridDim.x) {
        const int32_t row = list[k];
        const int64_t s = rowptr[row], len = rowptr[row + 1] - s;
        auto labels_from = [&](int64_t j0, int32_t (&l)[U]) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t j = j0 + u * kHugeThreads + threadIdx.x;
                l[u] = j < len ? col[s + j] : -1;
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (l[u] >= 0) l[u] = lab[l[u]];
        };
        unsigned long long best = 0;
        for (int64_t j0 = 0; j0 < len; j0 += U * kHugeThreads) {
            int32_t l[U];
            labels_from(j0, l);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                uint32_t votes;
                if (counts_label(l[u], lane, votes)) best = max(best, candidate(atomicAdd(&cnt[l[u]], votes) + votes, l[u]));
            }
        }
        label_row<kHugeThreads>(best, wave_best, row, lab, nxt, changed);
        __threadfence();  // (counts first, then zeros, then the next row's counts)
        __syncthreads();
        for (int64_t j0 = 0; j0 < len; j0 += U * kHugeThreads) {
            int32_t l[U];
            labels_from(j0, l);
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (l[u] >= 0) cnt[l[u]] = 0;
        }
        __threadfence();
        __syncthreads();
    }
    if (threadIdx.x == 0 && changed) atomicAdd(&tally->changed[round], changed);
}

// 1 where a label is in use (rank then holds, after an exclusive scan, the cluster's number)
__global__ __launch_bounds__(kThreads) void gp_mark_labels(const int32_t* __restrict__ even, const int32_t* __restrict__ odd, int64_t n,
                                                           const Tally* __restrict__ tally, uint32_t* __restrict__ rank)
{
    const int32_t* lab = rounds_that_count(tally->changed, kMaxRounds, n) & 1 ? odd : even;
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kThreads) rank[lab[i]] = 1;
}

// Cluster numbers in place of labels, and the clusters' sizes: a workgroup counts its rows in a table in LDS, a cluster
// that finds its place taken by another at once in memory (one atomic per wavefront and cluster queues at the counters of
// the large ones: a giant cluster of 490,000 rows 105 us, 50 clusters of 233,000 rows 381 us).
constexpr int kSizeTable = 2048;
__global__ __launch_bounds__(kThreads) void gp_number_clusters(int32_t* __restrict__ even, int32_t* __restrict__ odd, int64_t n,
                                                               const Tally* __restrict__ tally, const uint32_t* __restrict__ rank,
                                                               uint32_t* __restrict__ size)
{
    __shared__ int32_t key[kSizeTable];
    __shared__ uint32_t cnt[kSizeTable];
    int32_t* lab = rounds_that_count(tally->changed, kMaxRounds, n) & 1 ? odd : even;
    for (int j = threadIdx.x; j < kSizeTable; j += kThreads) {
        key[j] = -1;
        cnt[j] = 0;
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    for (int64_t i0 = ((int64_t)blockIdx.x * kThreads + threadIdx.x) - lane; i0 < n; i0 += (int64_t)gridDim.x * kThreads) {
        const int64_t i = i0 + lane;
        int32_t c = -1;
        if (i < n) {
            c = (int32_t)rank[lab[i]];
            lab[i] = c;
        }
        const int32_t one = __builtin_amdgcn_readfirstlane(c);  // (the first lane has a row)
        const unsigned long long same = __ballot(c == one);
        uint32_t rows = lane == 0 ? (uint32_t)__popcll(same) : 1;
        if (c < 0 || (c == one && lane != 0)) rows = 0;
        if (rows) {
            const uint32_t at = mix((uint32_t)c) % kSizeTable;
            const int32_t was = atomicCAS(&key[at], -1, c);
            if (was == -1 || was == c)
                atomicAdd(&cnt[at], rows);
            else
                atomicAdd(&size[c], rows);
        }
    }
    __syncthreads();
    for (int j = threadIdx.x; j < kSizeTable; j += kThreads)
        if (cnt[j]) atomicAdd(&size[key[j]], cnt[j]);
}

__global__ __launch_bounds__(kThreads) void gp_weigh_clusters(const int64_t* __restrict__ rowptr, const int32_t* __restrict__ col, int64_t n,
                                                              const int32_t* __restrict__ even, const int32_t* __restrict__ odd,
                                                              const uint32_t* __restrict__ size, Tally* __restrict__ tally)
{
    __shared__ unsigned long long part[2][kThreads / 64];
    const int32_t* lab = rounds_that_count(tally->changed, kMaxRounds, n) & 1 ? odd : even;
    const int lane = threadIdx.x & 63;
    const int64_t waves = (int64_t)gridDim.x * (kThreads / 64);
    unsigned long long inside = 0, weight_size = 0;
    for (int64_t tile = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6); tile * kTileRows < n; tile += waves) {
        const int64_t r0 = tile * kTileRows;
        const int rows = (int)min((int64_t)kTileRows, n - r0);
        const int64_t at = rowptr[r0 + min(lane, rows)];
        const int32_t own = lab[r0 + min(lane, rows - 1)];
        for (int r = 0; r < rows; ++r) {
            const int64_t s = __shfl(at, r, 64), e = __shfl(at, r + 1, 64);
            const int32_t mine = __shfl(own, r, 64);
            for (int64_t j = s + lane; j < e; j += 64) inside += lab[col[j]] == mine;
            if (lane == 0) weight_size += (unsigned long long)(e - s) * size[mine];
        }
    }
#pragma unroll
    for (int o = 32; o; o >>= 1) {
        inside += __shfl_xor(inside, o, 64);
        weight_size += __shfl_xor(weight_size, o, 64);
    }
    if (lane == 0) {
        part[0][threadIdx.x >> 6] = inside;
        part[1][threadIdx.x >> 6] = weight_size;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        unsigned long long sum = 0;
        for (int w = 0; w < kThreads / 64; ++w) sum += part[threadIdx.x][w];
        atomicAdd(threadIdx.x == 0 ? &tally->inside : &tally->weight_size, sum);
    }
}

__global__ __launch_bounds__(kThreads) void gp_clear_words(uint32_t* __restrict__ p, int64_t count)
{
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < count; i += (int64_t)gridDim.x * kThreads) p[i] = 0;
}

}  // namespace

bool cluster_rows_on_device(const gp_plan& P, RowClusters& C, hipStream_t stream)
{
    const int64_t n = P.n;
    if (P.nnz == 0 || !P.dev.col || P.rowptr.size() != (size_t)n + 1) return false;
    if ((double)P.nnz * (double)n >= 18e18) return false;  // (weight_size may reach their product, and holds less than 2^64)
    // one allocation: row pointers, two label lists, ranks (and the scan's words), sizes, the lists of longer rows, the tally
    const size_t words = (size_t)n, most_huge = (size_t)(P.nnz / kBigRow);
    const size_t rank_words = words + 1, scan_words = device_scan_scratch_words(n + 1);
    const size_t bytes = sizeof(Tally) + (words + 1) * sizeof(int64_t) + 4 * (2 * words + rank_words + scan_words + words + 2 * words + most_huge);
    char* base = nullptr;
    if (hipMalloc((void**)&base, bytes) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    struct Guard {
        void* p;
        ~Guard() { (void)hipFree(p); }
    } guard{base}, guard_counters{nullptr};
    int64_t* rowptr = (int64_t*)base;
    Tally* tally = (Tally*)(rowptr + words + 1);
    uint32_t* rank = (uint32_t*)(tally + 1);  // (tally, ranks and sizes lie together: cleared in one launch)
    uint32_t* size = rank + rank_words;
    uint32_t* scan = size + words;
    int32_t* even = (int32_t*)(scan + scan_words);
    int32_t* odd = even + words;
    int32_t* mid = odd + words;
    int32_t* big = mid + words;
    int32_t* huge = big + words;

    // (a setting of the current device's copy of the kernel: asked for by every call)
    if (hipFuncSetAttribute((const void*)gp_label_long_rows<1024, kBigTable>, hipFuncAttributeMaxDynamicSharedMemorySize, 2 * kBigTable * 4) !=
        hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    auto grid = [](int64_t items) { return dim3((unsigned)std::max<int64_t>(1, std::min<int64_t>((items + kThreads - 1) / kThreads, 256 * 8))); };
    const dim3 tiles = grid((n + kTileRows - 1) / kTileRows * 64);
    bool ok = hipMemcpyAsync(rowptr, P.rowptr.data(), (words + 1) * sizeof(int64_t), hipMemcpyHostToDevice, stream) == hipSuccess;
    const int64_t clear = (int64_t)(sizeof(Tally) / 4 + rank_words + words);
    hipLaunchKernelGGL(gp_clear_words, grid(clear), dim3(kThreads), 0, stream, (uint32_t*)tally, clear);
    hipLaunchKernelGGL(gp_first_labels, grid(n), dim3(kThreads), 0, stream, even, n);
    hipLaunchKernelGGL(gp_list_long_rows, dim3((unsigned)((n + kListRows - 1) / kListRows)), dim3(kThreads), 0, stream, rowptr, n, tally, mid, big, huge);
    // Huge rows, if there are any: counters for as many of them as go side by side, in up to 512 MiB or for one.
    uint32_t huge_rows = 0;
    ok = ok && hipMemcpyAsync(&huge_rows, &tally->huge_rows, sizeof(huge_rows), hipMemcpyDeviceToHost, stream) == hipSuccess;
    ok = (hipStreamSynchronize(stream) == hipSuccess) && ok;
    const int64_t side_by_side = std::min<int64_t>({(int64_t)huge_rows, 256, std::max<int64_t>(1, ((int64_t)512 << 20) / 4 / n)});
    uint32_t* counters = nullptr;
    if (!ok || (side_by_side > 0 && hipMalloc((void**)&counters, (size_t)(side_by_side * n) * 4) != hipSuccess)) {
        (void)hipGetLastError();
        return false;
    }
    guard_counters.p = counters;
    if (counters) hipLaunchKernelGGL(gp_clear_words, grid(side_by_side * n), dim3(kThreads), 0, stream, counters, side_by_side * n);
    for (int round = 0; round < kMaxRounds; ++round) {
        hipLaunchKernelGGL(gp_label_short_rows, tiles, dim3(kThreads), 0, stream, rowptr, P.dev.col, n, even, odd, round, tally);
        if (round == 0) continue;  // (that round takes rows of any length)
        hipLaunchKernelGGL((gp_label_long_rows<64, kMidTable>), dim3(256 * 16), dim3(64), 2 * kMidTable * 4, stream, rowptr, P.dev.col, n, even,
                           odd, round, tally, mid);
        hipLaunchKernelGGL((gp_label_long_rows<1024, kBigTable>), dim3(256), dim3(1024), 2 * kBigTable * 4, stream, rowptr, P.dev.col, n, even,
                           odd, round, tally, big);
        if (counters)
            hipLaunchKernelGGL(gp_label_huge_rows, dim3((unsigned)side_by_side), dim3(kHugeThreads), 0, stream, rowptr, P.dev.col, n, even, odd,
                               round, tally, huge, counters);
    }
    hipLaunchKernelGGL(gp_mark_labels, grid(n), dim3(kThreads), 0, stream, even, odd, n, tally, rank);
    ok = ok && device_exclusive_scan(rank, n + 1, scan, stream) == GP_OK;  // the last word: the number of clusters
    hipLaunchKernelGGL(gp_number_clusters, dim3((unsigned)std::min<int64_t>((n + kThreads - 1) / kThreads, 256)), dim3(kThreads), 0, stream, even, odd, n, tally, rank, size);
    hipLaunchKernelGGL(gp_weigh_clusters, dim3(std::min(tiles.x, 1024u)), dim3(kThreads), 0, stream, rowptr, P.dev.col, n, even, odd, size, tally);
    Tally t;
    uint32_t num = 0;
    C.label.resize(words);
    ok = ok && hipGetLastError() == hipSuccess && hipMemcpyAsync(&t, tally, sizeof(t), hipMemcpyDeviceToHost, stream) == hipSuccess &&
         hipMemcpyAsync(&num, rank + n, sizeof(num), hipMemcpyDeviceToHost, stream) == hipSuccess;
    ok = (hipStreamSynchronize(stream) == hipSuccess) && ok;
    if (ok) {
        const int rounds = rounds_that_count(t.changed, kMaxRounds, n);
        ok = hipMemcpyAsync(C.label.data(), rounds & 1 ? odd : even, words * sizeof(int32_t), hipMemcpyDeviceToHost, stream) == hipSuccess &&
             hipStreamSynchronize(stream) == hipSuccess;
    }
    if (!ok) {
        (void)hipGetLastError();
        return false;
    }
    C.num = (int32_t)num;
    C.inside_fraction = (double)t.inside / (double)P.nnz;
    C.typical_rows = (double)t.weight_size / (double)P.nnz;
    C.ready = true;
    return true;
}

}  // namespace gp
