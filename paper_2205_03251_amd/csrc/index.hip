// Device-side index of a population of prefix trees: the first steps of
// loading (Section 3.1 flattens each tree into one byte per node in prefix
// order).  For every tree it decides validity, and for every node of a valid
// tree it finds the end of the node's subtree and the node's parent.
//
// A node's step is +1 for a function (binary: it opens two child positions
// and fills one) and -1 for anything else.  E(k) is the sum of the steps of
// the positions before k, over the whole population.  The tree on [s, e) is
// valid iff each byte is a known function or a terminal below n_inputs,
// E(k) >= E(s) for s < k < e, and E(e) = E(s) - 1 (the count of open child
// positions never runs out early and ends exhausted).  The subtree of node k
// ends (exclusively) at the first j > k with E(j) < E(k): k + 1 for a
// terminal.  A function's first child follows it, the second starts where the
// first one's subtree ends.  The searches for the ends run per 4096-position
// block, in registers and in the block's minima in LDS; the few that leave the
// block continue in a min-tree of E (level 0 is E, each entry of level l the
// minimum of a group of kIxFan entries of level l - 1, so a search step reads
// one 64-byte group).  On request the Strahler
// number of every node follows, one level per pass over the subtree ranges,
// first within each block and then for the subtrees that leave theirs.
#include <algorithm>
#include <mutex>

#include "dev.h"

namespace gpe {

// Scratch of the allocation-free index entry point (layout in dev.h).  Host
// code never names it except to look up its device address: on each device
// the array has its own copy at its own address.
static __device__ __align__(256) int32_t scratch[kIxStaticWords];

hipError_t ix_static_scratch(int device, int32_t** out)
{
    static std::mutex mu;
    static int32_t* addr[256] = {};
    if (device < 0 || device >= 256) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(mu);
    if (!addr[device]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[device] = (int32_t*)p;
    }
    *out = addr[device];
    return hipSuccess;
}

__global__ __launch_bounds__(256) void k_fill_u8(uint8_t* dst, int64_t n, uint8_t v)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) dst[i] = v;
}

hipError_t launch_fill_u8(uint8_t* dst, int64_t n, uint8_t v, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    const int64_t grid = std::min<int64_t>(1024, (n + 255) / 256);
    hipLaunchKernelGGL(k_fill_u8, dim3((unsigned)grid), dim3(256), 0, s, dst, n, v);
    return hipGetLastError();
}

static_assert(kIxFan == 16, "a group is read as four 16-byte loads");

// Two int16 values (within +-32767) in one word, the first in the low half.
__device__ __forceinline__ int32_t ix_pack16(int32_t lo, int32_t hi)
{
    return (int32_t)(((uint32_t)lo & 0xffffu) | ((uint32_t)hi << 16));
}

__device__ __forceinline__ int32_t ix_e(const IxParams& q, int64_t k)
{
    return q.el[k] + q.boff[k / kIxBlock];
}

__device__ __forceinline__ bool ix_bad_byte(uint8_t b, int n_inputs)
{
    return (b & 0x80) ? (b & 0x7f) > 3 : (int)b >= n_inputs;
}

// Last tree t with offsets[t] <= k (offsets non-decreasing; any t in range
// otherwise).
__device__ __forceinline__ int64_t ix_tree_of(const IxParams& q, int64_t k)
{
    int64_t lo = 0, hi = q.n_trees;
    while (hi - lo > 1) {
        const int64_t mid = (lo + hi) >> 1;
        if (q.offsets[mid] <= k) lo = mid;
        else hi = mid;
    }
    return lo;
}

// The last tree t in [lo, hi] with offsets[t] <= k, or lo.
__device__ __forceinline__ int64_t ix_tree_in(const IxParams& q, int64_t lo, int64_t hi, int64_t k)
{
    ++hi;
    while (hi - lo > 1) {
        const int64_t mid = (lo + hi) >> 1;
        if (q.offsets[mid] <= k) lo = mid;
        else hi = mid;
    }
    return lo;
}

// Group g of min-tree level l (the kIxFan entries from g, g a multiple of
// kIxFan), read with four 16-byte loads (two for el); levels and el are
// padded to whole groups.  Entries past the level's length hold whatever the padding holds.
__device__ __forceinline__ void ix_load_group(const IxParams& q, int l, int64_t g, int32_t (&x)[kIxFan])
{
    if (l == 0) {
        // 16 int16 entries, two 16-byte loads
        const int4* src = (const int4*)(q.el + g);
        const int32_t add = q.boff[g / kIxBlock];   // a group never straddles a scan block
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int4 w = src[i];
            const int32_t u[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                x[8 * i + 2 * h] = (int32_t)(int16_t)(u[h] & 0xffff) + add;
                x[8 * i + 2 * h + 1] = (u[h] >> 16) + add;
            }
        }
        return;
    }
    const int4* src = (const int4*)(q.seg + q.lvl[2 * l] + g);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int4 w = src[i];
        x[4 * i] = w.x;
        x[4 * i + 1] = w.y;
        x[4 * i + 2] = w.z;
        x[4 * i + 3] = w.w;
    }
}

// The first index in [p, end of p's group) of level l whose value is below
// v, or -1.
__device__ __forceinline__ int64_t ix_scan_in(const int32_t (&x)[kIxFan], int64_t g, int64_t p, int64_t len,
                                             int32_t v)
{
    int64_t hit = -1;
#pragma unroll
    for (int i = kIxFan - 1; i >= 0; --i) {
        const int64_t idx = g + i;
        if (idx >= p && idx < len && x[i] < v) hit = idx;
    }
    return hit;
}

__device__ __forceinline__ int64_t ix_scan_group(const IxParams& q, int l, int64_t p, int32_t v)
{
    const int64_t g = p & ~(int64_t)(kIxFan - 1);
    int32_t x[kIxFan];
    ix_load_group(q, l, g, x);
    return ix_scan_in(x, g, p, q.lvl[2 * l + 1], v);
}

// First position at or after entry p of level l whose E is below v, or -1
// (p times kIxFan^l is the first position searched).  Going up, every
// position from there to the end of the current node's parent has been
// checked when a group scan fails, so the search continues at the parent's
// next sibling; going down, it takes the first child whose minimum is below v.
__device__ __forceinline__ int64_t ix_first_below_at(const IxParams& q, int l, int64_t p, int32_t v)
{
    int64_t hit = -1;
    for (;;) {
        if (p >= q.lvl[2 * l + 1]) return -1;
        hit = ix_scan_group(q, l, p, v);
        if (hit >= 0) break;
        if (l == q.top) return -1;
        p = p / kIxFan + 1;
        ++l;
    }
    while (l > 0 && hit >= 0) {
        --l;
        hit = ix_scan_group(q, l, hit * kIxFan, v);
    }
    return hit;
}

// Steps of one 4096-position block: el = exclusive prefix within the block,
// bsum = the block's total.  Positions past n step by 0.
__global__ __launch_bounds__(256) void k_ix_scan(IxParams q, int32_t* bsum)
{
    __shared__ int32_t wtot[4];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int64_t base = (int64_t)blockIdx.x * kIxBlock + (int64_t)tid * 16;
    uint32_t word[4] = {0, 0, 0, 0};
    if (base + 16 <= q.n) {
        const uint4 v = *(const uint4*)(q.ops + base);
        word[0] = v.x;
        word[1] = v.y;
        word[2] = v.z;
        word[3] = v.w;
    } else {
        for (int j = 0; j < 16; ++j)
            if (base + j < q.n) word[j >> 2] |= (uint32_t)q.ops[base + j] << (8 * (j & 3));
    }
    int32_t pre[16];
    int32_t run = 0;
    for (int j = 0; j < 16; ++j) {
        pre[j] = run;
        const uint32_t b = (word[j >> 2] >> (8 * (j & 3))) & 0xffu;
        run += base + j < q.n ? ((b & 0x80u) ? 1 : -1) : 0;
    }
    int32_t incl = run;
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
    }
    if (lane == 63) wtot[w] = incl;
    __syncthreads();
    int32_t wbase = 0;
    for (int i = 0; i < w; ++i) wbase += wtot[i];
    const int32_t excl = wbase + incl - run;
    int4* dst = (int4*)(q.el + base);
    for (int j = 0; j < 2; ++j)
        dst[j] = make_int4(ix_pack16(excl + pre[8 * j], excl + pre[8 * j + 1]),
                           ix_pack16(excl + pre[8 * j + 2], excl + pre[8 * j + 3]),
                           ix_pack16(excl + pre[8 * j + 4], excl + pre[8 * j + 5]),
                           ix_pack16(excl + pre[8 * j + 6], excl + pre[8 * j + 7]));
    if (tid == 255) bsum[blockIdx.x] = excl + run;
}

// Exclusive prefix of the block totals bsum[0 .. nb) into boff, boff[nb] =
// their sum (E(n) after the position scan), and el[nb * kIxBlock] = 0 so that
// E(n) = el[n] + boff[n / kIxBlock] also when n is a multiple of the block.
// One launch for a single group of kIxBlock totals, three for more: the prefix
// within each group (a workgroup per group, 16 a thread), whose sum then
// replaces the group's first total (read by then); the group sums scanned in
// place by one workgroup; each group's offset added.  bsum is left clobbered.
__global__ __launch_bounds__(256) void k_ix_top_local(IxParams q, int32_t* bsum, int64_t nb)
{
    __shared__ int32_t wtot[4];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int64_t g0 = (int64_t)blockIdx.x * kIxBlock, i0 = g0 + (int64_t)tid * 16;
    int32_t pre[16];
    int32_t run = 0;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        pre[j] = run;
        run += i0 + j < nb ? bsum[i0 + j] : 0;
    }
    int32_t incl = run;
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
    }
    if (lane == 63) wtot[w] = incl;
    __syncthreads();
    int32_t wbase = 0;
    for (int i = 0; i < w; ++i) wbase += wtot[i];
    const int32_t excl = wbase + incl - run;
#pragma unroll
    for (int j = 0; j < 16; ++j)
        if (i0 + j < nb) q.boff[i0 + j] = excl + pre[j];
    if (gridDim.x == 1) {
        if (tid == 255) {
            q.boff[nb] = excl + run;
            q.el[nb * kIxBlock] = 0;
        }
        return;
    }
    __syncthreads();                          // every total of the group read
    if (tid == 255) bsum[g0] = excl + run;
}

constexpr int kIxTopGroups = 256;         // groups of kIxBlock totals one workgroup scans

__global__ __launch_bounds__(kIxTopGroups) void k_ix_top_groups(IxParams q, int32_t* bsum, int64_t nb)
{
    __shared__ int32_t wtot[kIxTopGroups / 64];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int64_t ng = (nb + kIxBlock - 1) / kIxBlock;
    const int32_t v = tid < ng ? bsum[(int64_t)tid * kIxBlock] : 0;
    int32_t incl = v;
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
    }
    if (lane == 63) wtot[w] = incl;
    __syncthreads();
    int32_t wbase = 0;
    for (int i = 0; i < w; ++i) wbase += wtot[i];
    if (tid < ng) bsum[(int64_t)tid * kIxBlock] = wbase + incl - v;
    if (tid == kIxTopGroups - 1) {
        q.boff[nb] = wbase + incl;
        q.el[nb * kIxBlock] = 0;
    }
}

__global__ __launch_bounds__(256) void k_ix_top_add(IxParams q, const int32_t* bsum, int64_t nb)
{
    for (int64_t i = kIxBlock + (int64_t)blockIdx.x * 256 + threadIdx.x; i < nb; i += (int64_t)gridDim.x * 256)
        q.boff[i] += bsum[i / kIxBlock * kIxBlock];
}

static hipError_t launch_top(const IxParams& q, int32_t* bsum, int64_t nb, hipStream_t s)
{
    const int64_t ng = (nb + kIxBlock - 1) / kIxBlock;
    if (ng > kIxTopGroups) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_ix_top_local, dim3((unsigned)ng), dim3(256), 0, s, q, bsum, nb);
    if (ng > 1) {
        hipLaunchKernelGGL(k_ix_top_groups, dim3(1), dim3(kIxTopGroups), 0, s, q, bsum, nb);
        const int64_t grid = std::min<int64_t>(65536, (nb - kIxBlock + 255) / 256);
        hipLaunchKernelGGL(k_ix_top_add, dim3((unsigned)grid), dim3(256), 0, s, q, (const int32_t*)bsum, nb);
    }
    return hipGetLastError();
}

// Level l >= 1 of the min-tree: the minimum of each group of level l - 1.
__global__ __launch_bounds__(256) void k_ix_level(IxParams q, int l)
{
    const int64_t len = q.lvl[2 * l + 1], src_len = q.lvl[2 * (l - 1) + 1];
    for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p < len; p += (int64_t)gridDim.x * 256) {
        const int64_t g = p * kIxFan;
        int32_t x[kIxFan];
        ix_load_group(q, l - 1, g, x);
        int32_t m = INT32_MAX;
        for (int i = 0; i < kIxFan; ++i)
            if (g + i < src_len) m = min(m, x[i]);
        q.seg[q.lvl[2 * l] + p] = m;
    }
}

// valid[t] = 1 for a tree whose offsets are in order and inside [0, n];
// flags offsets that do not run from 0 to n without decreasing.
__global__ __launch_bounds__(256) void k_ix_init(IxParams q)
{
    for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < q.n_trees; t += (int64_t)gridDim.x * 256) {
        const int64_t s = q.offsets[t], e = q.offsets[t + 1];
        const bool inside = 0 <= s && s < e && e <= q.n;
        q.valid[t] = inside ? 1 : 0;
        if (e < s || (t == 0 && s != 0) || (t == q.n_trees - 1 && e != q.n)) *q.bad_offsets = 1;
    }
}

// The 16 bytes at p + k0 (zero past n), four to a word.
__device__ __forceinline__ void ix_bytes16(const uint8_t* p, int64_t k0, int64_t n, uint32_t (&w)[4])
{
    if (k0 + 16 <= n && (((uintptr_t)(p + k0)) & 15) == 0) {
        const uint4 v = *(const uint4*)(p + k0);
        w[0] = v.x;
        w[1] = v.y;
        w[2] = v.z;
        w[3] = v.w;
    } else {
        w[0] = w[1] = w[2] = w[3] = 0;
        for (int j = 0; j < 16; ++j)
            if (k0 + j < n) w[j >> 2] |= (uint32_t)p[k0 + j] << (8 * (j & 3));
    }
}

// Validity, in two parts.  Every byte a known opcode: one pass over the
// bytes, which looks a tree up only for a bad byte.  The count of open child
// positions never running out before the end and running out there: with
// steps of +-1, the first j > s with E(j) < E(s) is e, one search per tree.
__global__ __launch_bounds__(256) void k_ix_bytes(IxParams q, const int32_t* tfirst)
{
    const int64_t k0 = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 16;
    if (k0 >= q.n) return;
    uint32_t w[4];
    ix_bytes16(q.ops, k0, q.n, w);
    uint32_t bad = 0;
#pragma unroll
    for (int j = 0; j < 16; ++j)
        if (k0 + j < q.n && ix_bad_byte((uint8_t)(w[j >> 2] >> (8 * (j & 3))), q.n_inputs)) bad |= 1u << j;
    if (!bad) return;
    const int64_t b = k0 / kIxBlock, nb = (q.n + kIxBlock - 1) / kIxBlock;
    int64_t t = ix_tree_in(q, tfirst[b], b + 1 < nb ? tfirst[b + 1] : q.n_trees - 1, k0);
    int64_t s = q.offsets[t], e = q.offsets[t + 1];
    while (bad) {
        const int64_t k = k0 + (__ffs(bad) - 1);
        bad &= bad - 1;
        while (k >= e && t + 1 < q.n_trees) {
            ++t;
            s = q.offsets[t];
            e = q.offsets[t + 1];
        }
        if (0 <= s && s <= k && k < e) q.valid[t] = 0;
    }
}

__global__ __launch_bounds__(256) void k_ix_trees(IxParams q)
{
    for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < q.n_trees; t += (int64_t)gridDim.x * 256) {
        const int64_t s = q.offsets[t], e = q.offsets[t + 1];
        if (!(0 <= s && s < e && e <= q.n)) continue;           // refused by k_ix_init
        if (ix_first_below_at(q, 0, s + 1, ix_e(q, s)) != e) q.valid[t] = 0;
    }
}

// Within one block: E of its positions less the block's offset (the scan's
// el, which stays within +-kIxBlock), the minimum of each group of kIxFan
// (one thread's positions) and of each kIxFan of those.
struct alignas(16) IxBlockMins {
    int16_t e0[kIxBlock];
    int16_t m1[kIxBlock / kIxFan];
    int16_t m2[kIxBlock / kIxFan / kIxFan];
};
static_assert(kIxBlock == kIxFan * kIxFan * kIxFan, "a block is three min-tree levels");

// The kIxFan entries of a block level from g (a multiple of kIxFan), with
// two 16-byte LDS reads.
__device__ __forceinline__ void ix_lds_group(const int16_t* a, int g, int32_t (&x)[kIxFan])
{
    const int4* p = (const int4*)(a + g);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int4 w = p[i];
        const int32_t u[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            x[8 * i + 2 * h] = (int32_t)(int16_t)(u[h] & 0xffff);
            x[8 * i + 2 * h + 1] = u[h] >> 16;
        }
    }
}

// First index in [g + from, g + kIxFan) whose entry is below v, or -1.
__device__ __forceinline__ int ix_first_lt(const int32_t (&x)[kIxFan], int g, int from, int32_t v)
{
    int hit = kIxFan;
#pragma unroll
    for (int i = kIxFan - 1; i >= 0; --i)
        if (i >= from && x[i] < v) hit = i;
    return hit < kIxFan ? g + hit : -1;
}

// First block position whose E is below v after the group of position i
// (that group already searched), or -1.
__device__ __forceinline__ int ix_lds_first_below(const IxBlockMins& b, int i, int32_t v)
{
    int32_t x[kIxFan];
    const int g1 = i / kIxFan;
    ix_lds_group(b.m1, g1 & ~(kIxFan - 1), x);
    int h1 = ix_first_lt(x, g1 & ~(kIxFan - 1), (g1 & (kIxFan - 1)) + 1, v);
    if (h1 < 0) {
        ix_lds_group(b.m2, 0, x);
        const int h2 = ix_first_lt(x, 0, g1 / kIxFan + 1, v);
        if (h2 < 0) return -1;
        ix_lds_group(b.m1, kIxFan * h2, x);
        h1 = ix_first_lt(x, kIxFan * h2, 0, v);
        if (h1 < 0) return -1;
    }
    ix_lds_group(b.e0, kIxFan * h1, x);
    return ix_first_lt(x, kIxFan * h1, 0, v);
}

// tfirst[b] = the tree holding the first position of scan block b (bsum,
// free once the block offsets are summed, holds them).
__global__ __launch_bounds__(256) void k_ix_tfirst(IxParams q, int32_t* tfirst, int64_t nb)
{
    for (int64_t b = (int64_t)blockIdx.x * 256 + threadIdx.x; b < nb; b += (int64_t)gridDim.x * 256)
        tfirst[b] = (int32_t)ix_tree_of(q, b * kIxBlock);
}

constexpr int kIxQueue = 1024;            // block-leaving searches shared out per workgroup

// The end of position k of tree [s, e), whose E is v, when the search left
// the block: continued in the global min-tree from the level whose entries
// are whole blocks (or the top).
__device__ __forceinline__ int32_t ix_global_end(const IxParams& q, int64_t B, int64_t k, int64_t s, int64_t e,
                                                 int32_t v)
{
    const int L = q.top < 3 ? q.top : 3;
    const int64_t J = ix_first_below_at(q, L, (B + kIxBlock) >> (4 * L), v);
    return J > k && J <= e ? (int32_t)(J - s) : -1;
}

// Results of a block in LDS: a word in 16 left out, so that threads that
// write 16 positions each and threads that read consecutive ones both spread
// over the banks.
__device__ __forceinline__ int ix_slot(int i) { return i + (i >> 4); }

// Subtree end and parent of every position, one scan block per workgroup.
// The end of function k is the first j > k with E(j) < E(k).  Each thread
// settles what its own positions answer (in registers); the searches that go
// past them are listed and shared out over the workgroup, which runs them in
// the block's minima in LDS with every lane busy (run where they arise, a wave
// would step through every search any of its lanes needs); those that leave
// the block (for a random walk about the square root of the block's length)
// are queued and continued in the global min-tree, and a search that finds
// the queue full continues at once.
//
// Parents need no search.  A position after a function is its first child,
// and the position where that child's subtree ends is the second: the thread
// that holds a first child hands the parent on, through LDS, or in memory
// where the second child lies in a later block (whose own workgroup leaves
// the position out).  Results are gathered in LDS and written out in whole
// lines: written per position, a wave's stores spread over 64 lines and reach
// memory one partial line at a time.
//
// Bound by the searches' chains of LDS reads and by 9 bytes a node of memory.
// 1000 trees of 10000 to 1000000 nodes (215 million), the whole index: 2.19 ms
// with parents searched like the ends, 1.71 handed on; 10 million nodes 637 -> 608
// us with Strahler numbers.  36 KiB of LDS: four workgroups on a compute unit.
__global__ __launch_bounds__(256) void k_ix_links(IxParams q, const int32_t* tfirst)
{
    __shared__ IxBlockMins bm;
    __shared__ uint16_t work[kIxBlock];       // block positions searched in the block minima
    __shared__ uint16_t queue[kIxQueue];      // block positions searched in the global min-tree
    __shared__ int32_t res[kIxBlock + kIxBlock / 16];         // ends, then parents, tree-local (ix_slot)
    __shared__ int32_t n_work, queued;
    const int tid = threadIdx.x, p0 = tid * kIxFan;
    const int64_t B = (int64_t)blockIdx.x * kIxBlock, k0 = B + p0;
    const int64_t nb = (q.n + kIxBlock - 1) / kIxBlock;
    const int64_t t_lo = tfirst[blockIdx.x], t_hi = blockIdx.x + 1 < nb ? tfirst[blockIdx.x + 1] : q.n_trees - 1;
    const int here = (int)min<int64_t>(kIxBlock, q.n - B);
    uint32_t w[4];
    ix_bytes16(q.ops, k0, q.n, w);
    if (tid == 0) n_work = queued = 0;
    uint64_t nxt = 0;
    uint32_t fns = 0;                         // functions
    {
        int32_t ev[kIxFan];
        int32_t run = q.el[k0];               // as the scan: positions past n step by 0
#pragma unroll
        for (int j = 0; j < kIxFan; ++j) {
            ev[j] = run;
            const uint32_t f = (w[j >> 2] >> (8 * (j & 3) + 7)) & 1u;
            fns |= f << j;
            run += k0 + j < q.n ? (f ? 1 : -1) : 0;
        }
        int32_t mn = ev[0];
#pragma unroll
        for (int j = 1; j < kIxFan; ++j) mn = min(mn, ev[j]);
#pragma unroll
        for (int j = 0; j < kIxFan; j += 8)
            *(int4*)&bm.e0[p0 + j] =
                make_int4((ev[j] & 0xffff) | (ev[j + 1] << 16), (ev[j + 2] & 0xffff) | (ev[j + 3] << 16),
                          (ev[j + 4] & 0xffff) | (ev[j + 5] << 16), (ev[j + 6] & 0xffff) | (ev[j + 7] << 16));
        bm.m1[tid] = (int16_t)mn;
        // the search within the thread's own positions, four bits per
        // position: the distance less one, 15 when the answer lies outside
#pragma unroll
        for (int j = 0; j < kIxFan; ++j) {
            uint32_t f = 15;
#pragma unroll
            for (int m = kIxFan - 1; m > j; --m)
                if (ev[m] < ev[j]) f = (uint32_t)(m - j - 1);
            nxt |= (uint64_t)f << (4 * j);
        }
    }
    __syncthreads();
    if (tid < kIxFan) {
        int32_t x = bm.m1[tid * kIxFan];
        for (int i = 1; i < kIxFan; ++i) x = min(x, (int32_t)bm.m1[tid * kIxFan + i]);
        bm.m2[tid] = (int16_t)x;
    }
    const int32_t boff = q.boff[blockIdx.x];
    int64_t t0 = 0, s0 = 0, e0 = 0;           // the tree of the thread's first position
    bool one_tree = false;                    // the common case: all 16 positions in one valid tree
    if (k0 < q.n) {
        t0 = ix_tree_in(q, t_lo, t_hi, k0);
        s0 = q.offsets[t0];
        e0 = q.offsets[t0 + 1];
        one_tree = q.valid[t0] != 0 && 0 <= s0 && s0 <= k0 && k0 + kIxFan <= e0 && e0 <= q.n;
    }
    // the other threads' positions, one at a time: body(j, k, in a valid tree, its start and end)
    const auto each = [&](auto body) {
        int64_t t = t0, s = s0, e = e0;
        bool ok = q.valid[t] != 0;
#pragma unroll 1
        for (int j = 0; j < kIxFan; ++j) {
            const int64_t k = k0 + j;
            if (k >= q.n) break;
            while (k >= e && t + 1 < q.n_trees) {
                ++t;
                s = q.offsets[t];
                e = q.offsets[t + 1];
                ok = q.valid[t] != 0;
            }
            body(j, k, ok && 0 <= s && s <= k && k < e && e <= q.n, s, e);
        }
    };
    const auto fn_at = [&](int j) -> bool { return ((fns >> j) & 1u) != 0; };
    if (one_tree) {
        const int32_t base = (int32_t)(k0 - s0);
#pragma unroll
        for (int j = 0; j < kIxFan; ++j) {
            const uint32_t d = (uint32_t)(nxt >> (4 * j)) & 15u;
            int32_t r = base + j + 1;
            if (fn_at(j)) {
                r += (int32_t)d;
                if (d == 15) work[atomicAdd(&n_work, 1)] = (uint16_t)(p0 + j);      // overwrites it
            }
            res[ix_slot(p0 + j)] = r;
        }
    } else if (k0 < q.n) {
        each([&](int j, int64_t k, bool in, int64_t s, int64_t) {
            int32_t r = -1;
            if (in) {
                const uint32_t d = (uint32_t)(nxt >> (4 * j)) & 15u;
                r = (int32_t)(k + 1 - s);
                if (fn_at(j)) {
                    r += (int32_t)d;
                    if (d == 15) work[atomicAdd(&n_work, 1)] = (uint16_t)(p0 + j);
                }
            }
            res[ix_slot(p0 + j)] = r;
        });
    }
    __syncthreads();
    const int nw = n_work;
    for (int x = tid; x < nw; x += 256) {
        const int i = work[x];
        const int64_t k = B + i;
        const int32_t v = bm.e0[i];
        const int m = ix_lds_first_below(bm, i, v);
        const int64_t t = ix_tree_in(q, t_lo, t_hi, k);
        const int64_t s = q.offsets[t], e = q.offsets[t + 1];
        if (m >= 0) {
            res[ix_slot(i)] = B + m <= e ? (int32_t)(B + m - s) : -1;
        } else {
            const int slot = atomicAdd(&queued, 1);
            if (slot < kIxQueue) queue[slot] = (uint16_t)i;
            else res[ix_slot(i)] = ix_global_end(q, B, k, s, e, v + boff);
        }
    }
    __syncthreads();
    const int nq = min(queued, kIxQueue);
    for (int x = tid; x < nq; x += 256) {
        const int i = queue[x];
        const int64_t t = ix_tree_in(q, t_lo, t_hi, B + i);
        res[ix_slot(i)] = ix_global_end(q, B, B + i, q.offsets[t], q.offsets[t + 1], bm.e0[i] + boff);
    }
    __syncthreads();
    for (int x = tid; x < here; x += 256) q.end[B + x] = res[ix_slot(x)];
    int32_t en[kIxFan];
#pragma unroll
    for (int j = 0; j < kIxFan; ++j) en[j] = one_tree ? res[ix_slot(p0 + j)] : 0;
    __syncthreads();                          // the ends read; q.end written
    // First children, from the byte before; -2 where another thread hands the
    // parent on.
    const bool fn_before = k0 > 0 && k0 < q.n && (q.ops[k0 - 1] & 0x80) != 0;
    if (one_tree) {
        const int32_t base = (int32_t)(k0 - s0);
#pragma unroll
        for (int j = 0; j < kIxFan; ++j) {
            const bool first = j > 0 ? fn_at(j - 1) : fn_before && base > 0;
            res[ix_slot(p0 + j)] = first ? base + j - 1 : base + j > 0 ? -2 : -1;
        }
    } else if (k0 < q.n) {
        each([&](int j, int64_t k, bool in, int64_t s, int64_t) {
            const bool first = in && k > s && (j > 0 ? fn_at(j - 1) : fn_before);
            res[ix_slot(p0 + j)] = first ? (int32_t)(k - 1 - s) : in && k > s ? -2 : -1;
        });
    }
    __syncthreads();
    // position k of [s, e), a first child whose subtree ends at r
    const auto hand_on = [&](int64_t k, int64_t s, int64_t e, int64_t r) {
        if (r <= k || r >= e) return;
        if (r < B + kIxBlock) res[ix_slot((int)(r - B))] = (int32_t)(k - 1 - s);
        else q.parent[r] = (int32_t)(k - 1 - s);
    };
    if (one_tree) {
#pragma unroll
        for (int j = 0; j < kIxFan; ++j)
            if (j > 0 ? fn_at(j - 1) : fn_before && k0 > s0) hand_on(k0 + j, s0, e0, s0 + en[j]);
    } else if (k0 < q.n) {
        each([&](int j, int64_t k, bool in, int64_t s, int64_t e) {
            if (in && k > s && (j > 0 ? fn_at(j - 1) : fn_before)) hand_on(k, s, e, s + q.end[k]);
        });
    }
    __syncthreads();
    for (int x = tid; x < here; x += 256) {
        const int32_t r = res[ix_slot(x)];
        if (r != -2) q.parent[B + x] = r;
    }
}

// Trees [lo, hi] that scan block b may hold, for the Strahler passes: the
// per-block first trees are copied into the global min-tree's storage, free
// once ends and parents are written (with no min-tree levels the population
// has at most kIxFan positions, one block).
__device__ __forceinline__ void ix_block_trees(const IxParams& q, int64_t b, int64_t& lo, int64_t& hi)
{
    const int64_t nb = (q.n + kIxBlock - 1) / kIxBlock;
    if (q.top == 0) {
        lo = 0;
        hi = q.n_trees - 1;
        return;
    }
    lo = q.seg[b];
    hi = b + 1 < nb ? q.seg[b + 1] : q.n_trees - 1;
}

// Strahler numbers, one level per pass.  A node's number is at least k + 1
// iff its subtree holds a function whose two children both have at least k
// (numbers never decrease towards the root, and a node whose children differ
// takes the larger).  Pass k marks those functions, counts them with a prefix
// sum over positions, and raises every function whose subtree range holds one.
//
// k_ix_sblock runs the passes of one block of positions in LDS, all levels in
// one launch.  That settles every node whose subtree ends inside the block;
// the open ones (about 2 in a hundred of a random tree's functions) hold the
// largest number among their descendants in the block.  k_ix_sopen adds the
// descendants in the block where the subtree ends, and the passes over the
// whole population (k_ix_sflag, k_ix_supd) are left with the open nodes and
// with a count of one, in front of a whole block's, for a block that holds a
// number above the pass's level.  At 200 trees of 1000 to 300000 nodes (10
// million) a pass over all nodes took 30 to 95 us, the reading of all numbers
// and the prefix of marks being most of it, and 40 more for the host's look at
// its count; now k_ix_sblock takes 62 us, k_ix_sopen 21 and a pass 20 to 25, all
// latency.  The whole index with numbers: 958 -> 635 us.

// The open nodes (a bit for each position of a group of 16), the largest
// number in a block before each of its groups and in each block: after the
// blocks' first trees in the min-tree's storage, which has a word for each
// group (n > kIxBlock).
struct IxOpen {
    uint16_t* open;
    uint8_t* before;
    uint8_t* bmax;
};

__device__ __forceinline__ IxOpen ix_open(const IxParams& q)
{
    const int64_t nb = (q.n + kIxBlock - 1) / kIxBlock, ng = (q.n + 15) / 16;
    IxOpen o;
    o.open = (uint16_t*)(q.seg + nb);
    o.before = (uint8_t*)(o.open + ng);
    o.bmax = o.before + ng;
    return o;
}

// The larger of each byte pair (values below 128).
__device__ __forceinline__ uint32_t ix_max8(uint32_t a, uint32_t b)
{
    const uint32_t ge = ((a | 0x80808080u) - b) & 0x80808080u;
    const uint32_t m = ge - (ge >> 7);
    return (a & m) | (b & ~m);
}

__device__ __forceinline__ uint32_t ix_max_of(uint32_t a)
{
    a = ix_max8(a, a >> 16);
    return ix_max8(a, a >> 8) & 0xffu;
}

// end[k0 .. k0 + 16), with four 16-byte loads where aligned (k0 + 16 <= n).
__device__ __forceinline__ void ix_ends16(const IxParams& q, int64_t k0, int32_t (&en)[kIxFan])
{
    if ((((uintptr_t)(q.end + k0)) & 15) == 0) {
        const int4* p = (const int4*)(q.end + k0);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int4 v = p[i];
            en[4 * i] = v.x;
            en[4 * i + 1] = v.y;
            en[4 * i + 2] = v.z;
            en[4 * i + 3] = v.w;
        }
    } else {
#pragma unroll
        for (int i = 0; i < kIxFan; ++i) en[i] = q.end[k0 + i];
    }
}

// For each set bit j of m, body(k0 + j, tree start, tree end), walking the
// trees from tree t = [s, e), the one holding k0.
template <class Body>
__device__ __forceinline__ void ix_each_from(const IxParams& q, int64_t k0, uint32_t m, int64_t t, int64_t s, int64_t e,
                                             Body body)
{
    while (m) {
        const int j = __ffs(m) - 1;
        m &= m - 1;
        const int64_t k = k0 + j;
        while (k >= e && t + 1 < q.n_trees) {
            ++t;
            s = q.offsets[t];
            e = q.offsets[t + 1];
        }
        if (0 <= s && s <= k && k < e && e <= q.n) body(k, s, e);
    }
}

// The passes of one block in LDS.  Bound by the chain of a tree's lookup, the
// loads and four barriers a level, not by its 6 bytes a node (0.8 TB/s):
// eight blocks of 256 threads on a compute unit hide part of it, so the dense
// level 2 stands apart (inside the loop its unpacked ends are kept for all
// levels: 123 registers against 50, half the blocks, 78 us against 62).
__global__ __launch_bounds__(256) void k_ix_sblock(IxParams q)
{
    __shared__ uint4 s_num[kIxBlock / 16];       // the numbers, a byte each
    __shared__ uint4 s_endv[kIxBlock / 8];       // subtree ends in the block, 16 bits each (kIxBlock: there or beyond)
    __shared__ int32_t s_pre[257];               // marked before a group of 16
    __shared__ uint32_t s_bits[257];             // marked in it
    __shared__ int32_t wtot[4];
    uint8_t* num = (uint8_t*)s_num;
    uint16_t* ends = (uint16_t*)s_endv;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, p0 = tid * 16;
    const int64_t B = (int64_t)blockIdx.x * kIxBlock, k0 = B + p0;
    uint32_t sn[4] = {0u, 0u, 0u, 0u}, xs[8];
    uint32_t at = 0, open = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) xs[j] = (uint32_t)(p0 + 2 * j + 1) | ((uint32_t)(p0 + 2 * j + 2) << 16);
    if (k0 < q.n) {
        int64_t lo, hi;
        ix_block_trees(q, blockIdx.x, lo, hi);
        int64_t t = ix_tree_in(q, lo, hi, k0);
        int64_t s = q.offsets[t], e = q.offsets[t + 1];
        bool ok = q.valid[t] != 0;
        if (0 <= s && s <= k0 && k0 + kIxFan <= e && e <= q.n) {         // all 16 in one tree
            if (ok) {
                uint32_t ops[4];
                ix_bytes16(q.ops, k0, q.n, ops);
                const int32_t sb = (int32_t)max<int64_t>(s - B, -INT32_MAX), eb = (int32_t)min<int64_t>(e - B, INT32_MAX);
                int32_t en[kIxFan];
                ix_ends16(q, k0, en);
#pragma unroll
                for (int j = 0; j < kIxFan; ++j) {
                    const int32_t x = sb + min(en[j], INT32_MAX - kIxBlock);
                    if (x > p0 + j && x <= eb) {
                        const uint32_t f = (ops[j >> 2] >> (8 * (j & 3) + 7)) & 1u;
                        sn[j >> 2] |= (f + 1u) << (8 * (j & 3));         // a function is at least 2
                        at |= f << j;
                        if (x > kIxBlock) open |= 1u << j;
                        const uint32_t xl = (uint32_t)min(x, kIxBlock);
                        xs[j >> 1] = (j & 1) ? (xs[j >> 1] & 0xffffu) | (xl << 16) : (xs[j >> 1] & 0xffff0000u) | xl;
                    }
                }
            }
        } else {
            // through LDS, one position at a time
            s_num[tid] = make_uint4(0u, 0u, 0u, 0u);
            s_endv[2 * tid] = make_uint4(xs[0], xs[1], xs[2], xs[3]);
            s_endv[2 * tid + 1] = make_uint4(xs[4], xs[5], xs[6], xs[7]);
#pragma unroll 1
            for (int j = 0; j < kIxFan && k0 + j < q.n; ++j) {
                const int64_t k = k0 + j;
                while (k >= e && t + 1 < q.n_trees) {
                    ++t;
                    s = q.offsets[t];
                    e = q.offsets[t + 1];
                    ok = q.valid[t] != 0;
                }
                if (ok && 0 <= s && s <= k && k < e && e <= q.n) {
                    const int64_t x = s - B + q.end[k];
                    if (x > p0 + j && x <= e - B) {
                        const uint32_t f = q.ops[k] >> 7;
                        num[p0 + j] = (uint8_t)(f + 1u);
                        ends[p0 + j] = (uint16_t)min<int64_t>(x, kIxBlock);
                        at |= f << j;
                        if (x > kIxBlock) open |= 1u << j;
                    }
                }
            }
            const uint4 v = s_num[tid], x0 = s_endv[2 * tid], x1 = s_endv[2 * tid + 1];
            sn[0] = v.x, sn[1] = v.y, sn[2] = v.z, sn[3] = v.w;
            xs[0] = x0.x, xs[1] = x0.y, xs[2] = x0.z, xs[3] = x0.w;
            xs[4] = x1.x, xs[5] = x1.y, xs[6] = x1.z, xs[7] = x1.w;
        }
    }
    s_num[tid] = make_uint4(sn[0], sn[1], sn[2], sn[3]);
    s_endv[2 * tid] = make_uint4(xs[0], xs[1], xs[2], xs[3]);
    s_endv[2 * tid + 1] = make_uint4(xs[4], xs[5], xs[6], xs[7]);
    if (tid == 0) s_bits[256] = 0;
    __syncthreads();
    // `at`: this thread's functions at the level, the only ones that can be marked or raised
    uint32_t bits = 0;
    int32_t excl = 0;                                                    // marked in the block before p0
    // the prefix of the marks; false when the block has none
    const auto count = [&]() -> bool {
        if (!__syncthreads_or(bits != 0)) return false;
        const int32_t run = __popc(bits);
        int32_t incl = run;
        for (int o = 1; o < 64; o <<= 1) {
            const int32_t y = __shfl_up(incl, o, 64);
            if (lane >= o) incl += y;
        }
        if (lane == 63) wtot[w] = incl;
        __syncthreads();
        excl = incl - run;
        for (int i = 0; i < w; ++i) excl += wtot[i];
        s_pre[tid] = excl;
        s_bits[tid] = bits;
        if (tid == 255) s_pre[256] = excl + run;
        __syncthreads();
        return true;
    };
    // marks in [p0 + j, x)
    const auto marked = [&](int j, uint32_t x) -> bool {
        return s_pre[x >> 4] + __popc(s_bits[x >> 4] & ((1u << (x & 15)) - 1u)) > excl + __popc(bits & ((1u << j) - 1u));
    };
    const auto raise = [&](uint32_t raised) {
        if (raised) {
#pragma unroll
            for (int j = 0; j < kIxFan; ++j) sn[j >> 2] += ((raised >> j) & 1u) << (8 * (j & 3));
            s_num[tid] = make_uint4(sn[0], sn[1], sn[2], sn[3]);
        }
        at = raised;
        __syncthreads();
    };
    // level 2, where every function is: all 16 positions at once
    {
        const uint32_t x16 = tid < 255 ? ends[p0 + 16] : (uint32_t)kIxBlock, n16 = tid < 255 ? num[p0 + 16] : 0u;
        uint32_t nr[kIxFan];                                             // the right children's numbers
#pragma unroll
        for (int j = 0; j < kIxFan; ++j) {
            const uint32_t r = j + 1 < kIxFan ? (xs[(j + 1) >> 1] >> (16 * ((j + 1) & 1))) & 0xffffu : x16;
            nr[j] = r < kIxBlock ? num[r] : 0u;
        }
#pragma unroll
        for (int j = 0; j < kIxFan; ++j) {
            const uint32_t nl = j + 1 < kIxFan ? (sn[(j + 1) >> 2] >> (8 * ((j + 1) & 3))) & 0xffu : n16;
            if (nl >= 2 && nr[j] >= 2) bits |= 1u << j;
        }
        bits &= at;
        if (count()) {
            uint32_t raised = 0;
#pragma unroll
            for (int j = 0; j < kIxFan; ++j)
                if (marked(j, (xs[j >> 1] >> (16 * (j & 1))) & 0xffffu)) raised |= 1u << j;
            raise(raised & at);
        } else {
            at = 0;
        }
    }
    for (uint32_t level = 3; level < 64; ++level) {
        bits = 0;
        for (uint32_t m = at; m; m &= m - 1) {
            const int j = __ffs(m) - 1, l = p0 + j + 1;
            const int r = l < kIxBlock ? ends[l] : kIxBlock;             // the right child
            if (r < kIxBlock && num[l] >= level && num[r] >= level) bits |= 1u << j;
        }
        if (!count()) break;
        uint32_t raised = 0;
        for (uint32_t m = at; m; m &= m - 1) {
            const int j = __ffs(m) - 1;
            if (marked(j, ends[p0 + j])) raised |= 1u << j;
        }
        raise(raised);
    }
    if (k0 < q.n) {
        if (k0 + 16 <= q.n && (((uintptr_t)(q.sn + k0)) & 15) == 0) {
            *(uint4*)(q.sn + k0) = make_uint4(sn[0], sn[1], sn[2], sn[3]);
        } else {
#pragma unroll
            for (int j = 0; j < kIxFan; ++j)
                if (k0 + j < q.n) q.sn[k0 + j] = (uint8_t)(sn[j >> 2] >> (8 * (j & 3)));
        }
    }
    if (gridDim.x == 1) return;                                          // nothing is open
    const IxOpen o = ix_open(q);
    // the largest number up to each group
    int32_t mx = (int32_t)ix_max_of(ix_max8(ix_max8(sn[0], sn[1]), ix_max8(sn[2], sn[3])));
    for (int d = 1; d < 64; d <<= 1) {
        const int32_t y = __shfl_up(mx, d, 64);
        if (lane >= d) mx = max(mx, y);
    }
    __syncthreads();
    if (lane == 63) wtot[w] = mx;
    __syncthreads();
    int32_t before = __shfl_up(mx, 1, 64);
    if (lane == 0) before = 0;
    for (int i = 0; i < w; ++i) before = max(before, wtot[i]);
    if (k0 < q.n) {
        o.open[k0 / 16] = (uint16_t)open;
        o.before[k0 / 16] = (uint8_t)before;
    }
    if (tid == 255) o.bmax[blockIdx.x] = (uint8_t)max(before, mx);
}

// The open nodes of this thread's group at `level` (at any, 0).
__device__ __forceinline__ uint32_t ix_open_at(const IxParams& q, const IxOpen& o, int64_t k0, uint32_t level)
{
    const uint32_t open = k0 < q.n ? o.open[k0 / 16] : 0u;
    if (!open || level == 0) return open;
    uint32_t sn[4], m = 0;
    ix_bytes16(q.sn, k0, q.n, sn);
#pragma unroll
    for (int j = 0; j < kIxFan; ++j)
        if (((sn[j >> 2] >> (8 * (j & 3))) & 0xffu) == level) m |= 1u << j;
    return m & open;
}

// Open nodes take the largest number in the block where their subtree ends,
// up to the end: all of it is theirs.  Numbers that other threads raise in
// the same launch count as they are read: each is some descendant's or less.
__global__ __launch_bounds__(256) void k_ix_sopen(IxParams q)
{
    const int64_t k0 = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 16;
    const IxOpen o = ix_open(q);
    const uint32_t m = ix_open_at(q, o, k0, 0);
    if (!m) return;
    int64_t lo, hi;
    ix_block_trees(q, blockIdx.x, lo, hi);
    const int64_t t = ix_tree_in(q, lo, hi, k0);
    ix_each_from(q, k0, m, t, q.offsets[t], q.offsets[t + 1], [&](int64_t k, int64_t s, int64_t e) {
        const int64_t x = s + q.end[k];
        if (x <= k || x > e || x % kIxBlock == 0) return;
        const int64_t g = (x - 1) / 16;                                  // the last group with positions before x
        uint32_t v[4];
        ix_bytes16(q.sn, g * 16, q.n, v);
        const int in = (int)(x - g * 16);
        uint32_t a = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int b = in - 4 * i;                                    // bytes of this word before x
            a = ix_max8(a, b <= 0 ? 0u : b >= 4 ? v[i] : v[i] & ((1u << (8 * b)) - 1u));
        }
        const uint32_t most = max(ix_max_of(a), (uint32_t)o.before[g]);
        if (most > q.sn[k]) q.sn[k] = (uint8_t)most;
    });
}

// A pass over the open nodes: marks those with two children at level or
// more, with their prefix in el (its E values are not needed any more).
__global__ __launch_bounds__(256) void k_ix_sflag(IxParams q, int level, int32_t* bsum)
{
    __shared__ int32_t wtot[4];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int64_t base = ((int64_t)blockIdx.x * 256 + tid) * 16;
    const IxOpen o = ix_open(q);
    uint32_t bits = 0;
    // a function with both children at level or more is itself at level already
    const uint32_t m = ix_open_at(q, o, base, (uint32_t)level);
    if (m) {
        int64_t lo, hi;
        ix_block_trees(q, blockIdx.x, lo, hi);
        const int64_t t = ix_tree_in(q, lo, hi, base);
        ix_each_from(q, base, m, t, q.offsets[t], q.offsets[t + 1], [&](int64_t k, int64_t s, int64_t e) {
            if (k + 1 < e) {
                const int64_t r = s + q.end[k + 1];                  // the right child
                if (r > k + 1 && r < e && q.sn[k + 1] >= level && q.sn[r] >= level) bits |= 1u << (int)(k - base);
            }
        });
    }
    const int32_t above = o.bmax[blockIdx.x] > level ? 1 : 0;
    // most blocks mark nothing: their prefix is left unwritten and read as zero
    if (!__syncthreads_or(bits != 0)) {
        if (tid == 0) {
            bsum[blockIdx.x] = above;
            q.bempty[blockIdx.x] = 1;
        }
        return;
    }
    if (tid == 0) q.bempty[blockIdx.x] = 0;
    const int32_t run = __popc(bits);
    int32_t incl = run;
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
    }
    if (lane == 63) wtot[w] = incl;
    __syncthreads();
    int32_t wbase = 0;
    for (int i = 0; i < w; ++i) wbase += wtot[i];
    const int32_t excl = wbase + incl - run;
    int32_t pre[16];
    for (int j = 0; j < 16; ++j) pre[j] = excl + __popc(bits & ((1u << j) - 1u));
    int4* dst = (int4*)(q.el + base);
    for (int j = 0; j < 2; ++j)
        dst[j] = make_int4(ix_pack16(pre[8 * j], pre[8 * j + 1]), ix_pack16(pre[8 * j + 2], pre[8 * j + 3]),
                           ix_pack16(pre[8 * j + 4], pre[8 * j + 5]), ix_pack16(pre[8 * j + 6], pre[8 * j + 7]));
    if (tid == 255) bsum[blockIdx.x] = excl + run + above;
}

// Marked functions before position x (x <= n): a block that marked none
// holds no prefix of its own.
__device__ __forceinline__ int32_t ix_count_before(const IxParams& q, int64_t x)
{
    const int64_t b = x / kIxBlock;
    return q.bempty[b] ? q.boff[b] : ix_e(q, x);
}

// Raises the open nodes at level whose range holds a mark, or a whole block
// with a number above level (the count in front of the node's own block is
// left out: its part from the node on is in the node's number already).
__global__ __launch_bounds__(256) void k_ix_supd(IxParams q, int level)
{
    const int64_t k0 = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 16;
    const IxOpen o = ix_open(q);
    if (blockIdx.x == 0 && threadIdx.x == 0) q.bad_offsets[1] = q.boff[gridDim.x];
    const uint32_t m = ix_open_at(q, o, k0, (uint32_t)level);
    if (!m) return;
    int64_t lo, hi;
    ix_block_trees(q, blockIdx.x, lo, hi);
    const int64_t t = ix_tree_in(q, lo, hi, k0);
    const int32_t above = o.bmax[blockIdx.x] > level ? 1 : 0;
    ix_each_from(q, k0, m, t, q.offsets[t], q.offsets[t + 1], [&](int64_t k, int64_t s, int64_t e) {
        const int64_t x = s + q.end[k];                              // the subtree is [k, x)
        if (x > k && x <= e && ix_count_before(q, x) > ix_count_before(q, k) + above) q.sn[k] = (uint8_t)(level + 1);
    });
}

hipError_t launch_strahler_init(const IxParams& q, int64_t nb, hipStream_t s)
{
    if (q.top > 0) {
        const int64_t bg = std::min<int64_t>(65536, std::max<int64_t>(1, (nb + 255) / 256));
        hipLaunchKernelGGL(k_ix_tfirst, dim3((unsigned)bg), dim3(256), 0, s, q, q.seg, nb);
    }
    hipLaunchKernelGGL(k_ix_sblock, dim3((unsigned)nb), dim3(256), 0, s, q);
    if (nb > 1) hipLaunchKernelGGL(k_ix_sopen, dim3((unsigned)nb), dim3(256), 0, s, q);
    return hipGetLastError();
}

hipError_t launch_strahler_level(const IxParams& q, int level, int32_t* bsum, int64_t nb,
                                 hipStream_t s)
{
    hipLaunchKernelGGL(k_ix_sflag, dim3((unsigned)nb), dim3(256), 0, s, q, level, bsum);
    const hipError_t et = launch_top(q, bsum, nb, s);
    if (et != hipSuccess) return et;
    hipLaunchKernelGGL(k_ix_supd, dim3((unsigned)nb), dim3(256), 0, s, q, level);
    return hipGetLastError();
}

hipError_t launch_index(const IxParams& q, int32_t* bsum, int64_t nb, const int64_t* host_len, hipStream_t s)
{
    hipLaunchKernelGGL(k_ix_scan, dim3((unsigned)nb), dim3(256), 0, s, q, bsum);
    const hipError_t et = launch_top(q, bsum, nb, s);
    if (et != hipSuccess) return et;
    for (int l = 1; l <= q.top; ++l) {
        const int64_t len = host_len[l];
        const int64_t grid = std::min<int64_t>(65536, std::max<int64_t>(1, (len + 255) / 256));
        hipLaunchKernelGGL(k_ix_level, dim3((unsigned)grid), dim3(256), 0, s, q, l);
    }
    const int64_t tg = std::min<int64_t>(65536, std::max<int64_t>(1, (q.n_trees + 255) / 256));
    hipLaunchKernelGGL(k_ix_init, dim3((unsigned)tg), dim3(256), 0, s, q);
    const int64_t bg = std::min<int64_t>(65536, std::max<int64_t>(1, (nb + 255) / 256));
    hipLaunchKernelGGL(k_ix_tfirst, dim3((unsigned)bg), dim3(256), 0, s, q, bsum, nb);
    const int64_t pg = (q.n + 16 * 256 - 1) / (16 * 256);
    hipLaunchKernelGGL(k_ix_bytes, dim3((unsigned)pg), dim3(256), 0, s, q, (const int32_t*)bsum);
    hipLaunchKernelGGL(k_ix_trees, dim3((unsigned)tg), dim3(256), 0, s, q);
    hipLaunchKernelGGL(k_ix_links, dim3((unsigned)pg), dim3(256), 0, s, q, (const int32_t*)bsum);
    return hipGetLastError();
}

}  // namespace gpe
