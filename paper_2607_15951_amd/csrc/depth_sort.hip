// depth_sort.hip -- stable LSD radix sort of the per-Gaussian depth keys.
//
// The sort of Sec. 3.1 stage 3 orders (Gaussian, tile) pairs by the 64-bit
// key (tile << 32 | depth bits).  Every pair of one Gaussian carries the same
// 32 depth bits, so the least-significant digits of that LSD radix sort are
// applied here to the N Gaussians -- before duplication -- instead of to the
// K ~ 80 N pairs.  The tile digit is then one stable counting pass
// (tile_bin.hip) that writes each pair straight to its sorted position.
//
// Few keys take fewer launches (below).
//
// Several views are sorted at once as segments of one array (one segment per
// view, items v * n + i); no block straddles two segments.
//
// Each 8-bit pass is an LDS histogram per block, written as the block's 256
// contiguous counts (whole cache lines; a digit-major table would take 256
// scattered partial-line writes per block), and a stable scatter that ranks
// equal digits with wavefront ballots (lower lanes and earlier waves first) and
// places digit d of segment v at v * n + (the segment's items of smaller
// digits) + (d's items in the blocks before).  Those come from group sums that
// the histograms add to (32 blocks of a segment) and the block's own group's
// counts; for many keys from a launch between the two, one workgroup per
// (segment, digit) that scans its digit's counts over the blocks.  Digits are taken from sort_key(key), which orders
// depths as numbers (negative ones, behind the camera, first); keys of
// Gaussians without a finite depth are 0xFFFFFFFF and sink to the end.
// Values start as the Gaussian index, so ties in depth stay in index order.
#include "gs_internal.h"
#include "partials.h"

#include <algorithm>
#include <type_traits>

namespace gsmi {
namespace {

// Block b sorts part lb = b % bpv of segment v = b / bpv: items
// [v * n + lb * tile, min(.. + tile, (v + 1) * n)), tile = kSortBlock * kItems.
// The count buffer holds two tables of group sums [segment][group][digit]
// (passes use them in turn), then the block histograms [block][digit]; or the
// digit totals [segment][digit], the offset table [segment][digit][part], then
// the block histograms.
template <int kItems>
__device__ __forceinline__ void sort_block_range(unsigned block, int64_t n, int bpv, int64_t* begin, int64_t* end)
{
    constexpr int64_t tile = (int64_t)kSortBlock * kItems;
    const int v = (int)(block / (unsigned)bpv), lb = (int)(block % (unsigned)bpv);
    *begin = (int64_t)v * n + (int64_t)lb * tile;
    const int64_t seg_end = (int64_t)(v + 1) * n;
    *end = (*begin + tile < seg_end) ? *begin + tile : seg_end;
}

// Consecutive parts of a segment whose counts are also kept as one sum: a
// block then finds where its digits go from the sums of its segment's groups
// and the counts of its own group's parts (51 rows of 1 KB at 2.5M keys).
constexpr int kGroupParts = 32;
__host__ __device__ __forceinline__ int sort_groups(int bpv) { return (bpv + kGroupParts - 1) / kGroupParts; }
__device__ __forceinline__ int sort_group(unsigned block, int bpv)
{
    return (int)(block / (unsigned)bpv) * sort_groups(bpv) + (int)(block % (unsigned)bpv) / kGroupParts;
}

// Order-preserving map of a depth key to the sort key: float bits compare as
// unsigned integers only among non-negative floats, so negative depths
// (Gaussians behind the camera) are flipped below them; 0xFFFFFFFF (no finite
// depth) stays last.  On the non-negative depths of the pairs it keeps the
// order of the bits themselves.
__device__ __forceinline__ uint32_t sort_key(uint32_t b)
{
    if (b == 0xFFFFFFFFu) return b;
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// Valid lanes of this wave that hold the lane's digit.
__device__ __forceinline__ uint64_t same_digit_lanes(uint32_t d, bool valid)
{
    uint64_t m = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const bool bit = (d >> b) & 1u;
        const uint64_t bb = __ballot(bit);
        m &= bit ? bb : ~bb;
    }
    return m;
}

template <int kItems>
__global__ __launch_bounds__(kSortBlock) void radix_hist_kernel(const uint32_t* __restrict__ keys, int64_t n,
                                                                 int shift, uint32_t* __restrict__ hist,
                                                                 uint32_t* __restrict__ groups, int bpv,
                                                                 const uint32_t* skip, PartialSums sums)
{
    if (skip && *skip) return;   // the previous frame's order was reused
    // the first sums.n_views workgroups sum the projection's partials
    if ((int)blockIdx.x < sums.n_views) {
        sum_partials<kSortBlock>(sums, (int)blockIdx.x);
        return;
    }
    const unsigned block = blockIdx.x - (unsigned)sums.n_views;
    __shared__ uint32_t h[4][256];   // one private histogram per wave
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
#pragma unroll
    for (int w = 0; w < 4; ++w) h[w][tid] = 0;
    __syncthreads();
    int64_t begin, end;
    sort_block_range<kItems>(block, n, bpv, &begin, &end);
    // every key load issued before any is used (a load under its own branch
    // is waited for before the next one issues); past end, key begin is
    // loaded and dropped
    uint32_t kk[kItems];
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        const int64_t idx = begin + k * kSortBlock + tid;
        kk[k] = keys[idx < end ? idx : begin];
    }
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        const int64_t idx = begin + k * kSortBlock + tid;
        const bool valid = idx < end;
        const uint32_t d = valid ? (sort_key(kk[k]) >> shift) & 255u : 0u;
        const uint64_t m = __ballot(valid);
        if (m == 0) continue;
        // the high digits of nearby depths are mostly one value: a wave whose
        // items share it counts them with one atomic instead of 64 colliding
        const int first = __ffsll((long long)m) - 1;
        const uint32_t d0 = (uint32_t)__shfl((int)d, first, 64);
        if (__ballot(valid && d != d0) == 0) {
            if (lane == first) atomicAdd(&h[wave][d0], (uint32_t)__popcll(m));
        } else if (valid) {
            atomicAdd(&h[wave][d], 1u);
        }
    }
    __syncthreads();
    const uint32_t count = h[0][tid] + h[1][tid] + h[2][tid] + h[3][tid];
    hist[(int64_t)block * 256 + tid] = count;
    if (groups && count) atomicAdd(&groups[(int64_t)sort_group(block, bpv) * 256 + tid], count);
}

// Workgroup (v, d): exclusive scan of digit d's counts over the bpv blocks of
// segment v (hist[(v * bpv + b) * 256 + d]) into row (v, d) of the offset
// table, and the digit's total in totals[v * 256 + d].  Counts fit 32 bits
// (n_views * n < 2^32).
constexpr int kScanRowItems = 8;
__global__ __launch_bounds__(256) void radix_row_scan_kernel(const uint32_t* __restrict__ hist,
                                                              uint32_t* __restrict__ table,
                                                              uint32_t* __restrict__ totals, int bpv,
                                                              const uint32_t* skip)
{
    if (skip && *skip) return;
    __shared__ uint32_t s_wsum[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int v = (int)(blockIdx.x >> 8), d = (int)(blockIdx.x & 255u);
    const uint32_t* col = hist + (int64_t)v * bpv * 256 + d;   // block b's count at col[b * 256]
    uint32_t* row = table + (int64_t)blockIdx.x * bpv;
    uint32_t carry = 0u;
    for (int base = 0; base < bpv; base += 256 * kScanRowItems) {
        uint32_t x[kScanRowItems], run = 0u;
        const int j0 = base + tid * kScanRowItems;   // this thread's consecutive counts
#pragma unroll
        for (int k = 0; k < kScanRowItems; ++k) {
            x[k] = (j0 + k < bpv) ? col[(int64_t)(j0 + k) * 256] : 0u;
            run += x[k];
        }
        uint32_t incl = run;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t t = __shfl_up(incl, o, 64);
            if (lane >= o) incl += t;
        }
        if (lane == 63) s_wsum[wave] = incl;
        __syncthreads();
        uint32_t before = carry;
        for (int w = 0; w < wave; ++w) before += s_wsum[w];
        const uint32_t chunk_total = s_wsum[0] + s_wsum[1] + s_wsum[2] + s_wsum[3];
        uint32_t acc = before + incl - run;
#pragma unroll
        for (int k = 0; k < kScanRowItems; ++k) {
            if (j0 + k < bpv) row[j0 + k] = acc;
            acc += x[k];
        }
        carry += chunk_total;
        __syncthreads();   // s_wsum is reused by the next chunk
    }
    if (tid == 0) totals[blockIdx.x] = carry;
}

// Stable scatter of one block's items.  Item (round k, wave w, lane l) is
// idx = begin + k * kSortBlock + 64 w + l, so the input order is (k, w, l).
// Each wave ranks its items of a round among equal digits with eight ballots
// (lanes holding the same digit) and records the group's size in
// cnt[k][w][d]; one pass of 256 threads (one per digit) turns those counts
// into exclusive offsets in (k, w) order and the digits' totals into the
// block's digit starts.  Every item is then placed in LDS at its position in
// the block's stable digit order, and the block writes that order out with
// consecutive threads on consecutive positions of each digit's run: item i of
// digit d goes to base[d] + (i - start[d]).  The global writes come as whole
// runs instead of one scattered word per lane.
//
// With kPay every item also carries a payload word: read from pay_in, or in
// the first pass (pay_in null) packed from rect_in, and written to pay_out
// beside its value.  keys_out may be null (the last pass: the sorted keys
// are not needed).
template <int kItems, bool kPay, bool kGrouped, int kThreads = kSortBlock>
__global__ __launch_bounds__(kThreads) void radix_scatter_kernel(
    const uint32_t* __restrict__ keys_in, const uint32_t* __restrict__ vals_in, uint32_t* __restrict__ keys_out,
    uint32_t* __restrict__ vals_out, const ushort4* __restrict__ rect_in, const uint32_t* __restrict__ pay_in,
    uint32_t* __restrict__ pay_out, int64_t n, int shift, const uint32_t* __restrict__ hist,
    const uint32_t* __restrict__ groups, uint32_t* __restrict__ next_groups, const uint32_t* __restrict__ offsets,
    const uint32_t* __restrict__ totals, int bpv, const uint32_t* skip)
{
    constexpr int kWaves = kThreads / 64;
    constexpr int kParts = kThreads / 256;   // threads that share a digit's rows
    constexpr int kBlockItems = kItems * kThreads;   // = kSortBlock * (kBlockItems / kSortBlock): the block's part
    static_assert(kThreads % kSortBlock == 0, "whole 256-thread groups");
    if (skip && *skip) return;
    // the block's keys, values (and payloads) in digit order; before that,
    // the 16-bit ranking counts cnt[k][w][d] (at most kBlockItems)
    // in the same bytes, which keeps the block's LDS at 8 (12) bytes per item
    __shared__ uint32_t s_buf[(kPay ? 3 : 2) * kBlockItems];
    uint16_t(*cnt)[kWaves][256] = reinterpret_cast<uint16_t(*)[kWaves][256]>(s_buf);
    static_assert(kItems * kWaves * 256 * sizeof(uint16_t) <= sizeof(s_buf), "ranking counts fit the key buffer");
    static_assert(kBlockItems <= 65535, "16-bit ranking offsets");
    __shared__ uint32_t s_start[256], s_base[256], s_wsum[4], s_ssum[4];
    __shared__ uint32_t s_total[kGrouped ? kParts : 1][256], s_before[kGrouped ? kParts : 1][256];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int64_t begin, end;
    sort_block_range<kBlockItems / kSortBlock>(blockIdx.x, n, bpv, &begin, &end);
    for (int i = tid; i < kItems * kWaves * 128; i += kThreads) s_buf[i] = 0u;   // cnt, two counts per word
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    __syncthreads();
    uint32_t key[kItems], val[kItems], digit[kItems], rank[kItems];
    uint32_t pay[kPay ? kItems : 1];
    // all loads first (see radix_hist_kernel)
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        const int64_t idx = begin + k * kThreads + tid;
        const int64_t ic = idx < end ? idx : begin;
        key[k] = keys_in[ic];
        val[k] = vals_in ? vals_in[ic] : (uint32_t)idx;
        if constexpr (kPay) pay[k] = pay_in ? pay_in[ic] : pack_rect(rect_in[ic]);
    }
    // digit d's count in the segment and in the parts before this one
    const int v = (int)(blockIdx.x / (unsigned)bpv), lb = (int)(blockIdx.x % (unsigned)bpv);
    if constexpr (kGrouped) {
        const int q = tid >> 8, d = tid & 255, ng = sort_groups(bpv), own = lb / kGroupParts;
        const uint32_t* g = groups + (int64_t)v * ng * 256 + d;
        uint32_t total = 0u, before = 0u;
#pragma unroll 4
        for (int i = q; i < ng; i += kParts) {
            const uint32_t c = g[i * 256];
            total += c;
            before += i < own ? c : 0u;
        }
        const uint32_t* h = hist + ((int64_t)v * bpv + own * kGroupParts) * 256 + d;
#pragma unroll 4
        for (int i = q; i < lb - own * kGroupParts; i += kParts) before += h[i * 256];
        s_total[q][d] = total;
        s_before[q][d] = before;
    }
    // the next pass's group sums start at zero
    if (kGrouped && next_groups)
        for (int64_t i = (int64_t)blockIdx.x * kThreads + tid; i < (int64_t)(gridDim.x / bpv) * sort_groups(bpv) * 256;
             i += (int64_t)gridDim.x * kThreads)
            next_groups[i] = 0u;
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        const int64_t idx = begin + k * kThreads + tid;
        const bool valid = idx < end;
        if (!valid) key[k] = val[k] = 0u;
        const uint32_t d = (sort_key(key[k]) >> shift) & 255u;
        const uint64_t m = same_digit_lanes(d, valid);
        digit[k] = valid ? d : 256u;
        rank[k] = (uint32_t)__popcll(m & lt);
        // the group's first lane records its size (groups are disjoint)
        if (valid && rank[k] == 0) cnt[k][wave][d] = (uint16_t)__popcll(m);
    }
    __syncthreads();
    // threads d < 256: exclusive offsets of digit d over (round, wave), its
    // total, and the block's digit start (exclusive prefix of the totals);
    // then the segment's start of digit d (exclusive prefix of its totals)
    uint32_t run = 0u, seg_total = 0u, incl = 0u, seg_incl = 0u;
    if (tid < 256) {
#pragma unroll
        for (int k = 0; k < kItems; ++k)
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                const uint32_t c = cnt[k][w][tid];
                cnt[k][w][tid] = (uint16_t)run;
                run += c;
            }
        // the segment's count of digit d
        if constexpr (kGrouped) {
#pragma unroll
            for (int q = 0; q < kParts; ++q) seg_total += s_total[q][tid];
        } else {
            seg_total = totals[v * 256 + tid];
        }
        incl = run;
        seg_incl = seg_total;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t t = __shfl_up(incl, o, 64), u = __shfl_up(seg_incl, o, 64);
            if (lane >= o) {
                incl += t;
                seg_incl += u;
            }
        }
        if (lane == 63) {
            s_wsum[wave] = incl;
            s_ssum[wave] = seg_incl;
        }
    }
    __syncthreads();
    if (tid < 256) {
        uint32_t before = 0u, seg_before = (uint32_t)((int64_t)v * n);
        for (int w = 0; w < wave; ++w) {
            before += s_wsum[w];
            seg_before += s_ssum[w];
        }
        s_start[tid] = before + incl - run;
        if constexpr (kGrouped) {
#pragma unroll
            for (int q = 0; q < kParts; ++q) seg_before += s_before[q][tid];
        } else {
            seg_before += offsets[((int64_t)v * 256 + tid) * bpv + lb];
        }
        s_base[tid] = seg_before + seg_incl - seg_total;
    }
    __syncthreads();
    uint32_t local[kItems];
#pragma unroll
    for (int k = 0; k < kItems; ++k)
        local[k] = digit[k] < 256u ? s_start[digit[k]] + cnt[k][wave][digit[k]] + rank[k] : ~0u;
    __syncthreads();   // cnt is reused below
    uint32_t* s_key = s_buf;
    uint32_t* s_val = s_key + kBlockItems;
    uint32_t* s_pay = s_val + kBlockItems;   // kPay only
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        if (local[k] != ~0u) {
            s_key[local[k]] = key[k];
            s_val[local[k]] = val[k];
            if constexpr (kPay) s_pay[local[k]] = pay[k];
        }
    }
    __syncthreads();
    const int count = (int)(end - begin);
    for (int i = tid; i < count; i += kThreads) {
        const uint32_t kk = s_key[i];
        const uint32_t d = (sort_key(kk) >> shift) & 255u;
        const uint32_t pos = s_base[d] + ((uint32_t)i - s_start[d]);
        if (keys_out) keys_out[pos] = kk;
        vals_out[pos] = s_val[i];
        if constexpr (kPay) pay_out[pos] = s_pay[i];
    }
}

// One 8-bit pass: histogram, for many keys a scan of the counts, scatter.
template <int kItems, bool kGrouped>
void launch_sort_pass(const uint32_t* kin, const uint32_t* vin, uint32_t* kout, uint32_t* vout, const ushort4* rect,
                      const uint32_t* pin, uint32_t* pout, uint32_t* counts, int64_t n, int n_views, int shift,
                      int bpv, unsigned nblocks, const uint32_t* skip, hipStream_t s, const PartialSums& sums,
                      hipEvent_t sums_done)
{
    const int pass = shift / 8;
    const int64_t table = (int64_t)n_views * sort_groups(bpv) * 256;
    uint32_t* groups = kGrouped ? counts + (pass & 1) * table : nullptr;
    uint32_t* next = kGrouped && pass < 3 ? counts + ((pass + 1) & 1) * table : nullptr;
    uint32_t* totals = kGrouped ? nullptr : counts;
    uint32_t* offsets = kGrouped ? nullptr : counts + (int64_t)256 * n_views;
    uint32_t* hist = kGrouped ? counts + 2 * table : offsets + (int64_t)256 * nblocks;
    hipLaunchKernelGGL(radix_hist_kernel<kItems>, dim3(nblocks + (unsigned)sums.n_views), dim3(kSortBlock), 0, s, kin,
                       n, shift, hist, groups, bpv, skip, sums);
    if (sums_done) (void)hipEventRecord(sums_done, s);
    if (!kGrouped)
        hipLaunchKernelGGL(radix_row_scan_kernel, dim3(256u * (unsigned)n_views), dim3(256), 0, s,
                           (const uint32_t*)hist, offsets, totals, bpv, skip);
    // the scatter of a 16-key part runs as 1024 threads of 4 keys: the same
    // part, ranked by 16 waves of 4 rounds instead of 4 waves of 16 (0.161
    // against 0.165 ms for the four passes at 3M keys; parts of 8192 keys,
    // one 100 KB block per CU, took 0.20 ms)
    constexpr int kThreads = kItems == 16 ? 1024 : kSortBlock;
    constexpr int kPer = kItems * kSortBlock / kThreads;
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(nblocks), dim3(kThreads), 0, s, kin, vin, kout, vout, rect, pin, pout, n,
                           shift, (const uint32_t*)hist, (const uint32_t*)groups, next, (const uint32_t*)offsets,
                           (const uint32_t*)totals, bpv, skip);
    };
    if (pout) go(radix_scatter_kernel<kPer, true, kGrouped, kThreads>);
    else go(radix_scatter_kernel<kPer, false, kGrouped, kThreads>);
}

// ------------------------------------------------------- few keys
// Up to kCountedKeys keys sort in five launches, not twelve: a pass's scatter
// sums its segment's part histograms itself (at most 96 rows of 1 KB) and
// counts, while it writes its items, the next pass's digits per part of where
// they land.  Such a sort costs its launches and their latency: 5000 keys 35
// us (65 with three launches per pass), 40000 keys 41 (68), 65536 keys 49
// (67).  The counting adds up to one atomic per key and pass: 131072 keys
// would take 70 us (69), 262144 keys 89 (72).
// A segment of up to 4 x 1024 keys sorts in one launch, all four passes in LDS
// (1000 keys: 8.4 us, 33 with a launch per pass).
constexpr int kFusedThreads = 1024, kFusedWaves = kFusedThreads / 64;
constexpr int64_t kCountedKeys = 98304;

// One pass over a block's items in registers: ranks them by digit and leaves
// keys, values (and payloads) in LDS in the block's stable digit order.  Item
// (k, thread) is the block's item k * kFusedThreads + thread; valid[k] holds
// for the first count of them.
template <int kItems, bool kPay>
struct FusedLds {
    static constexpr int kPart = kItems * kFusedThreads;
    // in digit order; before that the ranking counts cnt[k][wave][digit]
    uint32_t buf[(kPay ? 3 : 2) * kPart];
    uint32_t start[256];    // the block's first item of a digit
    uint32_t total[256];    // and its items
    uint32_t wsum[4];
    __device__ __forceinline__ uint32_t* keys() { return buf; }
    __device__ __forceinline__ uint32_t* vals() { return buf + kPart; }
    __device__ __forceinline__ uint32_t* pays() { return buf + 2 * kPart; }
};

template <int kItems, bool kPay>
__device__ __forceinline__ void fused_order(FusedLds<kItems, kPay>& L, const uint32_t (&key)[kItems],
                                            const uint32_t (&val)[kItems], const uint32_t* pay, int count, int shift)
{
    uint16_t(*cnt)[kFusedWaves][256] = reinterpret_cast<uint16_t(*)[kFusedWaves][256]>(L.buf);
    static_assert(kItems * kFusedWaves * 256 * sizeof(uint16_t) <= sizeof(L.buf), "ranking counts fit");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int i = 0; i < 2 * kItems; ++i) L.buf[i * kFusedThreads + tid] = 0u;
    __syncthreads();
    uint32_t digit[kItems], rank[kItems];
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        const bool valid = k * kFusedThreads + tid < count;
        const uint32_t d = (sort_key(key[k]) >> shift) & 255u;
        const uint64_t m = same_digit_lanes(d, valid);
        digit[k] = valid ? d : 256u;
        rank[k] = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        if (valid && rank[k] == 0u) cnt[k][wave][d] = (uint16_t)__popcll(m);
    }
    __syncthreads();
    uint32_t run = 0u, incl = 0u;
    if (tid < 256) {
        uint32_t c[kItems * kFusedWaves];
#pragma unroll
        for (int j = 0; j < kItems * kFusedWaves; ++j) c[j] = cnt[j / kFusedWaves][j % kFusedWaves][tid];
#pragma unroll
        for (int j = 0; j < kItems * kFusedWaves; ++j) {
            cnt[j / kFusedWaves][j % kFusedWaves][tid] = (uint16_t)run;
            run += c[j];
        }
        L.total[tid] = run;
        incl = run;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t t = __shfl_up(incl, o, 64);
            if (lane >= o) incl += t;
        }
        if (lane == 63) L.wsum[wave] = incl;
    }
    __syncthreads();
    if (tid < 256) {
        uint32_t before = 0u;
        for (int w = 0; w < wave; ++w) before += L.wsum[w];
        L.start[tid] = before + incl - run;
    }
    __syncthreads();
    uint32_t local[kItems];
#pragma unroll
    for (int k = 0; k < kItems; ++k)
        local[k] = digit[k] < 256u ? L.start[digit[k]] + cnt[k][wave][digit[k]] + rank[k] : ~0u;
    __syncthreads();   // the counts' bytes are reused
#pragma unroll
    for (int k = 0; k < kItems; ++k)
        if (local[k] != ~0u) {
            L.keys()[local[k]] = key[k];
            L.vals()[local[k]] = val[k];
            if constexpr (kPay) L.pays()[local[k]] = pay[k];
        }
    __syncthreads();
}

// One block per segment of at most kItems * kFusedThreads keys.
template <int kItems, bool kPay>
__global__ __launch_bounds__(kFusedThreads) void radix_segment_kernel(const uint32_t* __restrict__ keys_in,
                                                                      uint32_t* __restrict__ vals_out,
                                                                      const ushort4* __restrict__ rect_in,
                                                                      uint32_t* __restrict__ pay_out, int n,
                                                                      const uint32_t* skip, PartialSums sums)
{
    if (skip && *skip) return;
    if ((int)blockIdx.x < sums.n_views) {
        sum_partials<kFusedThreads>(sums, (int)blockIdx.x);
        return;
    }
    __shared__ FusedLds<kItems, kPay> L;
    const int tid = threadIdx.x;
    const int64_t begin = (int64_t)(blockIdx.x - (unsigned)sums.n_views) * n;
    uint32_t key[kItems], val[kItems], pay[kPay ? kItems : 1];
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        const int i = k * kFusedThreads + tid;
        const int64_t ic = begin + (i < n ? i : 0);
        key[k] = keys_in[ic];
        val[k] = (uint32_t)ic;
        if constexpr (kPay) pay[k] = pack_rect(rect_in[ic]);
    }
    for (int shift = 0; shift < 32; shift += 8) {
        fused_order<kItems, kPay>(L, key, val, pay, n, shift);
        if (shift == 24) break;
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            const int i = k * kFusedThreads + tid;
            key[k] = L.keys()[i];   // past n: whatever is there, never used
            val[k] = L.vals()[i];
            if constexpr (kPay) pay[k] = L.pays()[i];
        }
        __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        const int i = k * kFusedThreads + tid;
        if (i < n) {
            vals_out[begin + i] = L.vals()[i];
            if constexpr (kPay) pay_out[begin + i] = L.pays()[i];
        }
    }
}

// Counts the first digit of every part, hist[part][digit], and clears the
// tables of the three passes that follow, which lie behind it.
__global__ __launch_bounds__(kFusedThreads) void radix_first_hist_kernel(const uint32_t* __restrict__ keys, int64_t n,
                                                                         uint32_t* __restrict__ hist, int bpv,
                                                                         const uint32_t* skip, PartialSums sums)
{
    if (skip && *skip) return;
    if ((int)blockIdx.x < sums.n_views) {
        sum_partials<kFusedThreads>(sums, (int)blockIdx.x);
        return;
    }
    const unsigned block = blockIdx.x - (unsigned)sums.n_views;
    __shared__ uint32_t h[4][256];
    const int tid = threadIdx.x;
    h[tid >> 8][tid & 255] = 0u;
    __syncthreads();
    int64_t begin, end;
    sort_block_range<kFusedThreads / kSortBlock>(block, n, bpv, &begin, &end);
    if (begin + tid < end) atomicAdd(&h[tid >> 8][sort_key(keys[begin + tid]) & 255u], 1u);
    __syncthreads();
    const int64_t at = (int64_t)block * 256, table = (int64_t)(gridDim.x - (unsigned)sums.n_views) * 256;
    const int t = tid >> 8, d = tid & 255;
    hist[t * table + at + d] = t == 0 ? h[0][d] + h[1][d] + h[2][d] + h[3][d] : 0u;
}

// One pass: stable scatter of the block's part by the digit at shift, whose
// counts per part are in hist; hist_next (null in the last pass) gets the
// counts of the next digit over the parts of the output.
template <bool kPay>
__global__ __launch_bounds__(kFusedThreads) void radix_fused_kernel(
    const uint32_t* __restrict__ keys_in, const uint32_t* __restrict__ vals_in, uint32_t* __restrict__ keys_out,
    uint32_t* __restrict__ vals_out, const ushort4* __restrict__ rect_in, const uint32_t* __restrict__ pay_in,
    uint32_t* __restrict__ pay_out, int64_t n, int shift, const uint32_t* __restrict__ hist,
    uint32_t* __restrict__ hist_next, int bpv, const uint32_t* skip)
{
    if (skip && *skip) return;
    constexpr int kPart = kFusedThreads;
    __shared__ FusedLds<1, kPay> L;
    __shared__ uint32_t s_total[4][256], s_before[4][256], s_base[256], s_ssum[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int64_t begin, end;
    sort_block_range<kPart / kSortBlock>(blockIdx.x, n, bpv, &begin, &end);
    const int v = (int)(blockIdx.x / (unsigned)bpv), lb = (int)(blockIdx.x % (unsigned)bpv);
    const int count = (int)(end - begin);
    const int64_t ic = tid < count ? begin + tid : begin;
    uint32_t key[1] = {keys_in[ic]}, val[1] = {vals_in ? vals_in[ic] : (uint32_t)ic}, pay[1];
    if constexpr (kPay) pay[0] = pay_in ? pay_in[ic] : pack_rect(rect_in[ic]);
    {   // digit d's count over the segment and over the parts before this one: every fourth part
        const int q = tid >> 8, d = tid & 255;
        const uint32_t* h = hist + (int64_t)v * bpv * 256 + d;
        uint32_t total = 0u, before = 0u;
#pragma unroll 8
        for (int b = q; b < bpv; b += 4) {
            const uint32_t c = h[b * 256];
            total += c;
            before += b < lb ? c : 0u;
        }
        s_total[q][d] = total;
        s_before[q][d] = before;
    }
    fused_order<1, kPay>(L, key, val, pay, count, shift);   // synchronises before and after
    uint32_t total = 0u, incl = 0u;
    if (tid < 256) {
        total = s_total[0][tid] + s_total[1][tid] + s_total[2][tid] + s_total[3][tid];
        incl = total;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t t = __shfl_up(incl, o, 64);
            if (lane >= o) incl += t;
        }
        if (lane == 63) s_ssum[wave] = incl;
    }
    __syncthreads();
    if (tid < 256) {
        uint32_t at = (uint32_t)((int64_t)v * n);
        for (int w = 0; w < wave; ++w) at += s_ssum[w];
        // less the block's start of the digit: item i goes to s_base[d] + i
        s_base[tid] = at + incl - total + s_before[0][tid] + s_before[1][tid] + s_before[2][tid] + s_before[3][tid] -
                      L.start[tid];
    }
    __syncthreads();
    uint32_t* next = hist_next ? hist_next + (int64_t)v * bpv * 256 : nullptr;
    const bool valid = tid < count;
    const uint32_t kk = L.keys()[valid ? tid : 0];
    const uint32_t sk = sort_key(kk) >> shift;
    const uint32_t pos = s_base[sk & 255u] + (uint32_t)tid;
    if (valid) {
        if (keys_out) keys_out[pos] = kk;
        vals_out[pos] = L.vals()[tid];
        if constexpr (kPay) pay_out[pos] = L.pays()[tid];
    }
    if (next) {
        // a few digits often hold most of a wave's items: those are counted
        // together, the rest lane by lane
        const uint32_t slot = (pos - (uint32_t)((int64_t)v * n)) / kPart * 256u + ((sk >> 8) & 255u);
        uint64_t left = __ballot(valid);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if (!left) break;
            const int f = __builtin_ctzll(left);
            const uint32_t first = (uint32_t)__builtin_amdgcn_readlane((int)slot, f);
            const uint64_t m = __ballot(slot == first) & left;
            if (lane == f) atomicAdd(&next[first], (uint32_t)__popcll(m));
            left &= ~m;
        }
        if ((left >> lane) & 1u) atomicAdd(&next[slot], 1u);
    }
}

// Items per thread with which a segment of n keys sorts in one launch, and
// whether n_views segments do in five.
int segment_items(int64_t n) { return n <= kFusedThreads ? 1 : (n <= 2 * kFusedThreads ? 2 : (n <= 4 * kFusedThreads ? 4 : 0)); }
bool fused_sort(int64_t n, int64_t n_views) { return n * n_views <= kCountedKeys; }

template <int kItems, bool kPay>
void launch_segment_sort(const uint32_t* keys_in, uint32_t* vals, const ushort4* rect, uint32_t* pay, int64_t n,
                         int n_views, const uint32_t* skip, hipStream_t s, const PartialSums& sums,
                         hipEvent_t sums_done)
{
    hipLaunchKernelGGL((radix_segment_kernel<kItems, kPay>), dim3((unsigned)(n_views + sums.n_views)),
                       dim3(kFusedThreads), 0, s, keys_in, vals, rect, pay, (int)n, skip, sums);
    if (sums_done) (void)hipEventRecord(sums_done, s);
}

template <bool kPay>
void launch_fused_sort(const uint32_t* keys_in, uint32_t* const (&keys)[2], uint32_t* const (&vals)[2],
                       const ushort4* rect, uint32_t* const (&pay)[2], uint32_t* counts, int64_t n, int n_views,
                       const uint32_t* skip, hipStream_t s, const PartialSums& sums, hipEvent_t sums_done)
{
    const int bpv = (int)((n + kFusedThreads - 1) / kFusedThreads);
    const unsigned blocks = (unsigned)bpv * (unsigned)n_views;
    const int64_t table = (int64_t)blocks * 256;
    hipLaunchKernelGGL(radix_first_hist_kernel, dim3(blocks + (unsigned)sums.n_views), dim3(kFusedThreads), 0, s,
                       keys_in, n, counts, bpv, skip, sums);
    if (sums_done) (void)hipEventRecord(sums_done, s);
    for (int pass = 0; pass < 4; ++pass) {
        const int to = pass & 1, from = to ^ 1;
        hipLaunchKernelGGL(radix_fused_kernel<kPay>, dim3(blocks), dim3(kFusedThreads), 0, s,
                           pass ? (const uint32_t*)keys[from] : keys_in, pass ? (const uint32_t*)vals[from] : nullptr,
                           pass < 3 ? keys[to] : nullptr, vals[to], rect, pass ? (const uint32_t*)pay[from] : nullptr,
                           pay[to], n, 8 * pass, (const uint32_t*)(counts + pass * table),
                           pass < 3 ? counts + (pass + 1) * table : nullptr, bpv, skip);
    }
}

// ------------------------------------------------- reuse of the previous order
// Between nearby frames few Gaussians change their tile (the data locality of
// Sec. 5.7, Table 5), but their depth order is another matter: a dense scene
// has depth gaps far below the depth change of a small camera step, so most
// adjacent pairs swap.  The previous frame's order (one view, same Gaussians)
// is therefore only tried, and cheaply: each item gets this frame's key in
// that order and the descents (adjacent pairs out of order) are counted.
//   no descent       the order holds (static camera, appearance-only
//                    changes): the radix passes are skipped;
//   a few descents   runs of kReuseBlock items are sorted in LDS twice
//                    (aligned, then shifted by half a run) and the result is
//                    checked; the passes are skipped if it holds;
//   more             the radix passes sort from scratch.
// Every decision is taken on the device (flags the kernels read), so the
// frame needs no host read and can be captured.  Whatever path runs, the
// order is the stable (depth, index) order: the check compares the composite
// (sort key << 32 | index), a strict total order.
constexpr int kReuseThreads = 1024;
constexpr int kReuseItems = 8;
constexpr int kReuseBlock = kReuseThreads * kReuseItems;   // items sorted together in LDS

// The gathered keys are sort keys (sort_key), as the radix passes compare.
// words[0] = 1 while the reused order holds (the radix passes' skip flag),
// words[1] = descents of the gathered previous order (churn), words[2] = 1
// when the local repair runs.  A repair is tried for at most n / kRepairFraction descents.
constexpr int64_t kRepairFraction = 256;
// One item per thread: item j takes this frame's key of prev[j], and each
// block counts its descents (pairs (j, j + 1) out of order, the pair across
// its end included) into partial[block].  No counter is shared: one atomic
// counter hit by every block serialises when most pairs swap.  The successor
// of lane l is lane l + 1's item; lane 63 loads its own.
__global__ __launch_bounds__(256) void order_gather_kernel(const uint32_t* __restrict__ keys,
                                                           const uint32_t* __restrict__ prev, int64_t n,
                                                           uint32_t* __restrict__ k_out, uint32_t* __restrict__ v_out,
                                                           uint32_t* words, uint32_t* __restrict__ partial)
{
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int lane = threadIdx.x & 63;
    const bool in = j < n;
    uint32_t p = prev[in ? j : 0];
    const bool tail = lane == 63 && j + 1 < n;
    uint32_t p1 = tail ? prev[j + 1] : 0u;
    const bool invalid = in && p >= (uint32_t)n;   // not an order of these items: sort from scratch
    p = p < (uint32_t)n ? p : 0u;
    p1 = p1 < (uint32_t)n ? p1 : 0u;
    const uint32_t k = sort_key(keys[p]);
    const uint32_t k1 = tail ? sort_key(keys[p1]) : 0u;
    if (in) {
        k_out[j] = k;
        v_out[j] = p;
    }
    uint32_t kn = __shfl_down(k, 1, 64), pn = __shfl_down(p, 1, 64);
    if (lane == 63) {
        kn = k1;
        pn = p1;
    }
    const uint64_t cur = ((uint64_t)k << 32) | p, next = ((uint64_t)kn << 32) | pn;
    uint32_t descents = (j + 1 < n && cur > next) ? 1u : 0u;
    if (invalid) words[0] = 0u;
    __shared__ uint32_t s_d[4];
    for (int o = 32; o > 0; o >>= 1) descents += __shfl_xor(descents, o, 64);
    if (lane == 0) s_d[threadIdx.x >> 6] = descents;
    __syncthreads();
    if (threadIdx.x == 0) partial[blockIdx.x] = s_d[0] + s_d[1] + s_d[2] + s_d[3];
}

// Sorts runs of kReuseBlock composite keys in LDS (bitonic network).  Run b
// covers [offset + b * kReuseBlock, ...); with kShifted the runs start half a
// run in, and one extra block copies the first half run unchanged.
// (The unshifted pass sorts in place: in and out may be the same arrays.)
template <bool kShifted>
__global__ __launch_bounds__(kReuseThreads) void order_local_sort_kernel(const uint32_t* k_in, const uint32_t* v_in,
                                                                        int64_t n, uint32_t* k_out, uint32_t* v_out,
                                                                        const uint32_t* words)
{
    if (!words[2]) return;   // no repair this frame
    __shared__ uint64_t s[kReuseBlock];
    const int tid = threadIdx.x;
    const int64_t half = kReuseBlock / 2;
    if (kShifted && blockIdx.x == gridDim.x - 1) {   // the head, already in place
        for (int64_t i = tid; i < half && i < n; i += kReuseThreads) {
            k_out[i] = k_in[i];
            v_out[i] = v_in[i];
        }
        return;
    }
    const int64_t base = (kShifted ? half : 0) + (int64_t)blockIdx.x * kReuseBlock;
#pragma unroll
    for (int k = 0; k < kReuseItems; ++k) {
        const int64_t i = base + k * kReuseThreads + tid;
        s[k * kReuseThreads + tid] = i < n ? (((uint64_t)k_in[i] << 32) | v_in[i]) : ~0ull;   // pads sort last
    }
    __syncthreads();
    for (int size = 2; size <= kReuseBlock; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
#pragma unroll
            for (int k = 0; k < kReuseBlock / 2 / kReuseThreads; ++k) {
                const int c = k * kReuseThreads + tid;   // pair index
                const int lo = 2 * stride * (c / stride) + (c % stride), hi = lo + stride;
                const bool up = (lo & size) == 0;
                const uint64_t a = s[lo], b = s[hi];
                if ((a > b) == up) {
                    s[lo] = b;
                    s[hi] = a;
                }
            }
            __syncthreads();
        }
    }
#pragma unroll
    for (int k = 0; k < kReuseItems; ++k) {
        const int64_t i = base + k * kReuseThreads + tid;
        if (i < n) {
            const uint64_t c = s[k * kReuseThreads + tid];
            k_out[i] = (uint32_t)(c >> 32);
            v_out[i] = (uint32_t)c;
        }
    }
}

// After the gather: no descent keeps the order as it is (the previous order
// in vals_b is this frame's order), a few start the repair, more give up.
__global__ __launch_bounds__(1024) void order_plan_kernel(uint32_t* words, const uint32_t* __restrict__ partial,
                                                           int blocks, int64_t n)
{
    // the descents: the gather blocks' counts summed
    __shared__ unsigned long long s_sum[16];
    unsigned long long t = 0;
    for (int b = threadIdx.x; b < blocks; b += 1024) t += partial[b];
    for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
    if ((threadIdx.x & 63) == 0) s_sum[threadIdx.x >> 6] = t;
    __syncthreads();
    if (threadIdx.x != 0) return;
    unsigned long long total = 0;
    for (int w = 0; w < 16; ++w) total += s_sum[w];
    const uint32_t d = (uint32_t)total;   // at most n - 1 < 2^32
    words[1] = d;
    const bool valid = words[0] != 0u;
    const bool repair = valid && d > 0u && (int64_t)d <= n / kRepairFraction;
    words[2] = repair ? 1u : 0u;
    words[0] = (valid && (d == 0u || repair)) ? 1u : 0u;
}

// Clears words[0] at any descent left after the two local sorts.
__global__ __launch_bounds__(256) void order_check_kernel(const uint32_t* __restrict__ k, const uint32_t* __restrict__ v,
                                                          int64_t n, uint32_t* words)
{
    if (!words[2]) return;
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j + 1 < n) {
        const uint64_t a = ((uint64_t)k[j] << 32) | v[j], b = ((uint64_t)k[j + 1] << 32) | v[j + 1];
        if (a > b) words[0] = 0u;
    }
}

// The rectangles in a reused order (see launch_order_pack).
__global__ __launch_bounds__(256) void order_pack_kernel(const uint32_t* __restrict__ order,
                                                         const ushort4* __restrict__ rect, int64_t n,
                                                         const uint32_t* words, uint32_t* __restrict__ pay)
{
    if (!words[0]) return;
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j < n) pay[j] = pack_rect(rect[order[j]]);
}

}  // namespace

hipError_t launch_order_pack(const uint32_t* vals_b, const ushort4* rect, int64_t n, const uint32_t* words,
                             uint32_t* pay_b, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(order_pack_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, vals_b, rect, n, words,
                       pay_b);
    return hipGetLastError();
}

bool depth_sort_items_supported(int items) { return items == 4 || items == 8 || items == 16; }

size_t order_reuse_words(int64_t n) { return (size_t)(kReuseWords + (n + 255) / 256); }

// From here on a sort whose width nobody set takes 16 keys per thread instead
// of 8: a digit's runs are twice as long.  Four passes of 8 and of 16: 74 and 75 us at 500K keys, 89
// and 82 at 1M, 100 and 97 at 1.2M, 180 and 165 at 3M, 699 and 588 at 16M.
constexpr int64_t kWideKeys = 800000;
// Up to here a pass goes without a launch that scans the counts: group sums
// take their place.  Four passes with the scan and with the group sums: 91 and
// 82 us at 1M keys, 123 and 114 at 2M, 170 and 170 at 3M, 268 and 278 at 6M, 610
// and 615 at 16M; and four launches less when the lists of the last frame hold
// (4.4 us each).
constexpr int64_t kGroupedKeys = 2500000;

size_t depth_sort_hist_elems(int64_t n, int n_views)
{
    // the block histograms, and the group sums in less than as much again,
    // sized for the smallest block (the most blocks) any supported width uses
    const int64_t tile = (int64_t)kSortBlock * 4;
    const int64_t bpv = (n + tile - 1) / tile;
    const int64_t V = n_views > 0 ? n_views : 1;
    const int64_t nb = bpv * V;
    const size_t passes = (size_t)(256 * (V + 2 * (nb > 0 ? nb : 1)));
    // few keys: one table per pass
    return fused_sort(n, V) ? std::max(passes, (size_t)(4 * 256 * V * ((n + kFusedThreads - 1) / kFusedThreads))) : passes;
}

// Items per thread that a sort of that many keys takes (items 0: not set).
static int sort_width(int64_t keys, int items) { return items ? items : (keys >= kWideKeys ? 16 : 8); }

size_t depth_sort_clear_words(int64_t n, int n_views, int items)
{
    if (n == 0 || segment_items(n) || fused_sort(n, n_views) || n * n_views > kGroupedKeys) return 0;
    const int64_t tile = (int64_t)kSortBlock * sort_width(n * n_views, items);
    return (size_t)(256 * n_views) * (size_t)sort_groups((int)((n + tile - 1) / tile));
}

hipError_t launch_order_reuse(const uint32_t* keys, uint32_t* keys_a, uint32_t* vals_a, uint32_t* keys_b,
                              uint32_t* vals_b, int64_t n, uint32_t* words, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipError_t e = launch_fill_u32(words, 0u, kReuseWords, s);
    if (e != hipSuccess) return e;
    e = launch_fill_u32(words, 1u, 1, s);
    if (e != hipSuccess) return e;
    const unsigned g256 = (unsigned)((n + 255) / 256);
    // previous order (vals_b) -> (this frame's keys, items) in a
    uint32_t* partial = words + kReuseWords;
    hipLaunchKernelGGL(order_gather_kernel, dim3(g256), dim3(256), 0, s, keys, (const uint32_t*)vals_b, n, keys_a,
                       vals_a, words, partial);
    hipLaunchKernelGGL(order_plan_kernel, dim3(1), dim3(1024), 0, s, words, (const uint32_t*)partial, (int)g256, n);
    const int64_t half = kReuseBlock / 2;
    const unsigned runs = (unsigned)((n + kReuseBlock - 1) / kReuseBlock);
    const unsigned runs_shifted = (unsigned)(n > half ? (n - half + kReuseBlock - 1) / kReuseBlock : 0) + 1u;
    hipLaunchKernelGGL(order_local_sort_kernel<false>, dim3(runs), dim3(kReuseThreads), 0, s, (const uint32_t*)keys_a,
                       (const uint32_t*)vals_a, n, keys_a, vals_a, (const uint32_t*)words);
    hipLaunchKernelGGL(order_local_sort_kernel<true>, dim3(runs_shifted), dim3(kReuseThreads), 0, s,
                       (const uint32_t*)keys_a, (const uint32_t*)vals_a, n, keys_b, vals_b, (const uint32_t*)words);
    hipLaunchKernelGGL(order_check_kernel, dim3(g256), dim3(256), 0, s, (const uint32_t*)keys_b, (const uint32_t*)vals_b,
                       n, words);
    return hipGetLastError();
}

// Sorts each of the n_views segments keys_in[v * n .. (v + 1) * n) (not
// modified) with values v * n + i, items keys per thread of a block (0: by
// their number).  Four
// passes: in -> a -> b -> a -> b, so the sorted values (and payloads) end in
// vals_b (pay_b); the last pass writes no keys.  With reuse_words (one view,
// after launch_order_reuse) every pass reads words[0] on the device and does
// nothing when the reused order holds.
hipError_t launch_depth_sort(const uint32_t* keys_in, uint32_t* keys_a, uint32_t* vals_a, uint32_t* keys_b,
                             uint32_t* vals_b, const ushort4* rect, uint32_t* pay_a, uint32_t* pay_b,
                             uint32_t* counts, int64_t n, int n_views, int items, const uint32_t* reuse_words,
                             hipStream_t s, const PartialSums* sums, hipEvent_t sums_done)
{
    if (n == 0 || n_views <= 0) return hipSuccess;
    items = sort_width(n * n_views, items);
    if (!depth_sort_items_supported(items) || (sums && reuse_words)) return hipErrorInvalidValue;
    const PartialSums no_sums{};
    const int64_t tile = (int64_t)kSortBlock * items;
    const int bpv = (int)((n + tile - 1) / tile);
    const unsigned nblocks = (unsigned)bpv * (unsigned)n_views;
    const uint32_t* kin = keys_in;
    const uint32_t* vin = nullptr;
    const uint32_t* pin = nullptr;   // the first pass packs from rect
    const uint32_t* skip = reuse_words;
    uint32_t* const keys[2] = {keys_a, keys_b};
    uint32_t* const vals[2] = {vals_a, vals_b};
    uint32_t* const pay[2] = {pay_a, pay_b};
    if (const int k = segment_items(n)) {
        const auto launch = k == 1   ? (rect ? launch_segment_sort<1, true> : launch_segment_sort<1, false>)
                            : k == 2 ? (rect ? launch_segment_sort<2, true> : launch_segment_sort<2, false>)
                                     : (rect ? launch_segment_sort<4, true> : launch_segment_sort<4, false>);
        launch(keys_in, vals_b, rect, pay_b, n, n_views, skip, s, sums ? *sums : no_sums, sums_done);
        return hipGetLastError();
    }
    if (fused_sort(n, n_views)) {
        (rect ? launch_fused_sort<true> : launch_fused_sort<false>)(keys_in, keys, vals, rect, pay, counts, n, n_views,
                                                                    skip, s, sums ? *sums : no_sums, sums_done);
        return hipGetLastError();
    }
    for (int pass = 0; pass < 4; ++pass) {
        const int shift = 8 * pass;
        const bool to_b = pass % 2 == 1;
        uint32_t* kout = pass == 3 ? nullptr : (to_b ? keys_b : keys_a);
        uint32_t* vout = to_b ? vals_b : vals_a;
        uint32_t* pout = rect ? (to_b ? pay_b : pay_a) : nullptr;
        const PartialSums& ps = pass == 0 && sums ? *sums : no_sums;
        const hipEvent_t ev = pass == 0 ? sums_done : nullptr;
        const auto pass_of = [&](auto W, auto G) {
            launch_sort_pass<decltype(W)::value, decltype(G)::value>(kin, vin, kout, vout, rect, pin, pout, counts, n,
                                                                     n_views, shift, bpv, nblocks, skip, s, ps, ev);
        };
        const auto grouped = [&](auto W) {
            if (n * n_views <= kGroupedKeys) pass_of(W, std::true_type{});
            else pass_of(W, std::false_type{});
        };
        switch (items) {
        case 4: grouped(std::integral_constant<int, 4>{}); break;
        case 8: grouped(std::integral_constant<int, 8>{}); break;
        default: grouped(std::integral_constant<int, 16>{}); break;
        }
        kin = kout;
        vin = vout;
        pin = pout;
    }
    return hipGetLastError();
}

}  // namespace gsmi
