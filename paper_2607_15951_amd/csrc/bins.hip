// bins.hip -- depth-ordered lists of the Gaussians over bins of up to 8x8
// screen tiles, which the blend walks.
//
// Every (Gaussian, tile) pair of Sec. 3.1 belongs to its tile's list, but a
// tile's pixels stop after a small part of it (at 3M Gaussians and 1080p the
// blend reads 6.5M of 236M pairs), so writing the per-tile lists cost more
// than reading them: 0.41 of a 1.03 ms frame.  The render therefore lists the
// Gaussians per bin of 1x1 to 8x8 tiles, each with the part of the bin its
// rectangle covers, and the blend picks its tile's entries out of the bin's
// list in order (blend_stage.h): the same entries at the same list positions.
// Binning and blend, per-tile lists and bins: 640 and 325 us of that frame;
// 3400 and 1250 us at 6M Gaussians and 3840x2160; 310 and 310 us for 2M small
// ones at 1080p (7.6 tiles a rectangle), whose frame takes as long as before.
// The per-tile lists themselves are written by tile_bin.hip when a caller
// asks for them.
//
// One workgroup takes a chunk of depth-sorted Gaussians of one view, each of
// its waves a consecutive part of it:
//   count    a 2D difference array over the view's bins in LDS (four atomics
//            per Gaussian whatever its size), summed to counts[bin][chunk];
//   scan     one device-wide exclusive scan: each chunk's cursor in each bin;
//   scatter  the waves count their own parts in the same way to get cursors
//            of their own; then each goes through its Gaussians 64 at a time.
//            Small ones: their (Gaussian, bin) entries are dealt out evenly
//            to the lanes, 64 at a time in order, and every entry goes to its
//            bin's cursor plus its rank among the window's entries of that
//            bin.  Large ones (most of them in most bins of their common
//            rectangle): bin by bin, a ballot of the Gaussians that touch it.
//            Either way each bin's list keeps the depth order.
// Grids of more bins than the waves' cursors fit in LDS are cut into bands of
// bin rows, and a workgroup takes one band of its chunk.
#include "gs_internal.h"

#include <type_traits>

namespace gsmi {
namespace {

// Bin grids whose cursors (12 bytes per bin and wave) a workgroup of kWaves
// waves keeps in LDS: up to 1080p at 4x4 tiles a bin and 4K at 8x8.  Larger
// grids are cut into bands of at most kBandBins bins (two workgroups a CU with
// the long rounds below), each workgroup going through its chunk's Gaussians
// for the part of them in its band.  One wave a chunk with its cursors in LDS
// up to 4096 bins, in the count table beyond, took 2.6 ms of scatter where the
// bands take 0.45 (1M Gaussians, 7680x4320), 41 where they take 0.26 (1M,
// 9216x9216) and 168 where they take 0.39 (100K, 16384x16384).
constexpr int kWaves = 4;
constexpr int kMaxBins = 768, kBandBins = 608;

// Entries that a round of the scatter stages in LDS, and its Gaussians, as
// multiples of these.  Twice as many where the bins are at their largest (so
// Gaussians take several each) and more than kLongBins: eight entries a bin and
// round are runs of half a cache line; but it leaves three workgroups a CU where
// there were five, two where there were three or four, and past 636 bins one
// where there were two.  Bins of
// 8x8 tiles, with 1M, 3M and 6M Gaussians of the power-law scene, once and
// twice as many, us:
//   135 bins  33  45 |  75  77 | 146 145      432 bins 100  75 | 192 177 | 398 352
//   240       46  74 | 101 123 | 199 232      510      116  88 | 227 213 | 509 420
//   260       50  79 | 108 129 | 211 246      570      222 171 | 300 228 | 609 447
//   299       81  62 | 153 137 | 302 268      627      318 217 | 357 253 | 751 507
//   375       92  69 | 176 160 | 358 309      680      369 233 | 387 479 | 803 964
// The line was drawn from 135 and 510 alone; by these it could lie at 280, and
// past 636 bins 1M Gaussians still gain and more lose.
// 510 bins of 4x4 tiles (2M small ones at 1080p): 72 and 94.
constexpr int kStage0 = 4096, kRoundItems0 = 512;
constexpr int kLongBins = 384;
static_assert(kBandBins >= ((kMaxBandTiles - 1) >> 3) + 1, "a band holds a row of bins of 8x8 tiles");
static_assert(kWaves * kMaxBins <= kStage0, "one Gaussian per wave fits a round");
static_assert(kMaxBins <= 1024 && 2 * kRoundItems0 <= 1024, "staged words hold 10 bits of each");

// A batch of 64 items goes bin by bin when each bin of its common rectangle
// is touched by more than this many of them on average.
constexpr uint32_t kDense = 24;

// LDS words that the lanes of one wave pass to each other.  Relaxed atomics
// keep every access in program order; a volatile access would also wait for
// the wave's global stores (1100 instead of about 100 cycles a step).
template <typename T>
__device__ __forceinline__ T lds_get(const T* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}
template <typename T>
__device__ __forceinline__ void lds_set(T* p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}

// Lane i receives the value of the DPP source lane, or 0 without one.
template <int kCtrl, int kRowMask>
__device__ __forceinline__ uint32_t dpp0(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, kCtrl, kRowMask, 0xF, false);
}

// Inclusive sum and maximum over the lanes up to this one: shifts by 1, 2, 4
// and 8 within rows of 16 lanes, then the rows' last lanes broadcast on.
__device__ __forceinline__ uint32_t wave_sum_scan(uint32_t x)
{
    x += dpp0<0x111, 0xF>(x);
    x += dpp0<0x112, 0xF>(x);
    x += dpp0<0x114, 0xF>(x);
    x += dpp0<0x118, 0xF>(x);
    x += dpp0<0x142, 0xA>(x);
    x += dpp0<0x143, 0xC>(x);
    return x;
}
__device__ __forceinline__ uint32_t wave_max_scan(uint32_t x)
{
    x = max(x, dpp0<0x111, 0xF>(x));
    x = max(x, dpp0<0x112, 0xF>(x));
    x = max(x, dpp0<0x114, 0xF>(x));
    x = max(x, dpp0<0x118, 0xF>(x));
    x = max(x, dpp0<0x142, 0xA>(x));
    x = max(x, dpp0<0x143, 0xC>(x));
    return x;
}

// Workgroup b -> chunk: block b runs on XCD b % 8, and each XCD takes every
// eighth group of kGroup consecutive chunks, whose output pieces are adjacent.
// (One contiguous run of chunks per XCD left one XCD with the far background,
// a tenth of the Gaussians of the 3M workload but two thirds of its entries.)
constexpr int kGroup = 4;
__device__ __forceinline__ int chunk_of_block()
{
    const int x = (int)(blockIdx.x & 7), j = (int)(blockIdx.x >> 3);
    return (j / kGroup * 8 + x) * kGroup + j % kGroup;
}

// Chunk c: view c / chunks1, part c % chunks1 of its keyed items (which open
// its segment of the depth order; those culled or off screen have an empty
// rectangle).  Returns false past the last view.
struct Chunk {
    int view, part;
    int64_t start, end;   // positions in the depth order
};
__device__ __forceinline__ bool chunk_range(const BinArgs& a, int c, Chunk& k)
{
    k.view = c / a.chunks1;
    k.part = a.chunks1 - 1 - c % a.chunks1;
    if (k.view >= a.n_views) return false;
    const int64_t seg = (int64_t)k.view * a.n, size = (int64_t)a.chunk;
    k.start = seg + (int64_t)k.part * size;
    const int64_t keyed = seg + (int64_t)a.view_counts[(int64_t)kViewCounters * k.view + 1];
    k.end = k.start + size < keyed ? k.start + size : keyed;
    return true;
}

// Rectangle of the item at position k of the depth order: x0 | x1 << 16 and
// y0 | y1 << 16 (tiles, exclusive ends); empty ones have x1 = 0.
__device__ __forceinline__ uint2 rect_words(ushort4 r)
{
    return make_uint2((uint32_t)r.x | ((uint32_t)r.z << 16), (uint32_t)r.y | ((uint32_t)r.w << 16));
}

// First bin and number of bins that tiles [lo, hi) of a row or column touch.
__device__ __forceinline__ void bin_span(uint32_t w, int shift, uint32_t& b0, uint32_t& nb)
{
    const uint32_t lo = w & 0xFFFFu, hi = w >> 16;
    b0 = lo >> shift;
    nb = hi ? ((hi - 1u) >> shift) - b0 + 1u : 0u;
}

// The entry's part of bin b along one axis: how far its tiles [lo, hi) stay
// clear of the bin's first and last tile, 0..7 each.
__device__ __forceinline__ void clip_span(uint32_t w, uint32_t b, int shift, uint32_t& at_first, uint32_t& at_last)
{
    const int lo = (int)(w & 0xFFFFu), hi = (int)(w >> 16), t0 = (int)(b << shift);
    at_first = (uint32_t)max(lo - t0, 0);
    at_last = (uint32_t)max(t0 + (1 << shift) - hi, 0);
}

// Bands of a grid of bins_x by bins_y bins, and the bin rows of each (the
// last one's may be fewer).
__host__ __device__ __forceinline__ int bin_bands(int bins_x, int bins_y)
{
    if (bins_x * bins_y <= kMaxBins) return 1;
    const int most = kBandBins / bins_x;
    return (bins_y + most - 1) / most;
}
__host__ __device__ __forceinline__ int band_rows(int bins_x, int bins_y)
{
    const int bands = bin_bands(bins_x, bins_y);
    return (bins_y + bands - 1) / bands;
}

// The rows of a view's bins that a workgroup takes: [y0, y0 + rows).
struct Band {
    int y0, rows;
};
template <bool kBanded>
__device__ __forceinline__ Band band_of_block(const ViewParams& vp)
{
    if constexpr (!kBanded) return {0, vp.bins_y};
    const int rows = band_rows(vp.bins_x, vp.bins_y), y0 = (int)blockIdx.y * rows;
    return {y0, min(rows, vp.bins_y - y0)};   // none past the view's last band
}

// The bins of one item, [bx0, bx0 + nbx) x [by0, by0 + nby), of a band with the
// rows counted from its first; none for an empty rectangle.
template <bool kBanded>
struct BinRect {
    uint32_t bx0, nbx, by0, nby;
    __device__ __forceinline__ BinRect(uint2 w, int shift, Band band)
    {
        bin_span(w.x, shift, bx0, nbx);
        bin_span(w.y, shift, by0, nby);
        if constexpr (kBanded) {
            const int lo = max((int)by0 - band.y0, 0), hi = min((int)(by0 + nby) - band.y0, band.rows);
            by0 = hi > lo ? (uint32_t)lo : 0u;
            nby = hi > lo ? (uint32_t)(hi - lo) : 0u;
            nbx = hi > lo ? nbx : 0u;
        }
    }
};

// Adds the item to a difference array over the grid, `wide` words a row.
template <bool kBanded>
__device__ __forceinline__ void diff_add(uint32_t* diff, int wide, const BinRect<kBanded>& r)
{
    if (r.nbx) {
        uint32_t* p = diff + r.by0 * wide + r.bx0;
        uint32_t* q = p + r.nby * wide;
        atomicAdd(p, 1u);
        atomicSub(p + r.nbx, 1u);
        atomicSub(q, 1u);
        atomicAdd(q + r.nbx, 1u);
    }
}

// diff[(by + 1) * wide] to counts in place (row y of the grid at y * wide),
// by one wave: down the columns, then along the rows.  Every row of
// differences sums to zero over its bins_x + 1 words, so one running sum over
// the whole grid restarts by itself at each row.
__device__ __forceinline__ void diff_sum(uint32_t* diff, int wide, int by, int lane)
{
    for (int x = lane; x < wide; x += 64) {
        uint32_t run = 0u;
        for (int y = 0; y < by; ++y) {
            run += diff[y * wide + x];
            diff[y * wide + x] = run;
        }
    }
    __builtin_amdgcn_wave_barrier();
    const int m = wide * by, per = (m + 63) / 64;
    const int b = lane * per, e = b + per < m ? b + per : m;
    uint32_t s = 0u;
    for (int i = b; i < e; ++i) s += diff[i];
    uint32_t run = wave_sum_scan(s) - s;
    for (int i = b; i < e; ++i) {
        run += diff[i];
        diff[i] = run;
    }
    __builtin_amdgcn_wave_barrier();
}

// Rectangle words of the items at k0 + 64 b + lane, b < kItems, empty past
// end; every load is issued before any is used (a load under its own branch
// is waited for before the next one issues).
template <int kItems>
__device__ __forceinline__ void load_rects(const BinArgs& a, int64_t k0, int64_t end, int lane, uint2 (&w)[kItems])
{
    if (a.sorted_pack) {
        uint32_t pk[kItems];
#pragma unroll
        for (int b = 0; b < kItems; ++b) {
            const int64_t k = k0 + b * 64 + lane;
            pk[b] = a.sorted_pack[k < end ? k : k0];
        }
#pragma unroll
        for (int b = 0; b < kItems; ++b) w[b] = rect_words(unpack_rect(pk[b]));
    } else {
        ushort4 r[kItems];
#pragma unroll
        for (int b = 0; b < kItems; ++b) {
            const int64_t k = k0 + b * 64 + lane;
            r[b] = a.sorted_rect[k < end ? k : k0];
        }
#pragma unroll
        for (int b = 0; b < kItems; ++b) w[b] = rect_words(r[b]);
    }
#pragma unroll
    for (int b = 0; b < kItems; ++b)
        if (k0 + b * 64 + lane >= end) w[b] = make_uint2(0u, 0u);
}

// The (Gaussian, bin) entries of a batch of 64 items in order, dealt to the
// lanes 64 at a time (a window).
struct Entry {
    uint32_t owner, bin;   // lane of the item, bin of the view
};
struct EntryWalk {
    uint32_t first, span;   // the lane's first entry; its bins bx0 | by0 << 10 | nbx << 20
    uint32_t total;         // of the batch (uniform)
    uint32_t carry;         // owner + 1 of the entry before the next window (uniform)
    bool some;

    template <bool kBanded>
    __device__ __forceinline__ EntryWalk(const BinRect<kBanded>& r)
    {
        const uint32_t cnt = r.nbx * r.nby, incl = wave_sum_scan(cnt);
        first = incl - cnt;
        span = r.bx0 | (r.by0 << 10) | (r.nbx << 20);
        some = cnt != 0u;
        total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        carry = 0u;
    }

    // The lane's entry of the window at e0 (meaningful below total).  flag:
    // 64 words of LDS of the wave's, zero between calls.
    __device__ __forceinline__ Entry window(uint32_t e0, int bx, int lane, uint32_t* flag)
    {
        // the items that start in this window mark their first entry; the
        // owner of an entry is the last mark at or before it
        if (some && first - e0 < 64u) lds_set(flag + (first - e0), (uint32_t)lane + 1u);
        __builtin_amdgcn_wave_barrier();
        uint32_t o = lds_get(flag + lane);
        lds_set(flag + lane, 0u);
        __builtin_amdgcn_wave_barrier();
        o = max(wave_max_scan(o), carry);
        carry = (uint32_t)__builtin_amdgcn_readlane((int)o, 63);
        Entry en;
        en.owner = o - 1u;
        const uint32_t sp = (uint32_t)__shfl((int)span, (int)en.owner, 64);
        const uint32_t k = e0 + (uint32_t)lane - (uint32_t)__shfl((int)first, (int)en.owner, 64);
        // k / nbx for k < 2^16: the quotient of k + 1/2 stays 1 / (2 nbx)
        // clear of the next integer, far above the float rounding
        const uint32_t nbx = sp >> 20;
        const uint32_t row = (uint32_t)(((float)k + 0.5f) * __builtin_amdgcn_rcpf((float)nbx));
        en.bin = (((sp >> 10) & 1023u) + row) * (uint32_t)bx + (sp & 1023u) + (k - row * nbx);
        return en;
    }
};

// Smallest value of a wave's lanes (uniform).
__device__ __forceinline__ uint32_t wave_min(uint32_t v)
{
    for (int o = 32; o > 0; o >>= 1) v = min(v, (uint32_t)__shfl_xor((int)v, o, 64));
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}

// Gathers the rectangles of grids too large to pack in depth order.
__global__ __launch_bounds__(256) void bins_gather_kernel(BinArgs a)
{
    if (a.skip && *a.skip) return;   // the last render's lists hold
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k < a.n * a.n_views) a.sorted_rect[k] = a.rect[a.sorted_idx[k]];
}

// counts[bin][chunk] of one chunk, for the bins of one band.
template <int kItems, bool kBanded>
__global__ __launch_bounds__(64 * kWaves) void bins_count_kernel(BinArgs a)
{
    if (a.skip && *a.skip) return;   // the last render's lists hold
    extern __shared__ uint32_t s_diff[];   // [rows + 1][bins_x + 1] of the largest band
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    Chunk ck;
    if (!chunk_range(a, chunk_of_block(), ck)) return;
    const ViewParams& vp = a.views[ck.view];
    const Band band = band_of_block<kBanded>(vp);
    if (kBanded && band.rows <= 0) return;
    const int bx = vp.bins_x, by = band.rows, wide = bx + 1, shift = vp.bin_shift;
    uint32_t* counts = a.table + ((int64_t)vp.bin_base + (int64_t)band.y0 * bx) * a.chunks1 + ck.part;
    for (int i = tid; i < wide * (by + 1); i += 64 * kWaves) s_diff[i] = 0u;
    __syncthreads();
    for (int64_t k0 = ck.start + wave * (kItems * 64); k0 < ck.end; k0 += kWaves * kItems * 64) {
        uint2 w[kItems];
        load_rects(a, k0, ck.end, lane, w);
#pragma unroll
        for (int b = 0; b < kItems; ++b) diff_add(s_diff, wide, BinRect<kBanded>(w[b], shift, band));
    }
    __syncthreads();
    if (wave == 0) diff_sum(s_diff, wide, by, lane);
    __syncthreads();
    for (int i = tid; i < bx * by; i += 64 * kWaves) counts[(int64_t)i * a.chunks1] = s_diff[i / bx * wide + i % bx];
}

// Span word of the blend: the part of bin (ex, ey) that the rectangle w covers.
__device__ __forceinline__ uint16_t span_word(uint2 w, uint32_t ex, uint32_t ey, int shift)
{
    uint32_t x0, x1, y0, y1;
    clip_span(w.x, ex, shift, x0, x1);
    clip_span(w.y, ey, shift, y0, y1);
    return (uint16_t)(x0 | (y0 << 4) | (x1 << 8) | (y1 << 12));
}

// Row of bin `bin` in a grid bx wide (both below 2^16), as in EntryWalk.
__device__ __forceinline__ uint32_t bin_row(uint32_t bin, float inv_bx)
{
    return (uint32_t)(((float)bin + 0.5f) * inv_bx);
}

// Positions of a batch's entries by the wave's cursors cur[bin], handed to
// put(position, lane of the item, bin) by the lanes that hold one; the
// cursors move on.  mask: a word per bin, zero between calls.
template <bool kBanded, typename Put>
__device__ __forceinline__ void place_batch(const BinRect<kBanded>& r, int bx, int lane, uint64_t lt, uint32_t* flag,
                                            uint64_t* mask, uint32_t* cur, Put put)
{
    EntryWalk ew(r);
    // bin by bin where the items touch most bins of their common rectangle: a
    // bin takes about a third of a window's issue and no LDS round trip
    if (ew.total > 64u * kDense) {
        const uint32_t xa = wave_min(r.nbx ? r.bx0 : 0xFFFFu), ya = wave_min(r.nby ? r.by0 : 0xFFFFu);
        const uint32_t xb = 0xFFFFu - wave_min(r.nbx ? 0xFFFFu - (r.bx0 + r.nbx) : 0xFFFFu);
        const uint32_t yb = 0xFFFFu - wave_min(r.nby ? 0xFFFFu - (r.by0 + r.nby) : 0xFFFFu);
        if (ew.total > kDense * (xb - xa) * (yb - ya)) {
            for (uint32_t y = ya; y < yb; ++y) {
                const bool in_row = y - r.by0 < r.nby;
                // 64 columns at a time, their cursors in the lanes
                for (uint32_t x64 = xa; x64 < xb; x64 += 64) {
                    const uint32_t row = y * (uint32_t)bx + x64, cols = min(xb - x64, 64u);
                    uint32_t c64 = (uint32_t)lane < cols ? lds_get(cur + row + lane) : 0u;
                    for (uint32_t q = 0; q < cols; ++q) {
                        const bool on = in_row && x64 + q - r.bx0 < r.nbx;
                        const uint64_t m = __ballot(on);
                        const uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)c64, (int)q);
                        if (on)
                            put(__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, c)),
                                (uint32_t)lane, row + q);
                        if ((uint32_t)lane == q) c64 = c + (uint32_t)__popcll(m);
                    }
                    if ((uint32_t)lane < cols) lds_set(cur + row + lane, c64);
                    __builtin_amdgcn_wave_barrier();
                }
            }
            return;
        }
    }
    if (ew.total == 0u) return;
    Entry e = ew.window(0u, bx, lane, flag);
    for (uint32_t e0 = 0; e0 < ew.total; e0 += 64) {
        const bool on = e0 + (uint32_t)lane < ew.total;
        // a wave's LDS operations take effect in order: every lane's bit is
        // in before any lane reads the mask
        uint64_t m = 0;
        uint32_t c = 0;
        if (on) {
            (void)__hip_atomic_fetch_or(mask + e.bin, (uint64_t)1 << lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
            __builtin_amdgcn_wave_barrier();
            m = lds_get(mask + e.bin);
            c = lds_get(cur + e.bin);
        }
        // the next window's entries while those reads are under way
        const Entry now = e;
        if (e0 + 64 < ew.total) e = ew.window(e0 + 64, bx, lane, flag);
        if (on) {
            const uint32_t pos = c + (uint32_t)__popcll(m & lt);
            if ((m >> lane) == 1ull) {   // the bin's last lane of the window moves the cursor on
                lds_set(cur + now.bin, pos + 1u);
                lds_set(mask + now.bin, (uint64_t)0);
            }
            put(pos, now.owner, now.bin);
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// The chunk's entries of one band to their places.  The chunk is taken in rounds of at most kStage entries
// that are put in bin order in LDS and written from there, consecutive lanes
// on consecutive places of a bin's list: written from the windows, every
// entry had a cache line of its own, and those partial-line stores bound the
// kernel (10M entries in 0.12 ms, 46M in 0.75 ms).  A round is 4 p
// consecutive Gaussians, p per wave; p halves while they do not fit and
// doubles while they would.
template <int kTimes, bool kBanded = false>
__global__ __launch_bounds__(64 * kWaves) void bins_scatter_kernel(BinArgs a)
{
    constexpr int kStage = kTimes * kStage0, kRoundItems = kTimes * kRoundItems0;
    if (a.skip && *a.skip) return;   // the last render's lists hold
    // each wave's masks (whose bytes first hold its difference array), each
    // wave's cursors, then each bin's place in its list
    extern __shared__ uint64_t s_dyn[];
    __shared__ uint32_t s_flag[kWaves][64];
    __shared__ uint32_t s_stage[kStage];   // item of the round | bin << 10
    __shared__ uint32_t s_item[kRoundItems];
    __shared__ uint2 s_rect[kRoundItems];
    __shared__ uint32_t s_sum[kWaves];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    Chunk ck;
    if (!chunk_range(a, chunk_of_block(), ck)) return;
    if (ck.start >= ck.end) return;
    const ViewParams& vp = a.views[ck.view];
    const Band band = band_of_block<kBanded>(vp);
    if (kBanded && band.rows <= 0) return;
    const int bx = vp.bins_x, by = band.rows, bins = bx * by, shift = vp.bin_shift, wide = bx + 1;
    const uint32_t* counts = a.table + ((int64_t)vp.bin_base + (int64_t)band.y0 * bx) * a.chunks1 + ck.part;
    uint64_t* mask = s_dyn + (int64_t)wave * a.lds_mask;
    uint32_t* diff = reinterpret_cast<uint32_t*>(mask);
    uint32_t* all = reinterpret_cast<uint32_t*>(s_dyn + (int64_t)kWaves * a.lds_mask);
    uint32_t* cur = all + wave * bins;
    uint32_t* base = all + kWaves * bins;
    uint32_t* flag = s_flag[wave];
    flag[lane] = 0u;
    for (int i = tid; i < bins; i += 64 * kWaves) base[i] = counts[(int64_t)i * a.chunks1];
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const float inv_bx = 1.0f / (float)bx;
    int p = min(a.chunk / kWaves, kRoundItems / kWaves);
    for (int64_t pos = ck.start; pos < ck.end;) {
        // the wave's items: batches of 64, or the first p lanes of one
        constexpr int kB = kRoundItems / kWaves / 64;
        uint2 w[kB];
        uint32_t g[kB], sum = 0u;
        const int64_t lo = pos + (int64_t)wave * p, hi = min(lo + p, ck.end);
#pragma unroll
        for (int b = 0; b < kB; ++b) {
            const int64_t k = lo + b * 64 + lane;
            const bool in = k < hi;
            w[b] = make_uint2(0u, 0u);
            g[b] = 0u;
            if (b * 64 < p) {   // uniform
                const int64_t kc = in ? k : ck.start;
                w[b] = a.sorted_pack ? rect_words(unpack_rect(a.sorted_pack[kc])) : rect_words(a.sorted_rect[kc]);
                g[b] = a.sorted_idx[kc];
                if (!in) w[b] = make_uint2(0u, 0u);
            }
            const BinRect<kBanded> r(w[b], shift, band);
            sum += r.nbx * r.nby;
        }
        const uint32_t incl = wave_sum_scan(sum);
        if (lane == 63) s_sum[wave] = incl;
        __syncthreads();
        const uint32_t total = s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3];
        if (kBanded && total == 0u) {   // uniform: nothing of these in the band
            pos += (int64_t)kWaves * p;
            if (p < kRoundItems / kWaves) p *= 2;
            __syncthreads();   // s_sum is written again
            continue;
        }
        if (total > (uint32_t)kStage) {   // uniform; p = 1 fits, 4 kMaxBins <= kStage
            p /= 2;
            __syncthreads();   // s_sum is written again
            continue;
        }
        // the waves' counts of each bin
        for (int i = lane; i < wide * (by + 1); i += 64) diff[i] = 0u;
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int b = 0; b < kB; ++b) {
            if (b * 64 >= p) break;
            diff_add(diff, wide, BinRect<kBanded>(w[b], shift, band));
            if (b * 64 + lane < p) {
                s_item[wave * p + b * 64 + lane] = g[b];
                s_rect[wave * p + b * 64 + lane] = w[b];
            }
        }
        __builtin_amdgcn_wave_barrier();
        diff_sum(diff, wide, by, lane);
        __syncthreads();
        // to cursors within the round's part of each bin, and its length
        for (int i = tid; i < bins; i += 64 * kWaves) {
            uint32_t run = 0u;
            const int at = i / bx * wide + i % bx;
#pragma unroll
            for (int v = 0; v < kWaves; ++v) {
                all[v * bins + i] = run;
                run += reinterpret_cast<uint32_t*>(s_dyn + (int64_t)v * a.lds_mask)[at];
            }
            base[bins + i] = run;
        }
        __syncthreads();
        // bin after bin: staged places; base becomes place in the list minus staged place
        if (wave == 0) {
            const int per = (bins + 63) / 64, i0 = lane * per, i1 = min(i0 + per, bins);
            uint32_t s = 0u;
            for (int i = i0; i < i1; ++i) s += base[bins + i];
            uint32_t run = wave_sum_scan(s) - s;
            for (int i = i0; i < i1; ++i) {
                const uint32_t len = base[bins + i];
#pragma unroll
                for (int v = 0; v < kWaves; ++v) all[v * bins + i] += run;
                base[i] -= run;
                base[bins + i] = run + len;   // undone below: the next round's place
                run += len;
            }
        }
        for (int i = lane; i < bins; i += 64) mask[i] = 0ull;
        __syncthreads();
#pragma unroll
        for (int b = 0; b < kB; ++b) {
            if (b * 64 >= p) break;
            const uint32_t first = (uint32_t)(wave * p + b * 64);
            place_batch(BinRect<kBanded>(w[b], shift, band), bx, lane, lt, flag, mask, cur,
                        [&](uint32_t at, uint32_t owner, uint32_t bin) { s_stage[at] = (first + owner) | (bin << 10); });
        }
        __syncthreads();
        for (uint32_t i = tid; i < total; i += 64 * kWaves) {
            const uint32_t e = s_stage[i], bin = e >> 10, k = e & 1023u, at = base[bin] + i;
            const uint32_t ey = bin_row(bin, inv_bx);
            if ((uint64_t)at < a.capacity) {
                a.items[at] = s_item[k];
                a.spans[at] = span_word(s_rect[k], bin - ey * (uint32_t)bx, ey + (uint32_t)band.y0, shift);
            }
        }
        __syncthreads();
        for (int i = tid; i < bins; i += 64 * kWaves) base[i] += base[bins + i];
        pos += (int64_t)kWaves * p;
        if (total <= (uint32_t)kStage / 3 && p < kRoundItems / kWaves) p *= 2;
    }
}

unsigned grid_of(int64_t chunks)
{
    constexpr int64_t all = 8 * kGroup;
    return (unsigned)((chunks + all - 1) / all * all);
}

// f with the items per lane of the count and whether the grids are cut in bands.
template <typename F>
void with_shape(const BinArgs& a, F f)
{
    auto items = [&](auto B) {
        switch (a.items1) {
        case 1: f(std::integral_constant<int, 1>{}, B); break;
        case 2: f(std::integral_constant<int, 2>{}, B); break;
        case 4: f(std::integral_constant<int, 4>{}, B); break;
        default: f(std::integral_constant<int, 8>{}, B); break;
        }
    };
    if (a.bands > 1) items(std::true_type{});
    else items(std::false_type{});
}

}  // namespace

// Tiles per bin edge (log2): about the edge of a Gaussian's rectangle in
// tiles (footprint: tiles per rectangle).  Smaller bins hold each Gaussian
// more often, larger ones make the blend pass over more entries of other
// tiles: with bins of 4x4 and 8x8 tiles the scatter and the blend took 232 +
// 208 and 75 + 223 us at 85 tiles a rectangle (3M, 1080p), 76 + 204 and 39 +
// 279 us at 7.6 (2M).  Not yet known, the footprint is taken from the resolution it grows
// with (85 tiles in the 3M workload at 1080p).
int bin_shift_of(int tiles_x, int tiles_y, float footprint)
{
    if (!(footprint > 0.f)) {
        const float edge = (float)std::max(tiles_x, tiles_y) / 13.f;
        footprint = edge * edge;
    }
    int shift = footprint >= 24.f ? 3 : (footprint >= 6.f ? 2 : (footprint >= 2.f ? 1 : 0));
    while (shift < 3 && (((tiles_x - 1) >> shift) + 1) * (((tiles_y - 1) >> shift) + 1) > kMaxBins) ++shift;
    return shift;
}

// Shape of the chunks: items per lane and rounds of a wave.  As few as keep
// the count table (bins x chunks words) at about one word per (view,
// Gaussian): a wave works through its 64-Gaussian batches one after another.
// The tuned width (8 the default) scales it.
constexpr int64_t kFullWaves = 16384, kTableSlack = 16384;
void bins_chunk_shape(int64_t n, int n_views, int64_t bins, int tuned, int* items1, int* chunk, int* chunks1)
{
    auto chunks = [&](int batches) {
        const int64_t size = (int64_t)batches * 64 * kWaves;
        return std::max<int64_t>((n + size - 1) / size, 1);
    };
    auto fits = [&](int batches) { return chunks(batches) == 1 || bins * chunks(batches) <= n * n_views + kTableSlack; };
    int batches = 1;   // per wave
    while (batches < 8 && n * n_views / (64 * batches) > kFullWaves) batches *= 2;
    while (!fits(batches)) batches *= 2;
    if (tuned > 8) batches *= 2;
    else if (tuned < 8 && batches > 1) batches /= 2;
    *items1 = std::min(batches, 8);
    *chunk = batches * 64 * kWaves;
    *chunks1 = (int)chunks(batches);
}

// Most count table words (bins x chunks) that bins_chunk_shape leaves for any
// bins up to that many: what fits, or a chunk a view; twice that at half the
// chunk size.
int64_t bins_count_bound(int64_t n, int n_views, int64_t bins, int tuned)
{
    return std::max<int64_t>(n * n_views + kTableSlack, bins) * (tuned < 8 ? 2 : 1);
}

BandShape bins_band_shape(int bins_x, int bins_y)
{
    const int rows = band_rows(bins_x, bins_y);
    return {bin_bands(bins_x, bins_y), rows * bins_x, (rows + 1) * (bins_x + 1)};
}

hipError_t launch_bins_count(const BinArgs& a, uint64_t* scan_scratch, hipStream_t s)
{
    const int64_t elems = a.bins * a.chunks1;
    if (a.n == 0) return launch_fill_u32(a.table, 0u, elems + 1, s);
    if (!a.sorted_pack)
        hipLaunchKernelGGL(bins_gather_kernel, dim3((unsigned)((a.n * a.n_views + 255) / 256)), dim3(256), 0, s, a);
    const dim3 grid(grid_of((int64_t)a.chunks1 * a.n_views), (unsigned)a.bands);
    with_shape(a, [&](auto I, auto B) {
        hipLaunchKernelGGL((bins_count_kernel<decltype(I)::value, decltype(B)::value>), grid, dim3(64 * kWaves),
                           (size_t)a.max_diff * sizeof(uint32_t), s, a);
    });
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_scan_exclusive(a.table, elems, scan_scratch, nullptr, a.table + elems, a.overflow, s, nullptr,
                                 a.skip);
}

hipError_t launch_bins_scatter(const BinArgs& a0, hipStream_t s)
{
    if (a0.n == 0) return hipSuccess;
    BinArgs a = a0;
    // 8-byte words of a wave's masks, which also hold its difference array
    a.lds_mask = std::max(a.max_bins, (a.max_diff + 1) / 2);
    const bool wide_rounds = a.min_shift == 3 && a.max_bins > kLongBins;
    const auto kernel = a.bands > 1 ? (wide_rounds ? bins_scatter_kernel<2, true> : bins_scatter_kernel<1, true>)
                                    : (wide_rounds ? bins_scatter_kernel<2> : bins_scatter_kernel<1>);
    hipLaunchKernelGGL(kernel, dim3(grid_of((int64_t)a.chunks1 * a.n_views), (unsigned)a.bands), dim3(64 * kWaves),
                       (size_t)kWaves * a.lds_mask * 8 + (size_t)(kWaves + 2) * a.max_bins * 4, s, a);
    return hipGetLastError();
}

}  // namespace gsmi
