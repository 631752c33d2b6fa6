// blend_stage.h -- staging of one list entry for the per-tile blend, shared
// by the forward (blend.hip) and backward (blend_backward.hip) kernels so that both
// see the same per-entry values and take the same inclusion decisions.
#pragma once

#include "gs_internal.h"

namespace gsmi {

constexpr float kLog2e = 1.4426950408889634f;

// The 4-bit mask of the tile's 8x8 quads in which the quadratic form
// A x^2 + 2 B x y + C y^2 (positive definite) of the offset from pixel to
// centre, (du, dv) minus the pixel, gets as small as limit.  The form is convex
// with its minimum at the origin, so over a quad's box of offsets it is least
// on an edge that faces the origin: the line x = xe or y = ye, where xe and ye
// are 0 clamped to the box (and 0 itself inside it).  On a line it is a 1D
// quadratic minimised in closed form, at y = -(B / C) x or x = -(B / A) y (bc =
// B / C and ba = B / A, computed once per entry: the rounding of the minimiser
// moves the value by a term quadratic in that rounding, far inside the
// margin).  The margin: 1e-5 of a bound on the size of the form's terms over
// the tile (2 |B x y| <= |B| (x^2 + y^2)), which covers the float rounding of
// every evaluation.  Two columns and two rows share their lines' terms, so the
// four quads take 75 vector instructions, where all four edges of each box and
// a test for the origin took about 200 of the 380 that stage 64 entries: the
// blend of 1M Gaussians at 1080p went from 216 to 203 us, of 6M at 3840x2160
// from 786 to 743, the 3M backward from 536 to 531.
__device__ __forceinline__ uint32_t quads_within(float du, float dv, float A, float B, float C, float bc, float ba,
                                                 float limit)
{
    const float xlo[2] = {du - 7.0f, du - 15.0f}, xhi[2] = {du, du - 8.0f};
    const float ylo[2] = {dv - 7.0f, dv - 15.0f}, yhi[2] = {dv, dv - 8.0f};
    const float ab = fabsf(B), B2 = 2.0f * B;
    const float S = (A + ab) * fmaxf(xhi[0] * xhi[0], xlo[1] * xlo[1]) +
                    (C + ab) * fmaxf(yhi[0] * yhi[0], ylo[1] * ylo[1]);
    const float most = limit + 1e-5f * (S + 1.0f);
    float fx[2], gx[2], my[2], fy[2], gy[2], mx[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const float xe = __builtin_amdgcn_fmed3f(0.0f, xlo[k], xhi[k]), ye = __builtin_amdgcn_fmed3f(0.0f, ylo[k], yhi[k]);
        fx[k] = A * xe * xe;   // on the line x = xe: fx + y (gx + C y), least at my
        gx[k] = B2 * xe;
        my[k] = -bc * xe;
        fy[k] = C * ye * ye;
        gy[k] = B2 * ye;
        mx[k] = -ba * ye;
    }
    uint32_t mask = 0u;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int c = q & 1, r = q >> 1;
        const float y = __builtin_amdgcn_fmed3f(my[c], ylo[r], yhi[r]), x = __builtin_amdgcn_fmed3f(mx[r], xlo[c], xhi[c]);
        const float f = fminf(fmaf(fmaf(C, y, gx[c]), y, fx[c]), fmaf(fmaf(A, x, gy[r]), x, fy[r]));
        mask |= f <= most ? 1u << q : 0u;
    }
    return mask;
}

// Stages one entry (its 48-byte record ra, rb, rc) for the tile with origin
// (ox, oy): v0 = centre - tile origin as a float hi/lo pair computed in double
// precision, v1 = conic scaled by -0.5 log2(e) (so alpha = opacity *
// exp2(A' dx^2 + B' dx dy + C' dy^2)) and opacity, v2 = colour and the list
// position.  Returns the 4-bit mask of the tile's 8x8 quads in which the entry
// can reach alpha 1/255 (a conservative bound: an entry outside it is skipped
// by every pixel of the quad).  v2.w holds the list position plus one (the
// n_contrib a pixel reports when this is its last composited entry).
__device__ __forceinline__ uint32_t stage_entry(const float4& ra, const float4& rb, const float4& rc, double ox,
                                                double oy, uint32_t pos, float4& v0, float4& v1, float4& v2)
{
    const double du = ((double)ra.x + (double)ra.z) - ox;
    const double dv = ((double)ra.y + (double)ra.w) - oy;
    const float du_hi = (float)du, dv_hi = (float)dv;
    // the minimisers' slopes need no correct rounding (see quads_within):
    // a hardware reciprocal, not two divisions
    const float bc = rb.y * __builtin_amdgcn_rcpf(rb.z), ba = rb.y * __builtin_amdgcn_rcpf(rb.x);
    // opacity * exp(-q / 2) >= 1/255 where q <= 2 ln(255 opacity): one log
    // per entry instead of an exp per quad, with a margin (1e-4 of the
    // threshold's size) that covers the 1e-5 relative margin on alpha, the
    // fast log's error and the per-pixel exp2's, so no quad a pixel reaches
    // is dropped
    const float lt = 2.0f * __logf(255.0f * rb.w);
    const float thr = lt + 1e-4f * (1.0f + fabsf(lt));
    const uint32_t qmask = quads_within(du_hi, dv_hi, rb.x, rb.y, rb.z, bc, ba, thr);
    v0 = make_float4(du_hi, dv_hi, (float)(du - (double)du_hi), (float)(dv - (double)dv_hi));
    v1 = make_float4(-0.5f * kLog2e * rb.x, -kLog2e * rb.y, -0.5f * kLog2e * rb.z, rb.w);
    v2 = make_float4(rc.x, rc.y, rc.z, __int_as_float((int)(pos + 1u)));
    return qmask;
}

// Alpha of a staged entry (e0, e1) at the pixel with tile offset (fx, fy),
// shared by the forward and the backward so that both take the same
// decisions: the offset to the centre as (hi - pixel) + lo, then
// opacity * E with E = exp2(dx (A' dx + B' dy) + C' dy^2), clamped to 0.99.
// Returns alpha; dx, dy and the falloff E (for the backward) on the side.
__device__ __forceinline__ float entry_alpha(const float4& e0, const float4& e1, float fx, float fy, float& dx,
                                             float& dy, float& E)
{
    dx = (e0.x - fx) + e0.z;
    dy = (e0.y - fy) + e0.w;
    const float pw = fmaf(fmaf(e1.x, dx, e1.y * dy), dx, (e1.z * dy) * dy);
    E = __builtin_amdgcn_exp2f(pw);
    return fminf(0.99f, e1.w * E);
}

// The entries of one tile, picked in order out of its bin's list by the 256
// threads of a workgroup.  A round passes over kRound entries of the bin, four
// consecutive ones per lane: an entry belongs to the tile when its part of
// the bin covers it, one subtraction per two entries (each 4-bit field of
// (tile | guard) - span keeps its guard bit when the tile lies inside the
// span on that side).  The picked items go to a ring in LDS; an entry's index
// in the ring's sequence is its position in the tile's list of Sec. 3.1.  A
// round is about 30 VALU instructions per wave and 256 entries, where staging
// takes 255 per 64 picked ones.
constexpr int kRound = 1024;
constexpr int kRing = 2048;

struct TilePick {
    uint32_t ring[kRing];
    uint32_t count[4];
};

// Four entries of a lane: which of them the tile takes, over the wave, and
// their items.
struct Pick4 {
    uint64_t m[4] = {0, 0, 0, 0};
    uint4 it = {0, 0, 0, 0};
    __device__ __forceinline__ uint32_t total() const
    {
        return (uint32_t)(__popcll(m[0]) + __popcll(m[1]) + __popcll(m[2]) + __popcll(m[3]));
    }
};

struct TileCursor {
    const uint32_t* items;
    const uint16_t* spans;
    // The bin's list: entries begin to end past base, a multiple of 4.  A bin
    // lists a Gaussian once, so end stays below 2^31 where base may be 2^32 less
    // a few, and nothing below (two rounds past the end at most) wraps.
    uint32_t base, begin, end;
    uint32_t cur;          // next round's first entry (a multiple of 4: whole groups are loaded)
    uint32_t tail;         // entries picked so far
    uint32_t key;          // the tile's place in the bin, guard bits set, twice

    __device__ __forceinline__ bool more() const { return cur < end; }

    // The lane's group of the round at c.  The last group may reach past the
    // list: the buffers hold whole groups; a lane past the last group loads
    // it again.
    __device__ __forceinline__ uint32_t group(uint32_t c) const
    {
        return min(c + 4u * threadIdx.x, (end - 1u) & ~3u);
    }
    __device__ __forceinline__ uint2 load_spans(uint32_t c) const
    {
        return *reinterpret_cast<const uint2*>(spans + (base + group(c)));
    }
    __device__ __forceinline__ uint4 load_items(uint32_t c) const
    {
        return *reinterpret_cast<const uint4*>(items + (base + group(c)));
    }

    __device__ __forceinline__ void start(const BinLists& lists, const ViewParams& vp, int tx, int ty)
    {
        const uint32_t* off = lists.off + lists.stride * (int64_t)bin_of_tile(vp, tx, ty);
        uint64_t b = off[0], e = off[lists.stride];
        if (e > lists.capacity) e = lists.capacity;
        if (b > e) b = e;
        items = lists.items;
        spans = lists.spans;
        // uniform values, kept scalar
        base = (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)b & ~3u));
        begin = (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)b & 3u));
        end = begin + (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(e - b));
        cur = begin < end ? 0u : end;
        tail = 0;
        const uint32_t edge = (1u << vp.bin_shift) - 1u, x = (uint32_t)tx & edge, y = (uint32_t)ty & edge;
        const uint32_t k = 0x8888u | x | (y << 4) | ((edge - x) << 8) | ((edge - y) << 12);
        key = k | (k << 16);
    }

    // The tile's entries among four, sp, of the round at c.
    __device__ __forceinline__ void pick4(uint2 sp, uint32_t c, Pick4& k) const
    {
        if (c < begin || c + kRound > end) {
            // entries outside the list: a span that covers no tile (8 in
            // every field, which borrows from none)
            const uint32_t i = c + 4u * threadIdx.x - begin, len = end - begin;
            sp.x = (i < len ? sp.x & 0xFFFFu : 0x8888u) | (i + 1u < len ? sp.x & 0xFFFF0000u : 0x88880000u);
            sp.y = (i + 2u < len ? sp.y & 0xFFFFu : 0x8888u) | (i + 3u < len ? sp.y & 0xFFFF0000u : 0x88880000u);
        }
        const uint32_t a = (key - sp.x) & 0x88888888u, b = (key - sp.y) & 0x88888888u;
        k.m[0] = __ballot((uint16_t)a == (uint16_t)0x8888u);
        k.m[1] = __ballot(a >= 0x88880000u);
        k.m[2] = __ballot((uint16_t)b == (uint16_t)0x8888u);
        k.m[3] = __ballot(b >= 0x88880000u);
    }

    // The lane's picks to the ring, from position pos of the wave's first.
    static __device__ __forceinline__ void write4(uint32_t* ring, const Pick4& k, uint32_t pos)
    {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            pos = __builtin_amdgcn_mbcnt_hi((uint32_t)(k.m[j] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)k.m[j], pos));
        const uint32_t item[4] = {k.it.x, k.it.y, k.it.z, k.it.w};
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (__builtin_amdgcn_inverse_ballot_w64(k.m[j])) {
                ring[pos & (kRing - 1)] = item[j];
                ++pos;
            }
    }

    // First half of a round: the picks and the wave's count.  (The picks are
    // the caller's, not the cursor's: as members they would hold registers
    // from one round to the next.)
    __device__ __forceinline__ void test(TilePick& pick, Pick4& p, int wave, int lane)
    {
        const uint2 sp = load_spans(cur);
        p.it = load_items(cur);
        pick4(sp, cur, p);
        const uint32_t n = p.total();
        if (lane == 0) pick.count[wave] = n;
        cur += kRound;
        // the items are here before the caller issues its gathers: waited for
        // in put(), they would make it wait for those as well
        __asm__ volatile("" : "+v"(p.it.x), "+v"(p.it.y), "+v"(p.it.z), "+v"(p.it.w));
    }

    // Second half, a barrier later: the picked items to the ring.
    __device__ __forceinline__ void put(TilePick& pick, const Pick4& p, int wave)
    {
        uint32_t pos = tail, n = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const uint32_t c = (uint32_t)__builtin_amdgcn_readfirstlane((int)pick.count[w]);
            pos += w < wave ? c : 0u;
            n += c;
        }
        write4(pick.ring, p, pos);
        tail += n;
    }

    // The first two rounds at once, into the empty ring, all loads together.
    __device__ __forceinline__ void begin_pick(TilePick& pick, int wave, int lane)
    {
        static_assert(kRing >= 2 * kRound, "two rounds fit");
        if (!more()) return;
        const uint32_t c = cur;
        const bool two = c + kRound < end;
        const uint2 sp = load_spans(c), sp2 = load_spans(c + kRound);   // past the list: its last group
        Pick4 p, p2;
        p.it = load_items(c);
        p2.it = load_items(c + kRound);
        pick4(sp, c, p);
        uint32_t n = p.total();
        pick4(sp2, c + kRound, p2);   // nothing past the list
        n |= p2.total() << 16;
        cur = two ? c + 2 * kRound : c + kRound;
        if (lane == 0) pick.count[wave] = n;
        __syncthreads();
        uint32_t before = 0, all = 0;   // both rounds' counts, 16 bits each (at most 1024)
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const uint32_t k = (uint32_t)__builtin_amdgcn_readfirstlane((int)pick.count[w]);
            before += w < wave ? k : 0u;
            all += k;
        }
        write4(pick.ring, p, before & 0xFFFFu);
        write4(pick.ring, p2, (all & 0xFFFFu) + (before >> 16));
        tail = (all & 0xFFFFu) + (all >> 16);
        __syncthreads();
    }

    // Whole rounds until target entries are picked or the list ends; every
    // thread of the workgroup takes part, and the ring is ready on return.
    __device__ __forceinline__ void fill(TilePick& pick, uint32_t target, int wave, int lane)
    {
        while (tail < target && more()) {
            Pick4 p;
            test(pick, p, wave, lane);
            __syncthreads();
            put(pick, p, wave);
            __syncthreads();
        }
    }
};

// Workgroup -> tile: tiles are cut into groups of `group` consecutive tiles
// (row-major), dealt to the 8 XCDs in turn (block b runs on XCD b % 8), so
// neighbouring tiles, which share list entries, share an XCD's L2.
__device__ __forceinline__ int blend_tile_of_block(int group)
{
    const int i = (int)(blockIdx.x >> 3);
    return ((i / group) * 8 + (int)(blockIdx.x & 7)) * group + i % group;
}

inline int blend_blocks(int64_t tiles, int group)
{
    return (int)(8 * group * ((tiles + 8 * group - 1) / (8 * group)));
}

// Workgroup -> tile when a dispatch order is given (heaviest tiles first,
// from the previous frame's per-tile work): block b takes order[b]; else the
// XCD groups above.
__device__ __forceinline__ int blend_tile(const uint32_t* order, int group)
{
    return order ? (int)order[blockIdx.x] : blend_tile_of_block(group);
}

inline int blend_grid(int64_t tiles, const uint32_t* order, int group)
{
    return order ? (int)tiles : blend_blocks(tiles, group);
}

}  // namespace gsmi
