// blend_backward.hip -- gradient of the per-tile front-to-back blend.
//
// The forward of Eq. 1 gives, per pixel, C = sum_j a_j T_j c_j + T_f bg with
// T_j = prod_{i<j} (1 - a_i) over the composited entries.  For a loss L with
// G = dL/dC and G_T = dL/dT_f, an entry j that the pixel composited gets
//   dL/dc_j = G a_j T_j
//   dL/da_j = G . (T_j c_j - (S_j + T_f bg) / (1 - a_j)) - G_T T_f / (1 - a_j)
// where S_j = sum_{k>j} a_k T_k c_k is the colour composited after j.  The
// pass is recomputed rather than stored: walking the list front to back with
// the forward's own arithmetic gives the same a_j and T_j, S_j is the
// forward's colour minus the running sum, and the walk stops at the pixel's
// n_contrib (one past its last composited entry).  With X_j = G . (S_j +
// T_f bg) + G_T T_f, dL/da_j = (T_{j+1} G . c_j - X_j) / (1 - a_j): the
// difference is rounded once.  (One running number per pixel for X_j, which
// the three of S_j give, saves 8 us of 540 but raises the errors: its steps do
// not mirror the forward's.)  Through a = min(0.99, opacity exp(p)) with p =
// -0.5 (A dx^2 + C dy^2) - B dx dy the gradient reaches the opacity, the conic
// and the centre; a clamped alpha passes none.
//
// Layout as the forward: one workgroup of four waves per 16x16 tile, one pixel
// per lane, entries staged through LDS with the same per-quad reach masks.
// Vector instructions bound it (92% of their issue rate), so an entry's sums
// over a wave are taken before what they share (the factors, for the conic all
// but the second moments of dL/dp), summed with as few
// cross-lane instructions as they need (below) and added into an LDS row of
// the staged entry; the rest is applied once per tile and entry, after the
// batch, on the way to nine atomic adds in HBM.  At 3M Gaussians and
// 1920x1080: 541 us, 672 with nine full gradients per pixel and a trading
// butterfly; four 640x480 views of 300K: 362 us, 498 so; 20K at 317x179: 163 us,
// 288 so.
// (Matrix instructions over 16 rows of moments of four entries took 246 us of
// the matrix cores at the first size and 811 us in all: their sums leave in
// more lanes than LDS atomics take quickly.)
#include "blend_stage.h"

namespace gsmi {
namespace {

constexpr float kLn2 = 0.69314718055994531f;
// Entries staged per batch: 20 KB of LDS with their sums, for seven workgroups a
// CU (192 and six: 1 to 3% slower at the three sizes above).
constexpr int kBackBatch = 128;
constexpr int kFlush = 256 / kGrad2d;   // entries whose sums are flushed at once

// The sums of an entry over a tile's pixels, with gp = dL/dp and w = a T, in
// the order in which wave_sum9 leaves them in the lanes.
enum { kSo, kSv, kSu, kSxx, kSxy, kSr, kSyy, kSg, kSb };   // dL/d(opacity), gp dp/dv / ln2, gp dp/du / ln2, gp dx^2, ...

struct BackLds {
    float4 s0[kBackBatch];   // du_hi, dv_hi, du_lo, dv_lo
    float4 s1[kBackBatch];   // A', B', C', opacity
    float4 s2[kBackBatch];   // r, g, b, list position
    uint32_t s_item[kBackBatch];
    float s_acc[kBackBatch][kGrad2d];
    uint32_t s_wave_keep[4];
    uint8_t s_mask[kBackBatch];
    TilePick pick;
};

// Half sums of two values at once: lanes 0-31 (even rows of 16 for the
// second) get a's, the others b's.  The swap trades a's upper half for b's
// lower one (a's odd rows for b's even ones), so one add sums both.
__device__ __forceinline__ float half_sums32(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float half_sums16(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Wave sums of nine values.  Two halving steps leave eight of them in two
// registers whose rows of 16 lanes hold one value each; DPP adds that write
// only some banks (groups of four lanes) then sum within the rows and pack the
// registers into one on the way: bank 0 of row r ends with value r, bank 2
// with value 4 + r, and bank 3, whose rows are summed last, with value 8 in
// row 3.  21 VALU instructions; the waits are the two states that DPP needs
// between a write and its use.  (A trading butterfly with lane selects took 50
// and five LDS exchanges, whole-row rotations of three registers 30.)
__device__ __forceinline__ float wave_sum9(const float (&g)[9])
{
    const float h0 = half_sums32(g[kSo], g[kSu]), h1 = half_sums32(g[kSv], g[kSxx]), h2 = half_sums32(g[kSxy], g[kSyy]),
                h3 = half_sums32(g[kSr], g[kSg]);
    const float q0 = half_sums16(h0, h1), q1 = half_sums16(h2, h3);
    float t, u = g[kSb];
    __asm__("s_nop 1\n\t"
            "v_add_f32_dpp %1, %1, %1 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
            "v_add_f32_dpp %0, %2, %2 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
            "v_add_f32_dpp %0, %3, %3 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"   // banks 2, 3: the second register
            "s_nop 1\n\t"
            "v_add_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
            "v_add_f32_dpp %0, %1, %1 row_half_mirror row_mask:0xf bank_mask:0x8\n\t"   // bank 3: the ninth value
            "s_nop 1\n\t"
            "v_add_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
            "s_nop 1\n\t"
            "v_add_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
            "s_nop 1\n\t"
            "v_add_f32_dpp %0, %0, %0 row_bcast:15 row_mask:0xa bank_mask:0x8\n\t"
            "s_nop 1\n\t"
            "v_add_f32_dpp %0, %0, %0 row_bcast:31 row_mask:0xc bank_mask:0x8"
            : "=&v"(t), "+v"(u)
            : "v"(q0), "v"(q1));
    return t;
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(7))) void blend_backward_kernel(BlendBackArgs a)
{
    __shared__ BackLds L;
    int tile = blend_tile(a.order, a.group);
    if (tile >= a.tiles) return;
    tile = __builtin_amdgcn_readfirstlane(tile);   // uniform: it and what follows from it stay scalar
    const int view = view_of_tile(a.views, a.n_views, (uint32_t)tile);
    const ViewParams& vp = a.views[view];
    const int width = vp.width, height = vp.height;
    const int local = tile - (int)vp.tile_base;
    const int tx = local % vp.tiles_x, ty = local / vp.tiles_x;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lx = (wave & 1) * 8 + (lane & 7), ly = (wave >> 1) * 8 + (lane >> 3);
    const int px = tx * kTile + lx, py = ty * kTile + ly;
    const bool inside = px < width && py < height;
    TileCursor tc;
    BinLists lists = a.lists;
    lists.stride = *a.stride;
    tc.start(lists, a.bin_views[view], tx, ty);
    const double ox = (double)(tx * kTile), oy = (double)(ty * kTile);
    const float fx = (float)lx, fy = (float)ly;

    // the pixel's loss gradient, its n_contrib, the colour composited over the
    // whole list without the background, and the part of X that is the same
    // for every entry: background and final transmittance
    float G0 = 0.f, G1 = 0.f, G2 = 0.f, S0 = 0.f, S1 = 0.f, S2 = 0.f, XT = 0.f;
    uint32_t nc = 0;
    if (inside) {
        const int64_t P = (int64_t)width * height, p = (int64_t)py * width + px;
        G0 = vp.grad_rgb[p];
        G1 = vp.grad_rgb[P + p];
        G2 = vp.grad_rgb[2 * P + p];
        nc = vp.out_nc[p];
        const float Tf = vp.out_T[p];
        S0 = vp.out_rgb[p] - Tf * a.bg[0];
        S1 = vp.out_rgb[P + p] - Tf * a.bg[1];
        S2 = vp.out_rgb[2 * P + p] - Tf * a.bg[2];
        XT = (G0 * a.bg[0] + G1 * a.bg[1] + G2 * a.bg[2] + (vp.grad_T ? vp.grad_T[p] : 0.f)) * Tf;
    }
    float Tr = 1.0f;
    // the lane's place among an entry's sums (wave_sum9)
    const bool holds = (lane & 7) == 0 || lane == 63;
    const int slot = lane == 63 ? 8 : ((lane & 8) >> 1) + (lane >> 4);
    float* const acc = &L.s_acc[0][slot];
    // the thread's gradient when the sums are flushed: which one, from which
    // sum, times what
    const int flush_j = tid / kGrad2d, flush_c = tid % kGrad2d;
    constexpr int kOf[kGrad2d] = {kSu, kSv, kSxx, kSxy, kSyy, kSo, kSr, kSg, kSb};
    int flush_of = 0;
#pragma unroll
    for (int c = 0; c < kGrad2d; ++c) flush_of = flush_c == c ? kOf[c] : flush_of;
    const float flush_by = flush_c < 2 ? kLn2 : (flush_c == 3 ? -1.0f : (flush_c < 5 ? -0.5f : 1.0f));

    // the forward's pipeline: entries picked two batches ahead, records one
    tc.begin_pick(L.pick, wave, lane);
    tc.fill(L.pick, 2 * kBackBatch, wave, lane);
    float4 na = make_float4(0.f, 0.f, 0.f, 0.f), nb = na, ncl = na;
    uint32_t item = 0u;
    if (tid < kBackBatch && (uint32_t)tid < tc.tail) {
        item = L.pick.ring[tid];
        const float4* rec = reinterpret_cast<const float4*>(a.splats + item);
        na = rec[0];
        nb = rec[1];
        ncl = rec[2];
    }
    // the last list position that a pixel of the wave, and of the tile, takes
    uint32_t wave_last = nc;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) wave_last = max(wave_last, (uint32_t)__shfl_xor((int)wave_last, o));
    wave_last = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_last);
    if (lane == 0) L.s_wave_keep[wave] = wave_last;
    __syncthreads();
    const uint32_t tile_last = (uint32_t)__builtin_amdgcn_readfirstlane(
        (int)max(max(L.s_wave_keep[0], L.s_wave_keep[1]), max(L.s_wave_keep[2], L.s_wave_keep[3])));
    if (tile_last == 0u) return;
    for (uint32_t b0 = 0; b0 < min(tc.tail, tile_last); b0 += kBackBatch) {
        __syncthreads();   // the previous batch's rows and the ring's picks
        const uint32_t tail = tc.tail, e = b0 + tid;
        uint32_t qmask = 0u;
        float4 v0, v1, v2;
        if (tid < kBackBatch && e < min(tail, tile_last)) qmask = stage_entry(na, nb, ncl, ox, oy, e, v0, v1, v2);
        const bool keep = qmask != 0u;
        const uint64_t km = __ballot(keep);
        if (lane == 0) L.s_wave_keep[wave] = (uint32_t)__popcll(km);
        __syncthreads();
        uint32_t before = 0u;
        int nk = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            if (w == wave) before = (uint32_t)nk;
            nk += __builtin_amdgcn_readfirstlane((int)L.s_wave_keep[w]);
        }
        if (keep) {
            const uint32_t at =
                __builtin_amdgcn_mbcnt_hi((uint32_t)(km >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)km, before));
            L.s0[at] = v0;
            L.s1[at] = v1;
            L.s2[at] = v2;
            L.s_mask[at] = (uint8_t)qmask;
            L.s_item[at] = item;
        }
        for (int k = tid; k < nk * kGrad2d; k += 256) (&L.s_acc[0][0])[k] = 0.f;
        const bool round = tail < b0 + 3 * kBackBatch && tc.more();
        Pick4 pk;
        if (round) tc.test(L.pick, pk, wave, lane);
        if (tid < kBackBatch && e + kBackBatch < tail) {
            item = L.pick.ring[(e + kBackBatch) & (kRing - 1)];
            const float4* rec = reinterpret_cast<const float4*>(a.splats + item);
            na = rec[0];
            nb = rec[1];
            ncl = rec[2];
        }
        __syncthreads();
        if (round) tc.put(L.pick, pk, wave);
        if (tc.tail < b0 + 3 * kBackBatch && tc.more()) {
            __syncthreads();   // every wave has read the round's counts
            tc.fill(L.pick, b0 + 3 * kBackBatch, wave, lane);
        }
        for (int q = 0; q < nk; q += 64) {
            const int jj = q + lane;
            uint64_t bits = __builtin_amdgcn_ballot_w64(jj < nk && ((L.s_mask[jj] >> wave) & 1u) &&
                                                        (uint32_t)__float_as_int(L.s2[jj].w) <= wave_last);
            while (bits) {
                const int j = q + __builtin_ctzll(bits);
                bits &= bits - 1;
                const float4 e0 = L.s0[j], e1 = L.s1[j], e2 = L.s2[j];
                float dx, dy, E;
                const float al = entry_alpha(e0, e1, fx, fy, dx, dy, E);
                // not past the pixel's last entry, and visible
                const bool take = (uint32_t)__float_as_int(e2.w) <= nc && al >= 1.0f / 255.0f;
                if (__builtin_amdgcn_ballot_w64(take) == 0) continue;
                float gp = 0.f, go = 0.f;   // dL/dp, p the exponent of exp, and dL/d(opacity)
                float g[9];
                g[kSr] = g[kSg] = g[kSb] = 0.f;
                if (take) {
                    const float gc = G0 * e2.x + G1 * e2.y + G2 * e2.z;
                    const float w = al * Tr;
                    S0 -= w * e2.x;   // colour composited after this entry
                    S1 -= w * e2.y;
                    S2 -= w * e2.z;
                    const float X = G0 * S0 + G1 * S1 + G2 * S2 + XT;
                    Tr = fmaf(-al, Tr, Tr);   // as the forward: Tr (1 - al), rounded once
                    const float inv = __builtin_amdgcn_rcpf(1.0f - al);   // 1 - al >= 0.01
                    const float ga = fmaf(gc, Tr, -X) * inv;
                    const float gm = e1.w * E <= 0.99f ? ga : 0.f;
                    gp = gm * al;
                    go = gm * E;
                    g[kSr] = G0 * w;
                    g[kSg] = G1 * w;
                    g[kSb] = G2 * w;
                }
                g[kSo] = go;
                // dp/d(dx) = -(A dx + B dy) = ln2 (2 A' dx + B' dy): formed per
                // pixel and in one fused step, since for a needle its two terms
                // cancel (from the sums of dx and dy, 25 us less at 3M, the
                // centres' errors are 2% larger; A' dx added to the sum that
                // the alpha holds already, and dL/d(opacity) as the sum of gp
                // over the opacity, are two instructions less, 577 against 583
                // us there, and a rounding or two more)
                const float cy = e1.z * dy;
                g[kSu] = gp * fmaf(e1.x + e1.x, dx, e1.y * dy);
                g[kSv] = gp * fmaf(e1.y, dx, cy + cy);
                const float gx = gp * dx, gy = gp * dy;
                g[kSxx] = gx * dx;
                g[kSxy] = gx * dy;
                g[kSyy] = gy * dy;
                const float v = wave_sum9(g);
                // (the row's offset stays scalar: as part of the address it
                // becomes a 64-bit multiply-add)
                int row = j * kGrad2d;
                __asm__("" : "+s"(row));
                if (holds) atomicAdd(acc + row, v);
            }
        }
        __syncthreads();
        // one set of atomic adds per staged entry and tile: thread 9 i + c adds
        // gradient c (u, v, A, B, C, opacity, r, g, b) of entries i, i + 28, ...
        if (tid < kFlush * kGrad2d) {
            for (int j = flush_j; j < nk; j += kFlush) {
                float v = L.s_acc[j][flush_of];
                v *= flush_by;
                if (v != 0.f) unsafeAtomicAdd(&a.grad2d[(int64_t)L.s_item[j] * kGrad2d + flush_c], v);
            }
        }
    }
}

}  // namespace

hipError_t launch_blend_backward(const BlendBackArgs& a, hipStream_t s)
{
    if (a.tiles <= 0) return hipSuccess;
    hipLaunchKernelGGL(blend_backward_kernel, dim3(blend_grid(a.tiles, a.order, a.group)), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace gsmi
