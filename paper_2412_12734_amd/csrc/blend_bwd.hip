// Backward blend (Alg. 1 backward with Alg. 2 adj-bilinear): one workgroup per tile walks the
// tile's pairs back to front in LDS batches, starting at the last pair any of its pixels
// blended. Each pixel starts from its saved T_final and S = T_final * bg and, for every splat
// it blended (index below its saved bound, alpha >= alpha_min), in reverse order:
//   T_k = T_{k+1} / (1 - alpha_k), w = alpha_k T_k, colour adjoint w g,
//   adj-bilinear -> texel gradients and (du, dv),
//   d alpha = g . (col T_k - S / (1 - alpha_k)), S += w col,
//   d o = d alpha G, dq = -G o d alpha (both zero where alpha was clamped to alpha_max),
//   uv branch: du += dq u, dv += dq v; low-pass branch: d(dx, dy) += dq 2 (dx, dy) / (2 var),
//   (u, v) = (rho0, rho1) / rho2 -> d rho -> d H (7 entries) and d(dx, dy) -> d c2 = -d(dx, dy).
//
// A lane owns one pixel (waves of 8 x 8 pixels). The list is taken in passes of 64 entries: each
// wave stages the entries' geometry for its own block, one entry per lane, and votes which can
// reach it; entries that reach some block of the tile get slots, in batches, for their texels and
// for the sums over pixels. Per splat and wave, the ten record gradients are summed by lane swaps
// and DPP adds; texel gradients are grouped by grid cell (with sigma = 0.5 the grid covers
// only the splat's core, so most blended pixels are border-clamped and share a few cells), one
// group after another, over the corners that the group weights and inside the rows of 16 lanes,
// until at most kLaneAddMax pixels are left, each of which adds its corners directly. After each
// batch the non-zero sums go to global memory with one float atomic each, and the next batch's
// texels are staged.
//
// The texel sums are 64-bit in LDS: ds_add_f64 serves 64 lanes with distinct addresses in 8.7 cycles
// of the CU's LDS (12 lanes 6.5, and 3 per lane on one address), where ds_add_f32 takes 3 cycles for
// every lane whatever the addresses (12 lanes 38, 64 lanes 193), which had made the LDS the limit.
// The record sums (ten lanes, once per step) are 32-bit: their last bits matter (see pixel_step). In
// 64 bits the step at 1M splats and 1080p took 1.825 ms against 1.834, too little to change them for.
// What bounds the kernel now is VALU issue where tiles fill the chip, and the latency of a wave's
// step where a few tiles hold the work. At 1M splats and 1080p 1.35 -> 1.10 ms, 3M splats on
// four 1080p views 14.5 -> 11.3, 16 uneven views with 4 x 4 grids 8.28 -> 6.9, 16 x 16 grids 2.33 ->
// 1.68, sides {2, 4, 8} 1.53 -> 1.20, 100k splats at 800 x 800 0.73 -> 0.55. (With the texels
// projected on the pixel's adjoint before the interpolation, one scalar for the colour behind and d c2
// formed once per batch the step took 3 to 4 % less, but its gradients had other last bits.)
#include "blend_common.h"

namespace gbb {

namespace {

// Per-pixel backward state and the outputs of one (pixel, splat) step.
struct PixState {
  float T, S0, S1, S2, g0, g1, g2;
  uint32_t last;
};

struct PixOut {
  int cell;          // first corner's index in the LDS texel layout (TexLayout)
  float wgt, fu, fv; // alpha T and the position inside the cell
  uint64_t in_u, in_v;  // lanes where |u| < sigma, |v| < sigma: not clamped to the border
  float rec[kRecGrad];  // record gradients
};

// One (pixel, splat) step of the reverse walk. `act`: the pixel blended this splat. A lane
// that did not runs the same arithmetic with a zero opacity, so that its weights, adjoints and
// state come out unchanged or zero without a branch; its u, v and 1 / rho2 are replaced by 0
// (they are infinite where rho2 = 0). Its cell is left unspecified.
// Every operation of the record gradients is written out, multiply-adds too. Sums of them can
// cancel, by chance or exactly (where the falloff is the low-pass's and one coordinate is clamped
// to the grid's border, the adjoint of that axis' scale is zero and what comes out is rounding
// alone), and Adam divides a gradient by its own size: another last bit here can move a parameter
// by a full step.
// s_g1, s_g2 and j: the splat's staged H. MIXED: gc holds the grid-coordinate constants of the
// splat's grid (grid_coord_c).
template <int N, bool MIXED>
__device__ __forceinline__ void pixel_step(const float4* s_g1, const float4* s_g2, int j,
                                           const float4* tex, const PixelEval& e, float inv,
                                           float u, float v, bool act, PixState& ps,
                                           const BlendParams& p, PixOut& o, const float4& gc) {
#pragma clang fp contract(off)
  const float alpha = act ? e.alpha : 0.f;
  const float inv1m = __builtin_amdgcn_rcpf(1.0f - alpha);
  ps.T = ps.T * inv1m;  // transmittance in front of this splat
  const float wgt = alpha * ps.T;
  o.wgt = wgt;
  float c[3], du = 0.f, dv = 0.f;
  if constexpr (N == 1) {
    const float4 t = tex[0];
    c[0] = t.x;
    c[1] = t.y;
    c[2] = t.z;
    o.cell = 0;
    o.fu = o.fv = 0.f;
  } else {
    int iu, iv;
    float fu, fv;
    if constexpr (MIXED) {
      grid_coord_c(u, gc, iu, fu);
      grid_coord_c(v, gc, iv, fv);
    } else {
      grid_coord<N>(u, p, iu, fu);
      grid_coord<N>(v, p, iv, fv);
    }
    o.fu = fu;
    o.fv = fv;
    o.cell = TexLayout<N>::at(iu, iv);
    float4 t00, t01, t10, t11;
    load_corners<TexLayout<N>::kRow>(tex + o.cell, t00, t01, t10, t11);
    const float tsc = MIXED ? gc.x : p.tex_scale;
    const float g[3] = {ps.g0, ps.g1, ps.g2};
    const float x0[3] = {t00.x, t00.y, t00.z}, x1[3] = {t01.x, t01.y, t01.z};
    const float y0[3] = {t10.x, t10.y, t10.z}, y1[3] = {t11.x, t11.y, t11.z};
    float dc[3], d[3], f[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const float xd = x1[k] - x0[k], yd = y1[k] - y0[k];
      const float a = __builtin_fmaf(fv, xd, x0[k]), b = __builtin_fmaf(fv, yd, y0[k]);
      dc[k] = wgt * g[k];
      d[k] = b - a;
      c[k] = __builtin_fmaf(fu, d[k], a);
      f[k] = __builtin_fmaf(1.f - fu, xd, fu * yd);
    }
    // fractional-position adjoints (Alg. 2), zero where the coordinate is clamped
    const float dfu = __builtin_fmaf(dc[2], d[2], __builtin_fmaf(dc[0], d[0], dc[1] * d[1]));
    const float dfv = __builtin_fmaf(dc[2], f[2], __builtin_fmaf(dc[0], f[0], dc[1] * f[1]));
    du = __builtin_amdgcn_inverse_ballot_w64(o.in_u) ? tsc * dfu : 0.f;
    dv = __builtin_amdgcn_inverse_ballot_w64(o.in_v) ? tsc * dfv : 0.f;
  }
  // d alpha = g . (colour T - S / (1 - alpha)), zero where the pixel did not blend the splat or
  // alpha was clamped to alpha_max
  const float a0 = __builtin_fmaf(c[0], ps.T, -(ps.S0 * inv1m)),
              a1 = __builtin_fmaf(c[1], ps.T, -(ps.S1 * inv1m)),
              a2 = __builtin_fmaf(c[2], ps.T, -(ps.S2 * inv1m));
  const float da = __builtin_fmaf(ps.g2, a2, __builtin_fmaf(ps.g0, a0, ps.g1 * a1));
  ps.S0 = __builtin_fmaf(wgt, c[0], ps.S0);
  ps.S1 = __builtin_fmaf(wgt, c[1], ps.S1);
  ps.S2 = __builtin_fmaf(wgt, c[2], ps.S2);
  const float dalpha = (act && e.oG <= p.alpha_max) ? da : 0.f;
  o.rec[9] = dalpha * e.G;
  // the falloff's adjoint goes to (u, v) or to the low-pass offset, selected without a branch
  const float dq = -e.oG * dalpha;
  const bool from_uv = __builtin_amdgcn_inverse_ballot_w64(e.uv_branch);
  const float dq_uv = from_uv ? dq : 0.f, dq_lp = from_uv ? 0.f : dq * p.lp_scale2;
  du = __builtin_fmaf(u, dq_uv, du);
  dv = __builtin_fmaf(v, dq_uv, dv);
  const float dr0 = du * inv, dr1 = dv * inv;
  const float dr2 = -__builtin_fmaf(u, du, v * dv) * inv;
  o.rec[0] = dr0 * e.dx;
  o.rec[1] = dr0 * e.dy;
  o.rec[2] = dr1 * e.dx;
  o.rec[3] = dr1 * e.dy;
  o.rec[4] = dr2 * e.dx;
  o.rec[5] = dr2 * e.dy;
  o.rec[6] = dr2;
  // (H read again from LDS: held through the step it would take six registers)
  __asm__ volatile("" : "+s"(j));
  const float4 h = s_g1[j], h2 = s_g2[j];
  // d c2: the low-pass term and the uv term through rho's dependence on the offset (the centre
  // enters both with a minus sign)
  o.rec[7] = __builtin_fmaf(-h2.x, dr2, __builtin_fmaf(-h.z, dr1,
                            __builtin_fmaf(dq_lp, -e.dx, -(h.x * dr0))));
  o.rec[8] = __builtin_fmaf(-h2.y, dr2, __builtin_fmaf(-h.w, dr1,
                            __builtin_fmaf(dq_lp, -e.dy, -(h.y * dr0))));
}

// w times the corner weights (00, 01, 10, 11) at (fu, fv). The multiply-adds are written out:
// contracted from w - w f they could leave a rounding residue instead of 0 at f = 1.
__device__ __forceinline__ void corner_weights(float w, float fu, float fv, float (&wc)[4]) {
  const float w1 = w * fu, w0 = __builtin_fmaf(-w, fu, w);
  wc[0] = __builtin_fmaf(-w0, fv, w0);
  wc[1] = w0 * fv;
  wc[2] = __builtin_fmaf(-w1, fv, w1);
  wc[3] = w1 * fv;
}

// Row of a cell index of the LDS texel layout.
template <int N>
__device__ __forceinline__ int cell_row(int cell) {
  return (int)((unsigned)cell / (unsigned)TexLayout<N>::kRow);
}

// Fields of a lane's packed places: first bit and width (a lane that owns no value of a kind holds
// bits that are never used).
struct PlaceField {
  int at, bits;
};
constexpr PlaceField kRec{0, 4}, kT12{8, 6}, kT6v{14, 3}, kT6u{17, 6}, kT3{23, 2};

__device__ __forceinline__ uint32_t place(PlaceField f, int x) {
  return ((uint32_t)x & ((1u << f.bits) - 1u)) << f.at;
}
__device__ __forceinline__ int place_of(PlaceField f, uint32_t places) {
  return (int)((places >> f.at) & ((1u << f.bits) - 1u));
}

// Adds the total that row_sums left in each owner lane to an LDS array at index base + offset (base
// uniform over the wave).
template <uint64_t OWNERS>
__device__ __forceinline__ void lds_add(double* array, int base, int offset, float tot) {
  base = __builtin_amdgcn_readfirstlane(base);
  __asm__ volatile("" : "+s"(base));  // a scalar add, not part of a 64-bit multiply-add
  if (__builtin_amdgcn_inverse_ballot_w64(OWNERS)) atomicAdd(array + offset + base, (double)tot);
}

// Pixels left to a wave step's cell grouping that are added one by one. Backward ms for 16 / 20 / 24
// / 32: 1M splats at 1080p 1.033 / 1.018 / 1.041 / 1.18, 3M splats at 4 x 1080p 11.9 / 10.9 / 10.8 /
// 11.6, 16 uneven views with 4 x 4 grids 6.00 / 6.17 / 6.28 / 6.92, 100k splats at 800 x 800 0.575 /
// 0.526 / 0.518 / 0.543. (Grouping every pixel of a step with more than 24: 3M splats 13.2, 100k
// 0.64.)
constexpr int kLaneAddMax = 20;

// Splats per batch: the number asked for, by default as many as let all tiles run at once, up to a
// whole pass; on more tiles fewer, where that lets another workgroup share a CU's 160 KB of LDS. On
// numbers of tiles between, where the crowded tiles of an uneven image are what the launch waits for,
// larger batches stay ahead beyond the tiles that all run at once: they meet fewer flushes.
// Backward times (of the step when it was 3 to 6 % lighter, but where "now" is said):
//  8 x 8 grids hold 2.7 KB per splat (texels and 64-bit sums) beside the pass's geometry: seven
//  splats and passes of 32 entries (3 KB) are 22.4 KB, seven workgroups. 6 of 64 / 7 of 32 / 8 of
//  64: 1.063 / 1.045 / 1.101 ms at 1M splats and 1080p, 11.4 / 10.8 / 11.9 at 3M splats on four
//  1080p views, but 324 / 323 / 286 us at 120k small splats on 999 tiles; 8 / 16 / 32 of 64 1.37 /
//  1.13 / 1.03 ms at 235k splats on 112 tiles. Sides {2, 4, 8}, now, 7 / 8 / 16: 300k splats on 1000
//  tiles 634 / 563 / 501 us, 100k on 1530 353 / 335 / 373, 300k on 1900 438 / 382 / 443, 500k on 2880
//  579 / 591 / 734.
//  4 x 4 grids, 16 / 24 / 32 splats: 16 uneven views of 1M splats 6.22 / 6.25 / 7.54 ms, 47k splats
//  on three uneven views 0.558 / 0.529 / -, 372k splats on 462 tiles 1.27 / - / 1.09.
//  2 x 2 grids, now, 8 / 16 / 32 / 64: 300k splats on 1000 tiles 396 / 335 / 295 / 277 us, 300k on
//  1900 281 / 242 / 219 / 202, 500k on 3600 648 / 610 / 584 / 587.
//  16 x 16 grids, 1 / 2 / 3 splats: 2.81 / 2.10 / 2.16 ms at 1M splats and 1080p, two in passes of
//  48 entries (six workgroups per CU instead of five) 1.63. Now, 2 / 3 / 4: 100k splats on 800 tiles
//  572 / 490 / 423 us, 300k on 1280 919 / 790 / 670, 100k on 1530 558 / 556 / 550, 300k small ones on
//  1900 635 / 540 / 590, on 2332 592 / 592 / 624, 300k on 2475 613 / 687 / 755, 500k on 3600 1829 / 2078
//  / 2293; 4 / 6 or 8 on 475 and 240 tiles 354 / 352 and 724 / 656. Sides {4, 8, 16}: 300k on 1000
//  tiles 1247 / 1012 / 865, 300k on 1900 860 / 673 / 749, 1M at 1080p 1570 / 1790 / 2033.
template <int N, bool MIXED>
int bwd_batch(int asked, int64_t tiles) {
  if (N == 1) return 64;
  if (N == 16)
    return tiles <= tiles_at_once(1) ? 8
           : tiles <= tiles_at_once(2) ? 6
           : tiles <= tiles_at_once(6) ? 4
           : tiles <= tiles_at_once(9) ? 3 : 2;
  if (N == 8) {
    if (asked == 0 && tiles <= tiles_at_once(MIXED ? 5 : 3))
      return tiles <= tiles_at_once(1) ? 32 : 16;
    return asked > 8 ? asked : tiles <= tiles_at_once(MIXED ? 8 : 5) ? 8 : 7;
  }
  if (N == 4) {
    if (asked == 0 && tiles <= tiles_at_once(2)) return 64;
    return asked != 0 && asked < 32 ? asked : tiles <= tiles_at_once(5) ? 32 : 24;
  }
  return asked != 0 ? asked : tiles <= tiles_at_once(6) ? 64 : 32;
}
template <int N, int B>
constexpr int bwd_pass_entries() {
  return N == 8 && B == 7 ? 32 : N >= 16 && B == 2 ? 48 : kPassEntries;
}

// Occupancy target: what the LDS allows (see above), at most 7 waves per SIMD (72 VGPRs): 8 (64
// VGPRs) spilled: 1M splats at 1080p 1.10 against 1.03 ms, 3M splats at 4 x 1080p 14.7 against
// 13.2.
template <int N, int B>
constexpr int bwd_min_waves() {
  return (N <= 2 && B <= 32) || N == 1 || (N == 4 && B <= 16) || (N == 8 && B <= 7) ? 7
         : N == 2 || (N == 4 && B == 24) || (N == 16 && B == 2)                     ? 6
         : (N == 4 && B == 32) || (N == 8 && B == 8)                                ? 5
                                                                                    : 1;
}

// Lanes that flush one splat's sums: as few as keep the number of reads per lane small, so that a
// wave flushes several splats side by side (one after another, each a chain of LDS reads, the
// flush was what bound tiles of many small splats).
template <int N, bool MIXED>
constexpr int flush_lanes() { return MIXED || N >= 16 ? 64 : N == 8 ? 32 : 16; }

// Depth-prefix split: on a tile that the prefix left open the block first walks the rest
// pass's list (the later splats) and then, with each pixel's T and S carried over in
// registers, the prefix pass's list; other tiles only walk the prefix list.
// MIXED: each splat has a grid side of its own (at most N), read from p.grid_n; its texel
// gradients go to its own n x n grid at p.grid_at.
template <int N, bool BF16, int B, bool MIXED>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(bwd_min_waves<N, B>())))
blend_bwd_kernel(const ViewDev* __restrict__ views, const SplatRec* __restrict__ rec,
                 PairList first, PairList rest, const uint32_t* __restrict__ open_bits,
                 const void* __restrict__ textures, BlendParams p,
                 const float* __restrict__ T_final, const float* __restrict__ d_rgb,
                 float* __restrict__ d_rec, float* __restrict__ d_tex) {
  constexpr int TEXG = 3 * N * N;
  constexpr int PE = bwd_pass_entries<N, B>();
  __shared__ GeoLds<PE> s_geo;
  __shared__ float4 s_tex[B * TexLayout<N>::kPerSplat];
  __shared__ __attribute__((aligned(16))) double s_gtex[B * TEXG];  // per slot
  __shared__ float s_rec[B * kRecGrad];  // per slot
  // the waves' votes of a pass, of which two can be in use at a time (a wave may vote on the
  // next pass while another still reads this one's)
  __shared__ uint64_t s_mask[2][4];
  __shared__ SlotList<PE> s_list;
  __shared__ uint32_t s_tile_last;

  const int tile = tile_of_block(p);
  if (tile >= p.total_tiles) return;
  const bool tile_open = open_bits && ((open_bits[tile >> 5] >> (tile & 31)) & 1u) != 0;
  const int vi = view_of_tile(views, p.n_views, tile);
  const ViewDev& V = views[vi];
  const uint32_t rec_base = (uint32_t)vi * (uint32_t)p.P;  // first record of the tile's view
  const int lt = tile - V.tile_base;
  const int tile_x0 = (lt % V.tiles_x) * p.tile_w;
  const int tile_y0 = (lt / V.tiles_x) * p.tile_h;

  const int tid = threadIdx.x, nthr = blockDim.x;
  // the wave index is uniform: keep it (and the wave block's geometry) in scalar registers
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int waves_x = p.tile_w >> 3;
  const int n_waves = nthr >> 6;
  const int bx = (w % waves_x) * 8, by = (w / waves_x) * 8;
  // pixel centres relative to the wave block's centre (exact half-integers); the block centre
  // relative to the tile's (wave-uniform integers)
  const float lx = (float)(lane & 7) - 3.5f, ly = (float)(lane >> 3) - 3.5f;
  const int tcx = tile_x0 + (p.tile_w >> 1), tcy = tile_y0 + (p.tile_h >> 1);
  const int kbx = tile_x0 + bx, kby = tile_y0 + by;  // the wave block's first pixel
  const float bcx = (float)(kbx + 4 - tcx), bcy = (float)(kby + 4 - tcy);
  // packed index of the lane's pixel, or -1 outside the view (recomputed when needed)
  auto pixel_index = [&]() -> int64_t {
    const int px = kbx + (lane & 7), py = kby + (lane >> 3);
    return (px < V.W && py < V.H) ? (int64_t)V.pix_base + (int64_t)py * V.W + px : -1;
  };
  PixState ps;
  {
    const int64_t pix = pixel_index();
    ps.T = 1.0f;
    ps.g0 = ps.g1 = ps.g2 = 0.f;
    if (pix >= 0) {
      ps.T = T_final[pix];
      ps.g0 = d_rgb[3 * pix + 0];
      ps.g1 = d_rgb[3 * pix + 1];
      ps.g2 = d_rgb[3 * pix + 2];
    }
    ps.S0 = ps.T * p.bg[0];
    ps.S1 = ps.T * p.bg[1];
    ps.S2 = ps.T * p.bg[2];
  }
  // the sum that this lane owns after the reductions: its place among a splat's record gradients, and
  // its offset from the first texel's first channel in the three kinds of texel group (four corners;
  // two texels along v, or along u; one texel), in one register: fields kRec, kT12, kT6v, kT6u, kT3
  // of lane_places. rec_owners: the lanes that own a record gradient.
  uint32_t places;
  uint64_t rec_owners;
  {
    const int rl = lane & 15;
    const int s12 = row_slot(12, rl), s6 = row_slot(6, rl), s3 = row_slot(3, rl);
    const int rs = record_slot(swap_sides(), rl);
    rec_owners = ballot(rs >= 0);
    places = place(kRec, rs) |
             place(kT12, 3 * ((s12 / 3 & 1) + (s12 / 6) * N) + s12 % 3) |
             place(kT6v, s6) |  // 3 (s6 / 3) + s6 % 3
             place(kT6u, 3 * (s6 / 3) * N + s6 % 3) | place(kT3, s3);
  }

  // the per-batch LDS sums start at zero; each batch's flush clears what it read
  // (the first barrier of the list loop orders these stores before any add)
  for (int e = tid; e < B * TEXG; e += nthr) s_gtex[e] = 0.0;
  for (int e = tid; e < B * kRecGrad; e += nthr) s_rec[e] = 0.f;
  // votes of waves that the workgroup does not have
  if (tid < 8 && (tid & 3) >= n_waves) s_mask[tid >> 2][tid & 3] = 0;
  int parity = 0;

#pragma unroll 1
  for (int li = tile_open ? 0 : 1; li < 2; ++li) {
    const PairList L = li == 0 ? rest : first;
    const uint32_t* __restrict__ pair_vals = L.pair_vals;
    const uint32_t start = L.ranges[2 * tile];
    uint32_t wave_last;  // one past the last pair that some pixel of the wave blended
    {
      const int64_t pix = pixel_index();
      ps.last = pix >= 0 ? L.n_last[pix] : start;
      uint32_t m = ps.last;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const uint32_t o = (uint32_t)__shfl_xor((int)m, d, 64);
        m = o > m ? o : m;
      }
      wave_last = __builtin_amdgcn_readfirstlane(m);
    }
    __syncthreads();  // every thread has read the previous list's bound
    if (tid == 0) s_tile_last = start;
    __syncthreads();
    if (lane == 0) atomicMax(&s_tile_last, wave_last);
    __syncthreads();
    const uint32_t tile_last = __builtin_amdgcn_readfirstlane(s_tile_last);

    // the record of the lane's entry of the pass that ends at `end`
    auto load_rec = [&](uint32_t end) {
      const int n = pass_size(start, end, PE);
      return lane < n ? pair_vals[end - (uint32_t)n + (uint32_t)lane] : rec_base;
    };
    uint32_t my_rec = load_rec(tile_last);  // loaded a pass ahead
    for (uint32_t pend = tile_last; pend > start;) {
      // a pass: entries [pbase, pend) of the list, one per lane
      const int n = pass_size(start, pend, PE);
      const uint32_t pbase = pend - (uint32_t)n;
      uint64_t mine = 0;
      EntryGrid eg{1, 0.f, 0};
      // wave 0 also stores what the blocks share of a splat's geometry
      if (w == 0 || pbase < wave_last) {
        bool may = false;
        const int e = fresh_tid() & 63;
        if (e < n) {
          const SplatRec R = rec[my_rec];
          const StagedGeo g = stage_geo(R, kbx + 4, kby + 4, tcx, tcy);
          s_geo.store(w, e, g);
          if constexpr (N == 1) {
            if (w == 0) s_tex[e] = one_texel<BF16>(textures, my_rec, rec_base, p.spec);
          }
          may = pbase + (uint32_t)e < wave_last &&
                block_may_contribute(g, bcx, bcy, kbx, kby, p);
        }
        mine = ballot(may);
      }
      if constexpr (MIXED) {
        if (lane < n) eg = entry_grid<N>(p, my_rec, rec_base);
      }
      if (lane == 0) s_mask[parity][w] = mine;
      __syncthreads();
      const PassVotes votes =
          pass_votes<true>(mine, s_mask[parity], lane, my_rec, s_list);
      my_rec = load_rec(pbase);
      parity ^= 1;

      auto batch_size = [&](int b0) { return votes.total - b0 < B ? votes.total - b0 : B; };
      auto stage_batch = [&](int b0) {
        if constexpr (N == 1)
          ;  // staged with the geometry
        else if constexpr (MIXED)
          stage_texels_mixed<N, BF16>(textures, s_list.entry + b0, s_list.rec + b0,
                                      batch_size(b0), s_tex, p.spec, eg);
        else
          stage_texels<N, BF16>(textures, s_list.rec + b0, rec_base, batch_size(b0), s_tex,
                                p.spec, fresh_tid());
      };
      if (N > 1 && votes.total > 0) {
        stage_batch(0);
        __syncthreads();
      }
      uint64_t ahead = ~0ull;  // entries that no batch has taken yet
      for (int b0 = 0; b0 < votes.total; b0 += B) {
        const int nb = batch_size(b0);
        const uint64_t batch =
            ahead & (~0ull << __builtin_amdgcn_readfirstlane((int)s_list.entry[b0 + nb - 1]));
        ahead &= ~batch;
        // the batch's splats that can reach the wave's block, walked back to front
        uint64_t todo = votes.mine & batch;
        while (todo != 0) {
          const int j = 63 - (int)__builtin_clzll(todo);
          todo &= ~(1ull << j);
          const uint32_t jg = pbase + (uint32_t)j;
          const uint64_t live = ballot(jg < ps.last);
          const StagedGeo g = s_geo.load(w, j);
          const PixelEval e = eval_splat(g, lx, ly, lx + bcx, ly + bcy, p);
          // lanes that blended this splat (a vote per compare: each is a lane mask already)
          const uint64_t pend_px = live & ballot(e.r2 != 0.0f) & ballot(e.alpha >= p.alpha_min);
          if (pend_px == 0) continue;  // no pixel of the wave blended it
          const bool act = __builtin_amdgcn_inverse_ballot_w64(pend_px);
          // the splat's slot: taken slots of the pass after this entry's
          const uint64_t after = votes.any >> 1 >> j;
          const int slot = popcount64(after) - b0;
          const float4* tex = s_tex + (N == 1 ? j : slot) * TexLayout<N>::kPerSplat;
          PixOut po;
          int n_side = N;
          float4 gc = make_float4(0.f, 0.f, 0.f, 0.f);
          if constexpr (MIXED) {
            n_side = __builtin_amdgcn_readlane(eg.n, j);
            const float hi = (float)(n_side - 1);
            gc = make_float4(
                __int_as_float(__builtin_amdgcn_readlane(__float_as_int(eg.scale), j)), 0.5f * hi,
                hi, __int_as_float(n_side > 2 ? n_side - 2 : 0));
          }
          const float inv = act ? e.inv : 0.f, u = act ? e.u : 0.f, v = act ? e.v : 0.f;
          po.in_u = ballot(fabsf(u) < p.sigma);  // (-sigma, sigma): one compare with |u|
          po.in_v = ballot(fabsf(v) < p.sigma);
          pixel_step<N, MIXED>(s_geo.g1, s_geo.g2, j, tex, e, inv, u, v, act, ps, p, po, gc);
          // Sums of the record gradients; the one lane that owns each adds it to the splat's slot.
          {
            const float tot = record_sums(po.rec);
            float* const at = s_rec + kRecGrad * slot;
            if (__builtin_amdgcn_inverse_ballot_w64(rec_owners))
              atomicAdd(at + place_of(kRec, places), tot);
          }

          // Texel gradients, grouped by cell over all pixels of the wave. A wave step that
          // blended few pixels (small or distant splats) adds each pixel's bilinear corners to
          // LDS directly; up to kLaneAddMax lanes this costs less than group passes.
          const int base = TEXG * slot;
          if constexpr (N == 1) {
            float red[3] = {po.wgt * (act ? ps.g0 : 0.f), po.wgt * (act ? ps.g1 : 0.f),
                            po.wgt * (act ? ps.g2 : 0.f)};
            const float tot = row_sums(red);
            lds_add<row_owners(3)>(s_gtex, base, place_of(kT3, places), tot);
          } else {
            // A group is every pending lane of the first pending lane's cell, so the loop ends
            // within 64 passes. Most groups lie where a coordinate is clamped to the grid's
            // border (with sigma = 0.5 the grid covers only the splat's core): there the weights
            // of the clamped axis are 0 and 1, the same for the whole group, and only two texels
            // or one take a sum (at 1M splats and 1080p one texel in 25 % of the groups, two in
            // 61 %). The clamped end follows from the cell when the axis has at least two
            // cells. Other lanes contribute through a zero adjoint.
            const uint64_t in_u = n_side > 2 ? po.in_u : ~0ull,
                           in_v = n_side > 2 ? po.in_v : ~0ull;
            const int key = act ? po.cell : -1;
#pragma unroll 1
            for (uint64_t left = pend_px; left != 0;) {
              if (popcount64(left) <= kLaneAddMax) {
                if (__builtin_amdgcn_inverse_ballot_w64(left)) {
                  double* const gb = s_gtex + base;
                  const int k00 = po.cell - cell_row<N>(po.cell);
                  float wc[4];
                  corner_weights(po.wgt, po.fu, po.fv, wc);
#pragma unroll
                  for (int q = 0; q < 4; ++q) {
                    if (wc[q] != 0.f) {
                      double* dst = gb + 3 * (k00 + (q & 1) + (q >> 1) * N);
                      atomicAdd(dst + 0, (double)(wc[q] * ps.g0));
                      atomicAdd(dst + 1, (double)(wc[q] * ps.g1));
                      atomicAdd(dst + 2, (double)(wc[q] * ps.g2));
                    }
                  }
                }
                break;
              }
              const int lead = __builtin_amdgcn_readlane(key, (int)__builtin_ctzll(left));
              const uint64_t members = ballot(key == lead);
              left &= ~members;
              // (adjoints, not weights, are zeroed: one that is not finite stays with its splats)
              const bool in = __builtin_amdgcn_inverse_ballot_w64(members);
              const float g0 = in ? ps.g0 : 0.f, g1 = in ? ps.g1 : 0.f, g2 = in ? ps.g2 : 0.f;
              const int lu = cell_row<N>(lead), lv = lead - lu * TexLayout<N>::kRow;
              // the texel row and column of a clamped coordinate
              const int bu = lu == 0 ? 0 : n_side - 1, bv = lv == 0 ? 0 : n_side - 1;
              if ((members & in_v) == 0) {
                if ((members & in_u) == 0) {
                  float red[3] = {po.wgt * g0, po.wgt * g1, po.wgt * g2};
                  const float tot = row_sums(red);
                  lds_add<row_owners(3)>(s_gtex, base + 3 * (bu * N + bv), place_of(kT3, places), tot);
                } else {
                  const float w1 = po.wgt * po.fu, w0 = __builtin_fmaf(-po.wgt, po.fu, po.wgt);
                  float red[6] = {w0 * g0, w0 * g1, w0 * g2,
                                  w1 * g0, w1 * g1, w1 * g2};
                  const float tot = row_sums(red);
                  lds_add<row_owners(6)>(s_gtex, base + 3 * (lu * N + bv), place_of(kT6u, places), tot);
                }
              } else if ((members & in_u) == 0) {
                const float w1 = po.wgt * po.fv, w0 = __builtin_fmaf(-po.wgt, po.fv, po.wgt);
                float red[6] = {w0 * g0, w0 * g1, w0 * g2,
                                w1 * g0, w1 * g1, w1 * g2};
                const float tot = row_sums(red);
                lds_add<row_owners(6)>(s_gtex, base + 3 * (bu * N + lv), place_of(kT6v, places), tot);
              } else {
                float wc[4], red[12];
                corner_weights(po.wgt, po.fu, po.fv, wc);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                  red[3 * q] = wc[q] * g0;
                  red[3 * q + 1] = wc[q] * g1;
                  red[3 * q + 2] = wc[q] * g2;
                }
                const float tot = row_sums(red);
                lds_add<row_owners(12)>(s_gtex, base + 3 * (lu * N + lv), place_of(kT12, places), tot);
              }
            }
          }
        }
        __syncthreads();
        // Flush: FL lanes take a slot, its sums go to global memory with one float atomic per
        // non-zero sum (consecutive lanes, consecutive addresses) and are left zero for the
        // next batch.
        constexpr int FL = flush_lanes<N, MIXED>(), PER = 64 / FL;
        const int ft = fresh_tid() & 63, fl = ft & (FL - 1);
        // (two waves share a slot of 768 sums where the batch has no slot for half of the waves)
        const int parts = N >= 16 && !MIXED && 2 * nb <= n_waves ? 2 : 1, part = w & (parts - 1);
        for (int j = w / parts * PER + (PER > 1 ? ft / FL : 0); j < nb; j += n_waves / parts * PER) {
          uint32_t r = s_list.rec[b0 + j];
          if constexpr (PER == 1) r = __builtin_amdgcn_readfirstlane(r);
          double* const gs = s_gtex + j * TEXG;
          const float rg = part == 0 && fl < kRecGrad ? s_rec[j * kRecGrad + fl] : 0.f;
          if (p.d_spec) {
            // the view-dependent colour of a record is added to every texel of its lookup, so
            // its adjoint over the tile is the sum of the record's texel sums, one per channel
            float sc[3] = {0.f, 0.f, 0.f};
            for (int t = fl + part * FL; t < N * N; t += parts * FL) {
              sc[0] += (float)gs[3 * t];
              sc[1] += (float)gs[3 * t + 1];
              sc[2] += (float)gs[3 * t + 2];
            }
            if constexpr (PER == 1) wave_sum_all<3>(sc);
            else row_sum_all<3>(sc);
            if constexpr (FL == 32) {
              for (float& x : sc) x += __shfl_xor(x, 16, 64);
            }
            const float x = fl == 0 ? sc[0] : fl == 1 ? sc[1] : sc[2];
            if (fl < 3 && x != 0.f) atomicAdd(&p.d_spec[4 * (int64_t)r + fl], x);
          }
          if constexpr (MIXED) {
            // the N x N sums hold the splat's n x n grid in rows and columns [0, n): lane i takes
            // values i, i + 64, ... of the grid's 3 n^2
            const int entry = __builtin_amdgcn_readfirstlane((int)s_list.entry[b0 + j]);
            const int n = __builtin_amdgcn_readlane(eg.n, entry);
            float* const dst = d_tex + readlane64(eg.first, entry);
            for (int i0 = fl; i0 < 3 * n * n; i0 += 3 * 64) {  // three reads at a time
              double x[3];
              int at[3];
#pragma unroll
              for (int k = 0; k < 3; ++k) {
                const int i = min(i0 + 64 * k, 3 * n * n - 1);
                const int t = i / 3, c = i - 3 * t, iu = div_side(t, n), iv = t - iu * n;
                at[k] = 3 * (iu * N + iv) + c;
                x[k] = gs[at[k]];
              }
#pragma unroll
              for (int k = 0; k < 3; ++k) {
                const int i = i0 + 64 * k;
                if (i < 3 * n * n && x[k] != 0.0) {
                  gs[at[k]] = 0.0;
                  atomicAdd(dst + i, (float)x[k]);
                }
              }
            }
          } else {
            float* const dst = d_tex + (int64_t)(r - rec_base) * TEXG;
            // (three reads at a time)
            constexpr int K = (TEXG + FL - 1) / FL, KU = K < 3 ? K : 3;
            for (int k0 = part * KU; k0 < K; k0 += parts * KU) {
              double x[KU];
#pragma unroll
              for (int k = 0; k < KU; ++k) {
                const int i = (k0 + k) * FL + fl;
                x[k] = (TEXG % FL == 0 && K % KU == 0) || i < TEXG ? gs[i] : 0.0;
              }
#pragma unroll
              for (int k = 0; k < KU; ++k) {
                const int i = (k0 + k) * FL + fl;
                if (x[k] != 0.0) {
                  gs[i] = 0.0;
                  atomicAdd(dst + i, (float)x[k]);
                }
              }
            }
          }
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          __builtin_amdgcn_wave_barrier();
          if (part == 0 && fl < kRecGrad) s_rec[j * kRecGrad + fl] = 0.f;
          if (fl < kRecGrad && rg != 0.f) atomicAdd(&d_rec[(int64_t)r * kRecGrad + fl], rg);
        }
        // the next batch's texels load while the atomics above drain
        if (b0 + B < votes.total) stage_batch(b0 + B);
        __syncthreads();
      }
      pend = pbase;
    }
  }  // lists
}

template <int N, bool BF16, bool MIXED = false>
hipError_t launch_np(const Plan& pl, const gb_splats& sp, const BlendParams& bp,
                     const ViewDev* views, const SplatRec* rec, const PairList& first,
                     const PairList& rest, const uint32_t* open_bits, const float* T_final,
                     const float* d_rgb, float* d_rec, float* d_tex, hipStream_t s) {
  const dim3 grid((unsigned)(bp.tile_order ? (int64_t)bp.total_tiles
                                           : tile_blocks(bp.total_tiles)));
  const dim3 block((unsigned)(pl.tile_w * pl.tile_h));
#define GBB_BWD_B(BB)                                                                          \
  case BB:                                                                                     \
    hipLaunchKernelGGL((blend_bwd_kernel<N, BF16, BB, MIXED>), grid, block, 0, s, views, rec,  \
                       first, rest, open_bits, sp.textures, bp, T_final, d_rgb, d_rec, d_tex); \
    break
  const int batch = bwd_batch<N, MIXED>(pl.batch_bwd, bp.total_tiles);
  if constexpr (N == 1) {
    switch (batch) { GBB_BWD_B(64); }
  } else if constexpr (N == 2) {
    switch (batch) {
      GBB_BWD_B(8);
      GBB_BWD_B(16);
      GBB_BWD_B(32);
      GBB_BWD_B(64);
      default: return hipErrorInvalidValue;
    }
  } else if constexpr (N == 4) {
    switch (batch) {
      GBB_BWD_B(8);
      GBB_BWD_B(16);
      GBB_BWD_B(24);
      GBB_BWD_B(32);
      GBB_BWD_B(64);
      default: return hipErrorInvalidValue;
    }
  } else if constexpr (N == 8) {
    switch (batch) {
      GBB_BWD_B(7);
      GBB_BWD_B(8);
      GBB_BWD_B(16);
      GBB_BWD_B(32);
      default: return hipErrorInvalidValue;
    }
  } else {
    switch (batch) {
      GBB_BWD_B(2);
      GBB_BWD_B(3);
      GBB_BWD_B(4);
      GBB_BWD_B(6);
      GBB_BWD_B(8);
      default: return hipErrorInvalidValue;
    }
  }
#undef GBB_BWD_B
  return hipGetLastError();
}

}  // namespace

hipError_t launch_blend_bwd(const Plan& pl, const gb_splats& sp, const gb_options& o,
                            const ViewDev* views, int n_views, const SplatRec* rec,
                            const PairList& first, const PairList& rest,
                            const uint32_t* open_bits, const uint32_t* tile_order,
                            const float* T_final, const float* d_rgb, float* d_rec,
                            float* d_tex, const float4* spec, float* d_spec, hipStream_t s) {
  BlendParams bp = make_blend_params(pl, o, n_views);
  bp.tile_order = tile_order;
  bp.spec = spec;
  bp.d_spec = d_spec;
  const bool bf = sp.tex_dtype == GB_BF16;
  if (sp.tex_side) {
    // grids of several sides in the N x N layout (N = 8 or 16, checked by the API)
    bp.grid_n = sp.tex_side;
    bp.grid_at = sp.tex_offset;
    if (pl.N == 16)
      return bf ? launch_np<16, true, true>(pl, sp, bp, views, rec, first, rest, open_bits,
                                               T_final, d_rgb, d_rec, d_tex, s)
                : launch_np<16, false, true>(pl, sp, bp, views, rec, first, rest, open_bits,
                                                T_final, d_rgb, d_rec, d_tex, s);
    return bf ? launch_np<8, true, true>(pl, sp, bp, views, rec, first, rest, open_bits,
                                            T_final, d_rgb, d_rec, d_tex, s)
              : launch_np<8, false, true>(pl, sp, bp, views, rec, first, rest, open_bits,
                                             T_final, d_rgb, d_rec, d_tex, s);
  }
  // One pixel per lane. Two pixels per lane (8 x 16 wave blocks) measured slower on the
  // 1M-splat 1080p workload (3.0 vs 2.3 ms): LDS limits such blocks to two waves per SIMD and
  // the per-wave cull is coarser.
#define GBB_BWD(NN)                                                                           \
  return bf ? launch_np<NN, true>(pl, sp, bp, views, rec, first, rest, open_bits, T_final, \
                                     d_rgb, d_rec, d_tex, s)                                  \
            : launch_np<NN, false>(pl, sp, bp, views, rec, first, rest, open_bits, T_final,\
                                      d_rgb, d_rec, d_tex, s)
  switch (pl.N) {
    case 1: GBB_BWD(1);
    case 2: GBB_BWD(2);
    case 4: GBB_BWD(4);
    case 8: GBB_BWD(8);
    case 16: GBB_BWD(16);
    default: return hipErrorInvalidValue;
  }
#undef GBB_BWD
}

}  // namespace gbb
