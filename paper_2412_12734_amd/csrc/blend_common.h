// Pieces shared by the forward and backward blend kernels: the launch parameters, the
// XCD-aware tile schedule, LDS staging of splat batches (geometry and texels) and the
// per-pixel evaluation of one splat (ray-splat uv, falloff, opacity, bilinear colour).
#pragma once

#include "device_util.h"
#include "gbb_internal.h"

namespace gbb {

// A float array zeroed by the forward's workgroups: n_head single floats up to the first
// 16-byte boundary, n_body float4s, then n_tail (at most 3) trailing floats.
struct ZeroRange {
  float* head;
  float4* body;
  float* tail;
  int64_t n_body;
  int32_t n_head, n_tail;
};

struct BlendParams {
  float tex_scale;    // (N - 1) / (2 sigma): uv -> grid coordinate slope
  float tex_offset;   // (N - 1) / 2
  float sigma;
  float alpha_min, alpha_max, t_min;
  float cull_alpha;   // 0.99 alpha_min: the per-wave cull's margin below alpha_min
  float lp_scale;     // 1 / (2 lowpass_var)
  float lp_scale2;    // 2 lp_scale
  float bg[3];
  int32_t tile_w, tile_h;
  int32_t n_views;
  int32_t P;          // splats per view: record v P + k is splat k seen from view v
  int32_t total_tiles;
  const uint32_t* tile_order;  // nullable: workgroup b takes tile tile_order[b]
  uint32_t* tile_work;         // nullable: per-tile blended span written by the forward
  // view-dependent colour of each record, added to every texel on staging (nullable), and
  // the backward's adjoint of it (nullable; xyz summed over the record's blended pixels)
  const float4* spec;
  float* d_spec;
  // colour grids of several sides (nullable: every grid is N x N): per splat its side and the
  // index of its first texel in the packed texture array
  const int32_t* grid_n;
  const int64_t* grid_at;
  // forward only: arrays that the workgroups zero while they blend (the coming backward's
  // texture and record gradients); an empty range zeroes nothing
  ZeroRange zero[2];
};

BlendParams make_blend_params(const Plan& pl, const gb_options& o, int n_views);

// Tile of a workgroup without a work order. Workgroups go to the eight XCDs in turn; each XCD takes
// every eighth run of kTileRun consecutive tiles, so that neighbouring tiles share an L2 (records and
// texels of the splats that cross them) while every XCD gets its share of the crowded part of the
// image. (One band of an eighth of the tiles per XCD left XCDs idle: 100k splats at 800 x 800 forward
// 268 -> 204 us, 444k splats on four views 1043 -> 727, 3M splats on four 1080p views 3.72 -> 3.51 ms;
// runs of 4 / 16 / 40 tiles 204 / 203 / 208 and 727 / 757 / 744.) With a work order the tiles with
// the most work start first.
constexpr int kTileRun = 4;

__host__ __device__ constexpr int64_t tile_blocks(int64_t tiles) {
  return (tiles + 8 * kTileRun - 1) / (8 * kTileRun) * (8 * kTileRun);
}

__device__ __forceinline__ int tile_of_block(const BlendParams& p) {
  const int b = blockIdx.x;
  if (p.tile_order) return b < p.total_tiles ? (int)p.tile_order[b] : p.total_tiles;
  const int q = b >> 3;
  return (q / kTileRun * 8 + (b & 7)) * kTileRun + q % kTileRun;
}

__device__ __forceinline__ int view_of_tile(const ViewDev* views, int n_views, int tile) {
  int v = 0;
  while (v + 1 < n_views && views[v + 1].tile_base <= tile) ++v;
  return v;
}

// Geometry of one staged splat for one wave's pixel block. With (lx, ly) a pixel's offset from
// the block centre (half-integers of at most 3.5 for 8 x 8 blocks, exact),
// rho = A + (h00 lx + h01 ly, h10 lx + h11 ly, h20 lx + h21 ly), where A is rho at the block
// centre, evaluated in pair precision. The float32 error of rho grows with the offset times
// |h|, so a centre per wave block (rather than per tile) keeps it at the block's size whatever
// the tile shape. The low-pass offset uses the tile centre: (ox, oy) = tile centre minus
// projected centre, so that a pixel's offset from the projected centre is (tx + ox, ty + oy)
// with (tx, ty) its offset from the tile centre.
//   g0 = (A0, A1, A2, opacity), g1 = (h00, h01, h10, h11), g2 = (h20, h21, ox, oy),
//   rect_x, rect_y: the record's pixel rectangle.
struct StagedGeo {
  float4 g0, g1, g2;
  int32_t rect_x, rect_y;
};

// (cx, cy): the block centre, (tx, ty) the tile centre, in pixel coordinates (integers: blocks
// and tiles have even sides).
__device__ __forceinline__ StagedGeo stage_geo(const SplatRec& r, int cx, int cy, int tx,
                                               int ty) {
  const f2 c2x{r.c2x_hi, r.c2x_lo}, c2y{r.c2y_hi, r.c2y_lo};
  const f2 ox = f2_sub(f2_of((float)cx), c2x);
  const f2 oy = f2_sub(f2_of((float)cy), c2y);
  f2 h[7];
#pragma unroll
  for (int i = 0; i < 7; ++i) h[i] = f2{r.h_hi[i], r.h_lo[i]};
  const f2 A0 = f2_add(f2_mul(h[0], ox), f2_mul(h[1], oy));
  const f2 A1 = f2_add(f2_mul(h[2], ox), f2_mul(h[3], oy));
  const f2 A2 = f2_add(f2_add(f2_mul(h[4], ox), f2_mul(h[5], oy)), h[6]);
  StagedGeo s;
  s.g0 = make_float4(f2_round(A0), f2_round(A1), f2_round(A2), r.opacity);
  s.g1 = make_float4(r.h_hi[0], r.h_hi[1], r.h_hi[2], r.h_hi[3]);
  s.g2 = make_float4(r.h_hi[4], r.h_hi[5], f2_round(f2_sub(f2_of((float)tx), c2x)),
                     f2_round(f2_sub(f2_of((float)ty), c2y)));
  s.rect_x = r.rect_x;
  s.rect_y = r.rect_y;
  return s;
}

// LDS copy of a pass's staged geometry for the (at most four) wave blocks of a tile: g1 and
// g2 once per splat, g0 once per (block, splat). 96 bytes per splat; reading one (block,
// splat) takes three 16-byte loads.
template <int B>
struct GeoLds {
  float4 g1[B];
  float4 g2[B];
  float4 g0[4][B];

  __device__ void store(int b, int j, const StagedGeo& g) {
    if (b == 0) {
      g1[j] = g.g1;
      g2[j] = g.g2;
    }
    g0[b][j] = g.g0;
  }
  __device__ StagedGeo load(int b, int j) const {
    StagedGeo g;
    g.g0 = g0[b][j];
    g.g1 = g1[j];
    g.g2 = g2[j];
    return g;
  }
};

// LDS texel layout per staged splat: N rows of N + 1 float4 (RGB + pad), so that texels
// (i, j) and (i + 1, j) fall into different LDS banks.
template <int N>
struct TexLayout {
  static constexpr int kRow = N + 1;
  static constexpr int kPerSplat = N == 1 ? 1 : N * (N + 1);
  // a 24-bit multiply (full rate; a 32-bit integer multiply is quarter rate): iu < N
  __device__ static int at(int iu, int iv) { return (int)__umul24((unsigned)iu, kRow) + iv; }
};

// The four corner texels of a cell, each as one 16-byte LDS read (5.6 cycles of the CU's LDS for a
// wave). Left to the compiler, which sees that the pad is unused, they become 12-byte reads, which
// take 9.1. (All four are asked for before the one point that uses the pads: a use after each read
// had put four LDS latencies one after another into every wave step.)
template <int ROW>
__device__ __forceinline__ void load_corners(const float4* t, float4& t00, float4& t01,
                                             float4& t10, float4& t11) {
  t00 = t[0];
  t01 = t[1];
  t10 = t[ROW];
  t11 = t[ROW + 1];
  __asm__ volatile("" : : "v"(t00.w), "v"(t01.w), "v"(t10.w), "v"(t11.w));
}

// Set bits of a uniform mask (two scalar counts).
__device__ __forceinline__ int popcount64(uint64_t x) {
  return __builtin_popcount((uint32_t)x) + __builtin_popcount((uint32_t)(x >> 32));
}

// A lane mask that is the same in every lane, kept in scalar registers.
__device__ __forceinline__ uint64_t uniform64(uint64_t x) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)x),
                 hi = __builtin_amdgcn_readfirstlane((uint32_t)(x >> 32));
  return (uint64_t)hi << 32 | lo;
}

// Most tiles that all run at once when `per_cu` workgroups share a CU (256 CUs): up to there the LDS
// that a larger batch takes costs nothing, and it saves barriers and trips to memory.
__host__ __device__ constexpr int64_t tiles_at_once(int per_cu) { return 256 * (int64_t)per_cu; }

// Entries (consecutive pairs of the tile's list) whose geometry one staging pass prepares: one
// per lane of each wave, which tests them against its own pixel block.
constexpr int kPassEntries = 64;

// Entries of the pass over what is left of a list, [b, end) in the forward (from its front) and in
// the backward (from its end). Pair slots go up to 2^32 - 16: a bound of 64 past a list's end can
// wrap, so that the passes count entries and compare the lane with the count.
__host__ __device__ constexpr int pass_size(uint32_t b, uint32_t end, int most) {
  return end - b < (uint32_t)most ? (int)(end - b) : most;
}

// The part of a staging pass that every wave works out alike from the waves' votes: `mine` marks
// the entries that can reach this wave's block, `any` those that can reach some block of the
// tile. Only the latter are given texel slots, in batches, so that a splat whose screen
// rectangle touches the tile but whose footprint does not (about half of them) costs a geometry
// test and nothing more. list.entry[slot] is the entry of each slot, by falling (REVERSE) or rising
// entry index, and list.rec[slot] its record (my_rec: the record of the lane's entry); every wave
// writes the same list and reads only what it has written itself.
template <int PE>
struct SlotList {
  uint32_t rec[PE];
  uint8_t entry[PE];
};

struct PassVotes {
  uint64_t mine, any;
  int total;  // set bits of any
};

template <bool REVERSE, int PE>
__device__ __forceinline__ PassVotes pass_votes(uint64_t mine, const uint64_t* s_mask, int lane,
                                                uint32_t my_rec, SlotList<PE>& list) {
  PassVotes v;
  v.mine = mine;
  v.any = uniform64((s_mask[0] | s_mask[1]) | (s_mask[2] | s_mask[3]));
  v.total = popcount64(v.any);
  if (__builtin_amdgcn_inverse_ballot_w64(v.any)) {
    const int below = (int)mbcnt(v.any);
    const int slot = REVERSE ? v.total - 1 - below : below;
    list.entry[slot] = (uint8_t)lane;
    list.rec[slot] = my_rec;
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  return v;
}

// The thread index as a value the compiler takes to be new: what a staging or flush phase
// derives from it is then computed in that phase, and does not sit in registers through the
// splat loop.
__device__ __forceinline__ int fresh_tid() {
  int t = (int)threadIdx.x;
  __asm__ volatile("" : "+v"(t));
  return t;
}

// Copies the texels of a batch of `nb` splats (even N) into LDS as float4 (RGB + pad) per texel.
// Slot j holds the splat of record recs[j] (a tile's records are all of the tile's view, so the
// splat is the record minus rec_base). A splat's 3 N^2 channel values split into groups of 12
// (four texels): each thread moves whole groups, three 16-byte (float32) or 8-byte (bfloat16)
// loads in, four LDS stores out.
// With spec != null each texel also gets the record's view-dependent colour spec[record]
// (the bilinear weights sum to one, so this adds that colour to the lookup).
template <int N, bool BF16>
__device__ __forceinline__ void stage_texels(const void* __restrict__ textures,
                                             const uint32_t* recs, uint32_t rec_base, int nb,
                                             float4* s_tex, const float4* __restrict__ spec,
                                             int tid) {
  constexpr int groups = 3 * N * N / 12;
#pragma unroll 1
  for (int gi = tid; gi < nb * groups; gi += (int)blockDim.x) {
    const int j = gi / groups, a = gi - j * groups;
    const uint32_t r = recs[j];
    const int64_t src = ((int64_t)(r - rec_base) * groups + a) * 3;
    const float4 sc = spec ? spec[r] : make_float4(0.f, 0.f, 0.f, 0.f);
    float v[12];
    if constexpr (BF16) {
      const uint2* t = reinterpret_cast<const uint2*>(textures) + src;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const uint2 x = t[k];
        v[4 * k + 0] = __uint_as_float(x.x << 16);
        v[4 * k + 1] = __uint_as_float(x.x & 0xffff0000u);
        v[4 * k + 2] = __uint_as_float(x.y << 16);
        v[4 * k + 3] = __uint_as_float(x.y & 0xffff0000u);
      }
    } else {
      const float4* t = reinterpret_cast<const float4*>(textures) + src;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const float4 x = t[k];
        v[4 * k + 0] = x.x;
        v[4 * k + 1] = x.y;
        v[4 * k + 2] = x.z;
        v[4 * k + 3] = x.w;
      }
    }
    float4* dst = s_tex + j * TexLayout<N>::kPerSplat;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int t = 4 * a + k, iu = t / N, iv = t - iu * N;
      dst[TexLayout<N>::at(iu, iv)] =
          spec ? make_float4(v[3 * k] + sc.x, v[3 * k + 1] + sc.y, v[3 * k + 2] + sc.z, 0.f)
               : make_float4(v[3 * k], v[3 * k + 1], v[3 * k + 2], 0.f);
    }
  }
}

// The texel of record r's splat where grids have one texel (N = 1), with the view-dependent colour
// as above. Such texels are staged with the pass's geometry, one per entry: they cost less than the
// second trip to memory that texels of chosen entries wait for.
template <bool BF16>
__device__ __forceinline__ float4 one_texel(const void* __restrict__ textures, uint32_t r,
                                            uint32_t rec_base, const float4* __restrict__ spec) {
  const int64_t i = 3 * (int64_t)(r - rec_base);
  float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
  if constexpr (BF16) {
    const uint16_t* t = reinterpret_cast<const uint16_t*>(textures) + i;
    x.x = bf16_to_f32(t[0]);
    x.y = bf16_to_f32(t[1]);
    x.z = bf16_to_f32(t[2]);
  } else {
    const float* t = reinterpret_cast<const float*>(textures) + i;
    x.x = t[0];
    x.y = t[1];
    x.z = t[2];
  }
  if (spec) {
    const float4 sc = spec[r];
    x.x += sc.x;
    x.y += sc.y;
    x.z += sc.z;
  }
  return x;
}

// Row and column of texel t (< 256) of an n-texel side (n <= 16): t / n as a multiply by
// ceil(2^16 / n) and a shift, exact in that range (checked for every t and n).
__device__ __forceinline__ int div_side(int t, int n) {
  return (int)(((uint32_t)t * (uint32_t)((65536 + n - 1) / n)) >> 16);
}

// Side of splat k's grid in a call with several sides, clamped to [1, N].
template <int N>
__device__ __forceinline__ int grid_side(const BlendParams& p, uint32_t k) {
  return min(max(p.grid_n[k], 1), N);
}

// What each lane holds of its entry of the pass in a call with grids of several sides: the
// grid's side, its uv -> grid slope and its first value in the texture array. The
// waves read an entry's values back with readlane (the entry is uniform over the wave).
struct EntryGrid {
  int n;
  float scale;
  int64_t first;
};

// Slope of the uv -> grid map of an n-texel side, formed as the host forms it for a uniform
// side (a call whose sides all equal N then matches the uniform path bit for bit).
__device__ __forceinline__ float grid_scale(int n, float sigma) {
  return (float)(n - 1) / (2.0f * sigma);
}

template <int N>
__device__ __forceinline__ EntryGrid entry_grid(const BlendParams& p, uint32_t r,
                                                uint32_t rec_base) {
  EntryGrid g;
  g.n = grid_side<N>(p, r - rec_base);
  g.scale = grid_scale(g.n, p.sigma);
  g.first = 3 * p.grid_at[r - rec_base];
  return g;
}

__device__ __forceinline__ int64_t readlane64(int64_t x, int lane) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)x, lane),
                 hi = (uint32_t)__builtin_amdgcn_readlane((int)(x >> 32), lane);
  return (int64_t)((uint64_t)hi << 32 | lo);
}

// Copies the texels of a batch of `nb` splats whose grids have sides of their own (at most N)
// into the N x N LDS layout: a splat's n x n texels go to rows and columns [0, n). Wave w takes
// slots w, w + nw, ...; lane i moves texels i, i + 64, ... of the grid (three channel values in,
// one 16-byte LDS store out: a third of the index arithmetic of moving single values), with the
// record's view-dependent colour (spec, nullable) added as in stage_texels. A one-texel grid is
// also copied to (0, 1), (1, 0) and (1, 1), so that the bilinear lookup, which reads the four
// corners of cell (0, 0) with weights (1, 0, 0, 0) there, reads finite values.
template <int N, bool BF16>
__device__ __forceinline__ void stage_texels_mixed(const void* __restrict__ textures,
                                                   const uint8_t* list, const uint32_t* recs,
                                                   int nb, float4* s_tex,
                                                   const float4* __restrict__ spec,
                                                   const EntryGrid& eg) {
  const int tid = fresh_tid(), lane = tid & 63, nw = (int)(blockDim.x >> 6);
  for (int j = __builtin_amdgcn_readfirstlane(tid >> 6); j < nb; j += nw) {
    const int e = __builtin_amdgcn_readfirstlane((int)list[j]);
    const int n = __builtin_amdgcn_readlane(eg.n, e);
    const int64_t base = readlane64(eg.first, e);
    const float4 sc = spec ? spec[recs[j]] : make_float4(0.f, 0.f, 0.f, 0.f);
    float4* dst = s_tex + j * TexLayout<N>::kPerSplat;
    // texel at value index i (its three channels), with the view-dependent colour added
    auto texel = [&](int64_t i) {
      float x0, x1, x2;
      if constexpr (BF16) {
        const uint16_t* t = reinterpret_cast<const uint16_t*>(textures) + i;
        x0 = bf16_to_f32(t[0]);
        x1 = bf16_to_f32(t[1]);
        x2 = bf16_to_f32(t[2]);
      } else {
        const float* t = reinterpret_cast<const float*>(textures) + i;
        x0 = t[0];
        x1 = t[1];
        x2 = t[2];
      }
      return make_float4(x0 + sc.x, x1 + sc.y, x2 + sc.z, 0.f);
    };
    if (n == 1) {
      if (lane < 4) dst[TexLayout<N>::at(lane >> 1, lane & 1)] = texel(base);  // corner lane
    } else {
      // one texel per lane and pass: its three channels in, one 16-byte LDS store out
      for (int t = lane; t < n * n; t += 64) {
        const int iu = div_side(t, n), iv = t - iu * n;
        dst[TexLayout<N>::at(iu, iv)] = texel(base + 3 * t);
      }
    }
  }
}

// Ray-splat solve and falloff of one splat at one pixel. The pixel can blend the splat where
// r2 != 0 and alpha >= alpha_min.
struct PixelEval {
  float dx, dy;       // pixel centre minus projected centre (float32; low-pass and gradients)
  float r2, inv;      // rho2 and 1 / rho2
  float u, v;
  float G;            // exp(-q)
  float oG;           // opacity times G
  float alpha;        // min(alpha_max, oG)
  uint64_t uv_branch;  // lanes whose q came from the uv Gaussian (else from the screen low-pass)
};

// (lx, ly): pixel centre minus the wave block's centre; (tx, ty): minus the tile's centre.
// Both falloff exponents are compared and scaled as 2 q (doubling is exact, so the result is
// that of q); each minimum is one instruction (fminf first canonicalises its operands), and
// the branch is a lane mask that only the backward asks for: 16 uneven views of 1M splats 12.52 -> 12.44
// ms, 3M splats on four 1080p views 16.67 -> 16.58.
__device__ __forceinline__ PixelEval eval_splat(const StagedGeo& s, float lx, float ly, float tx,
                                                float ty, const BlendParams& p) {
  PixelEval e;
  e.dx = tx + s.g2.z;
  e.dy = ty + s.g2.w;
  const float r0 = __builtin_fmaf(s.g1.y, ly, __builtin_fmaf(s.g1.x, lx, s.g0.x));
  const float r1 = __builtin_fmaf(s.g1.w, ly, __builtin_fmaf(s.g1.z, lx, s.g0.y));
  e.r2 = __builtin_fmaf(s.g2.y, ly, __builtin_fmaf(s.g2.x, lx, s.g0.z));
  e.inv = __builtin_amdgcn_rcpf(e.r2);
  e.u = r0 * e.inv;
  e.v = r1 * e.inv;
  const float q_uv = e.u * e.u + e.v * e.v;
  const float q_lp = (e.dx * e.dx + e.dy * e.dy) * p.lp_scale2;
  e.uv_branch = ballot(q_uv <= q_lp);
  float q;  // the smaller one; q_lp where q_uv is not a number
  __asm__("v_min_f32 %0, %1, %2" : "=v"(q) : "v"(q_uv), "v"(q_lp));
  e.G = __builtin_amdgcn_exp2f(q * (-0.5f * 1.4426950408889634f));
  e.oG = s.g0.w * e.G;
  __asm__("v_min_f32 %0, %1, %2" : "=v"(e.alpha) : "s"(p.alpha_max), "v"(e.oG));
  return e;
}

// Conservative test whether a staged splat can reach alpha >= alpha_min anywhere in a wave's
// bw x bh pixel block, staged for that block: (bx0, by0) is the block's first pixel and (cx, cy)
// its centre relative to the tile centre. rho is affine in the pixel offset, so its range over
// the block is exact; where rho2 keeps its sign, |u| >= min|rho0| / max|rho2| (likewise v), and
// the low-pass term is bounded by the block's distance to the projected centre. A splat is
// skipped only if even the largest possible opacity is clearly below alpha_min, so skipping
// never changes a result.
__device__ __forceinline__ bool block_may_contribute(const StagedGeo& s, float cx, float cy,
                                                     int bx0, int by0, const BlendParams& p,
                                                     int bw = 8, int bh = 8) {
  const int rx = s.rect_x, ry = s.rect_y;
  const int i0 = rx & 0xffff, i1 = rx >> 16, j0 = ry & 0xffff, j1 = ry >> 16;
  if (i1 < bx0 || i0 > bx0 + bw - 1 || j1 < by0 || j0 > by0 + bh - 1) return false;
  // half extents of the block's pixel centres
  const float ex = 0.5f * (float)(bw - 1), ey = 0.5f * (float)(bh - 1);
  const float h00 = s.g1.x, h01 = s.g1.y, h10 = s.g1.z, h11 = s.g1.w, h20 = s.g2.x, h21 = s.g2.y;
  const float r2c = s.g0.z;
  const float r2e = ex * fabsf(h20) + ey * fabsf(h21);
  if (!(fabsf(r2c) > 1.001f * r2e)) return true;  // the vanishing line may cross the block
  const float r0c = s.g0.x;
  const float r1c = s.g0.y;
  const float r0m = fmaxf(fabsf(r0c) - (ex * fabsf(h00) + ey * fabsf(h01)), 0.f);
  const float r1m = fmaxf(fabsf(r1c) - (ex * fabsf(h10) + ey * fabsf(h11)), 0.f);
  const float inv = 1.0f / (fabsf(r2c) + r2e);
  const float um = r0m * inv, vm = r1m * inv;
  const float q_uv = 0.5f * (um * um + vm * vm);
  const float dxm = fmaxf(fabsf(cx + s.g2.z) - ex, 0.f);
  const float dym = fmaxf(fabsf(cy + s.g2.w) - ey, 0.f);
  const float q_lp = (dxm * dxm + dym * dym) * p.lp_scale;
  const float q = fminf(q_uv, q_lp);
  return s.g0.w * __builtin_amdgcn_exp2f(-q * 1.4426950408889634f) >= p.cull_alpha;
}

// Grid coordinate of u on the corner-aligned N-texel grid (Alg. 2 with the cell index taken
// from the remapped coordinate and limited to N - 2 at the clamped top edge).
template <int N>
__device__ __forceinline__ void grid_coord(float u, const BlendParams& p, int& i, float& f) {
  const float up = fminf(fmaxf(__builtin_fmaf(u, p.tex_scale, p.tex_offset), 0.0f), (float)(N - 1));
  const int fi = (int)up;  // up >= 0, so truncation is the floor
  i = fi < N - 2 ? fi : N - 2;
  f = up - (float)i;
}

// Grid coordinate of u on a corner-aligned grid of n texels per side with slope `scale`
// (grid_scale): as grid_coord<N> with n in place of N (a uniform call's grids give the same
// results); one texel gives cell 0 with f = 0.
__device__ __forceinline__ void grid_coord_n(float u, float scale, int n, int& i, float& f) {
  const float hi = (float)(n - 1);
  const float up = fminf(fmaxf(__builtin_fmaf(u, scale, 0.5f * hi), 0.0f), hi);
  const int fi = (int)up;
  const int cmax = n > 2 ? n - 2 : 0;
  i = fi < cmax ? fi : cmax;
  f = up - (float)i;
}

// grid_coord_n from constants of the side, formed once per splat: gc holds the slope (grid_scale),
// the offset (n - 1) / 2, the upper clamp n - 1 and the largest cell index (its int bits). The same
// operations in the same order, so the same results.
__device__ __forceinline__ void grid_coord_c(float u, const float4& gc, int& i, float& f) {
  const float up = fminf(fmaxf(__builtin_fmaf(u, gc.x, gc.y), 0.0f), gc.z);
  const int fi = (int)up;
  const int cmax = __float_as_int(gc.w);
  i = fi < cmax ? fi : cmax;
  f = up - (float)i;
}

}  // namespace gbb
