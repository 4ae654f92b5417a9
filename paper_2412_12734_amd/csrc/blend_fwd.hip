// Forward blend (Alg. 1 forward with Alg. 2 bilinear): one workgroup per tile, one lane per
// pixel, each wave owning an 8 x 8 pixel block. The tile's depth-sorted splats are taken in passes
// of 64: each wave stages their geometry for its own block, one splat per lane, and votes which
// can reach it (a wave whose pixels have all terminated votes for none); the splats that reach
// some block have their texels staged into LDS in batches (bfloat16 decoded on staging) and are
// walked by the waves that they reach. The workgroup stops when every wave has terminated.
// Bound by VALU issue where tiles fill the chip, and by the latency of a wave's step (two LDS
// round trips) where they do not. Staging only the splats that reach a block and their geometry by
// all waves at once, the four corner texels in flight together, and the open pixels as a scalar
// lane mask (a flag per lane cost copies of the pixel's state around every branch): at 1M splats
// and 1080p 0.509 -> 0.370 ms, 16 x 16 grids 1.24 -> 0.76, sides {2, 4, 8} 0.745 -> 0.468, 3M splats
// on four 1080p views 4.91 -> 3.51, 350k small splats on 135 tiles 0.363 -> 0.229 (with the tile
// order and the batches of later lines of this file and of blend_common.h).
//
// Per pixel and splat: (u, v) from the centre-relative homography, G = exp(-min(q_uv, q_lp)),
// alpha = min(alpha_max, o G); alpha < alpha_min is skipped; if T (1 - alpha) < t_min the
// pixel ends without blending it; otherwise acc += alpha T bilinear(C, u, v), T *= 1 - alpha.
// Saved for the backward: T_final and one past the index of the last blended pair.
//
// Depth-prefix split: the prefix pass also marks every tile where some pixel is still open
// (not stopped by t_min) in a bitmap and saves those pixels' accumulated colour and done flag;
// the rest pass (REST) runs on marked tiles only and resumes from that state, so each pixel
// sees exactly the sequence of splats and operations of a single pass.
#include "blend_common.h"

namespace gbb {

namespace {

// With STATS the kernel also counts its work into stats[0..3]: blended pairs, pixels stopped
// by t_min, lane evaluations (64 per wave and evaluated splat) and staged (tile, splat) pairs;
// the rest pass also adds its blended pairs to stats[4].
// Occupancy target: eight waves per SIMD, or what the 160 KB of LDS per CU allows (a
// workgroup puts one wave on each of the CU's four SIMDs).
template <int N, int B>
constexpr int fwd_min_waves() {
  constexpr int lds = (int)sizeof(GeoLds<kPassEntries>) + 512 + B * TexLayout<N>::kPerSplat * 16;
  return 160 * 1024 / lds < 8 ? 160 * 1024 / lds : 8;
}

// Splats per batch: the number asked for; by default a whole pass, or as many as let all tiles run
// at once, and on more tiles as many as let eight workgroups share a CU's LDS beside the pass's 6 KB
// of geometry. 8 x 8 grids (1.1 KB of texels per splat), when a step still took 0.458 ms at 1M splats
// and 1080p, there and at 3M splats on four 1080p views: batches of 8 0.482 / 5.26, 12 0.458 / 4.75,
// 16 0.501 / 5.28; 350k small splats on 135 tiles, 12 / 64: 305 / 229 us. 4 x 4 grids, 372k small
// splats on 462 tiles, 32 / 64: 437 / 382 us. 2 x 2 grids, 8 / 16 / 32 / 64: 300k splats on 1000
// tiles 207 / 159 / 136 / 120 us, 500k on 3600 285 / 246 / 227 / 213. 16 x 16 grids (4.3 KB) at 1M
// splats: 2 0.915, 3 0.840, 4 0.854; 3 / 8 / 16 on 240 tiles 396 / 290 / 264 us, on 475 200 / 151 /
// 136; 3 / 8 on 1000 tiles 500 / 410, on 1900 427 / 400, on 3600 814 / 972 (8 is not taken beyond 768
// tiles yet). One-texel grids stage their texels with the geometry, a whole pass at once.
template <int N>
int fwd_batch(int asked, int64_t tiles) {
  if (N == 1) return 64;
  if (N == 16) return tiles <= tiles_at_once(2) ? 16 : tiles <= tiles_at_once(3) ? 8 : 3;
  if (asked != 0) return N == 8 && asked == 16 ? 12 : asked;
  if (N == 8) return tiles <= tiles_at_once(2) ? 64 : tiles <= tiles_at_once(3) ? 32 : 12;
  return N == 2 || tiles <= tiles_at_once(6) ? 64 : 32;
}

// This workgroup's slices of the arrays to zero (the coming backward's texture and record
// gradients). Called when the workgroup has finished blending, so that the stores drain
// while other workgroups blend, and without holding registers during the blend. The stores
// are non-temporal: the zeros are not read again before the backward's atomics, and kept out
// of the caches they do not evict the records and texels other workgroups are reading (at 1M
// splats and 1080p the forward took 0.533 ms with ordinary stores, 0.507 with these).
__device__ __forceinline__ void zero_range(const ZeroRange& z) {
  typedef float v4f __attribute__((ext_vector_type(4)));
  const int64_t per = (z.n_body + (int64_t)gridDim.x - 1) / (int64_t)gridDim.x;
  const int64_t lo = (int64_t)blockIdx.x * per;
  const int64_t hi = lo + per < z.n_body ? lo + per : z.n_body;
  v4f* const q = reinterpret_cast<v4f*>(z.body);
  for (int64_t i = lo + (int64_t)threadIdx.x; i < hi; i += (int64_t)blockDim.x)
    __builtin_nontemporal_store((v4f){0.f, 0.f, 0.f, 0.f}, q + i);
  if (blockIdx.x == 0) {
    if ((int)threadIdx.x < z.n_head) z.head[threadIdx.x] = 0.f;
    if ((int)threadIdx.x < z.n_tail) z.tail[threadIdx.x] = 0.f;
  }
}

__device__ __forceinline__ void zero_slice(const BlendParams& p) {
  zero_range(p.zero[0]);
  zero_range(p.zero[1]);
}

// MIXED: each splat has a grid side of its own (at most N), read from p.grid_n.
template <int N, bool BF16, int B, bool STATS, bool REST, bool MIXED>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(fwd_min_waves<N, B>())))
blend_fwd_kernel(const ViewDev* __restrict__ views, const SplatRec* __restrict__ rec,
                 const uint32_t* __restrict__ pair_vals, const uint32_t* __restrict__ ranges,
                 const void* __restrict__ textures, BlendParams p, float* __restrict__ rgb,
                 float* __restrict__ T_final, uint32_t* __restrict__ n_last, SplitState split,
                 unsigned long long* __restrict__ stats) {
  __shared__ GeoLds<kPassEntries> s_geo;
  __shared__ float4 s_tex[B * TexLayout<N>::kPerSplat];
  // the waves' votes of a pass, of which two can be in use at a time
  __shared__ uint64_t s_mask[2][4];
  __shared__ SlotList<kPassEntries> s_list;
  __shared__ uint64_t s_open[2][4];  // the waves' open pixels, likewise

  const int tile = tile_of_block(p);
  if (tile >= p.total_tiles) {
    if (!REST) zero_slice(p);
    return;
  }
  if (REST && !((split.open_bits[tile >> 5] >> (tile & 31)) & 1u)) return;
  const int vi = view_of_tile(views, p.n_views, tile);
  const ViewDev& V = views[vi];
  const int lt = tile - V.tile_base;
  const int tile_x0 = (lt % V.tiles_x) * p.tile_w;
  const int tile_y0 = (lt / V.tiles_x) * p.tile_h;

  const int tid = threadIdx.x;
  // the wave index is uniform: keep it (and the wave block's geometry) in scalar registers
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int waves_x = p.tile_w >> 3;
  const int n_waves = (int)(blockDim.x >> 6);
  const int bx = (w % waves_x) * 8, by = (w / waves_x) * 8;
  const int lxi = bx + (lane & 7), lyi = by + (lane >> 3);
  const int px = tile_x0 + lxi, py = tile_y0 + lyi;
  const bool inside = px < V.W && py < V.H;
  // pixel centre relative to the wave block's centre and to the tile's (exact half-integers)
  const float lx = (float)(lane & 7) - 3.5f;
  const float ly = (float)(lane >> 3) - 3.5f;
  const float tx = (float)lxi - 0.5f * (float)(p.tile_w - 1);
  const float ty = (float)lyi - 0.5f * (float)(p.tile_h - 1);
  const int tcx = tile_x0 + (p.tile_w >> 1), tcy = tile_y0 + (p.tile_h >> 1);

  const uint32_t rec_base = (uint32_t)vi * (uint32_t)p.P;  // first record of the tile's view
  const uint32_t start = ranges[2 * tile], end = ranges[2 * tile + 1];
  const int64_t pix = (int64_t)V.pix_base + (int64_t)py * V.W + px;  // valid if inside
  float T = 1.0f;
  float acc0 = 0.f, acc1 = 0.f, acc2 = 0.f;
  uint32_t last = start;
  bool done = !inside;  // before the list
  if (REST && inside) {
    const float4 sv = split.fwd_state[pix];
    acc0 = sv.x;
    acc1 = sv.y;
    acc2 = sv.z;
    done = sv.w != 0.f;
    T = T_final[pix];
  }
  // pixels still open, as a lane mask in scalar registers
  uint64_t open = ballot(!done);
  uint32_t st_blend = 0, st_eval = 0;
  bool st_term = false;
  const int kbx = tile_x0 + bx, kby = tile_y0 + by;  // the wave block's first pixel
  int parity = 0, open_set = 0;
  bool all_done = false;
  // whether some pixel of the tile is open; a barrier of the tile (two sets of masks: a wave may
  // set the next call's while another still reads this one's)
  auto tile_open = [&]() {
    uint64_t* const m = s_open[open_set];
    open_set ^= 1;
    if (lane == 0) m[w] = open;
    __syncthreads();
    return uniform64((m[0] | m[1]) | (m[2] | m[3])) != 0;
  };
  // entries of waves that the workgroup does not have
  if (tid < 8 && (tid & 3) >= n_waves) s_mask[tid >> 2][tid & 3] = s_open[tid >> 2][tid & 3] = 0;

  // the record of the lane's entry, loaded a pass ahead
  uint32_t my_rec = lane < pass_size(start, end, kPassEntries) ? pair_vals[start + (uint32_t)lane]
                                                               : rec_base;

  for (uint32_t b = start, n = 0; b < end && !all_done; b += n) {
    // a pass: entries [b, b + n) of the list, one per lane, for the wave's own block
    n = (uint32_t)pass_size(b, end, kPassEntries);
    if (STATS && tid == 0) atomicAdd(&stats[3], (unsigned long long)n);
    uint64_t mine = 0;
    EntryGrid eg{1, 0.f, 0};
    const bool wave_open = open != 0;
    // wave 0 also stores what the blocks share of a splat's geometry
    if (w == 0 || wave_open) {
      bool may = false;
      if (lane < (int)n) {
        const SplatRec R = rec[my_rec];
        const StagedGeo g = stage_geo(R, kbx + 4, kby + 4, tcx, tcy);
        s_geo.store(w, lane, g);
        if constexpr (N == 1) {
          if (w == 0) s_tex[lane] = one_texel<BF16>(textures, my_rec, rec_base, p.spec);
        }
        may = wave_open && block_may_contribute(g, (float)(kbx + 4 - tcx), (float)(kby + 4 - tcy),
                                                kbx, kby, p);
      }
      mine = ballot(may);
    }
    if constexpr (MIXED) {
      if (lane < (int)n) eg = entry_grid<N>(p, my_rec, rec_base);
    }
    if (lane == 0) s_mask[parity][w] = mine;
    __syncthreads();
    const PassVotes votes =
        pass_votes<false>(mine, s_mask[parity], lane, my_rec, s_list);
    if (lane < pass_size(b + n, end, kPassEntries)) my_rec = pair_vals[b + n + (uint32_t)lane];
    parity ^= 1;

    uint64_t ahead = ~0ull;  // entries that no batch has taken yet
    for (int b0 = 0; b0 < votes.total; b0 += B) {
      const int nb = votes.total - b0 < B ? votes.total - b0 : B;
      if constexpr (N == 1)
        ;  // staged with the geometry
      else if constexpr (MIXED)
        stage_texels_mixed<N, BF16>(textures, s_list.entry + b0, s_list.rec + b0, nb, s_tex,
                                    p.spec, eg);
      else
        stage_texels<N, BF16>(textures, s_list.rec + b0, rec_base, nb, s_tex, p.spec, tid);
      if constexpr (N > 1) __syncthreads();
      const uint64_t batch =
          ahead & (~0ull >> (63 - __builtin_amdgcn_readfirstlane((int)s_list.entry[b0 + nb - 1])));
      ahead &= ~batch;
      if (open != 0) {
        // the batch's splats that can reach the wave's block
        uint64_t todo = votes.mine & batch;
        while (todo != 0) {
          const int j = (int)__builtin_ctzll(todo);
          todo &= todo - 1;
          const StagedGeo g = s_geo.load(w, j);
          const PixelEval e = eval_splat(g, lx, ly, tx, ty, p);
          if (STATS) ++st_eval;
          // pixels that the splat stops, and those that blend it
          const uint64_t hit = open & ballot(e.r2 != 0.0f) & ballot(e.alpha >= p.alpha_min);
          const float Tn = T * (1.0f - e.alpha);
          const uint64_t stop = hit & ballot(Tn < p.t_min);
          open = uniform64(open & ~stop);
          const uint64_t blend = hit & ~stop;
          if (STATS && __builtin_amdgcn_inverse_ballot_w64(stop)) st_term = true;
          if (__builtin_amdgcn_inverse_ballot_w64(blend)) {
            if (STATS) ++st_blend;
            float c0, c1, c2;
            // the splat's slot: taken slots of the pass before this entry's
            const int slot = popcount64(votes.any & ((1ull << j) - 1ull)) - b0;
            const float4* tex = s_tex + (N == 1 ? j : slot) * TexLayout<N>::kPerSplat;
            if constexpr (N == 1) {
              const float4 t = tex[0];
              c0 = t.x;
              c1 = t.y;
              c2 = t.z;
            } else {
              int iu, iv;
              float fu, fv;
              if constexpr (MIXED) {
                const int ns = __builtin_amdgcn_readlane(eg.n, j);
                const float sc = __int_as_float(
                    __builtin_amdgcn_readlane(__float_as_int(eg.scale), j));
                grid_coord_n(e.u, sc, ns, iu, fu);
                grid_coord_n(e.v, sc, ns, iv, fv);
              } else {
                grid_coord<N>(e.u, p, iu, fu);
                grid_coord<N>(e.v, p, iv, fv);
              }
              float4 t00, t01, t10, t11;
              load_corners<TexLayout<N>::kRow>(tex + TexLayout<N>::at(iu, iv), t00, t01, t10, t11);
              const float a0 = t00.x + fv * (t01.x - t00.x), b0_ = t10.x + fv * (t11.x - t10.x);
              const float a1 = t00.y + fv * (t01.y - t00.y), b1 = t10.y + fv * (t11.y - t10.y);
              const float a2 = t00.z + fv * (t01.z - t00.z), b2 = t10.z + fv * (t11.z - t10.z);
              c0 = a0 + fu * (b0_ - a0);
              c1 = a1 + fu * (b1 - a1);
              c2 = a2 + fu * (b2 - a2);
            }
            const float wgt = e.alpha * T;
            acc0 += wgt * c0;
            acc1 += wgt * c1;
            acc2 += wgt * c2;
            T = Tn;
            last = b + (uint32_t)j + 1u;
          }
          if (open == 0) break;
        }
      }
      all_done = !tile_open();
      if (all_done) break;
    }
  }

  if (p.tile_work) {
    // the tile's blended span: from its first pair to one past the last pair any pixel
    // blended (the backward's work on this tile)
    __shared__ uint32_t s_span;
    if (tid == 0) s_span = 0u;
    __syncthreads();
    uint32_t span = last - start;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t o = (uint32_t)__shfl_xor((int)span, d, 64);
      span = o > span ? o : span;
    }
    if (lane == 0) atomicMax(&s_span, span);
    __syncthreads();
    if (tid == 0) p.tile_work[tile] = REST ? p.tile_work[tile] + s_span : s_span;
  }
  if (inside) {
    rgb[3 * pix + 0] = acc0 + T * p.bg[0];
    rgb[3 * pix + 1] = acc1 + T * p.bg[1];
    rgb[3 * pix + 2] = acc2 + T * p.bg[2];
    T_final[pix] = T;
    n_last[pix] = last;
  }
  if (!REST && split.open_bits) {
    // a tile with an open pixel takes part in the rest pass, if there is one
    if (tile_open()) {
      if (tid == 0) {
        atomicOr(&split.open_bits[tile >> 5], 1u << (tile & 31));
        atomicOr(split.any_open, 1u);
      }
      if (inside) {
        if (split.mode == kPrefixPass)
          split.fwd_state[pix] = make_float4(
              acc0, acc1, acc2, __builtin_amdgcn_inverse_ballot_w64(open) ? 0.f : 1.f);
        else
          split.n_last_rest[pix] = 0u;
      }
    }
  }
  if (STATS) {
    // per-wave totals (exact in float32: at most 64 x 2^17 per wave), one atomic each
    float red[2] = {(float)st_blend, st_term ? 1.f : 0.f};
    wave_sum_all<2>(red);
    if (lane == 0) {
      atomicAdd(&stats[0], (unsigned long long)red[0]);
      atomicAdd(&stats[1], (unsigned long long)red[1]);
      atomicAdd(&stats[2], 64ull * st_eval);
      if (REST) atomicAdd(&stats[4], (unsigned long long)red[0]);
    }
  }
  if (!REST) zero_slice(p);
}

template <int N, bool BF16, bool STATS, bool REST, bool MIXED>
hipError_t launch_n(const Plan& pl, const gb_splats& sp, const BlendParams& bp,
                    const ViewDev* views, const SplatRec* rec, const uint32_t* pair_vals,
                    const uint32_t* ranges, float* rgb, float* T_final, uint32_t* n_last,
                    const SplitState& split, unsigned long long* stats, hipStream_t s) {
  const dim3 grid((unsigned)(bp.tile_order ? (int64_t)bp.total_tiles
                                           : tile_blocks(bp.total_tiles)));
  const dim3 block((unsigned)(pl.tile_w * pl.tile_h));
#define GBB_FWD_B(BB)                                                                        \
  hipLaunchKernelGGL((blend_fwd_kernel<N, BF16, BB, STATS, REST, MIXED>), grid, block, 0, s,   \
                     views,                                                                   \
                     rec, pair_vals, ranges, sp.textures, bp, rgb, T_final, n_last, split,    \
                     stats)
  const int batch = fwd_batch<N>(pl.batch_fwd, bp.total_tiles);
  if constexpr (N == 1) {
    GBB_FWD_B(64);
  } else if constexpr (N == 16) {
    switch (batch) {
      case 16: GBB_FWD_B(16); break;
      case 8: GBB_FWD_B(8); break;
      default: GBB_FWD_B(3); break;
    }
  } else {
    switch (batch) {
      case 8: GBB_FWD_B(8); break;
      case 12: GBB_FWD_B(12); break;
      case 16: GBB_FWD_B(16); break;
      case 32: GBB_FWD_B(32); break;
      default: GBB_FWD_B(64); break;
    }
  }
#undef GBB_FWD_B
  return hipGetLastError();
}

template <int N, bool BF16, bool MIXED = false>
hipError_t launch_nb(const Plan& pl, const gb_splats& sp, const BlendParams& bp,
                     const ViewDev* views, const SplatRec* rec, const uint32_t* pair_vals,
                     const uint32_t* ranges, float* rgb, float* T_final, uint32_t* n_last,
                     const SplitState& split, unsigned long long* stats, hipStream_t s) {
  const bool rest = split.mode == kRestPass;
  if (stats)
    return rest ? launch_n<N, BF16, true, true, MIXED>(pl, sp, bp, views, rec, pair_vals,
                                                       ranges, rgb, T_final, n_last, split,
                                                       stats, s)
                : launch_n<N, BF16, true, false, MIXED>(pl, sp, bp, views, rec, pair_vals,
                                                        ranges, rgb, T_final, n_last, split,
                                                        stats, s);
  return rest ? launch_n<N, BF16, false, true, MIXED>(pl, sp, bp, views, rec, pair_vals, ranges,
                                                      rgb, T_final, n_last, split, stats, s)
              : launch_n<N, BF16, false, false, MIXED>(pl, sp, bp, views, rec, pair_vals,
                                                       ranges, rgb, T_final, n_last, split,
                                                       stats, s);
}

}  // namespace

// Split of a 4-byte aligned float array into single floats up to its first 16-byte boundary,
// 16-byte stores, and at most 3 trailing floats.
static ZeroRange zero_range_of(float* p, int64_t n) {
  ZeroRange z{nullptr, nullptr, nullptr, 0, 0, 0};
  if (!p || n <= 0) return z;
  int64_t head = (int64_t)((16 - (reinterpret_cast<uintptr_t>(p) & 15)) & 15) / 4;
  if (head > n) head = n;
  const int64_t body = (n - head) / 4;
  z.head = p;
  z.n_head = (int32_t)head;
  z.body = reinterpret_cast<float4*>(p + head);
  z.n_body = body;
  z.tail = p + head + 4 * body;
  z.n_tail = (int32_t)(n - head - 4 * body);
  return z;
}

BlendParams make_blend_params(const Plan& pl, const gb_options& o, int n_views) {
  BlendParams bp;
  const int N = pl.N;
  bp.tex_scale = (float)(N - 1) / (2.0f * o.sigma);
  bp.tex_offset = 0.5f * (float)(N - 1);
  bp.sigma = o.sigma;
  bp.alpha_min = o.alpha_min;
  bp.cull_alpha = 0.99f * o.alpha_min;
  bp.alpha_max = o.alpha_max;
  bp.t_min = o.t_min;
  bp.lp_scale = 1.0f / (2.0f * o.lowpass_var);
  bp.lp_scale2 = 2.0f * bp.lp_scale;
  bp.bg[0] = o.bg[0];
  bp.bg[1] = o.bg[1];
  bp.bg[2] = o.bg[2];
  bp.tile_w = pl.tile_w;
  bp.tile_h = pl.tile_h;
  bp.n_views = n_views;
  bp.P = pl.P;
  bp.total_tiles = (int32_t)pl.total_tiles;
  bp.tile_order = nullptr;
  bp.tile_work = nullptr;
  bp.spec = nullptr;
  bp.d_spec = nullptr;
  bp.grid_n = nullptr;
  bp.grid_at = nullptr;
  bp.zero[0] = ZeroRange{nullptr, nullptr, nullptr, 0, 0, 0};
  bp.zero[1] = ZeroRange{nullptr, nullptr, nullptr, 0, 0, 0};
  return bp;
}

hipError_t launch_blend_fwd(const Plan& pl, const gb_splats& sp, const gb_options& o,
                            const ViewDev* views, int n_views, const SplatRec* rec,
                            const uint32_t* pair_vals, const uint32_t* ranges, float* rgb,
                            float* T_final, uint32_t* n_last, const SplitState& split,
                            uint32_t* tile_work, const uint32_t* tile_order, const float4* spec,
                            unsigned long long* stats,
                            float* zero, int64_t zero_n, float* zero2, int64_t zero2_n,
                            hipStream_t s) {
  BlendParams bp = make_blend_params(pl, o, n_views);
  bp.tile_work = tile_work;
  bp.tile_order = tile_order;
  bp.spec = spec;
  if (split.mode != kRestPass) {
    bp.zero[0] = zero_range_of(zero, zero_n);
    bp.zero[1] = zero_range_of(zero2, zero2_n);
  }
  const bool bf = sp.tex_dtype == GB_BF16;
  if (sp.tex_side) {
    // grids of several sides, staged into the N x N layout (N = 8 or 16, checked by the API)
    bp.grid_n = sp.tex_side;
    bp.grid_at = sp.tex_offset;
    if (pl.N == 16)
      return bf ? launch_nb<16, true, true>(pl, sp, bp, views, rec, pair_vals, ranges, rgb,
                                            T_final, n_last, split, stats, s)
                : launch_nb<16, false, true>(pl, sp, bp, views, rec, pair_vals, ranges, rgb,
                                             T_final, n_last, split, stats, s);
    return bf ? launch_nb<8, true, true>(pl, sp, bp, views, rec, pair_vals, ranges, rgb, T_final,
                                         n_last, split, stats, s)
              : launch_nb<8, false, true>(pl, sp, bp, views, rec, pair_vals, ranges, rgb,
                                          T_final, n_last, split, stats, s);
  }
#define GBB_FWD(NN)                                                                          \
  return bf ? launch_nb<NN, true>(pl, sp, bp, views, rec, pair_vals, ranges, rgb, T_final,   \
                                  n_last, split, stats, s)                                   \
            : launch_nb<NN, false>(pl, sp, bp, views, rec, pair_vals, ranges, rgb, T_final,  \
                                   n_last, split, stats, s)
  switch (pl.N) {
    case 1: GBB_FWD(1);
    case 2: GBB_FWD(2);
    case 4: GBB_FWD(4);
    case 8: GBB_FWD(8);
    case 16: GBB_FWD(16);
    default: return hipErrorInvalidValue;
  }
#undef GBB_FWD
}

}  // namespace gbb
