// Tile rasteriser: front-to-back alpha blending of Eq. (6) with p_i(t) folded
// into each primitive's opacity (Sec. 3.2), and its backward pass.
//
// A tile is 16x16 pixels, four 8x8 quadrants, one pixel of a quadrant per lane
// of a wave. The tile's primitive list is staged through LDS in batches. While
// staging, each entry's alpha-floor ellipse (the pixels where
// opacity * exp(power) can reach 1/255) is tested against the quadrants; only
// the entries that can touch a quadrant are walked there. A skipped entry would
// have failed the 1/255 test at every pixel of the quadrant, so the blend is
// unchanged.
//
// The forward pass gives a wave one, two or all four quadrants of its tile. It
// is bound by instruction issue and by LDS reads: an entry's nine values come
// to every lane, 18 LDS cycles per wave and entry at 128 B per cycle, so one
// quadrant per wave (four waves per tile) keeps a CU's LDS as busy as its four
// SIMDs' vector ALUs. With four pixels per lane an entry is read once per tile
// and its offsets and half of its quadratic form are shared by two quadrants.
// Waves share nothing and meet at no barrier, and a quadrant whose pixels have
// all stopped is left out at once. 300k primitives, 8 views 1352x1014 (43.5k
// tiles): 444 -> 351 us against four waves per tile over lists staged by the
// workgroup.
//
// The forward pass keeps only the final transmittance and the number of list
// entries up to the last contributor per pixel. The backward pass walks the
// list back to front from there, recovering T_i = T_{i+1} / (1 - a_i), and
// works in two phases per group of primitives: (1) each pixel's dL/dpower and
// a_i T_i for the group go into LDS; (2) the lanes regroup as primitives x 16
// pixel columns and accumulate the per-primitive sums over the tile's pixels.
// A reduce-scatter per group combines the columns, leaving each of ten lanes
// of a primitive with one value of its gradient line, and those lanes add the
// tile's share with one FP64 atomic instruction into one 128-byte line. There
// are two kernels: one wave per tile (large launches), and several waves per
// tile in step at barriers: four, batches of 12 primitives (small launches), or
// eight in two roles, batches of 16 (the smallest).
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "shade.h"

namespace g4d {
namespace {

using shade::sc_fma;

// The gradient line's place for the number of tiles in which the record
// blended (with densification statistics on). An add in the same atomic
// instruction as the line's values: a plain store of a flag took the lines
// from the atomics in flight (four-wave backward of 500k primitives, 8 views:
// 1330 us without statistics, 1568 with the store, 1345 with the count).
constexpr int kBlendedSlot = 15;

// Backward LDS slots of one primitive's per-pixel values: pixel (row, col) of
// the tile sits at 16 row + (col ^ 8 [(row >> 1) & 1]); the x-halves of rows
// 2-3 of every four are swapped so that a wave's 8x8 quadrant (4 rows per
// half-wave) hits 32 distinct banks when writing, and 16 columns x 2
// primitives (stride 272 = 16 mod 32) do when reading.
constexpr int kGwStride = 256 + 16;
__device__ __forceinline__ int gw_slot(int row, int col) { return 16 * row + (col ^ (((row >> 1) & 1) << 3)); }

// log2 of opacity * exp(power) at offset (dx, dy) from the mean.
// sa = (u, v, A, B), sb = (C, log2 opacity, ., .) with
// A = -log2(e)/2 conic00, B = -log2(e) conic01, C = -log2(e)/2 conic11.
__device__ __forceinline__ float frag_log2(float dx, float dy, float4 sa, float4 sb) {
  return fmaf(dx, fmaf(sa.z, dx, sa.w * dy), fmaf(sb.x * dy, dy, sb.y));
}

// A record whose colour is NaN (its primitive has a non-finite 4DSH
// coefficient) is staged fully transparent: log2 opacity far below the 1/255
// floor at every pixel (finite, so its reciprocal stays finite), colour 0.
constexpr float kHiddenLog2 = -100.f;

__device__ __forceinline__ float staged_log2_opacity(const Record& r) {
  return isnan(r.c.x) ? kHiddenLog2 : __log2f(r.a.w);
}

__device__ __forceinline__ void stage_record(const Record& r, float4& sa, float4& sb, float4& sc) {
  const bool hide = isnan(r.c.x);
  sa = make_float4(r.a.x, r.a.y, -0.5f * kLog2e * r.b.x, -kLog2e * r.b.y);
  sb = make_float4(-0.5f * kLog2e * r.b.z, staged_log2_opacity(r), r.a.z, 0.f);
  sc = hide ? make_float4(0.f, 0.f, 0.f, 0.f) : make_float4(r.c.x, r.c.y, r.c.z, 0.f);
}

// For the backward, which divides by the opacity: that of a record with none (p(t)
// underflows; only with the ellipse cull off and t_cull near 0 is it binned) is
// held at the same place, so that its gradient is 0 instead of 0 / 0.
__device__ __forceinline__ float nonzero_log2_opacity(float l2o) { return fmaxf(l2o, kHiddenLog2); }

// Whether the record's alpha-floor ellipse (where opacity * exp(power) reaches
// 1/255) meets the 8x8 quadrant q of the tile, whose pixel centres span
// x0 + 8 (q & 1) + [0.5, 7.5], y0 + 8 (q >> 1) + [0.5, 7.5]. In the staged
// form a fragment counts when log2 opacity - Q(dx, dy) >= log2(1/255), with
// Q = A dx^2 + 2 B dx dy + C dy^2 (A = -sa.z, 2B = -sa.w, C = -sb.x), a
// convex quadratic: its minimum over the quadrant is zero when the quadrant
// holds the centre, else it lies on an edge, where Q is a 1D quadratic
// minimised at a clamped point. The bound is loosened (0.1 % + 0.01) so
// rounding never drops a blended pixel.
__device__ __forceinline__ bool quadrant_hit(const float4& sa, const float4& sb, float tile_x0, float tile_y0, int q) {
  const float lim = fmaf(sb.y - kLog2AlphaMin, 1.001f, 0.01f);
  if (!(lim > 0.f)) return false;
  const float A = -sa.z, B = -0.5f * sa.w, C = -sb.x;
  const float ex0 = tile_x0 + 8.f * (q & 1) + 0.5f - sa.x, ex1 = ex0 + 7.f;
  const float ey0 = tile_y0 + 8.f * (q >> 1) + 0.5f - sa.y, ey1 = ey0 + 7.f;
  if (ex0 <= 0.f && ex1 >= 0.f && ey0 <= 0.f && ey1 >= 0.f) return true;
  const auto Q = [&](float dx, float dy) { return fmaf(dx, fmaf(A, dx, 2.f * B * dy), C * dy * dy); };
  const float iA = __builtin_amdgcn_rcpf(A), iC = __builtin_amdgcn_rcpf(C);
  const float ya = __builtin_amdgcn_fmed3f(-B * ex0 * iC, ey0, ey1);
  const float yb = __builtin_amdgcn_fmed3f(-B * ex1 * iC, ey0, ey1);
  const float xa = __builtin_amdgcn_fmed3f(-B * ey0 * iA, ex0, ex1);
  const float xb = __builtin_amdgcn_fmed3f(-B * ey1 * iA, ex0, ex1);
  return fminf(fminf(Q(ex0, ya), Q(ex1, yb)), fminf(Q(xa, ey0), Q(xb, ey1))) <= lim;
}

// stage_record written to LDS in pieces that are whole registers of the loaded
// record (the empty asm statements keep the pieces from being merged into
// wider writes), so a record loaded a batch ahead needs no repacking moves,
// which would wait for the load right after issuing it.
__device__ __forceinline__ void stage_split(const Record& r, float l2o, float4* sa, float4* sb, float4* sc) {
  float2* pa = reinterpret_cast<float2*>(sa);
  pa[0] = make_float2(r.a.x, r.a.y);
  asm volatile("" ::: "memory");
  pa[1] = make_float2(-0.5f * kLog2e * r.b.x, -kLog2e * r.b.y);
  float* pb = reinterpret_cast<float*>(sb);
  pb[0] = -0.5f * kLog2e * r.b.z;
  pb[1] = l2o;
  asm volatile("" ::: "memory");
  pb[2] = r.a.z;
  asm volatile("" ::: "memory");
  pb[3] = 0.f;
  const bool hide = isnan(r.c.x);
  float* pc = reinterpret_cast<float*>(sc);
  pc[0] = hide ? 0.f : r.c.x;
  pc[1] = hide ? 0.f : r.c.y;
  pc[2] = hide ? 0.f : r.c.z;
}

__device__ __forceinline__ int find_view(const ViewDev* views, int n_views, int tile) {
  int lo = 0, hi = n_views - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (views[mid].tile_base <= tile) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// (the controls used here, row mirrors and quad permutations, read a lane of
// the same row for every lane, so the bound control changes nothing; with it
// set the compiler can fold the move into the add that uses it)
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)b, CTRL, 0xF, 0xF, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(b >> 32), CTRL, 0xF, 0xF, false);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Reduce-scatter of ten values over each 16-lane row: afterwards lane c holds
// the row sum of value slot(c), slot = 5 (c >> 3) + 3 ((c >> 2) & 1) +
// 2 ((c >> 1) & 1) + (c & 1), on lanes 0-2, 4-5, 8-10, 12-13 (slot -1
// elsewhere). Pairs: row mirror (c <-> 15 - c), half-row mirror, quad
// (c <-> 3 - c), quad (c <-> c ^ 1); each step keeps half of the values.
template <typename V>
__device__ __forceinline__ V row16_reduce_scatter10(const V (&q)[10], int c, int& slot) {
  const bool hi = c & 8, b = c & 4, cc = c & 2, d = c & 1;
  V r[6], s[4], t[2];
#pragma unroll
  for (int i = 0; i < 5; ++i) r[i] = (hi ? q[i + 5] : q[i]) + dpp<0x140>(hi ? q[i] : q[i + 5]);
  r[5] = 0;
#pragma unroll
  for (int i = 0; i < 3; ++i) s[i] = (b ? r[i + 3] : r[i]) + dpp<0x141>(b ? r[i] : r[i + 3]);
  s[3] = 0;
#pragma unroll
  for (int i = 0; i < 2; ++i) t[i] = (cc ? s[i + 2] : s[i]) + dpp<0x1B>(cc ? s[i] : s[i + 2]);
  const V out = (d ? t[1] : t[0]) + dpp<0xB1>(d ? t[0] : t[1]);
  const int e = 2 * (int)cc + (int)d;
  slot = (e <= (b ? 1 : 2)) ? 5 * (int)hi + 3 * (int)b + e : -1;
  return out;
}

__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, off, 64));
  return v;
}

__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v = min(v, (uint32_t)__shfl_xor((int)v, off, 64));
  return v;
}

// Work items of a launch: tile order[i] (or i) for i < n_items. Without a
// queue, workgroup b takes item b; with one, every workgroup of a grid sized
// to stay resident takes items from the counter at *queue (zero at launch)
// until they run out.
__device__ __forceinline__ bool next_item(const uint32_t* __restrict__ order, uint32_t n_items, uint32_t* queue,
                                          uint32_t* s_item, bool first, int& tile) {
  uint32_t item;
  if (queue) {
    __syncthreads();  // the previous item's LDS readers are done
    if (threadIdx.x == 0) *s_item = atomicAdd(queue, 1u);
    __syncthreads();
    item = *s_item;
  } else {
    if (!first) return false;
    item = blockIdx.x;
  }
  if (item >= n_items) return false;
  tile = order ? (int)order[item] : (int)item;
  return true;
}

// The front-to-back blend of one pixel per lane. A pixel that is done (or
// outside the image) has an infinite floor, so no fragment counts any more.
struct Blend {
  float T, C0, C1, C2, D, floor;
  uint32_t last;  // list position of the last contributor (~0: none)
};

// A staged list entry.
struct Entry {
  float u, v, A, B, C, l2o, z, r, g, b;
  uint32_t pos;
};
template <bool DEPTH>
__device__ __forceinline__ Entry staged_entry(const Record& s) {
  const float4 a = s.a;
  const float2 b = make_float2(s.b.x, s.b.y);
  const float4 c = s.c;
  return Entry{a.x, a.y, a.z, a.w, b.x, b.y, DEPTH ? s.b.z : 0.f, c.x, c.y, c.z, __float_as_uint(c.w)};
}

// One entry over one quadrant: p2 = log2 alpha, pos its list position. done
// is called when the quadrant's last pixel stops.
template <bool DEPTH, typename Done>
__device__ __forceinline__ void blend(Blend& s, float p2, const Entry& e, uint32_t pos, const Done& done) {
  uint64_t go = __ballot(p2 >= s.floor);  // the lanes it counts for
  if (!go) return;
  const float a = __builtin_amdgcn_fmed3f(__builtin_amdgcn_exp2f(p2), 0.f, kAlphaMax);
  const float Tn = fmaf(-a, s.T, s.T);
  const uint64_t stopped = go & __ballot(Tn < kTStop);
  if (__builtin_expect(stopped != 0ull, 0)) {
    asm volatile("");  // kept a branch: seldom taken
    s.floor = p2 >= s.floor && Tn < kTStop ? __builtin_inff() : s.floor;
    go &= ~stopped;
    if (!__any(s.floor < 0.f)) done();
  }
  // the valid lanes' updates, under their execution mask (in one piece: left
  // to itself the compiler tests the mask and branches around them)
  float w;
  uint64_t exec;
  if (DEPTH)
    asm("s_and_saveexec_b64 %[x0], %[m]\n\t"
        "v_mul_f32_e32 %[w], %[a], %[T]\n\t"
        "v_fmac_f32_e32 %[c0], %[w], %[x]\n\t"
        "v_fmac_f32_e32 %[c1], %[w], %[y]\n\t"
        "v_fmac_f32_e32 %[c2], %[w], %[zc]\n\t"
        "v_fmac_f32_e32 %[d], %[w], %[z]\n\t"
        "v_mov_b32_e32 %[T], %[n]\n\t"
        "v_mov_b32_e32 %[l], %[p]\n\t"
        "s_mov_b64 exec, %[x0]"
        : [x0] "=&s"(exec), [w] "=&v"(w), [T] "+v"(s.T), [c0] "+v"(s.C0), [c1] "+v"(s.C1), [c2] "+v"(s.C2),
          [d] "+v"(s.D), [l] "+v"(s.last)
        : [m] "s"(go), [a] "v"(a), [n] "v"(Tn), [x] "v"(e.r), [y] "v"(e.g), [zc] "v"(e.b), [z] "v"(e.z),
          [p] "v"(pos)
        : "scc");
  else
    asm("s_and_saveexec_b64 %[x0], %[m]\n\t"
        "v_mul_f32_e32 %[w], %[a], %[T]\n\t"
        "v_fmac_f32_e32 %[c0], %[w], %[x]\n\t"
        "v_fmac_f32_e32 %[c1], %[w], %[y]\n\t"
        "v_fmac_f32_e32 %[c2], %[w], %[zc]\n\t"
        "v_mov_b32_e32 %[T], %[n]\n\t"
        "v_mov_b32_e32 %[l], %[p]\n\t"
        "s_mov_b64 exec, %[x0]"
        : [x0] "=&s"(exec), [w] "=&v"(w), [T] "+v"(s.T), [c0] "+v"(s.C0), [c1] "+v"(s.C1), [c2] "+v"(s.C2),
          [l] "+v"(s.last)
        : [m] "s"(go), [a] "v"(a), [n] "v"(Tn), [x] "v"(e.r), [y] "v"(e.g), [zc] "v"(e.b), [p] "v"(pos)
        : "scc");
}

// DEPTH: whether the depth plane is written (otherwise its sum is compiled
// out). NQ: quadrants per wave: 4 (one wave per tile, four pixels per lane), 2
// (two waves, one over the tile's upper and one over its lower half) or 1.
// A wave takes 64 list entries at a time, a lane each, tests them against its
// quadrants and stages those that can touch any in LDS of its own, without gaps;
// then it walks them, reading each one's values once for all its quadrants.
template <bool DEPTH, int NQ>
__global__ void __launch_bounds__(256 / NQ) k_raster_forward(const uint32_t* __restrict__ order, uint32_t n_items,
                                                              uint32_t* queue, int n_views,
                                                              const ViewDev* __restrict__ views,
                                                              const uint2* __restrict__ ranges,
                                                              const uint32_t* __restrict__ ival,
                                                              const Record* __restrict__ recs, float bg0, float bg1,
                                                              float bg2, int channels, bool cull,
                                                              float* __restrict__ out_rgb,
                                                              float* __restrict__ out_depth,
                                                              float* __restrict__ out_alpha,
                                                              float* __restrict__ pix_t,
                                                              uint32_t* __restrict__ pix_last) {
  constexpr int kWaves = 4 / NQ;
  // staged: (u, v, A, B) (C, log2 opacity, z, -) (r, g, b, list position; with
  // several quadrants, the position's last six bits and the quadrants);
  // the walk reads up to four entries past the last
  __shared__ Record s_rec[kWaves][68];
  __shared__ uint32_t s_item;
  int tile;
  for (bool first = true; next_item(order, n_items, queue, &s_item, first, tile); first = false) {
  const int vi = find_view(views, n_views, tile);
  const ViewDev& vw = views[vi];
  const int lt = tile - vw.tile_base;
  const int tx = lt % vw.tiles_x, ty = lt / vw.tiles_x;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int q0 = wave * NQ;  // the wave's first quadrant
  const int px = tx * kTile + 8 * (q0 & 1) + (lane & 7), py = ty * kTile + 8 * (q0 >> 1) + (lane >> 3);
  const float tile_x0 = (float)(tx * kTile), tile_y0 = (float)(ty * kTile);
  const float fx[2] = {px + 0.5f, px + 8 + 0.5f};
  const float fy[2] = {py + 0.5f, py + 8 + 0.5f};
  const uint2 rg = ranges[tile];
  const uint32_t count = rg.y - rg.x;
  const uint32_t* list = ival + rg.x;

  Blend s[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const bool inside = px + 8 * (q & 1) < vw.width && py + 8 * (q >> 1) < vw.height;
    s[q] = Blend{1.f, 0.f, 0.f, 0.f, 0.f, inside ? kLog2AlphaMin : __builtin_inff(), ~0u};
  }
  uint32_t d = (uint32_t)lane < count ? list[lane] : 0u;
  for (uint32_t b0 = 0; b0 < count; b0 += 64) {
    uint32_t live = 0u;  // the quadrants with a pixel still going
#pragma unroll
    for (int q = 0; q < NQ; ++q) live |= __any(s[q].floor < 0.f) ? 1u << q : 0u;
    if (!live) break;
    uint32_t hits = 0u;  // per lane: the quadrants its entry can touch
    __builtin_amdgcn_wave_barrier();  // (compiler only: the wave's LDS accesses are in order)
    if (b0 + lane < count) {
      float4 sa, sb, sc;
      stage_record(recs[d], sa, sb, sc);
#pragma unroll
      for (int q = 0; q < NQ; ++q) hits |= !cull || quadrant_hit(sa, sb, tile_x0, tile_y0, q0 + q) ? 1u << q : 0u;
      // the entries that touch a live one, without gaps
      hits &= live;
      const uint64_t in = __ballot(hits != 0u);
      if (hits) {
        const uint32_t slot =
            __builtin_amdgcn_mbcnt_hi((uint32_t)(in >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)in, 0u));
        sc.w = __uint_as_float(NQ > 1 ? hits << 6 | lane : b0 + lane);
        Record& r = s_rec[wave][slot];
        r.a = sa;
        r.b = sb;
        r.c = sc;
      }
    }
    d = b0 + 64 + lane < count ? list[b0 + 64 + lane] : 0u;  // the next entries' records
    int left = __popcll(__ballot(hits != 0u));  // entries to walk
    __builtin_amdgcn_wave_barrier();
    const auto walk = [&](const Entry& e) {
      const uint32_t touch = NQ == 1 ? 1u : (uint32_t)__builtin_amdgcn_readfirstlane(e.pos) >> 6 & live;
      const uint32_t pos = NQ == 1 ? e.pos : (e.pos & 63u) | b0;
      const float dx[2] = {fx[0] - e.u, fx[1] - e.u};
      float row1[2], row2[2];
#pragma unroll
      for (int h = 0; h < (NQ + 1) / 2; ++h) {
        const float dy = fy[h] - e.v;
        row1[h] = e.B * dy;
        row2[h] = fmaf(e.C * dy, dy, e.l2o);
      }
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        if (NQ > 1 && !__builtin_expect((touch >> q) & 1u, 1)) continue;
        const float dq = dx[q & 1];
        const float p2 = fmaf(dq, fmaf(e.A, dq, row1[q >> 1]), row2[q >> 1]);
        blend<DEPTH>(s[q], p2, e, pos, [&] {
          live &= ~(1u << q);
          if (NQ == 1 || !live) left = 0;
        });
      }
    };
    const Record* stage = s_rec[wave];
    int off = 0;
    asm("" : "+v"(off));  // a vector register: the LDS address
    const auto at = [&](int k) {
      return staged_entry<DEPTH>(reinterpret_cast<const Record*>(reinterpret_cast<const char*>(stage) + off)[k]);
    };
    if constexpr (NQ == 1) {
      // few waves, so the longest list's instructions one after the other are
      // the launch's time: no bit scan over gaps (one view of 300k primitives 97
      // -> 84 us), and the next entry's LDS reads are in flight while one is
      // blended (with more quadrants that costs registers: 630 -> 655 us for 16
      // mixed views of 1M)
      if (left) {
        Entry e0 = at(0), e1;
        for (;;) {
          e1 = at(1);
          walk(e0);
          if (left < 2) break;
          e0 = at(2);
          walk(e1);
          if (left < 3) break;
          e1 = at(3);
          walk(e0);
          if (left < 4) break;
          e0 = at(4);
          walk(e1);
          if (left < 5) break;
          off += 4 * (int)sizeof(Record);
          left -= 4;
        }
      }
    } else {
      for (; left > 0; --left, off += (int)sizeof(Record)) walk(at(0));
    }
    __builtin_amdgcn_wave_barrier();
  }
  const long long hw = (long long)vw.width * vw.height;
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int x = px + 8 * (q & 1), y = py + 8 * (q >> 1);
    if (x >= vw.width || y >= vw.height) continue;
    const long long pl = (long long)y * vw.width + x;
    const long long pix = vw.pix_base + pl;
    float* rgb = out_rgb + channels * vw.pix_base + pl;
    rgb[0] = fmaf(s[q].T, bg0, s[q].C0);
    rgb[hw] = fmaf(s[q].T, bg1, s[q].C1);
    if (channels == 3) rgb[2 * hw] = fmaf(s[q].T, bg2, s[q].C2);
    if (DEPTH) out_depth[pix] = s[q].D;
    if (out_alpha) out_alpha[pix] = 1.f - s[q].T;
    pix_t[pix] = s[q].T;
    pix_last[pix] = s[q].last + 1u;
  }
  }  // items
}

// Whether a record's footprint is so elongated (condition number of its
// conic above ~100: 4 det < 0.04 trace^2) that its gradient must be summed in
// FP64: the short axis's share of dL/dconic is then a small part of much
// larger long-axis terms, which float32 tile sums would lose.
__device__ __forceinline__ bool ill_conditioned(const Record& r) {
  const float tr = r.b.x + r.b.z;
  const float det = fmaf(r.b.x, r.b.z, -r.b.y * r.b.y);
  return det < 0.01f * tr * tr;
}

// The ten values of a gradient line (dL/du, dL/dv, dL/dconic (3), dL/d(opacity
// p), dL/drgb (3), dL/dz) from one column's sums. Row moments are about the
// tile's middle row (offset m = k - 7.5) and moved to the primitive's centre:
// with dy = dc + m, sum g dy = dc Sg + Sgm and sum g dy^2 = dc^2 Sg + 2 dc Sgm
// + Sgmm. The 2D-mean, conic and opacity values are linear in the moments, so
// they are formed before the sum over the columns.
template <typename G, bool HAS_D>
__device__ __forceinline__ void form_line(G (&q)[10], bool live, const float4& pa, const float4& pb, G dx, G dc, G Sg,
                                          G Sgm, G Sgmm, float Sr, float Sgc, float Sb, float Sd) {
  const G Sgy = sc_fma(dc, Sg, Sgm);
  const G Sgyy = sc_fma(dc, sc_fma(dc, Sg, (G)2 * Sgm), Sgmm);
  const G k0 = live ? (G)pa.z * (G)(-2.f / kLog2e) : (G)0, k1 = live ? (G)pa.w * (G)(-1.f / kLog2e) : (G)0;
  const G k2 = live ? (G)pb.x * (G)(-2.f / kLog2e) : (G)0;
  const G iop = live ? (G)__builtin_amdgcn_exp2f(-pb.y) : (G)0;
  const G Sgx = dx * Sg, Sgxy = dx * Sgy;
  q[0] = sc_fma(k0, Sgx, k1 * Sgy);
  q[1] = sc_fma(k1, Sgx, k2 * Sgy);
  q[2] = (G)-0.5 * dx * Sgx;
  q[3] = -Sgxy;
  q[4] = (G)-0.5 * Sgyy;
  q[5] = Sg * iop;
  q[6] = Sr;
  q[7] = Sgc;
  q[8] = Sb;
  q[9] = HAS_D ? (G)Sd : (G)0;
}

// Phase 2 of the backward for primitive j2 of the staged batch and pixel
// column c2: its share of the tile sums over the rows of the quadrants where
// it blended, formed into the ten values of its gradient line (before the row
// sum). G is the type of the position moments and of the line (float, or
// double for ill-conditioned footprints); the colour and depth sums stay float.
template <typename G, bool HAS_D>
__device__ __forceinline__ void phase2_line(G (&q)[10], bool live, int j2, int c2, int tx, int ty,
                                            const float4* __restrict__ s_a, const float4* __restrict__ s_b,
                                            const uint32_t* __restrict__ s_act, const float* __restrict__ s_g,
                                            const float* __restrict__ s_w, const float4* __restrict__ s_pix) {
  // Row moments are taken about the tile's middle row (offset m = k - 7.5)
  // and moved to the primitive's centre afterwards: with dy = dc + m,
  // sum g dy = dc Sg + Sgm and sum g dy^2 = dc^2 Sg + 2 dc Sgm + Sgmm.
  G Sg = 0, Sgm = 0, Sgmm = 0;
  float Sr = 0.f, Sgc = 0.f, Sb = 0.f, Sd = 0.f;
  G dx = 0, dc = 0;
  if (live) {
    const float4 sa = s_a[j2];
    dx = (G)(tx * kTile + c2) + (G)0.5 - (G)sa.x;
    dc = (G)(ty * kTile) + (G)8 - (G)sa.y;
    const uint32_t act = (s_act[c2 >> 3] | (s_act[2 + (c2 >> 3)] << 16)) >> j2;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      if (!((act >> (16 * half)) & 1u)) continue;
#pragma unroll
      for (int k = 8 * half; k < 8 * half + 8; ++k) {
        const int p = k * 16 + c2;
        const int slot = j2 * kGwStride + gw_slot(k, c2);
        const float2 gw = make_float2(s_g[slot], s_w[slot]);
        const float4 pd = s_pix[p];
        const G g = gw.x;
        const G m = (G)k - (G)7.5;
        Sg += g;
        Sgm = sc_fma(g, m, Sgm);
        Sgmm = sc_fma(g, m * m, Sgmm);
        Sr = fmaf(gw.y, pd.x, Sr);
        Sgc = fmaf(gw.y, pd.y, Sgc);
        Sb = fmaf(gw.y, pd.z, Sb);
        if (HAS_D) Sd = fmaf(gw.y, pd.w, Sd);
      }
    }
  }
  form_line<G, HAS_D>(q, live, s_a[j2], s_b[j2], dx, dc, Sg, Sgm, Sgmm, Sr, Sgc, Sb, Sd);
}

// HAS_D / HAS_A: whether dL/d(depth) and dL/d(alpha) are given (otherwise
// their terms are compiled out). With loss.kind set, dl_rgb is the rendered
// image and the image loss is folded in (LossArgs).
template <bool HAS_D, bool HAS_A, bool PIPE>
__global__ void __launch_bounds__(PIPE ? 512 : 256, PIPE ? 4 : 5) k_raster_backward(
    const uint32_t* __restrict__ order, uint32_t n_items, uint32_t* queue, int n_views,
    const ViewDev* __restrict__ views, const uint2* __restrict__ ranges, const uint32_t* __restrict__ ival,
    const Record* __restrict__ recs, float bg0, float bg1, float bg2, const float* __restrict__ dl_rgb,
    const float* __restrict__ dl_depth, const float* __restrict__ dl_alpha, const float* __restrict__ pix_t,
    const uint32_t* __restrict__ pix_last, double* __restrict__ grad2d, bool mark_blended, bool cull,
    LossArgs loss) {
  // Entries per batch, staged batches and batches' products in LDS, the wave
  // that stages.
  //
  // Four waves: 12 entries rather than 16: the per-(primitive, pixel) buffers
  // then take 26 KB, the workgroup 31.6 KB of LDS, and with at most 96 VGPRs
  // (the launch bound) five workgroups share a CU instead of four; the backward
  // is bound by issue stalls more than by its instruction count, so the fifth
  // wave per SIMD outweighs the third more barriers per entry. The batch's 12
  // primitives also leave wave 0 free for the staging in phase 2.
  //
  // PIPE, eight waves in two roles, phase 2 of a batch beside phase 1 of the
  // next: the longest list's batches, one after the other, are the time of a
  // launch of few tiles. 76 KB of LDS, two workgroups per CU. Batches of 12 took
  // 39 us and of 8 (four workgroups per CU) 53 where 16 take 32.
  constexpr int kBatch = PIPE ? 16 : 12, kStages = PIPE ? 3 : 2, kProducts = PIPE ? 2 : 1, kStager = PIPE ? 4 : 0;
  __shared__ float4 s_a2[kStages][kBatch], s_b2[kStages][kBatch], s_c2[kStages][kBatch];
  __shared__ uint32_t s_d2[kStages][kBatch];
  __shared__ uint32_t s_qm2[kStages][kBatch];
  __shared__ uint32_t s_ill2[kStages];  // per staged batch: bit j when entry j's footprint is ill-conditioned
  __shared__ uint32_t s_act2[kProducts][4];  // per quadrant: bit j when entry j blended somewhere in it
  __shared__ float s_g2[kProducts][kBatch * kGwStride];  // dL/dpower per (primitive, pixel)
  __shared__ float s_w2[kProducts][kBatch * kGwStride];  // a_i T_i per (primitive, pixel)
  __shared__ float4 s_pix[256];
  __shared__ uint32_t s_max;
  __shared__ uint32_t s_item;
  __shared__ float s_loss[4];

  int tile;
  for (bool first = true; next_item(order, n_items, queue, &s_item, first, tile); first = false) {
  const int vi = find_view(views, n_views, tile);
  const ViewDev& vw = views[vi];
  const int lt = tile - vw.tile_base;
  const int tx = lt % vw.tiles_x, ty = lt / vw.tiles_x;
  const int wave = PIPE ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : threadIdx.x >> 6, lane = threadIdx.x & 63;
  const bool blends = !PIPE || wave < 4;
  const int lx = (wave & 1) * 8 + (lane & 7), ly = (wave >> 1 & 1) * 8 + (lane >> 3);
  const int p_self = ly * 16 + lx;                  // row-major pixel index within the tile
  const int q_self = gw_slot(ly, lx);               // this pixel's slot in s_g / s_w
  const int px = tx * kTile + lx, py = ty * kTile + ly;
  const bool inside = blends && px < vw.width && py < vw.height;
  const float fx = px + 0.5f, fy = py + 0.5f;
  const float tile_x0 = (float)(tx * kTile), tile_y0 = (float)(ty * kTile);
  const uint2 rg = ranges[tile];
  const int count = (int)(rg.y - rg.x);

  if (threadIdx.x == 0) s_max = 0u;
  float T = 1.f, gC0 = 0.f, gC1 = 0.f, gC2 = 0.f, gD = 0.f, gA = 0.f, lsum = 0.f;
  uint32_t last = 0;
  if (inside) {
    const long long hw = (long long)vw.width * vw.height;
    const long long pl = (long long)py * vw.width + px;
    const long long pix = vw.pix_base + pl;
    const float* g = dl_rgb + 3 * vw.pix_base + pl;
    if (loss.kind) {
      // with a folded loss the rgb input is the rendered image: the loss
      // term and dL/dC of each channel against the target, formed as the
      // image-loss kernel forms them
      const float* tg = loss.target + 3 * vw.pix_base + pl;
      lsum = shade::loss_term(loss.kind, g[0] - tg[0], loss.scale, gC0) +
             shade::loss_term(loss.kind, g[hw] - tg[hw], loss.scale, gC1) +
             shade::loss_term(loss.kind, g[2 * hw] - tg[2 * hw], loss.scale, gC2);
    } else {
      gC0 = g[0];
      gC1 = g[hw];
      gC2 = g[2 * hw];
    }
    if (HAS_D) gD = dl_depth[pix];
    if (HAS_A) gA = dl_alpha[pix];
    T = pix_t[pix];
    last = pix_last[pix];
  }
  if (blends) s_pix[p_self] = make_float4(gC0, gC1, gC2, gD);
  if (loss.kind && blends) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) lsum += __shfl_xor(lsum, off, 64);
    if (lane == 0) s_loss[wave] = lsum;
  }
  const uint32_t wave_last = wave_max_u32(last);
  // batches ending at or before every lane's last contributor need no
  // per-entry list-position test
  const uint32_t wave_first_last = wave_min_u32(last);
  __syncthreads();
  if (lane == 0 && wave_last) atomicMax(&s_max, wave_last);
  // the tile's loss, summed over its pixels
  if (loss.kind && threadIdx.x == 0) loss.part[tile] = s_loss[0] + s_loss[1] + s_loss[2] + s_loss[3];
  // Only the dot product of this pixel's output gradient with the colour,
  // depth and alpha of everything behind the current primitive (normalised by
  // the transmittance after it) enters dL/da; it starts at the background.
  float beta = fmaf(gC0, bg0, fmaf(gC1, bg1, gC2 * bg2));
  __syncthreads();
  const int max_last = (int)s_max;

  const int c2 = lane & 15;  // phase 2: pixel column
  const int b_first = ((max_last + kBatch - 1) / kBatch - 1) * kBatch;
  // Staging pipeline (lanes < kBatch of one wave): the record of the batch
  // after the one in LDS and the list index of the batch after that are in
  // flight, so no wait covers a load issued in the same batch.
  Record nxt;
  uint32_t nxt_d = 0, nn_d = 0;
  // Run by the whole wave: lanes < kBatch stage entry e0 + lane; then four
  // lanes per entry test its quadrants on the staged values (taken from the
  // staging lane by a shuffle) and a ballot gathers the four bits.
  auto stage = [&](int e0, int bb) {
    const int t = lane;
    const float l2o = nonzero_log2_opacity(staged_log2_opacity(nxt));
    if (t < kBatch && e0 + t < count) {
      stage_split(nxt, l2o, &s_a2[bb][t], &s_b2[bb][t], &s_c2[bb][t]);
      s_d2[bb][t] = nxt_d;
    }
    const int src = t >> 2;
    float4 qa, qb;
    qa.x = __shfl(nxt.a.x, src, 64);
    qa.y = __shfl(nxt.a.y, src, 64);
    qa.z = -0.5f * kLog2e * __shfl(nxt.b.x, src, 64);
    qa.w = -kLog2e * __shfl(nxt.b.y, src, 64);
    qb.x = -0.5f * kLog2e * __shfl(nxt.b.z, src, 64);
    qb.y = __shfl(l2o, src, 64);
    const bool hit = e0 + src < count && (!cull || quadrant_hit(qa, qb, tile_x0, tile_y0, t & 3));
    const uint64_t bits = __ballot(hit);
    if (t < kBatch) s_qm2[bb][t] = (uint32_t)(bits >> (4 * t)) & 0xFu;
    const uint64_t ill = __ballot(t < kBatch && e0 + t < count && ill_conditioned(nxt));
    if (t == 0) s_ill2[bb] = (uint32_t)ill & 0xFFFFu;
  };
  if (wave == kStager && b_first >= 0) {
    if (lane < kBatch && b_first + lane < count) {
      nxt_d = ival[rg.x + b_first + lane];
      nxt = recs[nxt_d];
    }
    stage(b_first, 0);
    const int e1 = b_first - kBatch + lane;
    if (lane < kBatch && e1 >= 0) {
      nxt_d = ival[rg.x + e1];
      nxt = recs[nxt_d];
    }
    const int e2n = e1 - kBatch;
    if (lane < kBatch && e2n >= 0) nn_d = ival[rg.x + e2n];
  }
  // ---- phase 1: this lane's pixel, back to front over the batch from b0 in
  // stage buffer sb, the products to buffer pb ----
  const auto phase1 = [&](int b0, int sb, int pb) {
    // the stage buffer's first entry as a vector register, so each entry's
    // LDS reads are immediate offsets from it
    int bv;
    asm volatile("v_mov_b32 %0, %1" : "=v"(bv) : "s"(sb * kBatch));
    const float4* s_a = &s_a2[0][0] + bv;
    const float4* s_b = &s_b2[0][0] + bv;
    const float4* s_c = &s_c2[0][0] + bv;
    const uint32_t* s_qm = s_qm2[sb];
    float *s_g = s_g2[pb], *s_w = s_w2[pb];
    // entries that can reach this wave's quadrant before its last contributor
    uint32_t todo;
    {
      const uint32_t qm = lane < kBatch ? s_qm[lane] : 0u;
      todo = (uint32_t)__ballot(((qm >> wave) & 1u) && (uint32_t)(b0 + lane) < wave_last);
    }
    uint32_t blended = 0u;
    // CHECK: test the entry's list position against this lane's last
    // contributor (not needed when the batch ends at or before every lane's)
    auto entry = [&](int j, const float4& sa, const float4& sb, const float4& sc, auto check) {
      const float p2 = frag_log2(fx - sa.x, fy - sa.y, sa, sb);
      const bool valid = (!decltype(check)::value || (uint32_t)(b0 + j) < last) && (p2 >= kLog2AlphaMin);
      if (!__any(valid)) return;
      const float G = __builtin_amdgcn_exp2f(p2);
      const float a = valid ? __builtin_amdgcn_fmed3f(G, 0.f, kAlphaMax) : 0.f;
      T = T * __builtin_amdgcn_rcpf(1.f - a);
      float dot = fmaf(gC0, sc.x, fmaf(gC1, sc.y, gC2 * sc.z));
      if (HAS_D) dot = fmaf(gD, sb.z, dot);
      if (HAS_A) dot += gA;
      const float s = dot - beta;
      beta = fmaf(a, s, beta);
      // dL/dpower = dL/da * a for an unclamped alpha (a = G), zero where the
      // clamp holds; a skipped fragment has a = 0
      const float w = a * T;
      const float g = G < kAlphaMax ? w * s : 0.f;
      s_g[j * kGwStride + q_self] = g;
      s_w[j * kGwStride + q_self] = w;
      blended |= 1u << j;
    };
    // back to front over the set entries; j is a constant in every unrolled
    // step, so the LDS addresses are immediate offsets
    if ((uint32_t)b0 + kBatch <= wave_first_last) {
#pragma unroll
      for (int j = kBatch - 1; j >= 0; --j) {
        if (!((todo >> j) & 1u)) continue;
        entry(j, s_a[j], s_b[j], s_c[j], std::false_type{});
      }
    } else {
#pragma unroll
      for (int j = kBatch - 1; j >= 0; --j) {
        if (!((todo >> j) & 1u)) continue;
        entry(j, s_a[j], s_b[j], s_c[j], std::true_type{});
      }
    }
    if (lane == 0) s_act2[pb][wave] = blended;
  };
  // ---- phase 2: primitive j2 = 4 rank + lane / 16, pixel column c2, rows of
  // active quadrants: the lane's value of the gradient line, if any ----
  const auto phase2 = [&](int rank, bool live, int sb, int pb, int& slot_q, double& val, uint32_t& d_atom) {
    const int j2 = 4 * rank + (lane >> 4);
    // FP64 sums for the waves whose four primitives include an
    // ill-conditioned footprint (wave-uniform)
    if ((s_ill2[sb] >> (4 * rank)) & 0xFu) {
      double q[10];
      phase2_line<double, HAS_D>(q, live, j2, c2, tx, ty, s_a2[sb], s_b2[sb],
                                  s_act2[pb], s_g2[pb], s_w2[pb], s_pix);
      val = row16_reduce_scatter10(q, c2, slot_q);
    } else {
      float q[10];
      phase2_line<float, HAS_D>(q, live, j2, c2, tx, ty, s_a2[sb], s_b2[sb],
                                  s_act2[pb], s_g2[pb], s_w2[pb], s_pix);
      val = (double)row16_reduce_scatter10(q, c2, slot_q);
    }
    // the record blended in this tile: one more lane counts it in the
    // gradient line's last value
    if (mark_blended && c2 == 15 && (((s_act2[pb][0] | s_act2[pb][1] | s_act2[pb][2] | s_act2[pb][3]) >> j2) & 1u)) {
      slot_q = kBlendedSlot;
      val = 1.0;
    }
    d_atom = s_d2[sb][j2];
  };
  // stages the batch from e0 in buffer sb and advances the loads
  const auto stage_next = [&](int e0, int sb) {
    stage(e0, sb);
    const int e1 = e0 - kBatch + lane;
    if (lane < kBatch && e1 >= 0) {
      nxt_d = nn_d;
      nxt = recs[nxt_d];
    }
    const int e2n = e1 - kBatch;
    if (lane < kBatch && e2n >= 0) nn_d = ival[rg.x + e2n];
  };
  // ten lanes of the primitive's row each add one value of its gradient
  // line, so a wave's atomics for a primitive share one 128-byte line
  const auto add_line = [&](bool live, int slot_q, double val, uint32_t d_atom) {
    if (live && slot_q >= 0 && val != 0.0)
      unsafeAtomicAdd(grad2d + (size_t)d_atom * kGrad2dStride + slot_q, val);
  };
  if constexpr (PIPE) {
    // one barrier per batch: waves 0-3 blend batch b0 while waves 4-7 sum the
    // one before, four primitives each, and wave 4 stages the next
    int sc = 0, sp = 2, cur = 0;  // stage buffers of this batch and the one before; product buffer of this one
    for (int b0 = b_first; b_first >= 0 && b0 > -2 * kBatch; b0 -= kBatch) {
      const int sn = sc == 2 ? 0 : sc + 1;
      __syncthreads();
      if (blends) {
        if (b0 >= 0) phase1(b0, sc, cur);
      } else {
        const bool live = b0 < b_first && b0 + kBatch + 4 * (wave - 4) + (lane >> 4) < count;
        int slot_q = -1;
        double val = 0.0;
        uint32_t d_atom = 0u;
        phase2(wave - 4, live, sp, cur ^ 1, slot_q, val, d_atom);
        // (the buffer was last read before the last barrier)
        if (wave == kStager && b0 >= kBatch) stage_next(b0 - kBatch, sn);
        add_line(live, slot_q, val, d_atom);
      }
      sp = sc;
      sc = sn;
      cur ^= 1;
    }
  } else {
    int buf = 0;
    for (int b0 = b_first; b0 >= 0; b0 -= kBatch, buf ^= 1) {
      __syncthreads();
      phase1(b0, buf, 0);
      __syncthreads();
      // Waves 1-3 sum four primitives each; wave 0, which stages the next
      // batch (into the other buffer, read by nobody until the next barrier),
      // none, so the waves reach that barrier together.
      const bool live = wave > 0 && b0 + 4 * (wave - 1) + (lane >> 4) < count;
      int slot_q = -1;
      double val = 0.0;
      uint32_t d_atom = 0u;
      if (wave > 0) phase2(wave - 1, live, buf, 0, slot_q, val, d_atom);
      if (wave == kStager && b0 >= kBatch) stage_next(b0 - kBatch, buf ^ 1);
      add_line(live, slot_q, val, d_atom);
    }
  }
  }  // items
}

// ---- the backward with one wave per tile ----
// Four pixels per lane, one of each quadrant, as in the forward with four
// quadrants per wave: an entry's values are read from LDS once per tile
// instead of once per quadrant, and the quadrants share its offsets. Groups of
// four entries alternate between phase 1 and phase 2 (lane 4 c + e sums entry
// e of the group over pixel column c) within the wave: no barrier, no idle
// wave. What bounds it is vector instruction issue (SQ counters: 0.93 of the
// launch); the kernel of four waves per tile moves 1.7 times the LDS
// instructions and keeps LDS and vector ALUs about equally busy. 10 KB of LDS
// and 128 registers let four waves share a SIMD. 300k primitives, 8 views
// 1352x1014: 1100 -> 862 us (with three waves per SIMD 1005, and 1045 with the
// LDS reads of phase 2 not all ahead of its sums).
constexpr int kWaveBatch = 4;
// LDS slots of the group's per-pixel values: the tile's left and right 8
// columns in planes of their own, in each an entry's 16 rows x 8 columns. A
// quadrant's write is 64 consecutive words (lane = pixel); a read of one row
// takes four entries x 16 columns at strides of 8 and 32 words mod 64, so all
// lanes hit distinct banks.
constexpr int kWavePrim = 128 + 8;
constexpr int kWavePlane = kWaveBatch * kWavePrim;
static_assert(kWavePrim % 64 == 8 && kWavePlane % 64 == 32, "bank-conflict-free strides");

using f32x4 = __attribute__((__vector_size__(4 * sizeof(float)))) float;

// Sum of ten values over the 16 columns c of lanes 4 c + e: two reduce-scatter
// steps over lane bits 5 and 4, each a register swap between wave halves (then
// rows) and an add, and an all-reduce of the three values left over the row's
// four columns. Lane 4 c + e ends with value line_slot(lane) of entry e
// (unspecified where that is -1).
__device__ __forceinline__ int line_slot(int lane) {
  const int b4 = (lane >> 4) & 1, i = (lane >> 2) & 3;
  return i < 3 - b4 ? 5 * (lane >> 5) + 3 * b4 + i : -1;
}
__device__ __forceinline__ float swap_add32(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float swap_add16(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float columns_reduce_scatter10(const float (&q)[10], int lane) {
  float r[5], s[3];
#pragma unroll
  for (int i = 0; i < 5; ++i) r[i] = swap_add32(q[i], q[i + 5]);
  s[0] = swap_add16(r[0], r[3]);
  s[1] = swap_add16(r[1], r[4]);
  s[2] = swap_add16(r[2], r[2]);
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    s[i] += dpp<0x128>(s[i]);  // row rotations by 8 and 4 lanes: the row's other three columns
    s[i] += dpp<0x124>(s[i]);
  }
  const int i = (lane >> 2) & 3;
  return i == 0 ? s[0] : (i == 1 ? s[1] : s[2]);
}
// The same for the FP64 lines of ill-conditioned footprints (seldom taken).
__device__ __forceinline__ double columns_reduce_scatter10(const double (&q)[10], int lane) {
  const int slot = line_slot(lane);
  double out = 0.0;
#pragma unroll
  for (int i = 0; i < 10; ++i) {
    double v = q[i];
#pragma unroll
    for (int off = 4; off < 64; off <<= 1) v += __shfl_xor(v, off, 64);
    out = slot == i ? v : out;
  }
  return out;
}

// v in the lanes of mask, else 0.
__device__ __forceinline__ float masked(float v, uint64_t mask) {
  float r;
  asm("v_cndmask_b32_e64 %0, 0, %1, %2" : "=v"(r) : "v"(v), "s"(mask));
  return r;
}

// One pixel's state back to front.
template <bool HAS_D, bool HAS_A>
struct BackPixel {
  float T, beta, g0, g1, g2, gD, gA;
  uint32_t last;
};

template <bool HAS_D, bool HAS_A>
__global__ void __launch_bounds__(64, 4) k_raster_backward_wave(
    const uint32_t* __restrict__ order, uint32_t n_items, uint32_t* queue, int n_views,
    const ViewDev* __restrict__ views, const uint2* __restrict__ ranges, const uint32_t* __restrict__ ival,
    const Record* __restrict__ recs, float bg0, float bg1, float bg2, const float* __restrict__ dl_rgb,
    const float* __restrict__ dl_depth, const float* __restrict__ dl_alpha, const float* __restrict__ pix_t,
    const uint32_t* __restrict__ pix_last, double* __restrict__ grad2d, bool mark_blended, bool cull, LossArgs loss) {
  // per (entry, pixel): dL/dpower, then a_i T_i
  __shared__ float s_gw[4 * kWavePlane];
  constexpr int kW = 2 * kWavePlane;
  __shared__ Record s_rec[32];           // staged: (u, v, A, B) (C, log2 opacity, z, record) (r, g, b, -)
  static_assert(4 * 256 <= 4 * kWavePlane, "the output gradients pass through s_gw");
  static_assert(sizeof(s_gw) + sizeof(s_rec) <= 10240, "16 workgroups per CU");

  int tile;
  uint32_t* s_item = reinterpret_cast<uint32_t*>(s_gw);  // between tiles
  for (bool first = true; next_item(order, n_items, queue, s_item, first, tile); first = false) {
  const int vi = find_view(views, n_views, tile);
  const ViewDev& vw = views[vi];
  const int lt = tile - vw.tile_base;
  const int tx = lt % vw.tiles_x, ty = lt / vw.tiles_x;
  const int lane = threadIdx.x;
  const int px = tx * kTile + (lane & 7), py = ty * kTile + (lane >> 3);
  const float tile_x0 = (float)(tx * kTile), tile_y0 = (float)(ty * kTile);
  const float fx[2] = {px + 0.5f, px + 8 + 0.5f};
  const float fy[2] = {py + 0.5f, py + 8 + 0.5f};
  const uint2 rg = ranges[tile];
  const uint32_t* list = ival + rg.x;

  BackPixel<HAS_D, HAS_A> s[4];
  uint32_t most[4], least[4];  // per quadrant: largest and smallest last contributor
  float lsum = 0.f;
  bool nf = false;
  // every load first, from the pixel or (outside the image) its nearest one
  const long long hw = (long long)vw.width * vw.height;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const long long pl = (long long)min(py + 8 * (q >> 1), vw.height - 1) * vw.width + min(px + 8 * (q & 1), vw.width - 1);
    const long long pix = vw.pix_base + pl;
    const float* g = dl_rgb + 3 * vw.pix_base + pl;
    s[q].g0 = g[0];
    s[q].g1 = g[hw];
    s[q].g2 = g[2 * hw];
    s[q].gD = HAS_D ? dl_depth[pix] : 0.f;
    s[q].gA = HAS_A ? dl_alpha[pix] : 0.f;
    s[q].T = pix_t[pix];
    s[q].last = pix_last[pix];
  }
  if (loss.kind) {
    // with a folded loss the rgb input is the rendered image: the loss term
    // and dL/dC of each channel against the target, formed as the image-loss
    // kernel forms them
    float tg[4][3];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const long long pl = (long long)min(py + 8 * (q >> 1), vw.height - 1) * vw.width + min(px + 8 * (q & 1), vw.width - 1);
      const float* t = loss.target + 3 * vw.pix_base + pl;
      tg[q][0] = t[0];
      tg[q][1] = t[hw];
      tg[q][2] = t[2 * hw];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float l = shade::loss_term(loss.kind, s[q].g0 - tg[q][0], loss.scale, s[q].g0) +
                      shade::loss_term(loss.kind, s[q].g1 - tg[q][1], loss.scale, s[q].g1) +
                      shade::loss_term(loss.kind, s[q].g2 - tg[q][2], loss.scale, s[q].g2);
      lsum += px + 8 * (q & 1) < vw.width && py + 8 * (q >> 1) < vw.height ? l : 0.f;
    }
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (px + 8 * (q & 1) >= vw.width || py + 8 * (q >> 1) >= vw.height)
      s[q] = BackPixel<HAS_D, HAS_A>{1.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0u};
    // only the dot product of the pixel's output gradient with the colour,
    // depth and alpha of everything behind the current primitive (normalised
    // by the transmittance after it) enters dL/da; it starts at the background
    s[q].beta = fmaf(s[q].g0, bg0, fmaf(s[q].g1, bg1, s[q].g2 * bg2));
    nf = nf || !isfinite(s[q].g0) || !isfinite(s[q].g1) || !isfinite(s[q].g2) || (HAS_D && !isfinite(s[q].gD));
    most[q] = __builtin_amdgcn_readfirstlane(wave_max_u32(s[q].last));
    least[q] = __builtin_amdgcn_readfirstlane(wave_min_u32(s[q].last));
  }
  const bool tile_nf = __any(nf);
  if (loss.kind) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) lsum += __shfl_xor(lsum, off, 64);
    if (lane == 0) loss.part[tile] = lsum;  // the tile's loss, summed over its pixels
  }
  // phase 2's left operand of row k: value lane & 3 (r, g, b, depth) of pixel
  // (k, lane >> 2)'s output gradient, turned through LDS
  float grad[16];
#pragma unroll
  for (int q = 0; q < 4; ++q)
    reinterpret_cast<float4*>(s_gw)[((lane >> 3) + 8 * (q >> 1)) * 16 + (lane & 7) + 8 * (q & 1)] =
        make_float4(s[q].g0, s[q].g1, s[q].g2, s[q].gD);
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int k = 0; k < 16; ++k) grad[k] = s_gw[64 * k + lane];
  __builtin_amdgcn_wave_barrier();

  const int total = (int)max(max(most[0], most[1]), max(most[2], most[3]));
  // the list from its last contributor to its front, 32 entries at a time:
  // lane i tests entry i against the upper two quadrants, lane 32 + i against
  // the lower two
  const int se = lane & 31, sq = (lane >> 5) * 2;
  const uint32_t most0 = sq ? most[2] : most[0], most1 = sq ? most[3] : most[1];
  int b0 = ((total + 31) / 32 - 1) * 32;
  uint32_t d = b0 >= 0 && b0 + se < total ? list[b0 + se] : 0u;
  for (; b0 >= 0; b0 -= 32) {
    uint32_t hits = 0u;  // per lane: which of its two quadrants the entry can touch, before their last contributors
    bool ill = false, clamp = false;
    __builtin_amdgcn_wave_barrier();
    const uint32_t p = (uint32_t)(b0 + se);
    if (p < (uint32_t)total) {
      const Record r = recs[d];
      float4 sa, sb, sc;
      stage_record(r, sa, sb, sc);
      sb.y = nonzero_log2_opacity(sb.y);
      sb.w = __uint_as_float(d);
      s_rec[se].a = sa;  // (both lanes of an entry write the same)
      s_rec[se].b = sb;
      s_rec[se].c = sc;
      hits = (p < most0 && (!cull || quadrant_hit(sa, sb, tile_x0, tile_y0, sq)) ? 1u : 0u) |
             (p < most1 && (!cull || quadrant_hit(sa, sb, tile_x0, tile_y0, sq + 1)) ? 2u : 0u);
      ill = ill_conditioned(r);
      clamp = ill || sb.y >= kLog2AlphaMax;
    }
    if (b0 >= 32) d = list[b0 - 32 + se];  // the next entries' records
    const uint64_t touched = __ballot(hits != 0u);
    uint32_t any = (uint32_t)touched | (uint32_t)(touched >> 32);
    const uint32_t ills = (uint32_t)__ballot(ill), clamps = (uint32_t)__ballot(clamp);
    __builtin_amdgcn_wave_barrier();
    while (any) {
      // ---- phase 1: up to four entries, back to front ----
      uint32_t js = 0u, acts = 0u;  // per entry of the group, 8 bits each: its staged index; the quadrants it blended in
      int n = 0;
      uint32_t group = 0u;
      do {
        const int j = 31 - __builtin_clz(any);
        any &= ~(1u << j);
        group |= 1u << j;
        const uint32_t touch = __builtin_amdgcn_readlane(hits, j) | __builtin_amdgcn_readlane(hits, j + 32) << 2;
        const uint32_t pos = b0 + j;
        const float4 sa = s_rec[j].a;
        const float2 sb = make_float2(s_rec[j].b.x, s_rec[j].b.y);
        const float z = HAS_D ? s_rec[j].b.z : 0.f;
        const float4 sc = s_rec[j].c;
        const float dx[2] = {fx[0] - sa.x, fx[1] - sa.x};
        float row1[2], row2[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const float dy = fy[h] - sa.y;
          row1[h] = sa.w * dy;
          row2[h] = fmaf(sb.x * dy, dy, sb.y);
        }
        float* gp = s_gw + n * kWavePrim + lane;
        uint32_t act = 0u;
        uint32_t clamped = (clamps >> j) & 1u;  // whether its alpha can reach the clamp
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int at = (q & 1) * kWavePlane + (q >> 1) * 64;
          uint64_t valid = 0ull;
          float p2 = 0.f;
          if (__builtin_expect((touch >> q) & 1u, 1)) {
            const float dq = dx[q & 1];
            p2 = fmaf(dq, fmaf(sa.z, dq, row1[q >> 1]), row2[q >> 1]);
            valid = __ballot(p2 >= kLog2AlphaMin);
            if (pos >= least[q]) {  // (entries before every lane's last contributor need no test)
              asm volatile("");
              valid &= __ballot(pos < s[q].last);
            }
          }
          if (__builtin_expect(valid == 0ull, 0)) {
            gp[at] = 0.f;
            gp[at + kW] = 0.f;
            continue;
          }
          const float G = __builtin_amdgcn_exp2f(p2);
          float a = masked(G, valid);
          asm("" : "+s"(clamped));  // tested anew each time: kept as a flag it would cost vector instructions
          if (__builtin_expect(clamped != 0u, 0)) {
            asm volatile("");
            a = fminf(a, kAlphaMax);
          }
          s[q].T = s[q].T * __builtin_amdgcn_rcpf(1.f - a);
          float dot = fmaf(s[q].g0, sc.x, fmaf(s[q].g1, sc.y, s[q].g2 * sc.z));
          if (HAS_D) dot = fmaf(s[q].gD, z, dot);
          if (HAS_A) dot += s[q].gA;
          const float t = dot - s[q].beta;
          s[q].beta = fmaf(a, t, s[q].beta);
          // dL/dpower = dL/da * a for an unclamped alpha (a = G), zero where
          // the clamp holds; a skipped fragment has a = 0
          const float w = a * s[q].T;
          float g = w * t;
          asm("" : "+s"(clamped));
          if (__builtin_expect(clamped != 0u, 0)) {
            asm volatile("");
            g = G < kAlphaMax ? g : 0.f;
          }
          gp[at] = g;
          gp[at + kW] = w;
          act |= 1u << q;
        }
        js |= (uint32_t)j << (8 * n);
        acts |= act << (8 * n);
        ++n;
      } while (n < kWaveBatch && any);
      __builtin_amdgcn_wave_barrier();
      // ---- phase 2: lane 4 c + e, entry e over pixel column c ----
      const int c = lane >> 2, e = lane & 3;
      const int je = (js >> (8 * e)) & 31;
      const uint32_t act = (acts >> (8 * e)) & 0xFu;
      const float4 pa = s_rec[je].a, pb = s_rec[je].b;
      const int at = (c >> 3) * kWavePlane + e * kWavePrim + (c & 7);
      const float* gp = s_gw + at;
      float gk[16], wk[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) wk[k] = gp[kW + 8 * k];
#pragma unroll
      for (int k = 0; k < 16; ++k) gk[k] = gp[8 * k];
      __builtin_amdgcn_sched_barrier(0);  // all reads in flight before the first sum
      // the colour and depth sums as 4x4x1 products of 16 blocks (block =
      // column): the pixel's output gradient times the four entries' a_i T_i,
      // one FMA each in the order of the rows, the tile's halves apart
      f32x4 sw[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        sw[0] = __builtin_amdgcn_mfma_f32_4x4x1f32(grad[k], wk[k], sw[0], 0, 0, 0);
        sw[1] = __builtin_amdgcn_mfma_f32_4x4x1f32(grad[8 + k], wk[8 + k], sw[1], 0, 0, 0);
      }
      // the row moments, rows k and 15 - k (at -m and m) together
      float Sg = 0.f, Sgm = 0.f, Sgmm = 0.f;
#pragma unroll
      for (int k = 8; k < 16; ++k) {
        const float m = (float)k - 7.5f, both = gk[k] + gk[15 - k];
        Sg += both;
        Sgm = fmaf(gk[k] - gk[15 - k], m, Sgm);
        Sgmm = fmaf(both, m * m, Sgmm);
      }
      if (tile_nf) {
        // a non-finite output gradient stays out of the sums of the entries
        // that did not blend in its quadrant (0 times it is NaN)
        if (!((act >> (c >> 3)) & 1u)) sw[0] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (!((act >> (2 + (c >> 3))) & 1u)) sw[1] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
      const f32x4 S = sw[0] + sw[1];
      // (the slots past the group's end hold what an earlier group left there;
      // their lanes' sums stay in their lanes and are not added)
      int slot = e < n ? line_slot(lane) : -1;
      bool add;
      double val;
      if (__builtin_expect((ills & group) != 0u, 0)) {
        // FP64 moments where the four include an ill-conditioned footprint
        double dg = 0.0, dgm = 0.0, dgmm = 0.0;
#pragma unroll 1
        for (int k = 0; k < 16; ++k) {
          const double g = gp[8 * k], m = (double)k - 7.5;
          dg += g;
          dgm = fma(g, m, dgm);
          dgmm = fma(g, m * m, dgmm);
        }
        double q[10];
        const double dx = (double)(tx * kTile + c) + 0.5 - (double)pa.x;
        const double dc = (double)(ty * kTile) + 8.0 - (double)pa.y;
        form_line<double, HAS_D>(q, true, pa, pb, dx, dc, dg, dgm, dgmm, S[0], S[1], S[2], S[3]);
        val = columns_reduce_scatter10(q, lane);
        add = val != 0.0;
      } else {
        float q[10];
        const float dx = (float)(tx * kTile + c) + 0.5f - pa.x;
        const float dc = (float)(ty * kTile) + 8.f - pa.y;
        form_line<float, HAS_D>(q, true, pa, pb, dx, dc, Sg, Sgm, Sgmm, S[0], S[1], S[2], S[3]);
        const float v = columns_reduce_scatter10(q, lane);
        add = v != 0.f;
        val = (double)v;
      }
      const uint32_t rec = __float_as_uint(pb.w);
      // the record blended in this tile: one more lane counts it in the
      // gradient line's last value
      if (mark_blended && c == 15 && e < n && act) {
        slot = kBlendedSlot;
        val = 1.0;
        add = true;
      }
      // ten lanes of an entry each add one value of its gradient line, so a
      // wave's atomics for an entry share one 128-byte line
      if (slot >= 0 && add) unsafeAtomicAdd(grad2d + (size_t)rec * kGrad2dStride + slot, val);
      __builtin_amdgcn_wave_barrier();
    }
  }
  }  // items
}

// Workgroups of Kernel that stay resident on the current device (looked up
// once per kernel, which has one workgroup size, and device: kernels of one
// signature hold from 16 waves a CU to 32, in workgroups of one wave to eight).
template <auto Kernel>
unsigned resident_grid(int threads) {
  constexpr int kDevs = 64;
  static std::atomic<unsigned> cached[kDevs] = {};
  int dev = 0, per_cu = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 1024;
  if (dev >= 0 && dev < kDevs)
    if (const unsigned g = cached[dev]) return g;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, Kernel, threads, 0) != hipSuccess || per_cu < 1 || cus < 1)
    return 1024;
  const unsigned g = (unsigned)(per_cu * cus);
  if (dev >= 0 && dev < kDevs) cached[dev] = g;
  return g;
}

// Grid of a launch over total_tiles items: one workgroup per item, or with
// a queue, `blocks` workgroups (-1: as many as stay resident).
template <auto Kernel>
unsigned item_grid(int threads, int total_tiles, uint32_t* queue, int blocks, hipStream_t s) {
  unsigned grid = (unsigned)total_tiles;
  if (queue) {
    const unsigned want = blocks > 0 ? (unsigned)blocks : resident_grid<Kernel>(threads);
    grid = std::min(grid, want);
    launch_fill_u32(queue, 1, 0u, s);
  }
  return grid;
}

template <bool DEPTH, int NQ>
void launch_fwd(int total_tiles, const uint32_t* order, uint32_t* queue, int blocks, int n_views,
                const ViewDev* views, const uint2* ranges, const uint32_t* ival, const Record* rec_sorted,
                const float* bg, int channels, bool cull, float* out_rgb, float* out_depth, float* out_alpha,
                float* pix_t, uint32_t* pix_last, hipStream_t s) {
  const unsigned grid = item_grid<k_raster_forward<DEPTH, NQ>>(256 / NQ, total_tiles, queue, blocks, s);
  hipLaunchKernelGGL((k_raster_forward<DEPTH, NQ>), dim3(grid), dim3(256 / NQ), 0, s, order, (uint32_t)total_tiles,
                     queue, n_views, views, ranges, ival, rec_sorted, bg[0], bg[1], bg[2], channels, cull, out_rgb,
                     out_depth, out_alpha, pix_t, pix_last);
}

}  // namespace

void launch_raster_forward(int total_tiles, const uint32_t* order, uint32_t* queue, int blocks, int n_views,
                           const ViewDev* views, const uint2* ranges, const uint32_t* ival,
                           const Record* rec_sorted, const float* bg, int channels, bool cull, float* out_rgb,
                           float* out_depth, float* out_alpha, float* pix_t, uint32_t* pix_last, hipStream_t s) {
  if (total_tiles == 0) return;
  // Quadrants per wave, by the waves that the launch would have (8192 stay
  // resident): wider waves share more work per entry, but leave a small launch
  // too few waves and a long tail. Measured (us, one / two / four quadrants per
  // wave; 300k primitives, views of 1352x1014), with the depth plane: 5.4k tiles 89 /
  // 119 / 179, 10.9k 128 / 147 / 193, 16.3k 159 / 170 / 207, 21.8k 212 / 197 / 252,
  // 32.6k 314 / 276 / 297, 43.5k 415 / 364 / 350; without: 80 / 112 / 170, 117 / 146 /
  // 189, 146 / 166 / 203, 186 / 189 / 230, 278 / 259 / 286, 364 / 340 / 331.
#define G4D_FWD(D, NQ)                                                                                            \
  launch_fwd<D, NQ>(total_tiles, order, queue, blocks, n_views, views, ranges, ival, rec_sorted, bg, channels, cull, \
                    out_rgb, out_depth, out_alpha, pix_t, pix_last, s)
  const bool d = out_depth != nullptr;
  if (total_tiles < 2 * 8192) {
    if (d) G4D_FWD(true, 1); else G4D_FWD(false, 1);
  } else if (total_tiles < 5 * 8192) {
    if (d) G4D_FWD(true, 2); else G4D_FWD(false, 2);
  } else {
    if (d) G4D_FWD(true, 4); else G4D_FWD(false, 4);
  }
#undef G4D_FWD
}

namespace {
template <bool HD, bool HA>
void launch_bwd(int total_tiles, const uint32_t* order, uint32_t* queue, int blocks, int n_views,
                const ViewDev* views, const uint2* ranges, const uint32_t* ival, const Record* rec_sorted,
                const float* bg, const float* dl_rgb, const float* dl_depth, const float* dl_alpha,
                const float* pix_t, const uint32_t* pix_last, double* grad2d, bool mark_blended, bool cull,
                const LossArgs& loss, hipStream_t s) {
  // One wave per tile once the launch has five times the 4096 such waves that
  // stay resident: fewer waves leave a tail of long tiles, each walked by one
  // wave. Measured (us, four waves per tile / one; 300k primitives at
  // 1352x1014): 5.4k tiles 200 / 320, 10.9k 290 / 365, 16.3k 421 / 458, 21.8k
  // 562 / 516, 32.6k 844 / 693, 43.5k 1100 / 862.
  // Below 2048 tiles two roles of waves (four waves per tile / two roles): 300
  // tiles 368 / 259, 690 174 / 122, 1200 199 / 143, 1900 138 / 134, 2961 162 / 165,
  // 5.4k 205 / 229; the 5k-primitive step's 520 tiles 45.6 / 32.
  if (total_tiles >= 5 * 4096) {
    const unsigned grid = item_grid<k_raster_backward_wave<HD, HA>>(64, total_tiles, queue, blocks, s);
    hipLaunchKernelGGL((k_raster_backward_wave<HD, HA>), dim3(grid), dim3(64), 0, s, order, (uint32_t)total_tiles,
                       queue, n_views, views, ranges, ival, rec_sorted, bg[0], bg[1], bg[2], dl_rgb, dl_depth, dl_alpha,
                       pix_t, pix_last, grad2d, mark_blended, cull, loss);
    return;
  }
  const bool pipe = total_tiles < 2048;
  const auto kernel = pipe ? k_raster_backward<HD, HA, true> : k_raster_backward<HD, HA, false>;
  const unsigned threads = pipe ? 512 : 256;
  const unsigned grid = pipe ? item_grid<k_raster_backward<HD, HA, true>>(512, total_tiles, queue, blocks, s)
                             : item_grid<k_raster_backward<HD, HA, false>>(256, total_tiles, queue, blocks, s);
  hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), 0, s, order, (uint32_t)total_tiles, queue, n_views, views,
                     ranges, ival, rec_sorted, bg[0], bg[1], bg[2], dl_rgb, dl_depth, dl_alpha, pix_t, pix_last,
                     grad2d, mark_blended, cull, loss);
}
}  // namespace

void launch_raster_backward(int total_tiles, const uint32_t* order, uint32_t* queue, int blocks, int n_views,
                            const ViewDev* views, const uint2* ranges, const uint32_t* ival,
                            const Record* rec_sorted, const float* bg, const float* dl_rgb, const float* dl_depth,
                            const float* dl_alpha, const float* pix_t, const uint32_t* pix_last, double* grad2d,
                            bool mark_blended, bool cull, const LossArgs& loss, hipStream_t s) {
  if (total_tiles == 0) return;
#define G4D_BWD(HD, HA)                                                                                          \
  launch_bwd<HD, HA>(total_tiles, order, queue, blocks, n_views, views, ranges, ival, rec_sorted, bg, dl_rgb,      \
                     dl_depth, dl_alpha, pix_t, pix_last, grad2d, mark_blended, cull, loss, s)
  if (dl_depth && dl_alpha) G4D_BWD(true, true);
  else if (dl_depth) G4D_BWD(true, false);
  else if (dl_alpha) G4D_BWD(false, true);
  else G4D_BWD(false, false);
#undef G4D_BWD
}

}  // namespace g4d
