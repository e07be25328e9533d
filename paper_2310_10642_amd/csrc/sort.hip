// Binning of active records into 16x16 tiles, ordered by (tile, depth).
//
// The tile rasteriser the paper adapts (Sec. 3.2, last paragraph of
// "Representation of 4D Gaussian") needs, per tile, the primitives whose
// footprint covers it in front-to-back order. This is an LSD radix sort on the
// composite key (global tile, depth, view*n + index), arranged so the low-order
// passes run on the active records before they are duplicated per tile:
//   1. stable 4-pass radix sort of the active records by float depth bits
//      (ties keep (view, index) order from the compaction scan);
//   2. emission of one (tile, record) instance per tile of the record's
//      rectangle that its alpha-floor ellipse reaches, in that order;
//   3. stable radix sort of the instances by global tile id.
// Every pass is stable, so the result equals a stable sort by (tile, depth)
// of the instances emitted in (view, index) order.
#include <utility>
#include "chain.h"
#include "g4d_common.h"

namespace g4d {
namespace {

constexpr int kThreads = 256;
constexpr int kItems = 16;
constexpr int kTileElems = kThreads * kItems;  // 4096 elements per block tile
static_assert(kTileElems == 4 * 1024, "the scan tile is four waves of 1024 elements");

__device__ __forceinline__ uint32_t dev_n(const uint32_t* n_dev, uint32_t n_max) {
  return n_dev ? min(*n_dev, n_max) : n_max;
}

// A record's footprint for binning: centre, conic, the bound L on
// Q = a dx^2 + 2 b dx dy + c dy^2 below which opacity * exp(-Q/2) reaches
// 1/255 (loosened by 0.1 % + 0.02 so FP32 rounding never drops a blended
// pixel), the ellipse's half-height ymax, the dy of its leftmost point ey
// (the rightmost is at -ey), and its tile rectangle. D = a c - b^2.
struct Footprint {
  float u, v, b, L, D, ia, ymax, ey;
  uint32_t x0, x1, y0, y1;
};

// Footprint and row_span are written with explicit rounding and no
// contraction, so the instance count of a record and its emission agree. The
// square roots are the hardware instruction (within about an ulp; it is the
// same instruction in both kernels, and far inside the spans' slack).
__device__ __forceinline__ Footprint footprint(const Record& r) {
#pragma clang fp contract(off)
  Footprint f;
  f.u = r.a.x;
  f.v = r.a.y;
  const float a = r.b.x, c = r.b.z;
  f.b = r.b.y;
  // 2 ln(255 opacity) = 2 ln2 (log2 opacity - log2(1/255))
  const float L0 = __fmul_rn(2.f * 0.69314718055994531f, __fsub_rn(__log2f(r.a.w), kLog2AlphaMin));
  f.L = __fmaf_rn(L0, 1.001f, 0.02f);
  const float p = __fmul_rn(f.b, f.b);
  f.D = __fsub_rn(__fmaf_rn(a, c, -p), __fmaf_rn(f.b, f.b, -p));  // product error recovered
  f.ia = __builtin_amdgcn_rcpf(a);
  const float iD = __builtin_amdgcn_rcpf(f.D);
  f.ymax = __builtin_amdgcn_sqrtf(fmaxf(__fmul_rn(__fmul_rn(f.L, a), iD), 0.f));
  const float xmax = __builtin_amdgcn_sqrtf(fmaxf(__fmul_rn(__fmul_rn(f.L, c), iD), 0.f));
  f.ey = __fmul_rn(__fmul_rn(f.b, xmax), __builtin_amdgcn_rcpf(c));
  if (!(f.L > 0.f) || !(f.D > 0.f) || !(f.ymax >= 0.f)) f.ymax = -1.f;  // no tile
  f.L = __fmul_rn(a, f.L);                           // kept as a L from here on
  const uint32_t rx = __float_as_uint(r.b.w), ry = __float_as_uint(r.c.w);
  f.x0 = rx & 0xFFFFu;
  f.x1 = rx >> 16;
  f.y0 = ry & 0xFFFFu;
  f.y1 = ry >> 16;
  return f;
}

// Tiles [xa, xb) of tile row ty whose pixel centres the ellipse Q <= L can
// reach, within the rectangle. Over the row's band of pixel-centre rows the
// ellipse's left edge x(dy) = (-b dy - sqrt(a L - D dy^2)) / a is convex and
// its right edge concave, so their extremes over the band sit at the
// leftmost / rightmost points clamped to the band. exact = false: the
// rectangle's whole row.
__device__ __forceinline__ void row_span(const Footprint& f, uint32_t ty, bool exact, uint32_t& xa, uint32_t& xb) {
#pragma clang fp contract(off)
  constexpr float kEps = 0.01f;  // px
  if (!exact) {
    xa = f.x0;
    xb = f.x1;
    return;
  }
  xa = xb = f.x0;
  const float band0 = __fsub_rn((float)(ty * kTile) + (0.5f - kEps), f.v);
  const float band1 = __fsub_rn((float)(ty * kTile) + (15.5f + kEps), f.v);
  const float lo = fmaxf(band0, -f.ymax), hi = fminf(band1, f.ymax);
  if (!(lo <= hi)) return;
  const float dl = fminf(fmaxf(f.ey, lo), hi), dr = fminf(fmaxf(-f.ey, lo), hi);
  const float sl = __builtin_amdgcn_sqrtf(fmaxf(__fsub_rn(f.L, __fmul_rn(f.D, __fmul_rn(dl, dl))), 0.f));
  const float sr = __builtin_amdgcn_sqrtf(fmaxf(__fsub_rn(f.L, __fmul_rn(f.D, __fmul_rn(dr, dr))), 0.f));
  const float left = __fadd_rn(f.u, __fmul_rn(__fsub_rn(-__fmul_rn(f.b, dl), sl), f.ia));
  const float right = __fadd_rn(f.u, __fmul_rn(__fadd_rn(-__fmul_rn(f.b, dr), sr), f.ia));
  // tile tx holds centres 16 tx + [0.5, 15.5]
  const float ta = ceilf(__fmul_rn(__fsub_rn(left, 15.5f + kEps), 1.f / kTile));
  const float tb = floorf(__fmul_rn(__fadd_rn(right, kEps - 0.5f), 1.f / kTile)) + 1.f;
  const float fx0 = (float)f.x0, fx1 = (float)f.x1;
  xa = (uint32_t)fminf(fmaxf(ta, fx0), fx1);
  xb = (uint32_t)fminf(fmaxf(tb, (float)xa), fx1);
}

// Exclusive scan of one value per thread across a block of T threads.
template <int T = kThreads>
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* s_wave, uint32_t& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t x = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t y = __shfl_up(x, off, 64);
    if (lane >= off) x += y;
  }
  if (lane == 63) s_wave[wave] = x;
  __syncthreads();
  uint32_t base = 0;
  total = 0;
#pragma unroll
  for (int w = 0; w < T / 64; ++w) {
    const uint32_t c = s_wave[w];
    base += (w < wave) ? c : 0u;
    total += c;
  }
  __syncthreads();
  return base + x - v;
}

// ---------------------------------------------------------------- scan ----
// The scan's block tile: wave w holds elements [1024 w, 1024 w + 1024) of the
// tile, and lane l the four 16-byte groups 256 j + 4 l (j = 0..3), so every
// load and store instruction of a wave covers 1 KB of consecutive words and
// the element order is (wave, group, lane, word). The arrays are the
// library's own 256-byte-aligned buffers, so a full tile's groups are aligned.
__device__ __forceinline__ size_t scan_group(int j) {
  return (size_t)(threadIdx.x >> 6) * 1024 + (size_t)j * 256 + (size_t)(threadIdx.x & 63) * 4;
}

__device__ __forceinline__ uint4 load_group(const uint32_t* __restrict__ p, size_t e, size_t n, bool full) {
  if (full) return *reinterpret_cast<const uint4*>(p + e);
  return make_uint4(e < n ? p[e] : 0u, e + 1 < n ? p[e + 1] : 0u, e + 2 < n ? p[e + 2] : 0u, e + 3 < n ? p[e + 3] : 0u);
}

__global__ void __launch_bounds__(kThreads) k_scan_reduce(const uint32_t* __restrict__ in, const uint32_t* n_dev,
                                                           uint32_t n_max, uint32_t* __restrict__ bsum) {
  __shared__ uint32_t s_wave[4];
  const uint32_t n = dev_n(n_dev, n_max);
  const size_t base = (size_t)blockIdx.x * kTileElems;
  if (base >= n) return;
  const bool full = base + kTileElems <= n;
  uint32_t acc = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint4 g = load_group(in, base + scan_group(j), n, full);
    acc += g.x + g.y + g.z + g.w;
  }
  uint32_t total;
  block_exclusive_scan(acc, s_wave, total);
  if (threadIdx.x == 0) bsum[blockIdx.x] = total;
}

// ---------------------------------------------------------- compaction ----
// The active pairs in (view, primitive) order: ckey = depth key, cval = pair
// id. The bits and a count per 256-pair group come from the preprocess; a
// workgroup takes 16 groups, four to a wave, which loads its 16 units' words
// at once and then writes each unit's keys as one run. Its first position is
// the sum of the groups before it: of whole 4096-group sums (coarse, when
// there are that many groups) and of the counts after them. view_end[v] gets
// the position after view v's last pair. hist (zeroed; or null): the keys'
// four digit counts are added to hist[4][256].
constexpr int kCompactGroups = 16;
constexpr int kCoarseGroups = kTileElems;  // groups per coarse sum
__global__ void __launch_bounds__(kThreads) k_compact(PairBits pb, const uint32_t* __restrict__ count,
                                                       uint32_t* __restrict__ hist,
                                                       const uint32_t* __restrict__ coarse, uint32_t groups,
                                                       const uint32_t* __restrict__ dkey, uint32_t* __restrict__ ckey,
                                                       uint32_t* __restrict__ cval, uint32_t* __restrict__ total,
                                                       uint32_t* __restrict__ view_end) {
  __shared__ uint32_t s_wave[4];
  __shared__ uint32_t s_hist[4][256];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t g0 = blockIdx.x * kCompactGroups;
  if (hist)
    for (int d = 0; d < 4; ++d) s_hist[d][threadIdx.x] = 0u;  // (a barrier follows)
  const uint32_t u0 = (g0 + 4 * wave) * 4, u_end = groups * 4;
  // lane j < 16: the wave's unit j
  uint2 act = make_uint2(0u, 0u), lst = make_uint2(0u, 0u);
  uint32_t first = 0u;
  if (lane < 16 && u0 + lane < u_end) {
    act = reinterpret_cast<const uint2*>(pb.active)[u0 + lane];
    lst = reinterpret_cast<const uint2*>(pb.listed)[u0 + lane];
    first = pb.first[u0 + lane];
  }
  const uint32_t before = (lane < 4 * wave && g0 + lane < groups) ? count[g0 + lane] : 0u;
  const uint32_t c0 = coarse ? g0 / kCoarseGroups * kCoarseGroups : 0u;
  uint32_t part = 0;
  if (coarse)
    for (uint32_t i = threadIdx.x; i < c0 / kCoarseGroups; i += kThreads) part += coarse[i];
  for (uint32_t i = c0 + threadIdx.x; i < g0; i += kThreads) part += count[i];
  uint32_t run;
  block_exclusive_scan(part, s_wave, run);  // contains barriers; run = the pairs before the block
  uint32_t b16 = before;
#pragma unroll
  for (int m = 8; m; m >>= 1) b16 += __shfl_xor(b16, m);
  run += (uint32_t)__builtin_amdgcn_readfirstlane((int)b16);
  const uint32_t vg = pb.units / 4;
  uint32_t v = (g0 + 4 * wave) / vg, g = (g0 + 4 * wave) - v * vg;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    if (u0 + j >= u_end) break;
    if (j % 4 == 0) {
      if (j) {
        if (++g == vg) ++v, g = 0;
      }
      if (g == 0 && v > 0 && lane == 0) view_end[v - 1] = run;
    }
    const uint32_t bx = (uint32_t)__builtin_amdgcn_readlane((int)act.x, j);
    const uint32_t by = (uint32_t)__builtin_amdgcn_readlane((int)act.y, j);
    if (((lane < 32 ? bx : by) >> (lane & 31)) & 1u) {
      const uint32_t below = __builtin_amdgcn_mbcnt_hi(by, __builtin_amdgcn_mbcnt_lo(bx, 0u));
      const uint32_t lx = (uint32_t)__builtin_amdgcn_readlane((int)lst.x, j);
      const uint32_t ly = (uint32_t)__builtin_amdgcn_readlane((int)lst.y, j);
      const uint32_t at = (uint32_t)__builtin_amdgcn_readlane((int)first, j) +
                          __builtin_amdgcn_mbcnt_hi(ly, __builtin_amdgcn_mbcnt_lo(lx, 0u));
      const uint32_t key = dkey[at];
      ckey[run + below] = key;
      cval[run + below] = v * (uint32_t)pb.n + g * 256u + 64u * (j % 4) + lane;
      if (hist) {
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          // (the top digits are often the whole wave's: one addition)
          const uint32_t digit = (key >> (8 * d)) & 255u;
          const uint32_t d0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)digit);
          const uint64_t in = __ballot(true), same = __ballot(digit == d0);
          if (d >= 2 && in == same) {
            if (below == 0) atomicAdd(&s_hist[d][d0], (uint32_t)__popcll(in));
          } else {
            atomicAdd(&s_hist[d][digit], 1u);
          }
        }
      }
    }
    run += (uint32_t)(__popc(bx) + __popc(by));
  }
  if (u0 < u_end && u0 + 16 >= u_end && lane == 0) {
    *total = run;
    view_end[v] = run;
  }
  if (hist) {
    __syncthreads();
    for (int d = 0; d < 4; ++d) {
      const uint32_t c = s_hist[d][threadIdx.x];
      if (c) atomicAdd(&hist[d * 256 + threadIdx.x], c);
    }
  }
}

// ---------------------------------------------------------- radix sort ----
// Workgroups are dispatched round-robin over the 8 XCDs; the sort's blocks
// take their ranges of tiles in XCD-major order, so the digit runs that
// consecutive ranges write next to each other come from one XCD's L2.
__device__ __forceinline__ uint32_t sort_block() {
  const uint32_t g = gridDim.x;
  return (g & 7u) ? blockIdx.x : (blockIdx.x & 7u) * (g >> 3) + (blockIdx.x >> 3);
}

__device__ __forceinline__ void block_range(uint32_t n, uint32_t tile, int grid, uint32_t& t0, uint32_t& t1) {
  const uint32_t tiles = (n + tile - 1) / tile;
  const uint32_t tpb = (tiles + grid - 1) / grid;
  t0 = min(sort_block() * tpb, tiles);
  t1 = min(t0 + tpb, tiles);
}

// K: uint32_t, or uint16_t for keys below 2^16 (the tile ids of a round).
// T threads, 16 keys each per tile (the scatter's tile).
template <typename K, int T>
__global__ void __launch_bounds__(T) k_rs_upsweep(const K* __restrict__ keys, const uint32_t* n_dev, uint32_t n_max,
                                                   int shift, int bits, uint32_t* __restrict__ counts) {
  constexpr int kWaves = T / 64, kElems = T * kItems;
  __shared__ uint32_t hist[kWaves][256];
  const uint32_t n = dev_n(n_dev, n_max);
  const int wave = threadIdx.x >> 6;
  for (int i = threadIdx.x; i < kWaves * 256; i += T) hist[i >> 8][i & 255] = 0u;
  __syncthreads();
  uint32_t t0, t1;
  block_range(n, kElems, gridDim.x, t0, t1);
  const uint32_t mask = (1u << bits) - 1u;
  for (uint32_t t = t0; t < t1; ++t) {
    const size_t tb = (size_t)t * kElems;
    if (tb + kElems <= n) {
      // full tile: 16-byte loads (four, or two of 16-bit keys), all in flight together
      constexpr int kVec = 16 / (int)sizeof(K);
      uint4 q[kItems / kVec];
#pragma unroll
      for (int i = 0; i < kItems / kVec; ++i)
        q[i] = reinterpret_cast<const uint4*>(keys + tb)[i * T + threadIdx.x];
#pragma unroll
      for (int i = 0; i < kItems / kVec; ++i) {
        const uint32_t w[4] = {q[i].x, q[i].y, q[i].z, q[i].w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (sizeof(K) == 4) {
            atomicAdd(&hist[wave][(w[j] >> shift) & mask], 1u);
          } else {
            atomicAdd(&hist[wave][((w[j] & 0xFFFFu) >> shift) & mask], 1u);
            atomicAdd(&hist[wave][(w[j] >> (16 + shift)) & mask], 1u);
          }
        }
      }
    } else {
      for (int i = 0; i < kItems; ++i) {
        const size_t idx = tb + (size_t)i * T + threadIdx.x;
        if (idx < n) atomicAdd(&hist[wave][((uint32_t)keys[idx] >> shift) & mask], 1u);
      }
    }
  }
  __syncthreads();
  const uint32_t d = threadIdx.x;
  if (T == 256 || d < 256u) {
    uint32_t c = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) c += hist[w][d];
    counts[(size_t)d * gridDim.x + sort_block()] = c;
  }
}

// One 256-thread block per digit: exclusive scan of counts[digit][0..grid) in
// place and the digit's total into digit_tot[digit]. Each thread takes eight
// consecutive counts of a 2048-count chunk, so a row of up to 2048 blocks'
// counts is one block-wide scan, and the small workgroup finds a CU beside
// another stream's work.
constexpr int kRowScanPer = 8;
__global__ void __launch_bounds__(kThreads) k_rs_rowscan(uint32_t* __restrict__ counts, int grid,
                                                         uint32_t* __restrict__ digit_tot) {
  __shared__ uint32_t s_wave[4];
  uint32_t* row = counts + (size_t)blockIdx.x * grid;
  uint32_t carry = 0;
  for (int c0 = 0; c0 < grid; c0 += kThreads * kRowScanPer) {
    const int b0 = c0 + (int)threadIdx.x * kRowScanPer;
    uint32_t v[kRowScanPer];
    uint32_t sum = 0;
#pragma unroll
    for (int i = 0; i < kRowScanPer; ++i) {
      v[i] = b0 + i < grid ? row[b0 + i] : 0u;
      sum += v[i];
    }
    uint32_t tot;
    uint32_t ex = carry + block_exclusive_scan(sum, s_wave, tot);  // contains barriers
#pragma unroll
    for (int i = 0; i < kRowScanPer; ++i) {
      if (b0 + i < grid) row[b0 + i] = ex;
      ex += v[i];
    }
    carry += tot;
  }
  if (threadIdx.x == 0) digit_tot[blockIdx.x] = carry;
}

// LDS of the stable scatter of one digit pass by T threads, ITEMS pairs each
// (T = 256: 30.7 KB with 16-bit keys, five workgroups per CU; 39.4 KB with
// 32-bit keys, four; T = 512: 59.4 KB with 16-bit keys, two).
template <typename K, int T, int ITEMS = kItems>
struct ScatterShared {
  static constexpr int kWaves = T / 64;
  static constexpr int kElems = T * ITEMS;
  K k[kElems];                 // the tile reordered by digit
  uint32_t v[kElems];
  uint32_t wcnt[kWaves][256];  // per wave and digit: count, then start
  uint32_t run[256];           // per digit: next output position of the block
  uint32_t tstart[256];        // per digit: start of its run in the reordered tile
  uint32_t wave[kWaves];
};

// Output positions of the block's digit runs: run[d] = (pairs of smaller
// digits in the whole pass) + (pairs of digit d in earlier blocks), from the
// per-(digit, block) exclusive scan `counts` and the digit totals.
template <typename K, int T>
__device__ __forceinline__ void scatter_begin(ScatterShared<K, T>& sh, const uint32_t* __restrict__ counts,
                                              const uint32_t* __restrict__ digit_tot, uint32_t grid, uint32_t block) {
  const uint32_t dg = threadIdx.x;
  uint32_t tot;
  const uint32_t base = block_exclusive_scan<T>(dg < 256u ? digit_tot[dg] : 0u, sh.wave, tot);
  if (dg < 256u) sh.run[dg] = base + counts[(size_t)dg * grid + block];
}

// One tile of up to ITEMS T (key, value) pairs stably reordered by digit in LDS:
// wave w holds pairs [64 ITEMS w, 64 ITEMS (w + 1)) of the tile, 64 at a time,
// step i in k[i], v[i]; the first nvalid pairs of the tile are valid. A lane's
// rank among equal digits comes from a ballot match over the digit bits.
// Returns the tile's pairs of digit threadIdx.x; a barrier has to follow.
// FULL: the tile holds ITEMS T valid pairs (the validity tests compile out).
// off.counted() gets the tile's digit counts as soon as they are known.
template <bool FULL, typename K, int T, int ITEMS, typename Offsets>
__device__ __forceinline__ uint32_t stage_tile(ScatterShared<K, T, ITEMS>& sh, uint32_t (&k)[ITEMS],
                                               const uint32_t (&v)[ITEMS], uint32_t nvalid, int shift, int bits,
                                               Offsets& off) {
  constexpr int kWaves = T / 64, kElems = T * ITEMS;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t mask = (1u << bits) - 1u;
  const uint32_t dg = threadIdx.x;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < 256 / 64; ++w) sh.wcnt[wave][w * 64 + lane] = 0u;
  __syncthreads();
  const uint32_t base = (uint32_t)wave * (ITEMS * 64);
  constexpr bool kPacked = sizeof(K) == 2;
  uint32_t rank[ITEMS];
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const bool valid = FULL || base + (uint32_t)i * 64 + lane < nvalid;
    const uint32_t d = (k[i] >> shift) & mask;
    // the lanes holding the same digit (a lane mask in two halves): per digit
    // bit, a lane keeps the lanes whose bit equals its own. S is the lane's
    // bit b as a whole-word mask, so each step is one compare for the ballot
    // and one three-input bit operation per half. Digits have at most 8
    // bits; bits above `bits` are zero in every lane.
    const uint64_t vb = __ballot(valid);
    uint32_t plo = (uint32_t)vb, phi = (uint32_t)(vb >> 32);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const int32_t S = (int32_t)(d << (31 - b)) >> 31;
      const uint64_t m = __ballot(S < 0);
      // x & ~(y ^ z): truth table 0x90 with operands (x, y, z)
      plo = __builtin_amdgcn_bitop3_b32(plo, (uint32_t)m, (uint32_t)S, 0x90);
      phi = __builtin_amdgcn_bitop3_b32(phi, (uint32_t)(m >> 32), (uint32_t)S, 0x90);
    }
    // equal-digit lanes below this one
    const uint32_t below = __builtin_amdgcn_mbcnt_hi(phi, __builtin_amdgcn_mbcnt_lo(plo, 0u));
    const uint32_t pre = sh.wcnt[wave][d];
    // a 16-bit key shares its register with its rank (< 4096). The empty asm
    // makes the rank final here: left to itself the compiler defers the sum
    // past the barrier and keeps each step's masks and count live until then
    if (kPacked) {
      k[i] |= (pre + below) << 16;
      asm volatile("" : "+v"(k[i]));
    } else {
      rank[i] = pre + below;
      asm volatile("" : "+v"(rank[i]));
    }
    // every lane of a digit writes the same count; in a full tile without a
    // branch, so the next step's ballots can overlap this step's LDS access
    const uint32_t cnt = pre + (uint32_t)(__popc(plo) + __popc(phi));
    if (FULL) sh.wcnt[wave][d] = cnt;
    else if (valid && below == 0) sh.wcnt[wave][d] = cnt;
  }
  __syncthreads();
  // per digit: tile-local start, then each wave's start inside it
  uint32_t c[kWaves], ctot = 0;
  if (T == 256 || dg < 256u) {
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      c[w] = sh.wcnt[w][dg];
      ctot += c[w];
    }
  }
  off.counted(ctot);
  uint32_t all;
  const uint32_t ts = block_exclusive_scan<T>(ctot, sh.wave, all);  // contains barriers
  if (T == 256 || dg < 256u) {
    uint32_t at = ts;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      sh.wcnt[w][dg] = at;
      at += c[w];
    }
    sh.tstart[dg] = ts;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const bool valid = FULL || base + (uint32_t)i * 64 + lane < nvalid;
    if (valid) {
      const uint32_t key = kPacked ? (k[i] & 0xFFFFu) : k[i];
      const uint32_t d = (key >> shift) & mask;
      const uint32_t lp = sh.wcnt[wave][d] + (kPacked ? k[i] >> 16 : rank[i]);
      if (lp < (uint32_t)kElems) {
        sh.k[lp] = (K)key;
        sh.v[lp] = v[i];
      }
    }
  }
  return ctot;
}

// Stable scatter of one tile: reordered by digit in LDS, so the global writes of
// each digit run are contiguous. Pairs go to run[d] + their rank among the
// block's pairs of digit d so far (bounded by n_out); with ranges (the last
// pass over the whole key) the keys are not written: each key's first and last
// position bound its range instead (a key >= n_ranges, which a consistent sort
// never produces, is skipped). off gives run[d]: ready() before the tile is
// written, done() after it.
template <bool FULL, typename K, int T, int ITEMS, typename Offsets>
__device__ __forceinline__ void scatter_tile(ScatterShared<K, T, ITEMS>& sh, uint32_t (&k)[ITEMS],
                                             const uint32_t (&v)[ITEMS], uint32_t nvalid, int shift, int bits,
                                             uint32_t n_out, K* __restrict__ keys_out,
                                             uint32_t* __restrict__ vals_out, uint2* __restrict__ ranges,
                                             uint32_t n_ranges, Offsets off) {
  constexpr int kElems = T * ITEMS;
  const uint32_t mask = (1u << bits) - 1u;
  const uint32_t ctot = stage_tile<FULL>(sh, k, v, nvalid, shift, bits, off);
  off.ready(ctot);
  __syncthreads();
  const uint32_t nt = FULL ? (uint32_t)kElems : min(nvalid, (uint32_t)kElems);
#pragma unroll 4
  for (int i = 0; i < ITEMS; ++i) {
    const uint32_t lp = (uint32_t)i * T + threadIdx.x;
    if (lp < nt) {
      const uint32_t key = sh.k[lp];
      const uint32_t d = (key >> shift) & mask;
      const uint32_t p = sh.run[d] + lp - sh.tstart[d];
      if (p < n_out) {  // always true for consistent counts; keeps a ranking fault in bounds
        if (ranges) {
          // the staged tile is ordered by key, so the first and last of each
          // key's run here bound its range
          if (key < n_ranges) {
            if (lp == 0 || sh.k[lp - 1] != key) atomicMin(&ranges[key].x, p);
            if (lp + 1 == nt || sh.k[lp + 1] != key) atomicMax(&ranges[key].y, p + 1);
          }
        } else {
          keys_out[p] = (K)key;
        }
        vals_out[p] = sh.v[lp];
      }
    }
  }
  __syncthreads();
  off.done(ctot);
}

// The block's own tiles one after the other: each moves the runs on.
template <typename Sh>
struct RunningOffsets {
  Sh& sh;
  __device__ __forceinline__ void counted(uint32_t) {}
  __device__ __forceinline__ void ready(uint32_t) {}
  __device__ __forceinline__ void done(uint32_t ctot) {
    if (Sh::kWaves == 4 || threadIdx.x < 256) sh.run[threadIdx.x] += ctot;
  }
};

// One digit pass over the pairs in memory: each block takes its range of
// scatter tiles in turn.
template <typename K, int T>
__global__ void __launch_bounds__(T) k_rs_downsweep(const K* __restrict__ keys_in,
                                                     const uint32_t* __restrict__ vals_in, K* __restrict__ keys_out,
                                                     uint32_t* __restrict__ vals_out, const uint32_t* n_dev,
                                                     uint32_t n_max, int shift, int bits,
                                                     const uint32_t* __restrict__ counts,
                                                     const uint32_t* __restrict__ digit_tot,
                                                     uint2* __restrict__ ranges, uint32_t n_ranges) {
  __shared__ ScatterShared<K, T> sh;
  constexpr uint32_t kElems = ScatterShared<K, T>::kElems;
  const uint32_t n = dev_n(n_dev, n_max);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  scatter_begin(sh, counts, digit_tot, gridDim.x, sort_block());
  uint32_t t0, t1;
  block_range(n, kElems, gridDim.x, t0, t1);
  RunningOffsets<ScatterShared<K, T>> off{sh};
  const uint32_t t_full = min(t1, n / kElems);
  for (uint32_t t = t0; t < t_full; ++t) {
    // a full tile (all but the last): no per-key bounds test
    uint32_t k[kItems], v[kItems];
    const size_t base = (size_t)t * kElems + (size_t)wave * (kItems * 64);
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
      const size_t idx = base + (size_t)i * 64 + lane;
      k[i] = (uint32_t)keys_in[idx];
      v[i] = vals_in[idx];
    }
    scatter_tile<true>(sh, k, v, kElems, shift, bits, n, keys_out, vals_out, ranges, n_ranges, off);
  }
  if (t0 < t1 && t_full < t1) {  // the block of the partial last tile
    uint32_t k[kItems], v[kItems];
    const size_t base = (size_t)t_full * kElems + (size_t)wave * (kItems * 64);
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
      const size_t idx = base + (size_t)i * 64 + lane;
      k[i] = (idx < n) ? (uint32_t)keys_in[idx] : 0u;
      v[i] = (idx < n) ? vals_in[idx] : 0u;
    }
    scatter_tile<false>(sh, k, v, n - t_full * kElems, shift, bits, n, keys_out, vals_out, ranges, n_ranges, off);
  }
}

// --------------------------------------------------------- small sorts ----
// Up to 8192 pairs sorted by one workgroup in one launch, digit by digit in
// LDS, in place of three launches per digit: four digits of 1000 pairs 49 -> 7 us.
constexpr int kSmallThreads = 1024;
constexpr uint32_t kSmallMax = 8 * kSmallThreads;

struct NoOffsets {
  __device__ __forceinline__ void counted(uint32_t) {}
};

// The first n pairs (pair at + 64 i of the thread in k[i], v[i]) put in order of
// the key bits [bit0, bit1); their keys stay in sh.k.
template <typename K, int ITEMS>
__device__ __forceinline__ void sort_small(ScatterShared<K, kSmallThreads, ITEMS>& sh, uint32_t (&k)[ITEMS],
                                           uint32_t (&v)[ITEMS], uint32_t at, uint32_t n, int bit0, int bit1) {
  NoOffsets off;
  for (int b = bit0; b < bit1; b += 8) {
    stage_tile<false>(sh, k, v, n, b, min(bit1 - b, 8), off);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      const uint32_t idx = at + 64u * i;
      k[i] = idx < n ? (uint32_t)sh.k[idx] : 0u;
      v[i] = idx < n ? sh.v[idx] : 0u;
    }
  }
}

// The n (from n_dev) pairs by the key bits [bit0, bit1) to (keys_out, vals_out),
// which may be the inputs; with ranges, each key's positions instead of the
// keys, as scatter_tile's.
template <typename K, int ITEMS>
__global__ void __launch_bounds__(kSmallThreads) k_rs_small(const K* keys_in, const uint32_t* vals_in, K* keys_out,
                                                            uint32_t* vals_out, const uint32_t* n_dev, uint32_t n_max,
                                                            int bit0, int bit1, uint2* __restrict__ ranges,
                                                            uint32_t n_ranges) {
  using Shared = ScatterShared<K, kSmallThreads, ITEMS>;
  __shared__ Shared sh;
  const uint32_t n = min(dev_n(n_dev, n_max), (uint32_t)Shared::kElems);
  const uint32_t at = (threadIdx.x >> 6) * (ITEMS * 64) + (threadIdx.x & 63);
  uint32_t k[ITEMS], v[ITEMS];
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const uint32_t idx = at + 64u * i;
    k[i] = idx < n ? (uint32_t)keys_in[idx] : 0u;
    v[i] = idx < n ? vals_in[idx] : 0u;
  }
  sort_small(sh, k, v, at, n, bit0, bit1);
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const uint32_t idx = at + 64u * i;
    if (idx >= n) break;
    vals_out[idx] = v[i];
    if (!ranges) {
      keys_out[idx] = (K)k[i];
    } else if (k[i] < n_ranges) {
      if (idx == 0 || sh.k[idx - 1] != (K)k[i]) ranges[k[i]].x = idx;
      if (idx + 1 == n || sh.k[idx + 1] != (K)k[i]) ranges[k[i]].y = idx + 1;
    }
  }
}

// ------------------------------------------------------- chained sort ----
// A digit pass in one launch, for the few tiles of a small depth sort, where
// the three launches of the passes above were latency: 17.7 us a pass -> 8.8
// for 88k pairs, 18.0 -> 9.5 for 400k slots with 200k active, 25 -> 22.5 for 525k;
// equal (24.5, 24) for 670k. Tiles of 8192, or 512 threads, took 10.6 and 9.1 for
// 88k; windows of 16 and 32 tiles 9.1 and 9.4.
// Workgroups take tiles by ticket, and a tile's place behind the earlier ones
// comes from what those have published per digit: their own count, then the sum
// up to and with them, a flag in the same word. A tile publishes its count before it
// waits, and waits only for tiles with smaller tickets, which running
// workgroups hold: every wait ends, whatever else occupies the device. The
// wait is bounded besides (chain_sum_before), for calls that share their
// scratch and overlap although they must not.
constexpr int kChainThreads = 1024, kChainItems = 4;  // tiles of 4096 pairs

struct ChainedOffsets {
  uint32_t base;     // thread d < 256: pairs of smaller digits
  uint32_t* run;     // LDS, per digit
  uint32_t* status;  // the pass's words [tile][256]
  uint32_t tile;
  __device__ __forceinline__ void publish(uint32_t word) {
    __hip_atomic_store(&status[(size_t)tile * 256 + threadIdx.x], word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ void counted(uint32_t ctot) {
    if (threadIdx.x < 256) publish((tile ? kChainCount : kChainSum) | ctot);
  }
  __device__ __forceinline__ void ready(uint32_t ctot) {
    if (threadIdx.x >= 256) return;
    const uint32_t sum = chain_sum_before((int)tile, kChainPolls, [&](int t) {
      return __hip_atomic_load(&status[(size_t)t * 256 + threadIdx.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    });
    if (tile) publish(kChainSum | (sum + ctot));
    run[threadIdx.x] = base + sum;
  }
  __device__ __forceinline__ void done(uint32_t) {}
};

__global__ void __launch_bounds__(kChainThreads) k_rs_chain(const uint32_t* __restrict__ keys_in,
                                                            const uint32_t* __restrict__ vals_in,
                                                            uint32_t* __restrict__ keys_out,
                                                            uint32_t* __restrict__ vals_out, const uint32_t* n_dev,
                                                            uint32_t n_max, int shift,
                                                            const uint32_t* __restrict__ hist,
                                                            uint32_t* __restrict__ ticket,
                                                            uint32_t* __restrict__ status) {
  constexpr int ITEMS = kChainItems;
  using Shared = ScatterShared<uint32_t, kChainThreads, ITEMS>;
  __shared__ Shared sh;
  __shared__ uint32_t s_tile;
  const uint32_t n = dev_n(n_dev, n_max), tiles = (n + Shared::kElems - 1) / Shared::kElems;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t all;
  const uint32_t base =
      block_exclusive_scan<kChainThreads>(threadIdx.x < 256 ? hist[threadIdx.x] : 0u, sh.wave, all);
  for (;;) {
    if (threadIdx.x == 0) s_tile = atomicAdd(ticket, 1u);
    __syncthreads();
    const uint32_t t = s_tile;
    if (t >= tiles) return;
    const size_t at = (size_t)t * Shared::kElems + (size_t)wave * (ITEMS * 64) + lane;
    uint32_t k[ITEMS], v[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      const size_t idx = at + (size_t)i * 64;
      k[i] = idx < n ? keys_in[idx] : 0u;
      v[i] = idx < n ? vals_in[idx] : 0u;
    }
    const ChainedOffsets off{base, sh.run, status, t};
    if (t + 1 < tiles || tiles * Shared::kElems == n)
      scatter_tile<true>(sh, k, v, Shared::kElems, shift, 8, n, keys_out, vals_out, nullptr, 0u, off);
    else
      scatter_tile<false>(sh, k, v, n - t * Shared::kElems, shift, 8, n, keys_out, vals_out, nullptr, 0u, off);
  }
}

// ------------------------------------------------------------- gather ----
// The tiles of a record (<= 2^20).
__device__ __forceinline__ uint32_t tile_count(const Record& r, bool exact) {
  const Footprint f = footprint(r);
  uint32_t cnt = 0;
  for (uint32_t ty = f.y0; ty < f.y1; ++ty) {
    uint32_t xa, xb;
    row_span(f, ty, exact, xa, xb);
    cnt += xb - xa;
  }
  return cnt;
}

__global__ void __launch_bounds__(kThreads) k_gather(const uint32_t* n_dev, uint32_t n_max,
                                                      const uint32_t* __restrict__ ids, PairBits pb,
                                                      const Record* __restrict__ rec,
                                                      Record* __restrict__ rec_sorted,
                                                      uint32_t* __restrict__ toff, bool exact,
                                                      uint32_t* __restrict__ bsum) {
  __shared__ uint32_t s_wave[4];
  const uint32_t n = dev_n(n_dev, n_max);
  const uint32_t d = blockIdx.x * blockDim.x + threadIdx.x;
  if (blockIdx.x * blockDim.x >= n) return;
  uint32_t cnt = 0;
  if (d < n) {
    const uint32_t id = ids[d], v = id / (uint32_t)pb.n;
    const Record r = rec[pair_place(pb, v, id - v * (uint32_t)pb.n)];
    rec_sorted[d] = r;
    cnt = tile_count(r, exact);
  }
  uint32_t total;
  const uint32_t ex = block_exclusive_scan(cnt, s_wave, total);  // <= 256 * 2^20 tiles
  if (d < n) toff[d] = ex;
  if (threadIdx.x == 0) bsum[blockIdx.x] = total;
}

// The instance total of n records to the device and, if asked for, the counts to
// the host, by a workgroup of 1024. The emission writes the instances of the
// records that it was launched for, and of those the ones below its capacity;
// the sort and the rasteriser would take as many as the total says.
__device__ __forceinline__ void write_totals(uint64_t sum, uint32_t n, uint32_t* total, unsigned long long* total64,
                                             const HostCounts& host) {
  const bool fits = n <= host.max_records && sum <= host.max_instances;
  if (threadIdx.x == 0) {
    *total = fits ? (uint32_t)sum : 0u;
    *total64 = sum;
  }
  if (!fits && host.guess_views)
    for (int v = threadIdx.x; v < host.n_views; v += 1024) host.guess_views[v].width = 0;
  if (host.counts) {
    if (threadIdx.x == 0) {
      host.counts[0] = n;
      host.counts[1] = (uint32_t)sum;
      host.counts[2] = (uint32_t)sum;
      host.counts[3] = (uint32_t)(sum >> 32);
    }
    for (int v = threadIdx.x; v < host.n_views; v += 1024) host.views[v] = host.view_end[v];
  }
}

// The gather's block sums to block offsets, in place, by one workgroup, 16
// sums per thread at a step (4M records); the total, also as 64 bits. The
// gather's blocks added it to one counter before, some 12 ns each, one after
// the other, and two passes over the records' counts made the offsets: 57 us
// with the gather for 0.7M records, 42 now (5 of them here; 10 for 6M records).
constexpr int kOffsetThreads = 1024;
__global__ void __launch_bounds__(kOffsetThreads) k_block_offsets(const uint32_t* n_dev, uint32_t n_max,
                                                                   uint32_t* __restrict__ bsum,
                                                                   uint32_t* __restrict__ total,
                                                                   unsigned long long* __restrict__ total64,
                                                                   HostCounts host) {
  __shared__ uint64_t s_wave[2][kOffsetThreads / 64];
  const uint32_t nb = (dev_n(n_dev, n_max) + kThreads - 1) / kThreads;
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint64_t carry = 0;
  int side = 0;
  for (uint32_t b0 = 0; b0 < nb; b0 += 16 * kOffsetThreads, side ^= 1) {
    const uint32_t e = b0 + 1024u * wave + 4u * lane;
    uint4 g[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) g[j] = load_group(bsum, (size_t)e + 256 * j, nb, e + 256 * j + 4 <= nb);
    uint64_t wsum = 0;
    uint32_t gx[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint64_t q = (uint64_t)g[j].x + g[j].y + g[j].z + g[j].w;
      uint64_t inc = q;
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const uint64_t y = __shfl_up(inc, off, 64);
        if (lane >= (uint32_t)off) inc += y;
      }
      gx[j] = (uint32_t)(wsum + inc - q);
      wsum += __shfl(inc, 63, 64);
    }
    if (lane == 0) s_wave[side][wave] = wsum;
    __syncthreads();
    uint64_t before = carry;
#pragma unroll
    for (uint32_t w = 0; w < kOffsetThreads / 64; ++w) {
      before += w < wave ? s_wave[side][w] : 0ull;
      carry += s_wave[side][w];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t i = e + 256 * j;
      uint4 o;
      o.x = (uint32_t)before + gx[j];
      o.y = o.x + g[j].x;
      o.z = o.y + g[j].y;
      o.w = o.z + g[j].z;
      if (i + 4 <= nb) {
        *reinterpret_cast<uint4*>(bsum + i) = o;
      } else {
        if (i < nb) bsum[i] = o.x;
        if (i + 1 < nb) bsum[i + 1] = o.y;
        if (i + 2 < nb) bsum[i + 2] = o.z;
      }
    }
  }
  write_totals(carry, dev_n(n_dev, n_max), total, total64, host);
}

// The depth sort, the gather and the offsets of up to 2048 pairs in one launch,
// by one workgroup, for images of up to 16 tile rows: a record's rows are one
// thread's, and the gather would be spread over the device. 67 -> 60 us a
// render of 1000 pairs against three launches, 81 -> 71 of 2000. By tile rows, 64
// pixels wide, 2000 footprints as tall as the image: 8 rows 120.2 -> 114.8, 16
// 122.1 -> 120.0, 24 124.5 -> 124.3, 32 125.6 -> 125.2 (of 1000, 5 us less at 16 and
// 4 at 32; small footprints 6 less throughout); an image may have 1024 rows.
constexpr uint32_t kSortGatherMax = 2 * kSmallThreads;
template <int ITEMS>
__global__ void __launch_bounds__(kSmallThreads) k_sort_gather(const uint32_t* __restrict__ keys, uint32_t* ids,
                                                               const uint32_t* n_dev, uint32_t n_max, PairBits pb,
                                                               const Record* __restrict__ rec,
                                                               Record* __restrict__ rec_sorted,
                                                               uint32_t* __restrict__ toff, bool exact,
                                                               uint32_t* __restrict__ boff,
                                                               uint32_t* __restrict__ total,
                                                               unsigned long long* __restrict__ total64,
                                                               HostCounts host) {
  __shared__ ScatterShared<uint32_t, kSmallThreads, ITEMS> sh;
  const uint32_t n = min(dev_n(n_dev, n_max), (uint32_t)(kSmallThreads * ITEMS));
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6, at = wave * (ITEMS * 64) + lane;
  uint32_t k[ITEMS], v[ITEMS];
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const uint32_t idx = at + 64u * i;
    k[i] = idx < n ? keys[idx] : 0u;
    v[i] = idx < n ? ids[idx] : 0u;
  }
  sort_small(sh, k, v, at, n, 0, 32);
  uint32_t before[ITEMS], wsum = 0;  // of the wave: <= 128 * 2^20
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const uint32_t idx = at + 64u * i;
    uint32_t c = 0;
    if (idx < n) {
      const uint32_t view = v[i] / (uint32_t)pb.n;
      const Record r = rec[pair_place(pb, view, v[i] - view * (uint32_t)pb.n)];
      rec_sorted[idx] = r;
      ids[idx] = v[i];
      c = tile_count(r, exact);
    }
    uint32_t inc = c;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t y = __shfl_up(inc, off, 64);
      if (lane >= (uint32_t)off) inc += y;
    }
    before[i] = wsum + inc - c;
    wsum += __shfl(inc, 63, 64);
  }
  __syncthreads();  // the sort's use of sh.wave is over
  if (lane == 0) sh.wave[wave] = wsum;
  __syncthreads();
  uint64_t base = 0, sum = 0;
#pragma unroll
  for (uint32_t w = 0; w < kSmallThreads / 64; ++w) {
    base += w < wave ? sh.wave[w] : 0u;
    sum += sh.wave[w];
  }
#pragma unroll
  for (int i = 0; i < ITEMS; ++i)
    if (at + 64u * i < n) toff[at + 64u * i] = (uint32_t)base + before[i];
  if (threadIdx.x < (n + kThreads - 1) / kThreads) boff[threadIdx.x] = 0u;
  write_totals(sum, n, total, total64, host);
}

// ---------------------------------------------------------------- emit ----
// One block per 64 or 128 consecutive records, whose tile rows it takes up to
// kEmitRows at a time (one record has no more). It lays the rows out in LDS
// (first tile, offset of the row's first instance by a block scan of the row
// widths) and, chunk by chunk, the row of the first of every four positions of
// the output, then a thread writes four instances at a time, walking the rows
// between them. (One instance at a time, and a search for the record of each
// instance of blocks with more rows: 267 us for 4M records, 80M instances, 554 for
// 5.7M, 236M; now 192 and 412, 3.4 TB/s of writes.)
constexpr int kEmitRows = 1024;    // 16384 pixels
constexpr int kEmitGroups = 2048;  // fours of a chunk

// K: the key type, uint16_t when the round's tile ids are below 2^16.
// kRecs: the records of a block.
template <typename K, int kRecs>
__global__ void __launch_bounds__(kThreads) k_emit(const uint32_t* n_dev, uint32_t n_max,
                                                    const uint32_t* __restrict__ toff,
                                                    const uint32_t* __restrict__ boff, const uint32_t* total,
                                                    uint32_t cap, const Record* __restrict__ rec_sorted,
                                                    const uint32_t* __restrict__ ids, uint32_t n_prims,
                                                    const ViewDev* __restrict__ views, bool exact,
                                                    K* __restrict__ ikey, uint32_t* __restrict__ ival,
                                                    uint2* __restrict__ ranges_init, uint32_t tiles) {
  __shared__ uint32_t offs[kRecs + 1];
  __shared__ uint32_t s_rbase[kRecs + 1];
  __shared__ uint32_t s_tb[kRecs], s_tw[kRecs];
  __shared__ Footprint s_fp[kRecs];
  __shared__ uint32_t s_row_off[kEmitRows + 1];  // first instance of each row (from the first record's on)
  __shared__ uint32_t s_row_tile[kEmitRows];     // global tile id of the row's first instance
  __shared__ uint8_t s_row_rec[kEmitRows];       // record of the row (block-relative, < kRecs)
  __shared__ uint16_t s_group_row[kEmitGroups];  // row of the first instance of each four of the chunk (< kEmitRows)
  static_assert(kRecs <= 256 && kEmitRows <= 65536, "narrow LDS maps: 18 or 22 KB, eight or seven workgroups per CU");
  __shared__ uint32_t s_wave[4];
  // the tile ranges that the sort's last pass fills start empty
  if (ranges_init)
    for (uint32_t t = blockIdx.x * kThreads + threadIdx.x; t < tiles; t += gridDim.x * kThreads)
      ranges_init[t] = make_uint2(0xFFFFFFFFu, 0u);
  const uint32_t n = dev_n(n_dev, n_max);
  const uint32_t d0 = blockIdx.x * kRecs;
  if (d0 >= n) return;
  const uint32_t nrec = min((uint32_t)kRecs, n - d0);
  const uint32_t tot = *total;
  uint32_t h = 0;
  if (threadIdx.x < kRecs) {
    const uint32_t d = d0 + threadIdx.x;
    offs[threadIdx.x] = d < n ? boff[d / kThreads] + toff[d] : tot;
    if (threadIdx.x == 0) {
      const uint32_t e = d0 + kRecs;
      offs[kRecs] = e < n ? boff[e / kThreads] + toff[e] : tot;
    }
    if (d < n) {
      const Footprint f = footprint(rec_sorted[d]);
      s_fp[threadIdx.x] = f;
      h = f.y1 - f.y0;
      const uint32_t v = ids[d] / n_prims;
      s_tb[threadIdx.x] = (uint32_t)views[v].tile_base;
      s_tw[threadIdx.x] = (uint32_t)views[v].tiles_x;
    }
  }
  uint32_t rows;
  const uint32_t rb = block_exclusive_scan(h, s_wave, rows);  // contains barriers
  if (threadIdx.x < kRecs) s_rbase[threadIdx.x] = rb;
  if (threadIdx.x == 0) s_rbase[kRecs] = rows;
  __syncthreads();
  const uint32_t lim = min(tot, cap);
  for (uint32_t r0 = 0, r1; r0 < nrec; r0 = r1) {
    // records [r0, r1): at least one, as a record has at most kEmitRows rows
    const uint32_t row0 = s_rbase[r0];
    r1 = nrec;
    if (rows - row0 > (uint32_t)kEmitRows)
      r1 = r0 + (uint32_t)__syncthreads_count(threadIdx.x >= r0 && threadIdx.x < nrec &&
                                              s_rbase[threadIdx.x + 1] - row0 <= (uint32_t)kEmitRows);
    const uint32_t rows_here = s_rbase[r1] - row0;
    // each record marks its rows with its block-relative index, so a row finds
    // its record with one LDS read
    if (threadIdx.x >= r0 && threadIdx.x < r1)
      for (uint32_t k = 0; k < h; ++k) s_row_rec[rb - row0 + k] = (uint8_t)threadIdx.x;
    __syncthreads();
    uint32_t carry = 0;
    for (uint32_t j0 = 0; j0 < rows_here; j0 += kThreads) {
      const uint32_t j = j0 + threadIdx.x;
      uint32_t w = 0;
      if (j < rows_here) {
        const int lo = s_row_rec[j];
        const Footprint& f = s_fp[lo];
        const uint32_t ty = f.y0 + (row0 + j - s_rbase[lo]);
        uint32_t xa, xb;
        row_span(f, ty, exact, xa, xb);
        w = xb - xa;
        s_row_tile[j] = s_tb[lo] + ty * s_tw[lo] + xa;
      }
      uint32_t tot_w;
      const uint32_t ex = block_exclusive_scan(w, s_wave, tot_w);  // contains barriers
      if (j < rows_here) s_row_off[j] = carry + ex;
      carry += tot_w;
    }
    if (threadIdx.x == 0) s_row_off[rows_here] = carry;
    __syncthreads();
    // instances [start, iend); the offsets' end is start + carry, as the counts
    // come from the same spans
    const uint32_t start = offs[r0], iend = min(min(offs[r1], lim), start + carry);
    const uint32_t g_end = (iend + 3) / 4;
    // (no instance of these records to write: the map would name no row)
    for (uint32_t c0 = start / 4; start < iend && c0 * 4 < iend; c0 += kEmitGroups) {
      if (c0 != start / 4) __syncthreads();  // the previous chunk's reads of the map are done
      const uint32_t c1 = min(c0 + (uint32_t)kEmitGroups, g_end);
      for (uint32_t j = threadIdx.x; j < rows_here; j += kThreads) {
        const uint32_t o0 = s_row_off[j], o1 = s_row_off[j + 1];
        const uint32_t a = max(o0 ? (start + o0 + 3) / 4 : start / 4, c0);
        const uint32_t b = o1 > o0 ? min((start + o1 + 3) / 4, c1) : 0u;
        for (uint32_t g = a; g < b; ++g) s_group_row[g - c0] = (uint16_t)j;
      }
      __syncthreads();
      for (uint32_t g = c0 + threadIdx.x; g < c1; g += kThreads) {
        uint32_t j = s_group_row[g - c0];
        uint32_t off = s_row_off[j], next = s_row_off[j + 1], tile = s_row_tile[j], rec = d0 + s_row_rec[j];
        const uint32_t i0 = max(g * 4, start), i1 = min(g * 4 + 4, iend);
        const auto step = [&](uint32_t i) {  // to instance i's row
          while (i - start >= next) {
            off = next;
            next = s_row_off[++j + 1];
            tile = s_row_tile[j];
            rec = d0 + s_row_rec[j];
          }
        };
        if (i1 - i0 == 4) {
          uint32_t k[4], v[4];
#pragma unroll
          for (uint32_t q = 0; q < 4; ++q) {
            step(i0 + q);
            k[q] = tile + (i0 + q - start - off);
            v[q] = rec;
          }
          *reinterpret_cast<uint4*>(ival + i0) = make_uint4(v[0], v[1], v[2], v[3]);
          if constexpr (sizeof(K) == 2)
            *reinterpret_cast<uint2*>(ikey + i0) = make_uint2(k[0] | k[1] << 16, k[2] | k[3] << 16);
          else
            *reinterpret_cast<uint4*>(ikey + i0) = make_uint4(k[0], k[1], k[2], k[3]);
        } else {
          for (uint32_t i = i0; i < i1; ++i) {
            step(i);
            ikey[i] = (K)(tile + (i - start - off));
            ival[i] = rec;
          }
        }
      }
    }
    if (r1 < nrec) __syncthreads();  // the rows are read before the next records' replace them
  }
}

// Ranges filled by the last radix pass: (max, 0) before it, and tiles it did
// not reach (no instances) set to (0, 0) after it.
__global__ void k_ranges_init(uint2* __restrict__ ranges, uint32_t tiles) {
  const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < tiles) ranges[t] = make_uint2(0xFFFFFFFFu, 0u);
}

__global__ void k_ranges_fix(uint2* __restrict__ ranges, uint32_t tiles) {
  const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= tiles) return;
  const uint2 r = ranges[t];
  if (r.x > r.y) ranges[t] = make_uint2(0u, 0u);
}

template <typename K>
__global__ void k_ranges(const uint32_t* n_dev, uint32_t n_max, const K* __restrict__ ikey,
                         uint2* __restrict__ ranges) {
  // four consecutive keys per thread
  const uint32_t n = dev_n(n_dev, n_max);
  const uint32_t i0 = 4u * (blockIdx.x * blockDim.x + threadIdx.x);
  if (i0 >= n) return;
  uint32_t k[6];  // k[0] = key before i0 (or none), k[1..4] = keys i0..i0+3, k[5] = key after
  for (int j = 0; j < 4; ++j) k[1 + j] = (i0 + j < n) ? (uint32_t)ikey[i0 + j] : 0xFFFFFFFFu;
  k[0] = i0 > 0 ? (uint32_t)ikey[i0 - 1] : 0xFFFFFFFFu;
  k[5] = (i0 + 4 < n) ? (uint32_t)ikey[i0 + 4] : 0xFFFFFFFFu;
#pragma unroll
  for (int j = 1; j <= 4; ++j) {
    const uint32_t i = i0 + j - 1;
    if (i >= n) break;
    if (i == 0 || k[j - 1] != k[j]) ranges[k[j]].x = i;
    if (i == n - 1 || k[j + 1] != k[j]) ranges[k[j]].y = i + 1;
  }
}

// Block sums (64-bit per thread), one atomic per block.
__global__ void __launch_bounds__(256) k_sum_u32(const uint32_t* __restrict__ in, uint64_t n,
                                                 unsigned long long* out) {
  __shared__ unsigned long long s_part[4];
  uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  unsigned long long acc = 0;
  for (; i < n; i += (uint64_t)gridDim.x * blockDim.x) acc += in[i];
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
  if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned long long tot = s_part[0] + s_part[1] + s_part[2] + s_part[3];
    if (tot) atomicAdd(out, tot);
  }
}

// Longest tile list: max over tiles of end - start, one atomic per block.
__global__ void __launch_bounds__(256) k_range_max(const uint2* __restrict__ ranges, uint32_t tiles, uint32_t* out) {
  __shared__ uint32_t s_part[4];
  uint32_t len = 0;
  for (uint32_t t = blockIdx.x * blockDim.x + threadIdx.x; t < tiles; t += gridDim.x * blockDim.x) {
    const uint2 r = ranges[t];
    len = max(len, r.y - r.x);
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) len = max(len, (uint32_t)__shfl_xor((int)len, off, 64));
  if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = len;
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t m = max(max(s_part[0], s_part[1]), max(s_part[2], s_part[3]));
    if (m) atomicMax(out, m);
  }
}

// Heavy-first tile order: key 255 - floor(16 log2(len + 1)), so that a
// stable sort of the keys lists tiles by decreasing list length in bins of
// ~4.4 %, keeping the natural order within a bin.
__device__ __forceinline__ uint32_t order_key(uint32_t len) {
  return 255u - min((uint32_t)(16.f * __log2f((float)len + 1.f)), 255u);
}

// The tiles' order keys. The same pass empties the ranges the last radix pass
// did not reach (fix, as k_ranges_fix) and raises *max_len to the longest list
// (as k_range_max).
__global__ void __launch_bounds__(256) k_order_keys(uint2* __restrict__ ranges, uint32_t tiles, bool fix,
                                                    uint32_t* __restrict__ keys, uint32_t* __restrict__ vals,
                                                    uint32_t* max_len) {
  __shared__ uint32_t s_part[4];
  const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  uint32_t len = 0;
  if (t < tiles) {
    uint2 r = ranges[t];
    if (fix && r.x > r.y) {
      r = make_uint2(0u, 0u);
      ranges[t] = r;
    }
    len = r.y - r.x;
    keys[t] = order_key(len);
    vals[t] = t;
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) len = max(len, (uint32_t)__shfl_xor((int)len, off, 64));
  if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = len;
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t m = max(max(s_part[0], s_part[1]), max(s_part[2], s_part[3]));
    if (m) atomicMax(max_len, m);
  }
}

// The same and its sort in one launch, by one workgroup, for up to kSmallMax
// tiles (four launches before: 21 -> 8.8 us for 5440 tiles, 17 -> 6 for 16).
__global__ void __launch_bounds__(kSmallThreads) k_order_small(uint2* __restrict__ ranges, uint32_t tiles, bool fix,
                                                               uint32_t* __restrict__ order, uint32_t* max_len) {
  constexpr int ITEMS = kSmallMax / kSmallThreads;
  __shared__ ScatterShared<uint16_t, kSmallThreads, ITEMS> sh;
  const uint32_t at = (threadIdx.x >> 6) * (ITEMS * 64) + (threadIdx.x & 63);
  uint32_t k[ITEMS], v[ITEMS], most = 0;
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const uint32_t t = at + 64u * i;
    k[i] = v[i] = 0u;
    if (t < tiles) {
      uint2 r = ranges[t];
      if (fix && r.x > r.y) {
        r = make_uint2(0u, 0u);
        ranges[t] = r;
      }
      most = max(most, r.y - r.x);
      k[i] = order_key(r.y - r.x);
      v[i] = t;
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) most = max(most, (uint32_t)__shfl_xor((int)most, off, 64));
  if (most && (threadIdx.x & 63) == 0) atomicMax(max_len, most);
  NoOffsets off;
  stage_tile<false>(sh, k, v, tiles, 0, 8, off);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const uint32_t t = threadIdx.x + (uint32_t)kSmallThreads * i;
    if (t < tiles) order[t] = sh.v[t];
  }
}

inline unsigned grid_for(uint64_t n, unsigned bs) { return (unsigned)((n + bs - 1) / bs); }

}  // namespace

size_t scan_scratch_words(size_t n_max) { return (n_max + kThreads - 1) / kThreads + 4; }

void launch_compact(const PairBits& pb, const uint32_t* count, int n_views, const uint32_t* dkey, uint32_t* ckey,
                    uint32_t* cval, uint32_t* hist, uint32_t* total, uint32_t* view_end, uint32_t* scratch,
                    hipStream_t s) {
  const uint32_t view_groups = pb.units / 4;
  if (view_groups == 0 || n_views == 0) {
    launch_fill_u32(total, 1, 0u, s);
    launch_fill_u32(view_end, (uint64_t)n_views, 0u, s);
    return;
  }
  const uint32_t groups = view_groups * (uint32_t)n_views;
  // up to 16384 groups (4M pairs) a workgroup adds the counts before it itself
  // (at most 64 loads per thread); beyond, a pass over the counts sums them by
  // the 4096 first
  const bool coarse = groups > 4 * (uint32_t)kCoarseGroups;
  if (coarse)
    hipLaunchKernelGGL(k_scan_reduce, dim3(grid_for(groups, kTileElems)), dim3(kThreads), 0, s, count, nullptr, groups,
                       scratch);
  hipLaunchKernelGGL(k_compact, dim3(grid_for(groups, kCompactGroups)), dim3(kThreads), 0, s, pb, count,
                     hist, coarse ? scratch : nullptr, groups, dkey, ckey, cval, total, view_end);
}

size_t radix_scratch_words(int grid) { return (size_t)256 * grid + 256; }

int radix_grid(uint32_t n_max, int max_blocks) {
  const int need = (int)grid_for(n_max, kTileElems);
  return need < 1 ? 1 : (need < max_blocks ? need : max_blocks);
}

int radix_passes(int bit0, int bit1) { return bit1 > bit0 ? (bit1 - bit0 + 7) / 8 : 0; }

// The digit passes, ping-ponging between the two buffer pairs; returns the
// pair that holds the result.
template <typename K, int T = kThreads>
std::pair<K*, uint32_t*> radix_passes_run(K* keys, uint32_t* vals, K* keys_alt, uint32_t* vals_alt,
                                          const uint32_t* n_dev, uint32_t n_max, int bit0, int bit1, int grid,
                                          uint32_t* scratch, hipStream_t s, uint2* last_ranges,
                                          uint32_t n_ranges) {
  if (n_max <= kSmallMax && bit1 > bit0) {
    const bool odd = radix_passes(bit0, bit1) & 1;
    K* ko = odd ? keys_alt : keys;
    uint32_t* vo = odd ? vals_alt : vals;
    const auto kernel = n_max <= kSmallMax / 8 ? k_rs_small<K, 1>
                        : n_max <= kSmallMax / 2 ? k_rs_small<K, 4> : k_rs_small<K, 8>;
    hipLaunchKernelGGL(kernel, dim3(1), dim3(kSmallThreads), 0, s, keys, vals, ko, vo, n_dev, n_max, bit0, bit1,
                       last_ranges, n_ranges);
    return {ko, vo};
  }
  // digits of equal width: 13 tile bits as 7 and 6 (two views of 300k primitives
  // 391 -> 386 us a render against 8 and 5), for longer runs in the first pass
  const int passes = radix_passes(bit0, bit1);
  const int step = passes ? (bit1 - bit0 + passes - 1) / passes : 8;
  K *kin = keys, *kout = keys_alt;
  uint32_t *vin = vals, *vout = vals_alt;
  for (int b = bit0; b < bit1; b += step) {
    const int bits = (bit1 - b) < step ? (bit1 - b) : step;
    hipLaunchKernelGGL((k_rs_upsweep<K, T>), dim3(grid), dim3(T), 0, s, kin, n_dev, n_max, b, bits, scratch);
    hipLaunchKernelGGL(k_rs_rowscan, dim3(256), dim3(kThreads), 0, s, scratch, grid, scratch + (size_t)256 * grid);
    hipLaunchKernelGGL((k_rs_downsweep<K, T>), dim3(grid), dim3(T), 0, s, kin, vin, kout, vout, n_dev, n_max, b,
                       bits, scratch, scratch + (size_t)256 * grid, b + step >= bit1 ? last_ranges : nullptr,
                       b + step >= bit1 && last_ranges ? n_ranges : 0u);
    std::swap(kin, kout);
    std::swap(vin, vout);
  }
  return {kin, vin};
}

void radix_sort(uint32_t* keys, uint32_t* vals, uint32_t* keys_alt, uint32_t* vals_alt, const uint32_t* n_dev,
                uint32_t n_max, int bit0, int bit1, int grid, uint32_t* scratch, hipStream_t s, bool copy_back,
                uint2* last_ranges, uint32_t n_ranges) {
  // an odd pass count ends with a copy back so the result is in (keys, vals),
  // unless the caller takes it from (keys_alt, vals_alt)
  const auto out = radix_passes_run(keys, vals, keys_alt, vals_alt, n_dev, n_max, bit0, bit1, grid, scratch, s,
                                    last_ranges, n_ranges);
  if (out.first != keys && copy_back) launch_copy_pairs(out.first, out.second, keys, vals, n_dev, n_max, s);
}

size_t chain_scratch_words(size_t n_max) {
  const size_t tile = (size_t)kChainThreads * kChainItems;
  return 4 * 256 + 64 + 4 * 256 * ((n_max + tile - 1) / tile);
}

void chain_sort(uint32_t* keys, uint32_t* vals, uint32_t* keys_alt, uint32_t* vals_alt, const uint32_t* n_dev,
                uint32_t n_max, uint32_t n_est, uint32_t* scratch, hipStream_t s) {
  const uint32_t tile = kChainThreads * kChainItems;
  const uint32_t tiles = grid_for(n_max, tile);
  uint32_t *hist = scratch, *tickets = scratch + 4 * 256, *status = tickets + 64;
  const dim3 grid(std::max(1u, std::min(grid_for(n_est, tile), 1024u)));
  for (int p = 0; p < 4; ++p) {
    hipLaunchKernelGGL(k_rs_chain, grid, dim3(kChainThreads), 0, s, keys, vals, keys_alt, vals_alt, n_dev,
                       n_max, 8 * p, hist + 256 * p, tickets + p, status + (size_t)p * tiles * 256);
    std::swap(keys, keys_alt);
    std::swap(vals, vals_alt);
  }
}

void radix_sort16(uint16_t* keys, uint32_t* vals, uint16_t* keys_alt, uint32_t* vals_alt, const uint32_t* n_dev,
                  uint32_t n_max, int bit0, int bit1, int grid, uint32_t* scratch, hipStream_t s,
                  uint2* last_ranges, uint32_t n_ranges) {
  // from 2^24 instances on, two 512-thread workgroups per CU with tiles of 8192:
  // digit runs of 32 instances write half as many partial cache lines, and
  // fewer lines are open at once, than with five 256-thread ones (per pass:
  // 109 -> 101 us for 26M instances, 186 -> 174 for 44M, 368 -> 325 for 80M,
  // 1139 -> 980 for 236M; equal at 14M, and at 3.4M 18.4 -> 21.4). Fewer if fewer
  // are asked for, and beyond the default of 1280 more in proportion (80M: 204
  // workgroups 455 us a pass, 409 366, 512 333, 819 364)
  if (n_max >= 1u << 24)
    radix_passes_run<uint16_t, 512>(keys, vals, keys_alt, vals_alt, n_dev, n_max, bit0, bit1,
                                    std::max(std::min(grid, 512), grid / 5 * 2), scratch, s, last_ranges, n_ranges);
  else
    radix_passes_run(keys, vals, keys_alt, vals_alt, n_dev, n_max, bit0, bit1, grid, scratch, s, last_ranges,
                     n_ranges);
}

void launch_gather(const uint32_t* n_dev, uint32_t n_max, const uint32_t* ids, const PairBits& pb,
                   const Record* rec, Record* rec_sorted, uint32_t* toff, bool exact, uint32_t* boff,
                   uint32_t* total, uint32_t* total64, const HostCounts& host, hipStream_t s) {
  if (n_max == 0) {
    launch_fill_u32(total, 1, 0u, s);
    launch_fill_u32(total64, 2, 0u, s);
    return;
  }
  hipLaunchKernelGGL(k_gather, dim3(grid_for(n_max, kThreads)), dim3(kThreads), 0, s, n_dev, n_max, ids, pb,
                     rec, rec_sorted, toff, exact, boff);
  hipLaunchKernelGGL(k_block_offsets, dim3(1), dim3(kOffsetThreads), 0, s, n_dev, n_max, boff, total,
                     reinterpret_cast<unsigned long long*>(total64), host);
}

bool sort_gather_fits(uint64_t pairs, int tile_rows) { return pairs <= kSortGatherMax && tile_rows <= 16; }

void launch_sort_gather(const uint32_t* n_dev, uint32_t n_max, const uint32_t* keys, uint32_t* ids,
                        const PairBits& pb, const Record* rec, Record* rec_sorted, uint32_t* toff, bool exact,
                        uint32_t* boff, uint32_t* total, uint32_t* total64, const HostCounts& host, hipStream_t s) {
  const auto kernel = n_max <= (uint32_t)kSmallThreads ? k_sort_gather<1> : k_sort_gather<2>;
  hipLaunchKernelGGL(kernel, dim3(1), dim3(kSmallThreads), 0, s, keys, ids, n_dev, n_max, pb, rec, rec_sorted, toff,
                     exact, boff, total, reinterpret_cast<unsigned long long*>(total64), host);
}

template <typename K>
void emit_keys(const uint32_t* n_dev, uint32_t n_max, const uint32_t* toff, const uint32_t* boff,
               const uint32_t* total, uint32_t cap, const Record* rec_sorted, const uint32_t* ids, int n_prims,
               const ViewDev* views, bool exact, K* ikey, uint32_t* ival, uint2* ranges_init, uint32_t tiles,
               hipStream_t s) {
  if (n_max == 0) {
    if (ranges_init) launch_ranges_init(ranges_init, tiles, s);
    return;
  }
  // many records: twice as many per block, for half the blocks' fixed steps (4M
  // 232 -> 192 us, 5.7M 462 -> 412; equal at 0.7M, and for one view's 88k, whose
  // nearest and largest footprints share a block, 13.4 -> 18.1)
  const bool many = n_max >= (1u << 20);
  const auto kernel = many ? k_emit<K, 128> : k_emit<K, 64>;
  hipLaunchKernelGGL(kernel, dim3(grid_for(n_max, many ? 128 : 64)), dim3(kThreads), 0, s, n_dev, n_max, toff, boff,
                     total, cap, rec_sorted, ids, (uint32_t)n_prims, views, exact, ikey, ival, ranges_init, tiles);
}

void launch_emit(const uint32_t* n_dev, uint32_t n_max, const uint32_t* toff, const uint32_t* boff,
                 const uint32_t* total, uint32_t cap, const Record* rec_sorted, const uint32_t* ids, int n_prims,
                 const ViewDev* views, bool exact,
                 uint32_t* ikey, uint32_t* ival, uint2* ranges_init, uint32_t tiles, hipStream_t s) {
  emit_keys(n_dev, n_max, toff, boff, total, cap, rec_sorted, ids, n_prims, views, exact, ikey, ival, ranges_init,
            tiles, s);
}

void launch_emit(const uint32_t* n_dev, uint32_t n_max, const uint32_t* toff, const uint32_t* boff,
                 const uint32_t* total, uint32_t cap, const Record* rec_sorted, const uint32_t* ids, int n_prims,
                 const ViewDev* views, bool exact,
                 uint16_t* ikey, uint32_t* ival, uint2* ranges_init, uint32_t tiles, hipStream_t s) {
  emit_keys(n_dev, n_max, toff, boff, total, cap, rec_sorted, ids, n_prims, views, exact, ikey, ival, ranges_init,
            tiles, s);
}

void launch_ranges_init(uint2* ranges, uint32_t tiles, hipStream_t s) {
  if (tiles) hipLaunchKernelGGL(k_ranges_init, dim3(grid_for(tiles, 256)), dim3(256), 0, s, ranges, tiles);
}

void launch_ranges_fix(uint2* ranges, uint32_t tiles, hipStream_t s) {
  if (tiles) hipLaunchKernelGGL(k_ranges_fix, dim3(grid_for(tiles, 256)), dim3(256), 0, s, ranges, tiles);
}

void launch_ranges(const uint32_t* n_dev, uint32_t n_max, const uint32_t* ikey, uint2* ranges, hipStream_t s) {
  if (n_max == 0) return;
  hipLaunchKernelGGL(k_ranges<uint32_t>, dim3(grid_for((n_max + 3) / 4, 256)), dim3(256), 0, s, n_dev, n_max, ikey,
                     ranges);
}

void launch_ranges(const uint32_t* n_dev, uint32_t n_max, const uint16_t* ikey, uint2* ranges, hipStream_t s) {
  if (n_max == 0) return;
  hipLaunchKernelGGL(k_ranges<uint16_t>, dim3(grid_for((n_max + 3) / 4, 256)), dim3(256), 0, s, n_dev, n_max, ikey,
                     ranges);
}

void launch_sum_u32(const uint32_t* in, uint64_t n, unsigned long long* out, hipStream_t s) {
  if (n == 0) return;
  unsigned g = grid_for(n, 256);
  if (g > 4096) g = 4096;
  hipLaunchKernelGGL(k_sum_u32, dim3(g), dim3(256), 0, s, in, n, out);
}

void launch_tile_order(uint2* ranges, uint32_t tiles, bool fix, uint32_t* keys, uint32_t* vals, uint32_t* keys_alt,
                       uint32_t* order, uint32_t* max_len, int sort_blocks, uint32_t* scratch, hipStream_t s) {
  if (tiles == 0) return;
  if (tiles <= kSmallMax) {
    hipLaunchKernelGGL(k_order_small, dim3(1), dim3(kSmallThreads), 0, s, ranges, tiles, fix, order, max_len);
    return;
  }
  hipLaunchKernelGGL(k_order_keys, dim3(grid_for(tiles, 256)), dim3(256), 0, s, ranges, tiles, fix, keys, vals,
                     max_len);
  // one 8-bit pass: the result lands in (keys_alt, order), no copy back
  radix_sort(keys, vals, keys_alt, order, nullptr, tiles, 0, 8, radix_grid(tiles, sort_blocks), scratch, s,
             /*copy_back=*/false);
}

void launch_range_max(const uint2* ranges, uint32_t tiles, uint32_t* out, hipStream_t s) {
  if (tiles == 0) return;
  unsigned g = grid_for(tiles, 1024);
  hipLaunchKernelGGL(k_range_max, dim3(g > 256 ? 256 : g), dim3(256), 0, s, ranges, tiles, out);
}

}  // namespace g4d
