// Per-primitive stages of the 4D Gaussian render. k_preprocess (all views of a
// batch at once): 4D covariance Sigma = R S S^T R^T with R = L(q_l) R(q_r)
// (Sec. 3.2, "Representation of 4D Gaussian"), temporal marginal and filter
// (Sec. 3.2 and Sec. 4.2), conditional 3D Gaussian at t (Sec. 3.2), EWA
// projection (Eqs. 3-4), footprint and tile rectangle -- and, for a flow
// render, the image-plane displacement of the conditional mean (Sec. 4.4).
// This geometry is evaluated in FP64 and every value a record holds is
// rounded to FP32 once, so a record differs from the exact value by that
// rounding alone and the cull, near-plane and rectangle decisions are those of
// the exact arithmetic.
// k_colour: the 4D spherindrical-harmonic colour (Sec. 3.2) of the active
// pairs, written into their records before the gather orders them by depth; it
// reads the coefficients of the primitives active in some view only.
// The backward is in preprocess_bwd.hip.
#include <cmath>

#include "shade.h"

namespace g4d {
namespace {

using namespace shade;

__device__ __forceinline__ bool finite4(float4 a) {
  return isfinite(a.x) && isfinite(a.y) && isfinite(a.z) && isfinite(a.w);
}

// A FP32 bound on Sigma_44 from above: Sigma_44 = sum_k (R_3k s_k)^2, every
// rounding of R_3k (sums of four products of unit-quaternion components, below
// 1e-6) taken against it, and a relative 1e-4 for the exponentials and the sum.
__device__ __forceinline__ float sigma44_bound(float4 ql, float4 qr, float4 ls) {
  const float nl = ql.x * ql.x + ql.y * ql.y + ql.z * ql.z + ql.w * ql.w;
  const float nr = qr.x * qr.x + qr.y * qr.y + qr.z * qr.z + qr.w * qr.w;
  // (squares that overflow or lose bits to underflow bound nothing)
  if (!(fminf(nl, nr) > 1e-30f && fmaxf(nl, nr) < 1e30f)) return INFINITY;
  const float il = rsqrtf(nl), ir = rsqrtf(nr);
  float L[4][4], Rr[4][4];
  isoclinic_left(make_float4(ql.x * il, ql.y * il, ql.z * il, ql.w * il), L);
  isoclinic_right(make_float4(qr.x * ir, qr.y * ir, qr.z * ir, qr.w * ir), Rr);
  const float e[4] = {ls.x, ls.y, ls.z, ls.w};
  float sum = 1e-30f;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    float r = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) r = fmaf(L[3][i], Rr[i][k], r);
    const float m = (fabsf(r) + 2e-6f) * expf(e[k]);
    sum = fmaf(m, m, sum);
  }
  return sum * 1.0001f;
}

// A wave per unit of 64 consecutive primitives, kPreViews views at a time,
// without barriers between the steps:
//   1. a lane per primitive: the views in which it can pass the temporal
//      filter, by a FP32 bound that never drops one (cull2 = -2 log t_cull,
//      enlarged), and the FP64 shape if there is any, kept in LDS;
//   2. a lane per such (view, primitive) pair: the exact filter, slice,
//      projection, footprint, record.
// The pairs come from ballots, so the lanes of the second step are full: with
// a thread per primitive and a loop over the views, a wave ran a view's ~300
// FP64 instructions whenever any of its 64 lanes was active. A pair's outputs
// do not depend on the lane that computes them.
// What a pair writes goes to its place in the unit's slab (64 n_views places),
// the unit's pairs one after the other in (view, primitive) order, so that a
// wave's 68 bytes per pair fill whole cache lines. Laid out by (view,
// primitive), with gaps at the culled pairs, it was bound by partial lines.
// 62 -> 16 us for one view of 300k primitives, 78 -> 31 for 8 of them, 375 ->
// 132 for 16 views of 1M, 605 -> 218 for 8 of 3M;
// the same kernel with gaps took 17, 48, 348 and 504;
// the colour kernels that read the pairs back, 92 -> 86, 560 -> 447, 917 -> 714.
constexpr int kPreViews = 16;
struct PreWave {
  double S[10][64];  // per primitive: Sigma (00 01 02 03 11 12 13 22 23 33)
  double opa[64];
  float4 mu[64];
  uint16_t pair[64 * kPreViews];  // view << 8 | primitive
  uint32_t act[kPreViews][2];     // the active pairs
};
__global__ void __launch_bounds__(256, 3) k_preprocess(RenderParams p, float cull2, PairBits pb,
                                                       uint32_t* __restrict__ group_count,
                                                       uint32_t* __restrict__ dkey,
                                                       Record* __restrict__ rec, float4* __restrict__ cdir,
                                                       uint32_t* __restrict__ zero, uint32_t n_zero) {
  __shared__ PreWave s_waves[4];
  __shared__ ViewDev s_view[kPreViews];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  PreWave& w = s_waves[wave];
  const uint32_t unit = blockIdx.x * 4 + wave;  // (there are whole groups of four units)
  const int gidx = (int)(unit * 64) + lane;
  const double t_cull = p.t_cull, near = p.near_plane;
  const uint64_t lower = (1ull << lane) - 1ull;
  // the words of the sort that follows
  for (uint32_t i = blockIdx.x * 256 + tid; i < n_zero; i += gridDim.x * 256) zero[i] = 0u;
  float s44 = 0.f, mu_t = 0.f;
  bool usable = false, any = false;
  float4 ls = make_float4(0.f, 0.f, 0.f, 0.f), qlf = ls, qrf = ls;
  if (gidx < p.n) {
    const float4 mu = p.means4[gidx];
    ls = p.log_scales4[gidx];
    qlf = p.q_left[gidx];
    qrf = p.q_right[gidx];
    const float logit = p.opacity_logit[gidx];
    // a primitive with a non-finite parameter is culled in every view (and counted)
    usable = finite4(mu) && finite4(ls) && finite4(qlf) && finite4(qrf) && isfinite(logit);
    if (usable) {
      s44 = sigma44_bound(qlf, qrf, ls);
      mu_t = mu.w;
      w.mu[lane] = mu;
      w.opa[lane] = (double)logit;  // (its sigmoid with the shape)
    } else if (p.nonfinite) {
      for (int vi = 0; vi < p.n_views; ++vi) atomicAdd(p.nonfinite + vi, 1u);
    }
  }
  bool have_shape = false;
  uint32_t place = unit * 64u * (uint32_t)p.n_views;  // the next pair's
  for (int vc = 0; vc < p.n_views; vc += kPreViews) {
    const int nv = min(kPreViews, p.n_views - vc);
    __syncthreads();  // the previous views are read
    for (int i = tid; i < nv * (int)(sizeof(ViewDev) / 4); i += 256)
      reinterpret_cast<uint32_t*>(s_view)[i] = reinterpret_cast<const uint32_t*>(p.views + vc)[i];
    if (lane < 2 * kPreViews) w.act[lane >> 1][lane & 1] = 0u;
    __syncthreads();
    // ---- 1. which pairs can pass the temporal filter ----
    uint32_t m = 0u;
    int pairs = 0;
    for (int v = 0; v < nv; ++v) {
      const float dt = s_view[v].t - mu_t, dt2 = dt * dt;
      // (a square out of float's range, or a NaN, is left to the exact test)
      const bool out = dt2 > cull2 * s44 && dt2 < 3e38f;
      const bool in = usable && !out;
      const uint64_t b = __ballot(in);
      if (in) w.pair[pairs + __popcll(b & lower)] = (uint16_t)(v << 8 | lane);
      if (lane == 0) {
        pb.listed[(size_t)(vc + v) * pb.units + unit] = b;
        pb.first[(size_t)(vc + v) * pb.units + unit] = place + (uint32_t)pairs;
      }
      pairs += (int)__popcll(b);
      m |= in ? 1u : 0u;
    }
    if (m && !have_shape) {
      Shape4T<double> sh;
      build_shape<double>(qlf, qrf, ls, sh);
      int k = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = i; j < 4; ++j) w.S[k++][lane] = sh.S[i][j];
      w.opa[lane] = 1.0 / (1.0 + exp(-w.opa[lane]));
      have_shape = true;
    }
    __builtin_amdgcn_wave_barrier();  // (the wave's LDS accesses are in order)
    // ---- 2. pairs ----
    for (int i = lane; i < pairs; i += 64) {
      const int v = w.pair[i] >> 8, c = w.pair[i] & 255;
      const ViewDev& vw = s_view[v];
      Shape4T<double> sh;
      int k = 0;
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int j = r; j < 4; ++j) {
          sh.S[r][j] = w.S[k++][c];
          sh.S[j][r] = sh.S[r][j];
        }
      sh.inv44 = 1.0 / sh.S[3][3];
      const double opa = w.opa[c];
      // temporal marginal and filter, slice, camera, EWA projection
      ViewGeomT<double> g;
      bool ok = view_geometry<double>(w.mu[c], sh, vw, t_cull, near, g);
      int x0 = 0, x1 = 0, y0 = 0, y1 = 0;
      if (ok) {
        // ---- footprint: integer 3-sigma radius, half-open tile rectangle ----
        const double mid = 0.5 * (g.a2 + g.c2);
        const double lmax = mid + sqrt(fmax(mid * mid - g.det, 0.0));
        const double rad = ceil(kSigmaExtent64 * sqrt(lmax));
        const double tx = vw.tiles_x, ty = vw.tiles_y;
        const double ft = 1.0 / kTile;  // a power of two: the product is exact
        x0 = (int)fmin(fmax(floor((g.u - rad) * ft), 0.0), tx);
        x1 = (int)fmin(fmax(floor((g.u + rad) * ft) + 1.0, 0.0), tx);
        y0 = (int)fmin(fmax(floor((g.v - rad) * ft), 0.0), ty);
        y1 = (int)fmin(fmax(floor((g.v + rad) * ft) + 1.0, 0.0), ty);
        ok = g.det > 0.0 && isfinite(g.u) && isfinite(g.v);
        if (p.ellipse_cull) {
          // Binning footprint: only tiles that can hold a pixel with
          // opacity * exp(power) >= 1/255, i.e. inside the ellipse
          // 1/2 d^T conic d <= ln(255 opacity); its bounding box has
          // half-widths sqrt(2 K Sigma2d_00), sqrt(2 K Sigma2d_11). Every other
          // tile of the 3-sigma rectangle would skip this primitive at every
          // pixel, so the blend is unchanged. The box only narrows the exact
          // rectangle, so it is formed in FP32 with slack for that and for the
          // FP32 evaluation of the fragments.
          const float K = __logf(255.f * (float)(opa * g.pt));
          ok = ok && K > -1e-4f;
          const float Kc = fmaxf(K, 0.f);
          const float hx = sqrtf(2.f * Kc * (float)g.a2) * 1.001f + 0.05f;
          const float hy = sqrtf(2.f * Kc * (float)g.c2) * 1.001f + 0.05f;
          const float uf = (float)g.u, vf = (float)g.v, ft = 1.f / kTile;
          const float bx = (float)vw.tiles_x + 1.f, by = (float)vw.tiles_y + 1.f;
          x0 = max(x0, (int)fminf(fmaxf(floorf((uf - hx) * ft), -1.f), bx));
          x1 = min(x1, (int)fminf(fmaxf(floorf((uf + hx) * ft) + 1.f, -1.f), bx));
          y0 = max(y0, (int)fminf(fmaxf(floorf((vf - hy) * ft), -1.f), by));
          y1 = min(y1, (int)fminf(fmaxf(floorf((vf + hy) * ft) + 1.f, -1.f), by));
        }
        ok = ok && (x1 > x0) && (y1 > y0);
      }
      if (!ok) continue;
      const uint32_t at = place + (uint32_t)i;
      const double z = g.pc[2];
      const float zf = (float)z;
      Record r;
      r.a = make_float4((float)g.u, (float)g.v, zf, (float)(opa * g.pt));
      r.b = make_float4((float)g.conic[0], (float)g.conic[1], (float)g.conic[2],
                        __uint_as_float((uint32_t)x0 | ((uint32_t)x1 << 16)));
      const float yr = __uint_as_float((uint32_t)y0 | ((uint32_t)y1 << 16));
      if (p.flow) {
        // Sec. 4.4: the conditional mean moves by v dt' / Sigma_44 (it is
        // linear in t); its projection moves by f (x' z - x z') / (z z') per axis
        const double sc = (double)p.flow_dt * sh.inv44;
        double dp[3];
#pragma unroll
        for (int a = 0; a < 3; ++a)
          dp[a] = sc * ((double)vw.rot[3 * a] * g.v3[0] + (double)vw.rot[3 * a + 1] * g.v3[1] +
                        (double)vw.rot[3 * a + 2] * g.v3[2]);
        const double z1 = z + dp[2];
        const bool front = z1 > near;
        const double q = front ? 1.0 / (z * z1) : 0.0;
        r.c = make_float4((float)(vw.fx * (dp[0] * z - g.pc[0] * dp[2]) * q),
                          (float)(vw.fy * (dp[1] * z - g.pc[1] * dp[2]) * q), 0.f, yr);
      } else {
        // colour: k_colour fills c.xyz from the view direction and t - mu_t
        r.c = make_float4(0.f, 0.f, 0.f, yr);
        cdir[at] = make_float4((float)g.dir[0], (float)g.dir[1], (float)g.dir[2], (float)g.dt);
      }
      rec[at] = r;
      dkey[at] = __float_as_uint(zf);  // z > near > 0: bit order = numeric order
      atomicOr(&w.act[v][c >> 5], 1u << (c & 31));
    }
    place += (uint32_t)pairs;
    __syncthreads();
    // the units' bits and the group's counts
    if (tid < nv * 8) {
      const int v = tid >> 3, k = tid & 7;
      const uint32_t word = s_waves[k >> 1].act[v][k & 1];
      pb.active[((size_t)(vc + v) * pb.units + 4 * blockIdx.x) * 2 + k] = word;
      uint32_t c = (uint32_t)__popc(word);  // a group's eight words are in eight adjacent lanes
      c += __shfl_xor(c, 1, 64);
      c += __shfl_xor(c, 2, 64);
      c += __shfl_xor(c, 4, 64);
      if (k == 0) group_count[(size_t)(vc + v) * gridDim.x + blockIdx.x] = c;
    }
    for (int v = 0; v < nv; ++v) any = any || ((w.act[v][lane >> 5] >> (lane & 31)) & 1u);
  }
  if (gidx < p.n) p.pany[gidx] = any ? 1 : 0;
}

// The primitives active in some view (in no particular order) and their
// number: 4096 per workgroup, one atomic each (at ~12.5 ns per atomic on one
// counter, one per wave of the preprocess took 50 us on 300k primitives).
__global__ void __launch_bounds__(256) k_list_active(const uint8_t* __restrict__ pany, int n,
                                                     uint32_t* __restrict__ list, uint32_t* __restrict__ list_n) {
  __shared__ uint32_t s_wave[4], s_base;
  const int i0 = (int)(blockIdx.x * 4096 + threadIdx.x * 16);
  uint32_t m = 0u;
  if (i0 + 16 <= n) {
    const uint4 q = *reinterpret_cast<const uint4*>(pany + i0);
    const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
    for (int j = 0; j < 16; ++j) m |= ((w[j >> 2] >> (8 * (j & 3))) & 1u) << j;
  } else {
    for (int j = 0; j < 16 && i0 + j < n; ++j) m |= (uint32_t)(pany[i0 + j] & 1) << j;
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t c = (uint32_t)__popc(m);
  uint32_t x = c;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t y = __shfl_up(x, off, 64);
    if (lane >= off) x += y;
  }
  if (lane == 63) s_wave[wave] = x;
  __syncthreads();
  if (threadIdx.x == 0) s_base = atomicAdd(list_n, s_wave[0] + s_wave[1] + s_wave[2] + s_wave[3]);
  __syncthreads();
  uint32_t at = s_base + x - c;
  for (int w = 0; w < wave; ++w) at += s_wave[w];
  while (m) {
    const int j = __ffs(m) - 1;
    m &= m - 1u;
    list[at++] = (uint32_t)(i0 + j);
  }
}

constexpr int kColourViews = 8;  // views that k_colour takes together

// 4D spherindrical-harmonic colour (Sec. 3.2) of the primitives active in
// some view (the list of them): a wave takes 16 listed primitives, a quad of
// lanes each, lane `sub` owning the basis functions lm = 4 sub + i and reading
// their coefficients straight from memory (the quad reads the primitive's
// coefficients once for all views, and in whole 16-byte pieces where they are
// aligned). The pairs of the 16 primitives in eight views at a time, up to 128:
//   1. a lane per view and primitive: its pair's place, listed in LDS;
//   2. a lane per listed pair: the basis and the Fourier terms, to LDS;
//   3. a quad per primitive, its pairs one after the other: the products with the
//      coefficients, summed over the quad.
// Vector instructions bounded it while each quad formed the bases of its own
// pairs (four times the same, and idle while another quad of the wave had
// more: 655 instructions a pair and lane, 270 of 355 us alone for 4M pairs). 355
// -> 255 us, beside the compaction and the depth sort 452 -> 329; 5.7M pairs 715
// -> 650; 0.7M 86 -> 66.
struct ColourPair {  // (a fifth 16 bytes also spreads the pairs over the banks)
  float4 basis[4];
  float2 cs;  // cs[1], cs[2]
  uint32_t place, pad;
};
__global__ void __launch_bounds__(256, 4) k_colour(RenderParams p, PairBits pb,
                                                const float4* __restrict__ cdir, Record* __restrict__ rec) {
  __shared__ ColourPair s_pairs[4][16 * kColourViews];  // 40 KB: four workgroups per CU
  ColourPair* pairs = s_pairs[threadIdx.x >> 6];
  const int nb = (p.sh_degree + 1) * (p.sh_degree + 1);
  const int nt = p.t_order + 1;
  const int K3 = nt * nb * 3;
  const uint32_t count = *p.plist_n;
  const int sub = threadIdx.x & 3, lane = threadIdx.x & 63;
  const uint32_t stride = (gridDim.x * blockDim.x) >> 2;
  for (uint32_t e0 = ((blockIdx.x * blockDim.x) >> 2); e0 < count; e0 += stride) {
    const uint32_t e = e0 + (threadIdx.x >> 2);
    const bool live = e < count;  // uniform per quad
    const int gidx = live ? (int)p.plist[e] : 0;
    float k[3][kBasisPerLane][3];
    if (live) load_own_coeffs(p.coeffs + (size_t)gidx * K3, sub, nb, nt, k);
    for (int v0 = 0; v0 < p.n_views; v0 += kColourViews) {
      // 1. lane `sub`: views v0 + sub and v0 + sub + 4
      uint32_t at[2], m = 0u;
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int v = v0 + sub + 4 * t;
        const bool there = live && v < p.n_views;
        at[t] = there ? pair_place(pb, v, gidx) : 0u;
        m |= (there && pair_active(pb, v, gidx) ? 1u : 0u) << (sub + 4 * t);
      }
      m |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0xB1, 0xF, 0xF, true);  // over the quad
      m |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0x4E, 0xF, 0xF, true);
      const uint32_t mine = (uint32_t)__popc(m);
      uint32_t upto = mine;  // inclusive scan over the quads
#pragma unroll
      for (int off = 4; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(upto, off, 64);
        if (lane >= off) upto += y;
      }
      const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)upto, 63), first = upto - mine;
      __builtin_amdgcn_wave_barrier();  // (the wave's LDS accesses are in order)
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int w = sub + 4 * t;
        if ((m >> w) & 1u) pairs[first + __popc(m & ((1u << w) - 1u))].place = at[t];
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      // 2.
      for (uint32_t i = lane; i < total; i += 64) {
        const float4 cd = cdir[pairs[i].place];
        float Y[16], cs[3] = {0.f, 0.f, 0.f};
#pragma unroll
        for (int jj = 0; jj < 16; ++jj) Y[jj] = 0.f;
        sh_eval(p.sh_degree, cd.x, cd.y, cd.z, Y);
        fourier_terms(p.t_order, cd.w, p.t_period, cs);
#pragma unroll
        for (int q = 0; q < 4; ++q) pairs[i].basis[q] = make_float4(Y[4 * q], Y[4 * q + 1], Y[4 * q + 2], Y[4 * q + 3]);
        pairs[i].cs = make_float2(cs[1], cs[2]);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      // 3.
      bool finite = true;
#pragma unroll
      for (int n = 0; n < 3; ++n)
#pragma unroll
        for (int i = 0; i < kBasisPerLane; ++i)
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            if (!live) k[n][i][c] = 0.f;
            finite = finite && isfinite(k[n][i][c]);
          }
      const bool bad = quad_any(!finite);
      for (uint32_t i = first; i < upto; ++i) {  // uniform per quad
        const float4 y4 = pairs[i].basis[sub];
        const float2 f = pairs[i].cs;
        const float y[kBasisPerLane] = {y4.x, y4.y, y4.z, y4.w};
        float col[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          float acc = 0.f;
#pragma unroll
          for (int j = 0; j < kBasisPerLane; ++j)
            acc = fmaf(y[j], fmaf(1.f, k[0][j][c], fmaf(f.x, k[1][j][c], f.y * k[2][j][c])), acc);
          col[c] = fmaxf(quad_sum(acc) + kColorOffset, 0.f);
        }
        // (a primitive with a non-finite coefficient is rendered transparent)
        const float o = bad ? __int_as_float(0x7FC00000) : sub == 0 ? col[0] : sub == 1 ? col[1] : col[2];
        if (sub < 3) reinterpret_cast<float*>(&rec[pairs[i].place].c)[sub] = o;
      }
      if (bad && sub == 0 && p.nonfinite)
        for (int w = 0; w < kColourViews; ++w)
          if ((m >> w) & 1u) atomicAdd(p.nonfinite + v0 + w, 1u);
    }
  }
}

}  // namespace

void launch_preprocess(const RenderParams& p, const PairBits& pb, uint32_t* group_count, uint32_t* dkey,
                       Record* rec, float4* cdir, uint32_t* zero, uint32_t n_zero, hipStream_t s) {
  if (p.n == 0) return;
  // -2 log t_cull, enlarged past every rounding of the FP32 test (infinite, so
  // that every pair is listed, for t_cull = 0)
  const float cull2 = (float)(-2.0 * std::log((double)p.t_cull) * 1.001 + 1e-5);
  hipLaunchKernelGGL(k_preprocess, dim3(pair_groups(p.n)), dim3(256), 0, s, p, cull2, pb, group_count, dkey, rec,
                     cdir, zero, n_zero);
}

// Workgroups of the kernels that walk the active-primitive list (64 listed
// primitives per workgroup and step): one step for up to 2^20 primitives,
// grid-stride beyond.
unsigned list_grid(int n) {
  const unsigned need = (unsigned)((n + kColourPrims - 1) / kColourPrims);
  return need < 1 ? 1 : (need < 16384 ? need : 16384);
}

void launch_colour(const RenderParams& p, const PairBits& pb, const float4* cdir, Record* rec, hipStream_t s) {
  if (p.n == 0 || p.flow) return;
  hipLaunchKernelGGL(k_list_active, dim3((unsigned)((p.n + 4095) / 4096)), dim3(256), 0, s, p.pany, p.n, p.plist,
                     p.plist_n);
  hipLaunchKernelGGL(k_colour, dim3(list_grid(p.n)), dim3(256), 0, s, p, pb, cdir, rec);
}

}  // namespace g4d
