// Internal declarations shared by the HIP translation units of libg4d.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace g4d {

constexpr int kTile = 16;                 // 16x16 pixel tiles
constexpr float kLowpass = 0.3f;          // EWA dilation, px^2
constexpr double kLowpass64 = 0.3;        // the same, for the FP64 forward geometry
constexpr float kFrustumSlack = 1.3f;     // Jacobian clamp, x half-fov
constexpr double kFrustumSlack64 = 1.3;
constexpr double kSigmaExtent64 = 3.0;
constexpr float kSigmaExtent = 3.0f;      // footprint radius in sigmas
constexpr float kAlphaMax = 0.99f;        // alpha clamp
constexpr float kTStop = 1e-4f;           // transmittance stop threshold
constexpr float kColorOffset = 0.5f;
// log2(1/255): fragments with log2(opacity * exp(power)) below this are skipped
constexpr float kLog2AlphaMin = -7.994353436858858f;
// log2(0.99) less a margin over the rounding of log2 and exp2: a fragment of a
// record whose log2 opacity is below this never reaches the alpha clamp, as its
// power is not positive. For elongated footprints (ill_conditioned) FP32 rounding
// can make it so by far more than the margin; for others the quadratic form is
// at least 1/200 of the sum of its terms' magnitudes, whose rounding is 1e-6 of it.
constexpr float kLog2AlphaMax = -0.0146f;
constexpr float kLog2e = 1.4426950408889634f;

// One view of a batch, device side.
struct ViewDev {
  int width, height, tiles_x, tiles_y;
  int tile_base;        // first global tile id of this view
  int pad0;
  long long pix_base;   // first pixel of this view in the concatenated planes
  float fx, fy, cx, cy;
  float rot[9];         // world -> camera rotation, row-major
  float trans[3];
  float center[3];      // camera position (world)
  float t;              // render time
  float lim_x, lim_y;   // Jacobian clamp limits on x/z, y/z
  double lim_x64, lim_y64;  // the same limits in FP64: 1.3 (W/2) / fx, 1.3 (H/2) / fy
};

// Doubles per active record in the screen-space gradient buffer: one 128-byte
// line holding dL/du, dL/dv, dL/dconic (3), dL/d(opacity p), dL/drgb (3),
// dL/dz, padding and (last) the count of tiles it blended in. The tiles' shares are added in
// FP64: a long footprint adds terms of both signs from many tiles, whose
// float32 sum would lose the small total.
constexpr int kGrad2dStride = 16;

// Per active (view, primitive) record used by binning and rasterisation.
// 3 x float4 = 48 bytes:
//   a: u, v, z, opacity * p(t)
//   b: conic00, conic01, conic11, rect x range (x0 | x1 << 16, as float bits)
//   c: r, g, b, rect y range (y0 | y1 << 16, as float bits)
struct Record {
  float4 a, b, c;
};

struct RenderParams {
  int n;                // primitives
  int n_views;
  int sh_degree, t_order;
  float t_period, t_cull, near_plane;
  float bg[3];
  const float4* means4;
  const float4* log_scales4;
  const float4* q_left;
  const float4* q_right;
  const float* opacity_logit;
  const float* coeffs;
  const ViewDev* views;
  int flow;             // 1: records carry the image-plane flow over flow_dt instead of the colour
  float flow_dt;
  // 1 (default): a record's rectangle is cut to the box of its alpha-floor
  // ellipse and records that can never reach alpha 1/255 are culled; 0: the
  // plain 3-sigma rectangle and no opacity cull (the reference footprint rule)
  int ellipse_cull;
  // per-view counters of (view, primitive) pairs culled for a non-finite
  // parameter, indexed by the view within the call (null: not counted)
  uint32_t* nonfinite;
  // written by the preprocess: per primitive, 1 when it is active in some
  // view of the call; by the colour pass: the list of those primitives (in no
  // particular order) and its length (zero before)
  uint8_t* pany;
  uint32_t* plist;
  uint32_t* plist_n;
};

// Per-primitive densification accumulators (all null: off).
struct DensifyStats {
  float* uv_grad_norm_sum;
  float* t_grad_abs_sum;
  int32_t* blend_count;
};

// The (view, primitive) pairs of a call. A unit is 64 consecutive primitives,
// a group four units; there are whole groups. Per view and unit: a bit per
// active pair, a bit per listed pair (one that a bound of the temporal filter
// let through; the active ones among them), and the place of its first listed
// pair. The pairs of a unit take consecutive places in (view, primitive) order
// from 64 n_views unit on: dkey, rec and cdir are indexed by place.
struct PairBits {
  int n;
  uint32_t units;    // per view
  uint32_t* active;  // [n_views][units][2]
  uint64_t* listed;  // [n_views][units]
  uint32_t* first;   // [n_views][units]
};
inline uint32_t pair_groups(int n) { return (uint32_t)(((int64_t)n + 255) / 256); }
#ifdef __HIPCC__
// The place of an active pair.
__device__ __forceinline__ uint32_t pair_place(const PairBits& pb, uint32_t view, uint32_t gidx) {
  const size_t u = (size_t)view * pb.units + (gidx >> 6);
  return pb.first[u] + (uint32_t)__popcll(pb.listed[u] & ((1ull << (gidx & 63)) - 1ull));
}
#endif

// ---- launchers (preprocess.hip) ----
// group_count: the active pairs of each view's groups; cdir: view direction,
// t - mu_t. dkey, rec and cdir are written for the active pairs.
// zero[0..n_zero) is set to zero (nothing if null).
void launch_preprocess(const RenderParams& p, const PairBits& pb, uint32_t* group_count, uint32_t* dkey,
                       Record* rec, float4* cdir, uint32_t* zero, uint32_t n_zero, hipStream_t s);
// Lists the primitives active in some view (p.plist), then the 4DSH colour of
// every active pair into its record, before the gather orders the records by
// depth; nothing in flow mode.
void launch_colour(const RenderParams& p, const PairBits& pb, const float4* cdir, Record* rec, hipStream_t s);
// ---- launchers (preprocess_bwd.hip) ----
size_t preprocess_backward_scratch_floats(size_t n_records);
// Workgroups of the kernels that walk the active-primitive list of n primitives.
unsigned list_grid(int n);
// slot: space for the pairs' map view * n + index -> depth position.
void launch_preprocess_backward(const RenderParams& p, const PairBits& pb, int32_t* slot, const double* grad2d,
                                const uint32_t* n_records_dev, uint32_t n_records_max, const uint32_t* ids,
                                const Record* recs, float* scratch, float* g_means4, float* g_log_scales4,
                                float* g_q_left, float* g_q_right, float* g_opacity_logit, float* g_coeffs,
                                bool accumulate, const DensifyStats& stats, hipStream_t s);

// ---- launchers (loss.hip) ----
void launch_image_loss(int kind, uint64_t n, const float* img, const float* tgt, float scale, float* loss,
                       float* grad, hipStream_t s);

// ---- launchers (sort.hip) ----
// Scratch words of the compaction and the gather for n_max pairs.
size_t scan_scratch_words(size_t n_max);
// The active pairs in (view, primitive) order: ckey[i] = dkey[place], cval[i] =
// view * n + primitive; their number in *total, and after each view's last in view_end[view].
// scratch: scan scratch words. hist: null, or 4 * 256 zeroed words that get the
// keys' digit counts.
void launch_compact(const PairBits& pb, const uint32_t* count, int n_views, const uint32_t* dkey, uint32_t* ckey,
                    uint32_t* cval, uint32_t* hist, uint32_t* total, uint32_t* view_end, uint32_t* scratch,
                    hipStream_t s);
// Stable sort of the n (from n_dev) pairs by 32-bit keys in four single-launch
// passes; the result is in (keys, vals). The scratch words start zeroed but
// for the keys' digit counts in the first 4 * 256 (the compaction's hist).
// n_est sizes the grid (any gives the same result).
size_t chain_scratch_words(size_t n_max);
void chain_sort(uint32_t* keys, uint32_t* vals, uint32_t* keys_alt, uint32_t* vals_alt, const uint32_t* n_dev,
                uint32_t n_max, uint32_t n_est, uint32_t* scratch, hipStream_t s);
// LSD radix sort of (key, value) pairs on bits [bit0, bit1) in 8-bit passes
// that ping-pong via alt; the result ends in keys/vals, copied back after an
// odd number of passes unless copy_back is false (then it is in the alt pair).
// With last_ranges (n_ranges entries, keys < 2^bit1, bit0 = 0, at least one
// pass, ranges set to (~0u, 0) by launch_ranges_init or the emission) the last
// pass writes no keys: it bounds each key's run in last_ranges[key] instead
// (launch_ranges_fix then empties the unused); a key >= n_ranges is skipped.
size_t radix_scratch_words(int grid);
int radix_grid(uint32_t n_max, int max_blocks);
int radix_passes(int bit0, int bit1);
void radix_sort(uint32_t* keys, uint32_t* vals, uint32_t* keys_alt, uint32_t* vals_alt, const uint32_t* n_dev,
                uint32_t n_max, int bit0, int bit1, int grid, uint32_t* scratch, hipStream_t s,
                bool copy_back = true, uint2* last_ranges = nullptr, uint32_t n_ranges = 0);
// The same with 16-bit keys (bit1 <= 16), without the copy back: after an odd
// number of passes the result is in (keys_alt, vals_alt).
void radix_sort16(uint16_t* keys, uint32_t* vals, uint16_t* keys_alt, uint32_t* vals_alt, const uint32_t* n_dev,
                  uint32_t n_max, int bit0, int bit1, int grid, uint32_t* scratch, hipStream_t s,
                  uint2* last_ranges = nullptr, uint32_t n_ranges = 0);
void launch_ranges_init(uint2* ranges, uint32_t tiles, hipStream_t s);
void launch_ranges_fix(uint2* ranges, uint32_t tiles, hipStream_t s);
// Pinned host words that get the counts by the launch that finds them (nothing
// if null, or for no pairs): the records, the instance total, and as 64 bits,
// and a copy of view_end.
struct HostCounts {
  uint32_t* counts;  // [4]
  uint32_t* views;   // [n_views]
  const uint32_t* view_end;
  int n_views;
  // The records and instances that the stages enqueued behind the counts can
  // hold (they may be guesses): beyond either, *total is zero, so that those
  // stages see no instance, and the n_views views at guess_views (if not null)
  // get no width, so that the forward rasteriser writes no pixel of them. (With a
  // word of its own to tell it, or an impossible range in every tile, the
  // rasteriser took 615 -> 627 us for 16 mixed views of 1M primitives.)
  uint32_t max_records = 0xFFFFFFFFu;
  uint64_t max_instances = 0xFFFFFFFFull;
  ViewDev* guess_views = nullptr;
};
// Depth-ordered records and the place of each record's first instance: toff[d] from its 256-record
// block's start boff[d / 256]. The instance total in *total (zero beyond host's
// limits), and as 64 bits (to detect 32-bit overflow) in total64[0..1]. boff:
// scan scratch words.
// exact: count only the rectangle's tiles the record's alpha-floor ellipse reaches.
void launch_gather(const uint32_t* n_dev, uint32_t n_max, const uint32_t* ids, const PairBits& pb,
                   const Record* rec, Record* rec_sorted, uint32_t* toff, bool exact, uint32_t* boff,
                   uint32_t* total, uint32_t* total64, const HostCounts& host, hipStream_t s);
// For few pairs and images of few tile rows: the sort of the (key, id) pairs by
// the whole key and the gather of the result, in one launch.
bool sort_gather_fits(uint64_t pairs, int tile_rows);
void launch_sort_gather(const uint32_t* n_dev, uint32_t n_max, const uint32_t* keys, uint32_t* ids,
                        const PairBits& pb, const Record* rec, Record* rec_sorted, uint32_t* toff, bool exact,
                        uint32_t* boff, uint32_t* total, uint32_t* total64, const HostCounts& host, hipStream_t s);
// Instances beyond min(*total, cap) are not written; exact as for launch_gather.
// Keys are 16-bit when the round's tile ids are below 2^16, else 32-bit. With
// ranges_init, the launch also sets ranges_init[0..tiles) to (~0u, 0), the
// start state of the ranges the sort's last pass fills.
void launch_emit(const uint32_t* n_dev, uint32_t n_max, const uint32_t* toff, const uint32_t* boff,
                 const uint32_t* total, uint32_t cap, const Record* rec_sorted, const uint32_t* ids, int n_prims,
                 const ViewDev* views, bool exact,
                 uint32_t* ikey, uint32_t* ival, uint2* ranges_init, uint32_t tiles, hipStream_t s);
void launch_emit(const uint32_t* n_dev, uint32_t n_max, const uint32_t* toff, const uint32_t* boff,
                 const uint32_t* total, uint32_t cap, const Record* rec_sorted, const uint32_t* ids, int n_prims,
                 const ViewDev* views, bool exact,
                 uint16_t* ikey, uint32_t* ival, uint2* ranges_init, uint32_t tiles, hipStream_t s);
void launch_ranges(const uint32_t* n_dev, uint32_t n_max, const uint32_t* ikey, uint2* ranges, hipStream_t s);
void launch_ranges(const uint32_t* n_dev, uint32_t n_max, const uint16_t* ikey, uint2* ranges, hipStream_t s);

// ---- launchers (raster.hip) ----
// order (nullable): the tiles in the order workgroups take them, e.g.
// heaviest lists first. queue (nullable): a device counter; then `blocks`
// workgroups (-1: as many as stay resident) take tiles from it in that order
// until they run out (zeroed before the launch); otherwise one workgroup per
// tile.
// channels: 3 (rgb planes) or 2 (the first two record colour values, e.g. flow).
// cull: waves walk only the entries whose alpha-floor ellipse meets their
// quadrant (false: every entry; same results).
// (Nothing is written of a view of no width.)
void launch_raster_forward(int total_tiles, const uint32_t* order, uint32_t* queue, int blocks, int n_views,
                           const ViewDev* views, const uint2* ranges, const uint32_t* ival,
                           const Record* rec_sorted, const float* bg, int channels, bool cull, float* out_rgb,
                           float* out_depth, float* out_alpha, float* pix_t, uint32_t* pix_last, hipStream_t s);
// The image loss folded into the backward rasteriser: with kind (1 = L1,
// 2 = L2) the rgb input is the rendered image, dL/dC is formed from it and
// target as launch_image_loss forms it, and part[tile] (the launch's tile id)
// receives the tile's unscaled loss sum. kind 0: the rgb input is dL/dC.
struct LossArgs {
  int kind;
  const float* target;
  float scale;
  float* part;
};
void launch_raster_backward(int total_tiles, const uint32_t* order, uint32_t* queue, int blocks, int n_views,
                            const ViewDev* views, const uint2* ranges, const uint32_t* ival,
                            const Record* rec_sorted, const float* bg, const float* dl_rgb, const float* dl_depth,
                            const float* dl_alpha, const float* pix_t, const uint32_t* pix_last, double* grad2d,
                            bool mark_blended, bool cull, const LossArgs& loss, hipStream_t s);
// *loss += scale * sum(part[0..n)) (one workgroup, fixed order).
void launch_loss_partials(const float* part, uint32_t n, float scale, float* loss, hipStream_t s);
void launch_sum_u32(const uint32_t* in, uint64_t n, unsigned long long* out, hipStream_t s);
void launch_range_max(const uint2* ranges, uint32_t tiles, uint32_t* out, hipStream_t s);
// Tile ids by decreasing list length (stable within ~4.4 % length bins) into
// order, through the scratch keys, vals and keys_alt. With fix it first
// empties the ranges the last radix pass did not reach (as launch_ranges_fix),
// and it raises *max_len to the longest list (as launch_range_max).
void launch_tile_order(uint2* ranges, uint32_t tiles, bool fix, uint32_t* keys, uint32_t* vals, uint32_t* keys_alt,
                       uint32_t* order, uint32_t* max_len, int sort_blocks, uint32_t* scratch, hipStream_t s);

// ---- launchers (optim.hip) ----
constexpr int kAdamGroups = 6;
struct AdamGroups {
  float* param[kAdamGroups];
  const float* grad[kAdamGroups];
  uint64_t end[kAdamGroups];  // cumulative element counts
  float lr[kAdamGroups];
};
// bc1 = 1 - beta1^step, bc2 = 1 - beta2^step; m, v: [end[5]] moment buffers.
void launch_adam(const AdamGroups& a, float b1, float b2, float eps, float bc1, float bc2, float* m, float* v,
                 hipStream_t s);
// out[k] = mu_i + R_i S_i z[k], i = idx[k]; NaN rows for i outside [0, n).
void launch_split_sample(const RenderParams& p, uint64_t count, const int32_t* idx, const float* z, float* out,
                         hipStream_t s);

// ---- launchers (util.hip) ----
// Views reach the device through kernel arguments, never a host copy.
// The views to the device; the spans of words are set to zero by the same launch.
constexpr int kZeroSpans = 3;
struct ZeroWords {
  uint32_t* p[kZeroSpans];
  uint32_t n[kZeroSpans];
};
void launch_set_views(const ViewDev* host, int n, ViewDev* dev, ZeroWords zero, hipStream_t s);
void launch_fill_u32(uint32_t* p, uint64_t n, uint32_t value, hipStream_t s);
// Zeroes floats_per_item (a multiple of 4) floats per item for min(*n_dev, max_items) items.
void launch_zero_counted(float* p, const uint32_t* n_dev, uint32_t floats_per_item, uint64_t max_items,
                         hipStream_t s);
// If the 64-bit instance total at inst64 exceeds cap: *overflow = 1 and
// *n_inst = 0. Then, with a_tot: *a_tot += *a and *(uint64*)i_tot64 += *n_inst
// (one thread).
void launch_cap_check(const uint32_t* inst64, uint32_t* n_inst, uint32_t* overflow, uint64_t cap, hipStream_t s,
                      const uint32_t* a = nullptr, uint32_t* a_tot = nullptr, uint32_t* i_tot64 = nullptr);
void launch_copy_pairs(const uint32_t* ka, const uint32_t* va, uint32_t* kb, uint32_t* vb, const uint32_t* n_dev,
                       uint32_t n_max, hipStream_t s);

}  // namespace g4d
