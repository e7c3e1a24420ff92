// Host-side launch plumbing shared by the kernel translation units.
#pragma once
#include <vector>

#include "nbvh_internal.h"

namespace nbvh {

// HIP event pairs around kernel groups, recorded on the launch stream while a
// profiling window is open (nbvh_profile_begin / nbvh_profile_end).
struct Profiler {
  bool on = false;
  std::vector<hipEvent_t> ev;  // 2 per record
  std::vector<int> kid;
  size_t used = 0;
  static constexpr size_t kMax = 16384;
};

class ProfScope {
 public:
  ProfScope(Profiler* p, int kid, hipStream_t s) : p_(p), idx_((size_t)-1), s_(s) {
    if (p_ && p_->on && p_->used < p_->kid.size()) {
      idx_ = p_->used++;
      p_->kid[idx_] = kid;
      (void)hipEventRecord(p_->ev[2 * idx_], s_);
    }
  }
  ~ProfScope() {
    if (idx_ != (size_t)-1) (void)hipEventRecord(p_->ev[2 * idx_ + 1], s_);
  }

 private:
  Profiler* p_;
  size_t idx_;
  hipStream_t s_;
};

// Device state block (nbvh_state_bytes() bytes, caller-owned).
struct DevState {
  int64_t step;
  int64_t skipped;
  float loss_scale;
  uint32_t flags;
  float last_loss[4];
  uint64_t last_n_segments;
  uint32_t nonfinite_pending;  // set by producers of this step's gradient
  uint32_t pad0;
  unsigned long long n_evaluated;  // segments evaluated by queries
  uint32_t pad[4];
};

struct LaunchCtx {
  hipStream_t stream;
  hipStream_t side;                // the context's second stream (nullable)
  hipEvent_t ev_fork, ev_join;     // fork to and join from `side`
  const Node* nodes;
  DevState* state;
  DevCfg cfg;
  int precision;
  float* params;
  void* params_lp;
  float* adam_m;
  float* adam_v;
  float* grad;
  void* aux;  // weight copies and FP8 scales (aux_total_bytes)
  bool fp8;   // queries and forward run the MLP in FP8 (weights and scales in aux)
  uint32_t n_nodes;
  int stack_depth;  // inner levels of the N-BVH: entries of a traversal stack
  int n_cu;
  // training hyper-parameters
  float w_hit, w_t, w_normal, w_albedo;
  float lr, beta1, beta2, eps, loss_scale;
  Profiler* prof;
  nbvh_tuning tune;
};

nbvh_status check_launch(const char* what);
void set_error(const char* fmt, ...);

__global__ void k_zero_u32(uint32_t* p, uint32_t n);
__global__ void k_zero_f32(float* p, uint64_t n);

// BF16 queries read the MLP weights in fragment order. The copies are made in
// every query, as the caller may have written the shadow since the last one, by
// workgroups of its traversal beside those of the rays: a launch of its own
// would take 3 us. Queries of one context on several streams write the same
// values.
struct WeightCopy {
  const void* src;  // the BF16 shadow of the parameters
  void* dst;        // the copies
  uint32_t blocks;  // workgroups of 256 threads, 16 bytes a thread (0: nothing to copy)
};

inline WeightCopy weight_copy(const LaunchCtx& L) {
  if (L.precision != NBVH_BF16 || L.fp8) return WeightCopy{nullptr, nullptr, 0};
  return WeightCopy{L.params_lp, (char*)L.aux + wf16_off(L.cfg), (uint32_t)((L.cfg.n_wf / 8 + 255) / 256)};
}

// workgroups of 256 rays
__host__ __device__ inline uint32_t ray_blocks(uint32_t n_rays) { return (uint32_t)(((uint64_t)n_rays + 255) / 256); }

__device__ inline void order_weights(const DevCfg& c, const WeightCopy& wc, uint32_t block) {
  const uint64_t e = ((uint64_t)block * 256 + threadIdx.x) * 8;  // eight columns of a row: a lane's part of a fragment
  if (e >= c.n_wf) return;
  int k = 0;
  while (k < c.hidden && e >= c.wf_off[k + 1]) ++k;
  const uint32_t K = (uint32_t)c.fan_in[k], at = (uint32_t)(e - c.wf_off[k]) / 8, lane = at & 63u, frag = at >> 6;
  const uint32_t n = frag / (K / 32) * 16 + (lane & 15u), col = frag % (K / 32) * 32 + (lane >> 4) * 8;
  if (n < (uint32_t)c.fan_out[k])  // the last rows of a padded tile hold nothing
    *(uint4*)((uint16_t*)wc.dst + e) = *(const uint4*)((const uint16_t*)wc.src + c.w_off[k] + (uint64_t)n * K + col);
}

// A permutation of the rays (launch_ray_order): the traversal's counting pass
// takes them in perm order; inv[r] is ray r's position in perm.
struct RayOrder {
  const uint32_t* perm;
  const uint32_t* inv;
};
size_t ray_order_bytes(uint64_t n);
// order: tuning query_order (0 leaves both pointers null); ws: ray_order_bytes(n)
nbvh_status launch_ray_order(const LaunchCtx& L, const nbvh_ray* rays, uint32_t n, int order, void* ws,
                             RayOrder* out);

// `staging` (traverse_staging_bytes(n_rays), required with `segs`): sorted
// per-ray runs kept by the counting pass so that the compaction copies them
// instead of walking again. `order` (nullable): a permutation the counting
// pass follows. `active_order_ws` (nullable, ray_order_bytes(n_rays)): with
// an active list and tuning query_order, sort the list by key once it is
// built instead. With `active` (the list of rays with a segment,
// in ray order; its length goes to *n_active, and the query's eight ray-queue
// counters after it are cleared), `segs`, scratch_pos
// (n_rays + 1 words) and scratch_sums2 (like scratch_sums) are required, and
// the query's weight copies are made.
size_t traverse_staging_bytes(uint64_t n_rays);
nbvh_status launch_traverse(const LaunchCtx& L, const nbvh_ray* rays, uint32_t n_rays, uint32_t* offsets,
                            nbvh_segment* segs, uint64_t capacity, nbvh_hit* hits, uint32_t* active,
                            uint32_t* n_active, uint32_t* scratch_counts, uint32_t* scratch_sums, float* staging,
                            const RayOrder* order = nullptr,
                            void* active_order_ws = nullptr, uint32_t* scratch_pos = nullptr,
                            uint32_t* scratch_sums2 = nullptr);

// z_trace / u_trace (nullable): each evaluated segment's logits [cap][n_out]
// and FP32 copy of its LDS feature row [cap][n_in] (not in FP8), at the
// segment's queue position; rows of segments not evaluated are untouched.
// own_queue: the segments come from launch_traverse, so each names its ray.
nbvh_status launch_query_eval(const LaunchCtx& L, const nbvh_ray* rays, const uint32_t* offsets,
                              const nbvh_segment* segs, const uint32_t* active, const uint32_t* n_active,
                              uint32_t* counter, nbvh_hit* hits, uint32_t n_rays_bound, uint64_t capacity,
                              float* z_trace = nullptr, float* u_trace = nullptr, bool own_queue = true);

nbvh_status launch_query_eval_batch(const LaunchCtx* Ls, int n_obj, const DevCfg* cfgs_dev, const uint32_t* const* offsets,
                                    const nbvh_segment* const* segs, const uint32_t* const* active,
                                    const uint32_t* const* n_active, uint32_t* const* counters, nbvh_hit* per_obj,
                                    nbvh_hit* hits, const nbvh_ray* rays, uint32_t n_rays, uint64_t capacity);

nbvh_status launch_first_hits(const LaunchCtx& L, const nbvh_ray* rays, uint32_t n, const float* u,
                              const float* accept, nbvh_probe* probes, uint32_t* leaf_out, uint32_t* n_out,
                              uint32_t* leaf_hits);

size_t group_ws_bytes(uint64_t n);
nbvh_status launch_group_by_leaf(const LaunchCtx& L, uint32_t n_leaves, const nbvh_probe* in, const uint32_t* ids,
                                 uint32_t n, nbvh_probe* out, uint32_t* ids_out, void* ws);

nbvh_status launch_leaf_loss(const LaunchCtx& L, const nbvh_probe* probes, const nbvh_label* labels,
                             const uint32_t* leaf_ids, uint32_t n, float* z, float* leaf_loss, uint32_t* leaf_count);

nbvh_status launch_active_rays(const LaunchCtx& L, const uint32_t* offsets, uint32_t n_rays, nbvh_hit* hits,
                               uint32_t* active, uint32_t* misc);

nbvh_status launch_encode(const LaunchCtx& L, const nbvh_probe* probes, uint32_t n, float* u);

nbvh_status launch_forward(const LaunchCtx& L, const nbvh_probe* probes, uint32_t n, float* z);

// FP8 calibration: weight scales from the FP32 master weights, activation
// scales from an FP32 forward of the given segments, then E4M3 weights.
nbvh_status launch_calibrate_fp8(const LaunchCtx& L, const nbvh_probe* probes, uint32_t n);

// training
size_t train_ws_bytes(const DevCfg& c, int precision, uint64_t max_batch, const nbvh_tuning& tune);
// out[0..n] = exclusive prefix sums of in[0..n) (out[n] = total); sums needs
// n / 1024 + 2 words
nbvh_status launch_exclusive_scan(hipStream_t s, const uint32_t* in, uint32_t n, uint32_t* out, uint32_t* sums);
nbvh_status launch_train_fwd_bwd(const LaunchCtx& L, const nbvh_probe* probes, const nbvh_label* labels,
                                 const float* dz_in, uint32_t n, float* loss_dev, void* ws, size_t ws_bytes,
                                 bool apply_grad);
nbvh_status launch_loss(const LaunchCtx& L, const float* z, const nbvh_label* labels, uint32_t n, float* loss_dev,
                        float* dz, void* ws, size_t ws_bytes);
nbvh_status launch_optimizer(const LaunchCtx& L, bool reset, bool shadow_only);
nbvh_status launch_unscale_grad(const LaunchCtx& L, float* out, bool clear);
nbvh_status launch_node_rank(hipStream_t s, const float* loss, const uint32_t* count, const uint32_t* hits, uint32_t n,
                             uint64_t n_rays, float* rank);
nbvh_status launch_acceptance(hipStream_t s, const float* rank, uint32_t n, float floor_, float* accept);

}  // namespace nbvh
