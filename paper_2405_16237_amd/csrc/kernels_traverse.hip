// N-BVH traversal (Sec. 5): per-lane stack, two child slab tests per visit,
// count -> exclusive scan -> fill into a compacted segment queue, each ray's
// run sorted front to back by (t0, leaf id).
//
// The slab test is binary32 with one rounding per operation (this file is
// built with FP contraction off) and correctly rounded reciprocals; because
// every inner box is the exact union of its children and each operation is
// monotone in the box bounds, the tree visits exactly the leaves an
// every-leaf test reports, with bit-identical intervals.
#include "launch.h"

namespace nbvh {

struct RayPre {
  float o[3], d[3], inv[3];
  float tmin, tmax;
  bool neg[3];  // the direction's sign bit: the far plane of the slab is lo
};

// inv = 1 / d, also where d is zero (inv = +-inf; see slab).
__device__ inline RayPre load_ray(const nbvh_ray* rays, uint32_t r) {
  const float4* p = (const float4*)(rays + r);
  float4 a = p[0], b = p[1];
  RayPre R;
  R.o[0] = a.x;
  R.o[1] = a.y;
  R.o[2] = a.z;
  R.tmin = a.w;
  R.d[0] = b.x;
  R.d[1] = b.y;
  R.d[2] = b.z;
  R.tmax = b.w;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    R.inv[k] = 1.0f / R.d[k];
    R.neg[k] = __float_as_uint(R.d[k]) >> 31;
  }
  return R;
}

// hit iff tn <= tf; axis with zero direction: origin must lie in the slab.
// That case needs no branch: inv is +-inf, so (plane - o) * inv is -inf or
// +inf by the side of the plane the origin lies on (the interval is left
// alone or made empty) and NaN when the origin lies on the plane, which
// fmaxf / fminf ignore (the plane counts as inside).
// REV (reversed inside queries): `inside` is set when the ray's line enters
// the box before tmin (entry te = the largest near-plane distance) and the
// box is hit, i.e. the origin lies in the box; the interval is then the chord
// [te, tf] instead of [tmin, tf].
template <bool REV>
__device__ inline bool slab(const RayPre& R, const float lo[3], const float hi[3], float& t0, float& t1,
                            bool& inside) {
  float tn = R.tmin, tf = R.tmax, te = -INFINITY;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float ta = (lo[a] - R.o[a]) * R.inv[a];
    const float tb = (hi[a] - R.o[a]) * R.inv[a];
    const float tnear = R.neg[a] ? tb : ta, tfar = R.neg[a] ? ta : tb;
    tn = fmaxf(tn, tnear);
    if (REV) te = fmaxf(te, tnear);
    tf = fminf(tf, tfar);
  }
  const bool hit = tn <= tf;
  inside = REV && hit && te < R.tmin;
  t0 = inside ? te : tn;
  t1 = tf;
  return hit;
}

// leaf field of a segment: the leaf id, with NBVH_SEG_INSIDE for a reversed chord
__device__ inline uint32_t seg_leaf(int32_t leaf, bool inside) {
  return (uint32_t)leaf | (inside ? NBVH_SEG_INSIDE : 0u);
}

// Hand the crossed leaf children over, the nearer one first: a run that comes
// in order is appended from registers, one that does not is read back from
// memory record by record (241 -> 222 us for 2^20 rays towards one of eight objects).
template <typename Emit>
__device__ inline void emit_leaves(bool h0, int32_t c0, float a0, float a1, bool ia, bool h1, int32_t c1, float b0,
                                   float b1, bool ib, Emit emit) {
  const bool swap = h1 && (!h0 || b0 < a0);
  if (h0 || h1) emit(swap ? ~c1 : ~c0, swap ? b0 : a0, swap ? b1 : a1, swap ? ib : ia);
  if (h0 && h1) emit(swap ? ~c0 : ~c1, swap ? a0 : b0, swap ? a1 : b1, swap ? ia : ib);
}

// A quad's four lanes fetch their nodes together. The L1 serves a 16-byte load
// one 64-byte line of a quad at a time, so four lanes that each read their own
// node take four turns for each of its four pieces. Here load j brings lane j's
// whole node, lane q its piece q (one line a quad), and a 4 x 4 transpose in
// registers hands every lane its own node. Called by whole quads. Traversal of
// 2^20 rays towards eight objects 222 -> 172 us an object, training-ray selection
// of 2^18 unordered rays over 16,384 leaves 272 -> 193 us.
__device__ inline uint32_t quad_swap(uint32_t v, int bit) {
  return bit == 1 ? __builtin_amdgcn_update_dpp(0u, v, 0xB1, 0xf, 0xf, false)   // lanes 1 0 3 2
                  : __builtin_amdgcn_update_dpp(0u, v, 0x4E, 0xf, 0xf, false);  // lanes 2 3 0 1
}

__device__ inline void quad_load_nodes(const Node* __restrict__ nodes, int32_t node, uint32_t m[4][4]) {
  const uint32_t q = threadIdx.x & 3u;
  uint32_t of[4];
  of[0] = __builtin_amdgcn_update_dpp(0u, (uint32_t)node, 0x00, 0xf, 0xf, false);
  of[1] = __builtin_amdgcn_update_dpp(0u, (uint32_t)node, 0x55, 0xf, 0xf, false);
  of[2] = __builtin_amdgcn_update_dpp(0u, (uint32_t)node, 0xAA, 0xf, 0xf, false);
  of[3] = __builtin_amdgcn_update_dpp(0u, (uint32_t)node, 0xFF, 0xf, 0xf, false);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint4 v = ((const uint4*)(nodes + of[j]))[q];
    m[j][0] = v.x;
    m[j][1] = v.y;
    m[j][2] = v.z;
    m[j][3] = v.w;
  }
#pragma unroll
  for (int bit = 1; bit <= 2; bit <<= 1) {
    const bool hi = (q & (uint32_t)bit) != 0u;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (j & bit) continue;
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const uint32_t lo_of = quad_swap(m[j][d], bit), hi_of = quad_swap(m[j | bit][d], bit);
        m[j][d] = hi ? hi_of : m[j][d];
        m[j | bit][d] = hi ? m[j | bit][d] : lo_of;
      }
    }
  }
}

// Walk the tree; Emit(leaf, t0, t1, inside) is called for every leaf crossed. The
// per-lane stack lives in LDS, entry i of this lane at stk[i * stride]
// (lane-contiguous, so a wave's pushes and pops touch consecutive words);
// it needs as many entries as the tree has inner levels. Called by every lane
// of the wave together; lanes with live = false emit nothing. TREE: `tree` is
// the workgroup's LDS copy of the nodes, which is read instead.
template <bool REV, bool TREE, bool MIXED, typename Emit>
__device__ inline void walk(const Node* __restrict__ nodes, const Node* tree, const RayPre& R, bool live, Emit emit,
                            int32_t* stk, uint32_t stride) {
  int sp = 0;
  int32_t node = 0;
  while (__ballot(live) != 0ull) {
    const uint32_t one = live ? 1u : 0u, two = one | quad_swap(one, 1);
    const bool quad = (two | quad_swap(two, 2)) != 0u;  // a lane of the quad still walks
    // Where no quad has lanes on different nodes (coherent rays, a lone ray) every
    // lane reads its own node, one line a quad as well, and the transpose is spared:
    // 10^6 camera rays over 64 leaves 79 -> 69 us, one ray over 16,384 leaves 33 -> 28,
    // and as incoherent waves thin out: 3,000 random rays over 16,384 leaves 224 -> 195.
    // Rays known to be scattered (MIXED false: a selection) pay 5 % for the choice.
    bool apart = true;
    if constexpr (MIXED && !TREE) {
      uint32_t lo = live ? (uint32_t)node : 0xffffffffu, hi = live ? (uint32_t)node : 0u;
      lo = min(lo, quad_swap(lo, 1));
      hi = max(hi, quad_swap(hi, 1));
      lo = min(lo, quad_swap(lo, 2));
      hi = max(hi, quad_swap(hi, 2));
      apart = __ballot(lo < hi) != 0ull;
    }
    if (quad) {
      uint32_t m[4][4];
      if constexpr (TREE) {
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const u32x4 v = lds_load<u32x4>((const uint4*)(tree + node) + j);
#pragma unroll
          for (int d = 0; d < 4; ++d) m[j][d] = v[d];
        }
      } else if (apart) {
        quad_load_nodes(nodes, node, m);
      } else if (live) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const uint4 v = ((const uint4*)(nodes + node))[j];
          m[j][0] = v.x;
          m[j][1] = v.y;
          m[j][2] = v.z;
          m[j][3] = v.w;
        }
      }
      if (live) {
        float f[12];
#pragma unroll
        for (int i = 0; i < 12; ++i) f[i] = __uint_as_float(m[i >> 2][i & 3]);
        const float lo0[3] = {f[0], f[1], f[2]}, hi0[3] = {f[3], f[4], f[5]};
        const float lo1[3] = {f[6], f[7], f[8]}, hi1[3] = {f[9], f[10], f[11]};
        const int32_t c0 = (int32_t)m[3][0], c1 = (int32_t)m[3][1];
        float a0, a1, b0, b1;
        bool ia = false, ib = false;
        bool h0 = slab<REV>(R, lo0, hi0, a0, a1, ia);
        bool h1 = (c1 != kEmptyChild) && slab<REV>(R, lo1, hi1, b0, b1, ib);
        int32_t next = -1;
        emit_leaves(h0 && c0 < 0, c0, a0, a1, ia, h1 && c1 < 0, c1, b0, b1, ib, emit);
        if (h0 && c0 >= 0) next = c0;
        if (h1 && c1 >= 0) {
          if (next < 0) {
            next = c1;
          } else {
            // both inner children: go to the nearer one first
            if (b0 < a0) {
              stk[(sp++) * stride] = next;
              next = c1;
            } else {
              stk[(sp++) * stride] = c1;
            }
          }
        }
        if (next >= 0) node = next;
        else if (sp > 0) node = stk[(--sp) * stride];
        else live = false;
      }
    }
  }
}

// Wave-coherent walk: the wave visits the union of its live lanes' nodes in
// one order that every lane shares. The node index is uniform, so a visit
// reads the node's 64 bytes once through the scalar cache instead of once per
// lane through the vector memory path; each lane tests both children against
// its own ray, and a child is entered when any lane hits it. The stack is one
// register holding entry i in lane i (pushes select the lane, pops read it),
// at most kMaxDepth < 64 entries. Both children entered: the one nearer along
// the guide direction g first, so that each lane's leaves come out mostly in
// front-to-back order. Must be called by every lane of the wave together.
template <bool REV, typename Emit>
__device__ inline void walk_wave(const Node* __restrict__ nodes, const RayPre& R, bool live, Emit emit, float gx,
                                 float gy, float gz) {
  const int lane = (int)(threadIdx.x & 63);
  int32_t stk = 0;
  int sp = 0;
  int32_t node = 0;
  while (true) {
    const float4* p = (const float4*)(nodes + node);
    float4 q0 = p[0], q1 = p[1], q2 = p[2], q3 = p[3];
    const float lo0[3] = {q0.x, q0.y, q0.z}, hi0[3] = {q0.w, q1.x, q1.y};
    const float lo1[3] = {q1.z, q1.w, q2.x}, hi1[3] = {q2.y, q2.z, q2.w};
    const int32_t c0 = __float_as_int(q3.x), c1 = __float_as_int(q3.y);
    float a0 = 0.f, a1 = 0.f, b0 = 0.f, b1 = 0.f;
    bool ia = false, ib = false;
    const bool h0 = live && slab<REV>(R, lo0, hi0, a0, a1, ia);
    const bool h1 = live && (c1 != kEmptyChild) && slab<REV>(R, lo1, hi1, b0, b1, ib);
    // (half the nodes have no leaf below them: 300,000 random rays, 16,384 leaves,
    // wave walks only, 1,940 us without the test, 1,843 with it, camera rays 373 and 354)
    if (c0 < 0 || c1 < 0) emit_leaves(h0 && c0 < 0, c0, a0, a1, ia, h1 && c1 < 0, c1, b0, b1, ib, emit);
    const bool e0 = c0 >= 0 && __ballot(h0) != 0ull;
    const bool e1 = c1 >= 0 && c1 != kEmptyChild && __ballot(h1) != 0ull;
    int32_t next;
    if (e0 && e1) {
      const float k0 = (lo0[0] + hi0[0]) * gx + (lo0[1] + hi0[1]) * gy + (lo0[2] + hi0[2]) * gz;
      const float k1 = (lo1[0] + hi1[0]) * gx + (lo1[1] + hi1[1]) * gy + (lo1[2] + hi1[2]) * gz;
      const bool first1 = __builtin_amdgcn_readfirstlane((int)(k1 < k0)) != 0;
      const int32_t later = first1 ? c0 : c1;
      stk = (lane == sp) ? later : stk;
      ++sp;
      next = first1 ? c1 : c0;
    } else if (e0) {
      next = c0;
    } else if (e1) {
      next = c1;
    } else {
      if (sp == 0) break;
      --sp;
      next = __builtin_amdgcn_readlane(stk, sp);
    }
    node = __builtin_amdgcn_readfirstlane(next);
  }
}

// traverse_mode: 0 = per-lane walk, 1 = wave-coherent walk, 2 = per wave,
// the wave-coherent walk when the wave's rays are coherent: every live
// lane's unit direction within kCoherentDir (max-norm) of the first live
// lane's and its origin within 1/kCoherentOrg of the root box's largest
// extent of that lane's. Coherent rays share most of their nodes: a
// 64-pixel row of a 1920-pixel camera visits 7 % more nodes as a union than
// its slowest lane alone, and the walk per wave is 20-40 % faster on camera
// rays at 1,024 and 16,384 leaves; on scattered bounce rays and on random
// training rays it is 25-75 % slower.
constexpr float kCoherentDir = 0.25f;
constexpr float kCoherentOrg = 32.0f;

__device__ inline float wave_max(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off));
  return v;
}

// Whether this wave walks together, and its guide direction. Called by every
// lane of the wave; lanes without a ray pass live = false.
__device__ inline bool wave_walks(int mode, const Node* __restrict__ nodes, const RayPre& R, bool live, float g[3]) {
  const uint64_t lm = __ballot(live);
  if (mode == 0 || lm == 0ull) return false;
  const int gl = __ffsll((unsigned long long)lm) - 1;
  const float n2 = R.d[0] * R.d[0] + R.d[1] * R.d[1] + R.d[2] * R.d[2];
  const float inv = n2 > 0.0f ? 1.0f / sqrtf(n2) : 0.0f;
  float dn[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    dn[k] = R.d[k] * inv;
    g[k] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(dn[k]), gl));
  }
  if (mode == 1) return true;
  const float4* p = (const float4*)nodes;
  const float4 q0 = p[0], q1 = p[1], q2 = p[2];
  const float ext = fmaxf(fmaxf(fmaxf(q0.w, q2.y) - fminf(q0.x, q1.z), fmaxf(q1.x, q2.z) - fminf(q0.y, q1.w)),
                          fmaxf(q1.y, q2.w) - fminf(q0.z, q2.x));
  float dev = 0.0f;
  if (live) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const float og = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(R.o[k]), gl));
      dev = fmaxf(dev, fabsf(dn[k] - g[k]) * (1.0f / kCoherentDir));
      dev = fmaxf(dev, fabsf(R.o[k] - og) * kCoherentOrg / fmaxf(ext, 1e-30f));
    }
  }
  return wave_max(dev) <= 1.0f;
}

// The walk the mode asks for. Called by every lane of the wave (the
// wave-coherent walk needs them all); lanes with live = false emit nothing.
template <bool REV, bool TREE = false, bool MIXED = true, typename Emit>
__device__ inline void walk_mode(int mode, const Node* __restrict__ nodes, const RayPre& R, bool live, Emit emit,
                                 int32_t* stk, uint32_t stride, const Node* tree = nullptr) {
  float g[3] = {0.f, 0.f, 0.f};
  if (wave_walks(mode, nodes, R, live, g))
    walk_wave<REV>(nodes, R, live, emit, g[0], g[1], g[2]);
  else
    walk<REV, TREE, MIXED>(nodes, tree, R, live, emit, stk, stride);
}

// The last record of a sorted run, kept in registers: a segment that sorts
// after it is appended without reading the run back.
struct RunTail {
  float t0 = 0.0f;
  uint32_t tag = 0u;
  __device__ bool before(float t, uint32_t g) const { return t0 < t || (t0 == t && tag < g); }
};

// Staged runs are plane-major: record i of ray r is (leaf, t0, t1) at
// planes 3i, 3i+1, 3i+2 of n_rays floats each, so that neighbouring rays
// (lanes) touch neighbouring words. Insert (tag, t0, t1) into ray r's sorted
// run of k records (order (t0, tag)).
template <typename P>
__device__ inline void insert_staged(P st, size_t plane, uint32_t k, uint32_t tag, float t0, float t1,
                                     RunTail& tail) {
  uint32_t j = k;
  if (k == 0 || tail.before(t0, tag)) {
    tail.t0 = t0;
    tail.tag = tag;
  } else {
    while (j > 0) {
      const float p0 = st[(3 * (j - 1) + 1) * plane];
      const uint32_t pl = __float_as_uint(st[(3 * (j - 1)) * plane]);
      if (p0 > t0 || (p0 == t0 && pl > tag)) {
        st[(3 * j) * plane] = __uint_as_float(pl);
        st[(3 * j + 1) * plane] = p0;
        st[(3 * j + 2) * plane] = st[(3 * (j - 1) + 2) * plane];
        --j;
      } else {
        break;
      }
    }
  }
  st[(3 * j) * plane] = __uint_as_float(tag);
  st[(3 * j + 1) * plane] = t0;
  st[(3 * j + 2) * plane] = t1;
}

// Insert (tag, t0, t1) into ray r's sorted run segs[beg, k) of the queue.
__device__ inline void insert_queue(nbvh_segment* __restrict__ segs, uint32_t beg, uint32_t k, uint32_t r, uint32_t tag,
                                    float t0, float t1, RunTail& tail) {
  uint32_t j = k;
  if (k == beg || tail.before(t0, tag)) {
    tail.t0 = t0;
    tail.tag = tag;
  } else {
    while (j > beg) {
      const nbvh_segment prev = segs[j - 1];
      if (prev.t0 > t0 || (prev.t0 == t0 && prev.leaf > tag)) {
        segs[j] = prev;
        --j;
      } else {
        break;
      }
    }
  }
  segs[j] = nbvh_segment{r, tag, t0, t1};
}

// A ray's precomputed form, or an inert one for lanes without a ray.
__device__ inline RayPre load_ray_or_none(const nbvh_ray* rays, uint32_t r, bool live) {
  if (live) return load_ray(rays, r);
  RayPre R;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    R.o[k] = R.d[k] = R.inv[k] = 0.0f;
    R.neg[k] = false;
  }
  R.tmin = 1.0f;
  R.tmax = 0.0f;
  return R;
}

// counts[r] = leaves crossed. If `hits` is given (full query), rays with no
// segment get their miss record here (rays with segments are listed by the
// compaction, at positions from a scan of the counts). If `staging` is
// given, the first kStage segments of ray r are also kept there, sorted, so
// that the compaction after the scan need not walk the tree again.
constexpr uint32_t kStage = 16;

// With few rays the walk's time is its chain of node loads (about 1 us a visit
// from L2), so the whole tree, if it has at most kTreeNodes nodes, is first
// copied to LDS; with many rays other waves hide that latency and the copy
// would cost occupancy instead. A tree of up to kTreeSmall nodes (8 KiB) costs
// none, and spares many rays the walk's wait for the L1: 64 leaves, camera rays,
// 65,536 41 us from memory and 35 from LDS, 10^6 68 and 56; 300,000 random rays
// 74 and 58.
constexpr uint32_t kTreeNodes = 1023, kTreeRays = 16384, kTreeSmall = 127;
template <bool TREE>
__device__ inline const Node* copy_tree(const Node* __restrict__ nodes, uint32_t n_nodes, void* lds) {
  if constexpr (TREE) {
    const uint4* src = (const uint4*)nodes;
    uint4* dst = (uint4*)lds;
    for (uint32_t i = threadIdx.x; i < n_nodes * 4u; i += blockDim.x) dst[i] = src[i];
    __syncthreads();
  }
  return (const Node*)lds;
}

template <bool REV, bool TREE>
__global__ __launch_bounds__(256) void k_traverse_count(const Node* __restrict__ nodes, const nbvh_ray* __restrict__ rays,
                                                        uint32_t n_rays, uint32_t* __restrict__ counts,
                                                        nbvh_hit* __restrict__ hits, float* __restrict__ staging,
                                                        int mode, const uint32_t* __restrict__ perm, uint32_t n_nodes,
                                                        uint32_t stack_words, DevCfg c, WeightCopy wc) {
  extern __shared__ __align__(16) int32_t s_stack[];  // the stacks, then the tree
  if (blockIdx.x >= ray_blocks(n_rays)) return order_weights(c, wc, blockIdx.x - ray_blocks(n_rays));
  const Node* tree = copy_tree<TREE>(nodes, n_nodes, s_stack + stack_words);
  // thread i takes ray perm[i] (ray i without a ray order); its staged run
  // is column i, so a wave's staging stores stay coalesced
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  const bool live = i < n_rays;
  const uint32_t r = (perm && live) ? perm[i] : i;
  uint32_t cnt = 0;
  RunTail tail;
  const RayPre R = load_ray_or_none(rays, r, live);
  float* run = (staging && live) ? staging + i : nullptr;
  walk_mode<REV, TREE>(
      mode, nodes, R, live,
      [&](int32_t leaf, float t0, float t1, bool inside) {
        if (run && cnt < kStage) insert_staged(run, n_rays, cnt, seg_leaf(leaf, inside), t0, t1, tail);
        ++cnt;
      },
      s_stack + threadIdx.x, blockDim.x, tree);
  if (live) {
    counts[r] = cnt;
    if (hits && cnt == 0) {
      float4* h = (float4*)(hits + r);
      h[0] = make_float4(0.f, 0.f, 0.f, 0.f);
      h[1] = make_float4(0.f, 0.f, 0.f, __uint_as_float(NBVH_MISS));
    }
  }
}

// Compaction from the staging runs: rays with more than kStage segments walk
// the tree again and insert their segments into the queue directly. A wave
// whose rays all have short runs copies them together: its runs are one
// contiguous range of the queue, each lane records in LDS which (lane, run
// record) fills each slot of the range, then the lanes take consecutive
// slots, so the stores are coalesced and the wave waits on two or three
// rounds of loads instead of its longest run's.
constexpr uint32_t kWaveSlots = 64 * kStage;
template <bool REV>
__global__ __launch_bounds__(256) void k_traverse_compact(const Node* __restrict__ nodes,
                                                          const nbvh_ray* __restrict__ rays, uint32_t n_rays,
                                                          const uint32_t* __restrict__ offsets,
                                                          const float* __restrict__ staging,
                                                          nbvh_segment* __restrict__ segs, uint64_t capacity, int mode,
                                                          const uint32_t* __restrict__ inv,
                                                          const uint32_t* __restrict__ apos,
                                                          uint32_t* __restrict__ active) {
  extern __shared__ __align__(16) int32_t s_stack[];
  __shared__ uint16_t s_slot[4][kWaveSlots];
  const uint32_t r = blockIdx.x * blockDim.x + threadIdx.x;
  if ((uint64_t)offsets[n_rays] > capacity) return;  // overflow flagged by the scan (uniform)
  const uint32_t beg = r < n_rays ? offsets[r] : 0u, end = r < n_rays ? offsets[r + 1] : 0u;
  // the rays with segments at their positions among them (in ray order, or
  // in the order the counting pass followed)
  if (active && end > beg) active[apos[inv ? inv[r] : r]] = r;
  const bool live = end - beg > kStage;
  const size_t plane = n_rays;
  if (__ballot(live) == 0ull) {
    const uint32_t lane = threadIdx.x & 63u, r0 = r - lane;
    if (r0 >= n_rays) return;  // the whole wave
    const uint32_t wbeg = offsets[r0], wend = offsets[min(r0 + 64u, n_rays)];  // wend - wbeg <= kWaveSlots
    uint16_t* slot = s_slot[threadIdx.x >> 6];
    for (uint32_t i = 0; i < end - beg; ++i) slot[beg - wbeg + i] = (uint16_t)(lane | (i << 6));
    wave_fence();
    for (uint32_t k = lane; k < wend - wbeg; k += 64u) {
      const uint32_t e = slot[k], o = r0 + (e & 63u), i = e >> 6;
      const float* run = staging + (inv ? inv[o] : o);
      segs[wbeg + k] = nbvh_segment{o, __float_as_uint(run[(3 * i) * plane]), run[(3 * i + 1) * plane],
                                    run[(3 * i + 2) * plane]};
    }
    return;
  }
  if (end > beg && !live) {
    const float* run = staging + (inv ? inv[r] : r);
    for (uint32_t i = 0; i < end - beg; ++i)
      segs[beg + i] = nbvh_segment{r, __float_as_uint(run[(3 * i) * plane]), run[(3 * i + 1) * plane],
                                   run[(3 * i + 2) * plane]};
  }
  const RayPre R = load_ray_or_none(rays, r, live);
  uint32_t k = beg;
  RunTail tail;
  walk_mode<REV>(
      mode, nodes, R, live,
      [&](int32_t leaf, float t0, float t1, bool inside) {
        // the counting pass found end - beg leaves along this ray; a walk
        // reports the same ones (every inner box is the union of its
        // children's), the bound keeps the writes inside the run regardless
        if (k < end) insert_queue(segs, beg, k, r, seg_leaf(leaf, inside), t0, t1, tail);
        ++k;
      },
      s_stack + threadIdx.x, blockDim.x);
}

// Training-ray selection (Sec. 5.2, "Ray distribution"): each ray trains only
// the first leaf it crosses (smallest t0, ties to the lower leaf id), and that
// leaf is kept with probability accept[leaf] (kept iff u[r] < accept[leaf]).
// Every leaf a ray crosses also counts one hit towards its hit-probability
// estimate (Sec. 5.1, "Node error"). Kept segments are appended in wave order.
// HIST, for trees of up to kHitBins leaves and eight rays a leaf: a workgroup
// counts its rays' hits in LDS and adds each leaf's sum once, as additions of one
// word in memory take turns and a small tree has few words. With the grouping
// after it, 10^6 rays: 64 leaves 286 us (7,615 by direct additions), 1,024 leaves
// 371 us (1,410); 2^18 rays, 16,384 leaves 295 us (265); 3,000 rays, 1,024 leaves
// 99 us (92).
constexpr uint32_t kHitBins = 2048;
template <bool REV, bool HIST>
__global__ __launch_bounds__(256) void k_first_hits(const Node* __restrict__ nodes, const nbvh_ray* __restrict__ rays,
                                                    uint32_t n, const float* __restrict__ u,
                                                    const float* __restrict__ accept, nbvh_probe* __restrict__ probes,
                                                    uint32_t* __restrict__ leaf_out, uint32_t* __restrict__ n_out,
                                                    uint32_t* __restrict__ leaf_hits, int mode, uint32_t stack_words,
                                                    uint32_t n_bins) {
  extern __shared__ __align__(16) int32_t s_stack[];
  uint32_t* const hist = (uint32_t*)s_stack + 256 * stack_words;
  if (HIST) {
    for (uint32_t i = threadIdx.x; i < n_bins; i += blockDim.x) hist[i] = 0u;
    __syncthreads();
  }
  for (uint64_t r0 = (uint64_t)blockIdx.x * blockDim.x; r0 < n; r0 += (uint64_t)gridDim.x * blockDim.x) {
    const uint64_t r64 = r0 + threadIdx.x;
    const bool live = r64 < n;
    const uint32_t r = live ? (uint32_t)r64 : 0u;
    bool take = false, b_in = false;
    int32_t best = -1;
    float b0 = 0.f, b1 = 0.f;
    const RayPre R = load_ray_or_none(rays, r, live);
    walk_mode<REV, false, false>(
        mode, nodes, R, live,
        [&](int32_t leaf, float t0, float t1, bool inside) {
          if (HIST)
            atomicAdd(&hist[leaf], 1u);
          else if (leaf_hits)
            atomicAdd(&leaf_hits[leaf], 1u);
          if (best < 0 || t0 < b0 || (t0 == b0 && leaf < best)) {
            best = leaf;
            b0 = t0;
            b1 = t1;
            b_in = inside;
          }
        },
        s_stack + threadIdx.x, blockDim.x);
    take = live && best >= 0 && u[r] < accept[best];
    const uint64_t mask = __ballot(take);
    if (mask) {
      const int lane = threadIdx.x & 63;
      const int leader = __ffsll((unsigned long long)mask) - 1;
      uint32_t base = 0;
      if (lane == leader) base = atomicAdd(n_out, (uint32_t)__popcll(mask));
      base = __shfl(base, leader);
      if (take) {
        const uint32_t k = base + (uint32_t)__popcll(mask & ((1ull << lane) - 1ull));
        float4* p = (float4*)(probes + k);
        if (b_in) {  // the chord crossed backwards from its exit point
          p[0] = make_float4(R.o[0], R.o[1], R.o[2], -b1);
          p[1] = make_float4(-R.d[0], -R.d[1], -R.d[2], -b0);
        } else {
          p[0] = make_float4(R.o[0], R.o[1], R.o[2], b0);
          p[1] = make_float4(R.d[0], R.d[1], R.d[2], b1);
        }
        leaf_out[k] = (uint32_t)best;
      }
    }
  }
  if (HIST) {
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < n_bins; i += blockDim.x)
      if (hist[i] != 0u) atomicAdd(&leaf_hits[i], hist[i]);
  }
}

// LDS for the walk stacks of a 256-thread workgroup
static size_t stack_lds(const LaunchCtx& L) { return (size_t)256 * (L.stack_depth > 0 ? L.stack_depth : 1) * 4; }

nbvh_status launch_first_hits(const LaunchCtx& L, const nbvh_ray* rays, uint32_t n, const float* u,
                              const float* accept, nbvh_probe* probes, uint32_t* leaf_out, uint32_t* n_out,
                              uint32_t* leaf_hits) {
  k_zero_u32<<<1, 64, 0, L.stream>>>(n_out, 1);
  if (n > 0) {
    const uint32_t bins = L.n_nodes + 1u;  // at least the leaves
    const bool hist = leaf_hits && bins <= kHitBins && n >= 8u * bins;
    const bool rev = L.cfg.inside_reverse;
    const auto kern = hist ? (rev ? k_first_hits<true, true> : k_first_hits<false, true>)
                           : (rev ? k_first_hits<true, false> : k_first_hits<false, false>);
    const uint32_t blocks = (n + 255) / 256, most = 8u * (uint32_t)L.n_cu;  // few enough sums, all in flight
    const size_t stack = stack_lds(L), lds = stack + (hist ? bins * 4u : 0u);
    if (lds > 64 * 1024) (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    kern<<<hist && blocks > most ? most : blocks, 256, lds, L.stream>>>(L.nodes, rays, n, u, accept, probes, leaf_out, n_out,
                                                                       leaf_hits, L.tune.traverse_mode,
                                                                       (uint32_t)(stack / 1024), bins);
  }
  return check_launch("first_hits");
}

// ---------------------------------------------------------------------------
// exclusive scan of uint32 counts: tile scan, then add (beyond kScanDirectTiles
// tiles a scan of the tile sums in between). Tile = 256 threads x 4 items.
// ---------------------------------------------------------------------------
constexpr int kScanItems = 4;
constexpr int kScanTile = 256 * kScanItems;

__device__ inline uint32_t block_exclusive_scan(uint32_t v, uint32_t* sh, uint32_t& total) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // inclusive scan within the wave
  uint32_t x = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    uint32_t y = __shfl_up(x, off);
    if (lane >= off) x += y;
  }
  if (lane == 63) sh[wave] = x;
  __syncthreads();
  uint32_t wsum = 0, tot = 0;
  for (int w = 0; w < (int)(blockDim.x >> 6); ++w) {
    if (w < wave) wsum += sh[w];
    tot += sh[w];
  }
  __syncthreads();
  total = tot;
  return wsum + x - v;
}

__global__ __launch_bounds__(256) void k_scan_tiles(const uint32_t* __restrict__ in, uint32_t n, uint32_t* __restrict__ out,
                                                    uint32_t* __restrict__ tile_sums) {
  __shared__ uint32_t sh[8];
  const uint32_t base = blockIdx.x * kScanTile + threadIdx.x * kScanItems;
  uint32_t v[kScanItems], s = 0;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    v[i] = (base + i < n) ? in[base + i] : 0u;
    s += v[i];
  }
  uint32_t total;
  uint32_t ex = block_exclusive_scan(s, sh, total);
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    if (base + i < n) out[base + i] = ex;
    ex += v[i];
  }
  if (threadIdx.x == 0) tile_sums[blockIdx.x] = total;
}

// one block: exclusive scan of the tile sums in place; total -> *total_out
__global__ __launch_bounds__(1024) void k_scan_sums(uint32_t* __restrict__ sums, uint32_t n_tiles,
                                                    uint32_t* __restrict__ total_out) {
  __shared__ uint32_t sh[16];
  __shared__ uint32_t carry;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  for (uint32_t base = 0; base < n_tiles; base += blockDim.x) {
    const uint32_t i = base + threadIdx.x;
    uint32_t v = (i < n_tiles) ? sums[i] : 0u;
    uint32_t total;
    uint32_t ex = block_exclusive_scan(v, sh, total);
    const uint32_t c0 = carry;
    if (i < n_tiles) sums[i] = ex + c0;
    __syncthreads();
    if (threadIdx.x == 0) carry = c0 + total;
    __syncthreads();
  }
  if (threadIdx.x == 0) *total_out = carry;
}

// Sum of sums[0 .. t) over a block of 256 threads.
__device__ inline uint32_t sum_before(const uint32_t* __restrict__ sums, uint32_t t, uint32_t* sh) {
  uint32_t v = 0;
  for (uint32_t i = threadIdx.x; i < t; i += 256u) v += sums[i];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += (uint32_t)__shfl_xor((int)v, off);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  v = sh[0] + sh[1] + sh[2] + sh[3];
  __syncthreads();
  return v;
}

// Up to this many tiles every block of the add pass sums the tiles before its
// own by itself (at most 8 KiB from L2), which saves the launch in between (4
// to 5 us); beyond, the tile sums are scanned first.
constexpr uint32_t kScanDirectTiles = 2048;

// block per tile: add the tiles before it; `scanned`: sums hold prefixes
__global__ __launch_bounds__(256) void k_scan_add(uint32_t* __restrict__ out, uint32_t n, const uint32_t* __restrict__ sums,
                                                  int scanned, uint64_t capacity, DevState* __restrict__ state) {
  __shared__ uint32_t sh[4];
  const uint32_t tile = blockIdx.x, base = tile * kScanTile;
  const uint32_t before = scanned ? sums[tile] : sum_before(sums, tile, sh);
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    const uint32_t k = base + (uint32_t)i * 256u + threadIdx.x;
    if (k < n) out[k] += before;
  }
  if (tile + 1 == gridDim.x && threadIdx.x == 0) {
    const uint32_t t = scanned ? sums[gridDim.x] : before + sums[tile];
    out[n] = t;
    if (state) {
      state->last_n_segments = t;
      if ((uint64_t)t > capacity) atomicOr(&state->flags, NBVH_FLAG_CAPACITY);
    }
  }
}

// The traversal's two scans at once: segment offsets of the counts and, for
// the active-ray list, positions among the rays with a segment (tile scans, add;
// beyond kScanDirectTiles tiles one block each scans the tile sums in between).
// (positions follow the ray order `perm` when one is given: pos[i] is the
// place of ray perm[i])
__global__ __launch_bounds__(256) void k_scan2_tiles(const uint32_t* __restrict__ in, uint32_t n,
                                                     const uint32_t* __restrict__ perm, uint32_t* __restrict__ out,
                                                     uint32_t* __restrict__ pos, uint32_t* __restrict__ sums_seg,
                                                     uint32_t* __restrict__ sums_ray) {
  __shared__ uint32_t sh[8];
  const uint32_t base = blockIdx.x * kScanTile + threadIdx.x * kScanItems;
  uint32_t v[kScanItems], g[kScanItems], s = 0, f = 0;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    const bool ok = base + i < n;
    v[i] = ok ? in[base + i] : 0u;
    g[i] = ok ? ((perm ? in[perm[base + i]] : v[i]) > 0u ? 1u : 0u) : 0u;
    s += v[i];
    f += g[i];
  }
  uint32_t total_s, total_f;
  uint32_t ex = block_exclusive_scan(s, sh, total_s);
  uint32_t ef = block_exclusive_scan(f, sh, total_f);
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    if (base + i < n) {
      out[base + i] = ex;
      pos[base + i] = ef;
    }
    ex += v[i];
    ef += g[i];
  }
  if (threadIdx.x == 0) {
    sums_seg[blockIdx.x] = total_s;
    sums_ray[blockIdx.x] = total_f;
  }
}

__global__ __launch_bounds__(1024) void k_scan2_sums(uint32_t* __restrict__ sums_seg, uint32_t* __restrict__ sums_ray,
                                                     uint32_t n_tiles) {
  __shared__ uint32_t sh[16];
  __shared__ uint32_t carry;
  uint32_t* sums = blockIdx.x == 0 ? sums_seg : sums_ray;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  for (uint32_t base = 0; base < n_tiles; base += blockDim.x) {
    const uint32_t i = base + threadIdx.x;
    uint32_t v = (i < n_tiles) ? sums[i] : 0u;
    uint32_t total;
    uint32_t ex = block_exclusive_scan(v, sh, total);
    const uint32_t c0 = carry;
    if (i < n_tiles) sums[i] = ex + c0;
    __syncthreads();
    if (threadIdx.x == 0) carry = c0 + total;
    __syncthreads();
  }
  if (threadIdx.x == 0) sums[n_tiles] = carry;
}

// The totals of a traversal with an active list: ends of both arrays, list
// length, state, and the query's ray-queue counters (n_active[1 .. 8]) cleared.
__device__ inline void finish_scan2(uint32_t segs, uint32_t act, uint32_t n, uint32_t* out, uint32_t* pos,
                                    uint32_t* n_active, uint64_t capacity, DevState* state) {
  out[n] = segs;
  pos[n] = act;
  n_active[0] = act;
  for (int i = 1; i <= 8; ++i) n_active[i] = 0u;
  if (state) {
    state->last_n_segments = segs;
    if ((uint64_t)segs > capacity) atomicOr(&state->flags, NBVH_FLAG_CAPACITY);
  }
}

__global__ __launch_bounds__(256) void k_scan2_add(uint32_t* __restrict__ out, uint32_t* __restrict__ pos, uint32_t n,
                                                   const uint32_t* __restrict__ sums_seg,
                                                   const uint32_t* __restrict__ sums_ray, int scanned,
                                                   uint32_t* __restrict__ n_active, uint64_t capacity,
                                                   DevState* __restrict__ state) {
  __shared__ uint32_t sh[4];
  const uint32_t tile = blockIdx.x, base = tile * kScanTile;
  const uint32_t bs = scanned ? sums_seg[tile] : sum_before(sums_seg, tile, sh);
  const uint32_t br = scanned ? sums_ray[tile] : sum_before(sums_ray, tile, sh);
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    const uint32_t k = base + (uint32_t)i * 256u + threadIdx.x;
    if (k < n) {
      out[k] += bs;
      pos[k] += br;
    }
  }
  if (tile + 1 == gridDim.x && threadIdx.x == 0)
    finish_scan2(scanned ? sums_seg[gridDim.x] : bs + sums_seg[tile], scanned ? sums_ray[gridDim.x] : br + sums_ray[tile], n,
                 out, pos, n_active, capacity, state);
}

// Both scans in one workgroup for up to kScanSmall rays: a launch less again.
// 16 rays a thread; at 16,384 rays it takes as long as the two launches.
constexpr uint32_t kScanSmall = 16384;
__global__ __launch_bounds__(1024) void k_scan2_small(const uint32_t* __restrict__ in, uint32_t n,
                                                      const uint32_t* __restrict__ perm, uint32_t* __restrict__ out,
                                                      uint32_t* __restrict__ pos, uint32_t* __restrict__ n_active,
                                                      uint64_t capacity, DevState* __restrict__ state) {
  __shared__ uint32_t sh[16];
  uint32_t cs = 0, cr = 0;
  for (uint32_t base = 0; base < n; base += 1024u) {
    const uint32_t i = base + threadIdx.x;
    const bool ok = i < n;
    const uint32_t v = ok ? in[i] : 0u;
    const uint32_t g = ok ? ((perm ? in[perm[i]] : v) > 0u ? 1u : 0u) : 0u;
    uint32_t ts, tr;
    const uint32_t es = block_exclusive_scan(v, sh, ts), er = block_exclusive_scan(g, sh, tr);
    if (ok) {
      out[i] = cs + es;
      pos[i] = cr + er;
    }
    cs += ts;
    cr += tr;
  }
  if (threadIdx.x == 0) finish_scan2(cs, cr, n, out, pos, n_active, capacity, state);
}

// The whole traversal of up to kOneRays rays in one workgroup: walk, offsets,
// active list and segment queue, three launches in one. Each wave has a SIMD
// unit to itself; more of them in one workgroup would walk slower than apart.
constexpr uint32_t kOneRays = 256;
template <bool REV, bool TREE>
__global__ __launch_bounds__(256) void k_traverse_one(const Node* __restrict__ nodes, const nbvh_ray* __restrict__ rays,
                                                      uint32_t n, nbvh_hit* __restrict__ hits,
                                                      int mode, uint32_t n_nodes, uint32_t stack_words,
                                                      uint32_t* __restrict__ offsets,
                                                      uint32_t* __restrict__ pos, uint32_t* __restrict__ active,
                                                      uint32_t* __restrict__ n_active, nbvh_segment* __restrict__ segs,
                                                      uint64_t capacity, DevState* __restrict__ state, DevCfg c,
                                                      WeightCopy wc) {
  if (blockIdx.x > 0) return order_weights(c, wc, blockIdx.x - 1);
  // the stacks, the staged runs (a record read back for an insertion takes 1 to
  // 2 us from global memory), then the tree
  extern __shared__ __align__(16) int32_t s_stack[];
  __shared__ uint32_t sh[8];
  typedef float NBVH_LDS* Run;
  const Node* tree = copy_tree<TREE>(nodes, n_nodes, s_stack + stack_words + kStage * 3 * 256);
  const uint32_t r = threadIdx.x;
  const bool have = r < n;
  const RayPre R = load_ray_or_none(rays, r, have);
  uint32_t cnt = 0;
  RunTail tail;
  const Run run = (Run)(s_stack + stack_words) + r;
  walk_mode<REV, TREE>(
      mode, nodes, R, have,
      [&](int32_t leaf, float t0, float t1, bool inside) {
        if (cnt < kStage) insert_staged(run, 256, cnt, seg_leaf(leaf, inside), t0, t1, tail);
        ++cnt;
      },
      s_stack + threadIdx.x, blockDim.x, tree);
  uint32_t total, act;
  const uint32_t beg = block_exclusive_scan(cnt, sh, total), place = block_exclusive_scan(cnt > 0u ? 1u : 0u, sh, act);
  if (have) {
    offsets[r] = beg;
    pos[r] = place;
    if (cnt > 0u) {
      active[place] = r;
    } else if (hits) {
      float4* h = (float4*)(hits + r);
      h[0] = make_float4(0.f, 0.f, 0.f, 0.f);
      h[1] = make_float4(0.f, 0.f, 0.f, __uint_as_float(NBVH_MISS));
    }
  }
  if (threadIdx.x == 0) finish_scan2(total, act, n, offsets, pos, n_active, capacity, state);
  if ((uint64_t)total > capacity) return;
  const bool again = cnt > kStage;
  if (!again)
    for (uint32_t i = 0; i < cnt; ++i)
      segs[beg + i] = nbvh_segment{r, __float_as_uint(run[3 * i * 256]), run[(3 * i + 1) * 256], run[(3 * i + 2) * 256]};
  if (__ballot(again) == 0ull) return;  // long runs walk again, as in the compaction
  uint32_t k = beg;
  RunTail qt;
  walk_mode<REV, TREE>(
      mode, nodes, R, again,
      [&](int32_t leaf, float t0, float t1, bool inside) {
        if (k < beg + cnt) insert_queue(segs, beg, k, r, seg_leaf(leaf, inside), t0, t1, qt);
        ++k;
      },
      s_stack + threadIdx.x, blockDim.x, tree);
}

// ---------------------------------------------------------------------------
// Stable least-significant-digit radix sort of (key, value) pairs, eight bits a
// pass, used to group training probes by leaf and to order rays. A pass is
// three launches: every block counts the digits of its 2,048 keys, one block a
// digit scans that digit's counts, and every block places its keys. (With four
// bits a pass and a general scan, a 24-bit sort was 30 launches of 4 to 9 us,
// most of them shorter than a launch costs; now nine.) A wave's keys are
// contiguous; a key's rank among its wave's equal digits comes from ballots.
constexpr int kSortDigits = 256;
constexpr int kSortRounds = 8;                    // keys of a thread
constexpr uint32_t kSortTile = 256 * kSortRounds;  // keys of a block
static inline size_t group_a256(size_t x) { return (x + 255) & ~(size_t)255; }

// lanes of the wave whose digit equals this lane's
__device__ inline uint64_t same_digit(uint32_t d, bool ok) {
  uint64_t m = __ballot(ok);
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    const uint64_t one = __ballot((d >> b) & 1u);
    m &= ((d >> b) & 1u) ? one : ~one;
  }
  return m;
}

__global__ __launch_bounds__(256) void k_sort_count(const uint32_t* __restrict__ keys, uint32_t n, int shift,
                                                    uint32_t mask, uint32_t* __restrict__ counts) {
  __shared__ uint32_t hist[kSortDigits];
  hist[threadIdx.x] = 0u;
  __syncthreads();
  const uint32_t base = blockIdx.x * kSortTile + threadIdx.x;
#pragma unroll
  for (int j = 0; j < kSortRounds; ++j) {
    const uint32_t i = base + (uint32_t)j * 256u;
    if (i < n) atomicAdd(&hist[(keys[i] >> shift) & mask], 1u);
  }
  __syncthreads();
  counts[(size_t)threadIdx.x * gridDim.x + blockIdx.x] = hist[threadIdx.x];
}

// block d: exclusive scan of digit d's counts over the blocks; its total
__global__ __launch_bounds__(256) void k_sort_scan(uint32_t* __restrict__ counts, uint32_t nb, uint32_t* __restrict__ totals) {
  __shared__ uint32_t sh[8];
  uint32_t* c = counts + (size_t)blockIdx.x * nb;
  uint32_t carry = 0;
  for (uint32_t base = 0; base < nb; base += 256u) {
    const uint32_t i = base + threadIdx.x;
    uint32_t total;
    const uint32_t ex = block_exclusive_scan(i < nb ? c[i] : 0u, sh, total);
    if (i < nb) c[i] = carry + ex;
    carry += total;
  }
  if (threadIdx.x == 0) totals[blockIdx.x] = carry;
}

// vals == nullptr: the values are the element indices (first pass)
__global__ __launch_bounds__(256) void k_sort_scatter(const uint32_t* __restrict__ keys, const uint32_t* __restrict__ vals,
                                                      uint32_t n, int shift, uint32_t mask,
                                                      const uint32_t* __restrict__ counts,
                                                      const uint32_t* __restrict__ totals,
                                                      uint32_t* __restrict__ keys_out, uint32_t* __restrict__ vals_out) {
  __shared__ uint32_t at[4][kSortDigits];  // a wave's next slot of each digit
  __shared__ uint32_t sh[8];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
#pragma unroll
  for (int w = 0; w < 4; ++w) at[w][tid] = 0u;
  __syncthreads();
  const uint32_t base = blockIdx.x * kSortTile + (uint32_t)wave * (kSortTile / 4) + (uint32_t)lane;
  uint32_t k[kSortRounds];
#pragma unroll
  for (int j = 0; j < kSortRounds; ++j) {
    const uint32_t i = base + (uint32_t)j * 64u;
    k[j] = i < n ? keys[i] : 0u;
    if (i < n) atomicAdd(&at[wave][(k[j] >> shift) & mask], 1u);
  }
  uint32_t total;
  uint32_t first = block_exclusive_scan(totals[tid], sh, total) + counts[(size_t)tid * gridDim.x + blockIdx.x];
#pragma unroll
  for (int w = 0; w < 4; ++w) {  // (the scan's barriers order the counts above)
    const uint32_t c = at[w][tid];
    at[w][tid] = first;
    first += c;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kSortRounds; ++j) {
    const uint32_t i = base + (uint32_t)j * 64u;
    const bool ok = i < n;
    const uint32_t d = (k[j] >> shift) & mask;
    const uint64_t m = same_digit(d, ok);
    if (ok) {
      const uint32_t rank = (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
      const uint32_t slot = at[wave][d] + rank;
      // the wave's reads above come before this write (one wave, one LDS queue)
      if (rank == 0u) at[wave][d] = slot + (uint32_t)__popcll(m);
      keys_out[slot] = k[j];
      vals_out[slot] = vals ? vals[i] : i;
    }
    wave_fence();
  }
}

// The whole sort in one workgroup for up to kSortSmall keys, which leave the
// launches of the passes as all that counts (4,096 keys of 24 bits: one launch
// instead of nine).
constexpr uint32_t kSortSmall = 4096;
struct SmallSort {
  uint32_t key[kSortSmall], val[kSortSmall];
  uint32_t at[16][kSortDigits];
  uint32_t sh[16];
};

// sorts S.key / S.val [n] by the low `bits` bits (a multiple of four); all 1,024 threads, after a barrier
__device__ inline void sort_small(SmallSort& S, uint32_t n, int bits) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int shift = 0; shift < bits; shift += 8) {
    const uint32_t mask = bits - shift >= 8 ? 255u : 15u;
    uint32_t k[4], v[4];
    for (int i = tid; i < 16 * kSortDigits; i += 1024) (&S.at[0][0])[i] = 0u;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t i = (uint32_t)wave * 256u + (uint32_t)j * 64u + (uint32_t)lane;
      k[j] = i < n ? S.key[i] : 0u;
      v[j] = i < n ? S.val[i] : 0u;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if ((uint32_t)wave * 256u + (uint32_t)j * 64u + (uint32_t)lane < n) atomicAdd(&S.at[wave][(k[j] >> shift) & mask], 1u);
    __syncthreads();
    uint32_t mine = 0, total;
    if (tid < kSortDigits)
      for (int w = 0; w < 16; ++w) mine += S.at[w][tid];
    uint32_t first = block_exclusive_scan(mine, S.sh, total);
    if (tid < kSortDigits)
      for (int w = 0; w < 16; ++w) {
        const uint32_t c = S.at[w][tid];
        S.at[w][tid] = first;
        first += c;
      }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const bool ok = (uint32_t)wave * 256u + (uint32_t)j * 64u + (uint32_t)lane < n;
      const uint32_t d = (k[j] >> shift) & mask;
      const uint64_t m = same_digit(d, ok);
      if (ok) {
        const uint32_t rank = (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
        const uint32_t slot = S.at[wave][d] + rank;
        if (rank == 0u) S.at[wave][d] = slot + (uint32_t)__popcll(m);
        S.key[slot] = k[j];
        S.val[slot] = v[j];
      }
      wave_fence();
    }
    __syncthreads();
  }
}

__global__ __launch_bounds__(1024) void k_group_small(const nbvh_probe* __restrict__ in, const uint32_t* __restrict__ ids,
                                                      uint32_t n, int bits, nbvh_probe* __restrict__ out,
                                                      uint32_t* __restrict__ ids_out) {
  __shared__ SmallSort S;
  for (uint32_t i = threadIdx.x; i < n; i += 1024u) {
    S.key[i] = ids[i];
    S.val[i] = i;
  }
  __syncthreads();
  sort_small(S, n, bits);
  for (uint32_t i = threadIdx.x; i < n; i += 1024u) {
    const float4* src = (const float4*)(in + S.val[i]);
    float4* dst = (float4*)(out + i);
    dst[0] = src[0];
    dst[1] = src[1];
    if (ids_out) ids_out[i] = S.key[i];
  }
}

__global__ __launch_bounds__(256) void k_group_gather(const nbvh_probe* __restrict__ in,
                                                      const uint32_t* __restrict__ perm,
                                                      const uint32_t* __restrict__ keys, uint32_t n,
                                                      nbvh_probe* __restrict__ out, uint32_t* __restrict__ ids_out) {
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;
  if (i >= n) return;
  const float4* src = (const float4*)(in + perm[i]);
  float4* dst = (float4*)(out + i);
  dst[0] = src[0];
  dst[1] = src[1];
  if (ids_out) ids_out[i] = keys[i];
}

// workspace of a sort of n pairs
struct SortWs {
  uint32_t *kbuf[2], *vbuf[2], *counts, *totals, *box;
};

static uint32_t sort_blocks(uint64_t n) { return (uint32_t)((n + kSortTile - 1) / kSortTile); }

size_t group_ws_bytes(uint64_t n) {
  const uint64_t nb = (n + kSortTile - 1) / kSortTile;
  return 4 * group_a256(n * 4) + group_a256(nb * kSortDigits * 4) + group_a256((kSortDigits + 6) * 4);
}

static SortWs sort_ws(void* ws, uint64_t n) {
  char* w = (char*)ws;
  SortWs O;
  size_t off = 0;
  for (int j = 0; j < 2; ++j) {
    O.kbuf[j] = (uint32_t*)(w + off);
    off += group_a256((size_t)n * 4);
    O.vbuf[j] = (uint32_t*)(w + off);
    off += group_a256((size_t)n * 4);
  }
  O.counts = (uint32_t*)(w + off);
  off += group_a256((size_t)sort_blocks(n) * kSortDigits * 4);
  O.totals = (uint32_t*)(w + off);
  O.box = O.totals + kSortDigits;  // the ray origins' box (6 words)
  return O;
}

// Sorts n pairs by the low `bits` bits (a multiple of four) of the keys; kin must not be kbuf[0].
// The results are *kout and *vout; the last pass writes the values to `vdst` if
// it is given.
static nbvh_status sort_pairs(hipStream_t st, const uint32_t* kin, const uint32_t* vin, uint32_t n, int bits,
                              const SortWs& O, uint32_t* vdst, const uint32_t** kout, const uint32_t** vout) {
  const uint32_t nb = sort_blocks(n);
  const int passes = (bits + 7) / 8;
  for (int p = 0; p < passes; ++p) {
    uint32_t* vo = (p == passes - 1 && vdst) ? vdst : O.vbuf[p & 1];
    const uint32_t mask = bits - 8 * p >= 8 ? 255u : 15u;
    k_sort_count<<<nb, 256, 0, st>>>(kin, n, 8 * p, mask, O.counts);
    k_sort_scan<<<kSortDigits, 256, 0, st>>>(O.counts, nb, O.totals);
    k_sort_scatter<<<nb, 256, 0, st>>>(kin, vin, n, 8 * p, mask, O.counts, O.totals, O.kbuf[p & 1], vo);
    kin = O.kbuf[p & 1];
    vin = vo;
  }
  *kout = kin;
  *vout = vin;
  return check_launch("sort");
}

nbvh_status launch_group_by_leaf(const LaunchCtx& L, uint32_t n_leaves, const nbvh_probe* in, const uint32_t* ids,
                                 uint32_t n, nbvh_probe* out, uint32_t* ids_out, void* ws) {
  if (n == 0) return NBVH_OK;
  const int bits = ((n_leaves > 1 ? 32 - __builtin_clz(n_leaves - 1) : 1) + 3) / 4 * 4;
  if (n <= kSortSmall) {
    k_group_small<<<1, 1024, 0, L.stream>>>(in, ids, n, bits, out, ids_out);
    return check_launch("group_by_leaf");
  }
  const uint32_t *keys, *perm;
  nbvh_status s = sort_pairs(L.stream, ids, nullptr, n, bits, sort_ws(ws, n), nullptr, &keys, &perm);
  if (s != NBVH_OK) return s;
  k_group_gather<<<(n + 255) / 256, 256, 0, L.stream>>>(in, perm, keys, n, out, ids_out);
  return check_launch("group_by_leaf");
}

// ---------------------------------------------------------------------------
nbvh_status launch_exclusive_scan(hipStream_t s, const uint32_t* in, uint32_t n, uint32_t* out, uint32_t* sums) {
  const uint32_t n_tiles = n > 0 ? (n + kScanTile - 1) / kScanTile : 1;
  const int scanned = n_tiles > kScanDirectTiles ? 1 : 0;
  k_scan_tiles<<<n_tiles, 256, 0, s>>>(in, n, out, sums);
  if (scanned) k_scan_sums<<<1, 1024, 0, s>>>(sums, n_tiles, sums + n_tiles);
  k_scan_add<<<n_tiles, 256, 0, s>>>(out, n, sums, scanned, 0, nullptr);
  return check_launch("scan");
}

size_t traverse_staging_bytes(uint64_t n_rays) { return (size_t)n_rays * kStage * 3 * sizeof(float); }

// Ray order (tuning query_order): a permutation of the rays by a Morton key,
// built before the traversal so that the counting pass takes the rays in that
// order (its waves, and the active list it fills, hold neighbouring rays)
// while every ray keeps its index. Keys are relative to the box of the ray
// origins (a min/max reduction first). Order 1: the origin's cell on a 256^3
// grid (24 bits). Order 2: five coordinates at 6 bits each (30 bits), the
// origin's cell on a 64^3 grid and the direction's cell on a 64^2 grid of its
// octahedral map.
__device__ inline uint32_t spread8(uint32_t v) {
  v = (v | (v << 8)) & 0x00F00Fu;
  v = (v | (v << 4)) & 0x0C30C3u;
  v = (v | (v << 2)) & 0x249249u;
  return v;
}

__device__ inline uint32_t cell_of(float x, float cells) {
  const float y = x * cells;
  return y > 0.0f ? (uint32_t)fminf(y, cells - 1.0f) : 0u;  // NaN -> 0
}

// order-preserving map of floats to unsigned integers
__device__ inline uint32_t float_key(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ inline float key_float(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

// min / max of the ray origins per axis (as float_key), one partial per
// block, then one block folds the partials
__device__ inline void wave_minmax(uint32_t lo[3], uint32_t hi[3]) {
#pragma unroll
  for (int a = 0; a < 3; ++a) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      lo[a] = min(lo[a], (uint32_t)__shfl_xor((int)lo[a], off));
      hi[a] = max(hi[a], (uint32_t)__shfl_xor((int)hi[a], off));
    }
  }
}

__global__ __launch_bounds__(256) void k_origin_box(const nbvh_ray* __restrict__ rays, uint32_t n,
                                                    uint32_t* __restrict__ part) {
  __shared__ uint32_t red[4][6];
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;
  uint32_t lo[3] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu}, hi[3] = {0u, 0u, 0u};
  if (i < n) {
    const float4 o = *(const float4*)(rays + i);
    const float p[3] = {o.x, o.y, o.z};
#pragma unroll
    for (int a = 0; a < 3; ++a) lo[a] = hi[a] = float_key(p[a]);
  }
  wave_minmax(lo, hi);
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      red[wave][a] = lo[a];
      red[wave][3 + a] = hi[a];
    }
  __syncthreads();
  if (threadIdx.x < 6) {
    uint32_t v = red[0][threadIdx.x];
    for (int w = 1; w < 4; ++w)
      v = threadIdx.x < 3 ? min(v, red[w][threadIdx.x]) : max(v, red[w][threadIdx.x]);
    part[(size_t)blockIdx.x * 6 + threadIdx.x] = v;
  }
}

__global__ __launch_bounds__(256) void k_origin_box_fold(const uint32_t* __restrict__ part, uint32_t n_parts,
                                                         uint32_t* __restrict__ box) {
  __shared__ uint32_t red[4][6];
  uint32_t lo[3] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu}, hi[3] = {0u, 0u, 0u};
  for (uint32_t b = threadIdx.x; b < n_parts; b += 256u)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      lo[a] = min(lo[a], part[(size_t)b * 6 + a]);
      hi[a] = max(hi[a], part[(size_t)b * 6 + 3 + a]);
    }
  wave_minmax(lo, hi);
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      red[wave][a] = lo[a];
      red[wave][3 + a] = hi[a];
    }
  __syncthreads();
  if (threadIdx.x < 6) {
    uint32_t v = red[0][threadIdx.x];
    for (int w = 1; w < 4; ++w)
      v = threadIdx.x < 3 ? min(v, red[w][threadIdx.x]) : max(v, red[w][threadIdx.x]);
    box[threadIdx.x] = v;
  }
}

// Morton key of a ray within the box of the ray origins
__device__ inline uint32_t order_key(const nbvh_ray* __restrict__ rays, uint32_t r, const uint32_t* box, int order) {
  const float4* p = (const float4*)(rays + r);
  const float4 o = p[0];
  const float ov[3] = {o.x, o.y, o.z};
  float org[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float lo = key_float(box[a]), hi = key_float(box[3 + a]);
    org[a] = hi > lo ? (ov[a] - lo) / (hi - lo) : 0.0f;
  }
  uint32_t key = 0u;
  if (order == 1) {
#pragma unroll
    for (int a = 0; a < 3; ++a) key |= spread8(cell_of(org[a], 256.0f)) << a;
  } else {
    const float4 d = p[1];
    // octahedral map of the direction onto [-1, 1]^2
    const float l1 = fabsf(d.x) + fabsf(d.y) + fabsf(d.z);
    float u = l1 > 0.0f ? d.x / l1 : 0.0f, v = l1 > 0.0f ? d.y / l1 : 0.0f;
    if (d.z < 0.0f) {
      const float uu = (1.0f - fabsf(v)) * (u >= 0.0f ? 1.0f : -1.0f);
      v = (1.0f - fabsf(u)) * (v >= 0.0f ? 1.0f : -1.0f);
      u = uu;
    }
    const uint32_t q[5] = {cell_of(org[0], 64.0f), cell_of(org[1], 64.0f), cell_of(org[2], 64.0f),
                           cell_of(0.5f * (u + 1.0f), 64.0f), cell_of(0.5f * (v + 1.0f), 64.0f)};
#pragma unroll
    for (int b = 0; b < 6; ++b)
#pragma unroll
      for (int k = 0; k < 5; ++k) key |= ((q[k] >> b) & 1u) << (5 * b + k);
  }
  return key;
}

// key of ray idx[i] (ray i without a list); entries at or past *n_valid (when
// given) get the largest key, so a stable sort keeps them behind the others
__global__ __launch_bounds__(256) void k_order_keys(const nbvh_ray* __restrict__ rays, const uint32_t* __restrict__ idx,
                                                    const uint32_t* __restrict__ n_valid, uint32_t n,
                                                    const uint32_t* __restrict__ box, int order,
                                                    uint32_t* __restrict__ keys) {
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;
  if (i >= n) return;
  keys[i] = (n_valid && i >= *n_valid) ? 0xFFFFFFFFu : order_key(rays, idx ? idx[i] : i, box, order);
}

// Box, keys and sort in one workgroup for up to kSortSmall rays; the sorted
// indices go to `out` (which may be idx) and, if given, their inverse to inv.
__global__ __launch_bounds__(1024) void k_order_small(const nbvh_ray* __restrict__ rays, const uint32_t* idx,
                                                      const uint32_t* __restrict__ n_valid, uint32_t n, int order,
                                                      uint32_t* out, uint32_t* __restrict__ inv) {
  __shared__ SmallSort S;
  __shared__ uint32_t red[16][6], box[6];
  uint32_t lo[3] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu}, hi[3] = {0u, 0u, 0u};
  for (uint32_t i = threadIdx.x; i < n; i += 1024u) {
    const float4 o = *(const float4*)(rays + i);
    const float p[3] = {o.x, o.y, o.z};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      lo[a] = min(lo[a], float_key(p[a]));
      hi[a] = max(hi[a], float_key(p[a]));
    }
  }
  wave_minmax(lo, hi);
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      red[threadIdx.x >> 6][a] = lo[a];
      red[threadIdx.x >> 6][3 + a] = hi[a];
    }
  __syncthreads();
  if (threadIdx.x < 6) {
    uint32_t v = red[0][threadIdx.x];
    for (int w = 1; w < 16; ++w) v = threadIdx.x < 3 ? min(v, red[w][threadIdx.x]) : max(v, red[w][threadIdx.x]);
    box[threadIdx.x] = v;
  }
  __syncthreads();
  const uint32_t valid = n_valid ? *n_valid : n;
  for (uint32_t i = threadIdx.x; i < n; i += 1024u) {
    const uint32_t r = idx && i < valid ? idx[i] : i;  // entries past the list's end hold nothing
    S.val[i] = r;
    S.key[i] = i < valid ? order_key(rays, r, box, order) : 0xFFFFFFFFu;
  }
  __syncthreads();
  sort_small(S, n, order == 1 ? 24 : 32);
  for (uint32_t i = threadIdx.x; i < n; i += 1024u) {
    out[i] = S.val[i];
    if (inv) inv[S.val[i]] = i;
  }
}

__global__ __launch_bounds__(256) void k_invert(const uint32_t* __restrict__ perm, uint32_t n,
                                                uint32_t* __restrict__ inv) {
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;
  if (i < n) inv[perm[i]] = i;
}

size_t ray_order_bytes(uint64_t n) { return group_ws_bytes(n); }

// The rays idx (all n, or the first *n_valid entries of a list) in key order:
// *sorted, written to `vout` when it is given.
static nbvh_status sort_rays(const LaunchCtx& L, const nbvh_ray* rays, const uint32_t* idx, const uint32_t* n_valid,
                             uint32_t n, int order, const SortWs& O, uint32_t* vout, const uint32_t** sorted) {
  const uint32_t nb = (n + 255) / 256;
  // the origins' box over all rays; its per-block partials use the digit counts' space
  k_origin_box<<<nb, 256, 0, L.stream>>>(rays, n, O.counts);
  k_origin_box_fold<<<1, 256, 0, L.stream>>>(O.counts, nb, O.box);
  k_order_keys<<<nb, 256, 0, L.stream>>>(rays, idx, n_valid, n, O.box, order, O.kbuf[1]);
  const uint32_t* keys = nullptr;
  return sort_pairs(L.stream, O.kbuf[1], idx, n, order == 1 ? 24 : 32, O, vout, &keys, sorted);  // 24- or 30-bit keys
}

// The permutation (grouped queries: one order for every object).
nbvh_status launch_ray_order(const LaunchCtx& L, const nbvh_ray* rays, uint32_t n, int order, void* ws,
                             RayOrder* out) {
  out->perm = out->inv = nullptr;
  if (n == 0 || order == 0) return NBVH_OK;
  const SortWs O = sort_ws(ws, n);
  uint32_t* inv = O.kbuf[0];  // the keys are not needed after the sort
  const uint32_t* perm = O.vbuf[0];
  if (n <= kSortSmall) {
    k_order_small<<<1, 1024, 0, L.stream>>>(rays, nullptr, nullptr, n, order, O.vbuf[0], inv);
  } else {
    nbvh_status s = sort_rays(L, rays, nullptr, nullptr, n, order, O, nullptr, &perm);
    if (s != NBVH_OK) return s;
    k_invert<<<(n + 255) / 256, 256, 0, L.stream>>>(perm, n, inv);
  }
  out->perm = perm;
  out->inv = inv;
  return check_launch("ray order");
}

// The active list of one object's query, reordered in place after the
// counting pass (the pass keeps the rays' own order, so its loads and
// stores stay coalesced; only the evaluation follows the key order).
static nbvh_status order_active_list(const LaunchCtx& L, const nbvh_ray* rays, uint32_t n, uint32_t* active,
                                     const uint32_t* n_active, int order, void* ws) {
  if (n <= kSortSmall) {
    k_order_small<<<1, 1024, 0, L.stream>>>(rays, active, n_active, n, order, active, nullptr);
    return check_launch("ray order");
  }
  const uint32_t* sorted = nullptr;
  return sort_rays(L, rays, active, n_active, n, order, sort_ws(ws, n), active, &sorted);
}

nbvh_status launch_traverse(const LaunchCtx& L, const nbvh_ray* rays, uint32_t n_rays, uint32_t* offsets,
                            nbvh_segment* segs, uint64_t capacity, nbvh_hit* hits, uint32_t* active,
                            uint32_t* n_active, uint32_t* scratch_counts, uint32_t* scratch_sums, float* staging,
                            const RayOrder* order,
                            void* active_order_ws, uint32_t* scratch_pos, uint32_t* scratch_sums2) {
  if (segs && !staging) return set_error("traversal staging buffer missing"), NBVH_ERR_INVALID_ARG;
  if (active && (!n_active || !segs || !scratch_pos || !scratch_sums2))
    return set_error("active-ray list without its buffers"), NBVH_ERR_INVALID_ARG;
  ProfScope ps(L.prof, NBVH_K_TRAVERSE, L.stream);
  const uint32_t grid = ray_blocks(n_rays);
  const WeightCopy wc = active ? weight_copy(L) : WeightCopy{nullptr, nullptr, 0};  // a query follows
  const uint32_t stack_words = 256u * (uint32_t)(L.stack_depth > 0 ? L.stack_depth : 1);
  const bool in_lds = L.n_nodes <= (n_rays <= kTreeRays ? kTreeNodes : kTreeSmall) && L.tune.traverse_mode != 1;
  const size_t lds = (size_t)stack_words * 4 + (in_lds ? (size_t)L.n_nodes * sizeof(Node) : 0);
  if (active && !order && n_rays > 0 && n_rays <= kOneRays) {
    auto kern = L.cfg.inside_reverse ? (in_lds ? k_traverse_one<true, true> : k_traverse_one<true, false>)
                                     : (in_lds ? k_traverse_one<false, true> : k_traverse_one<false, false>);
    const size_t one = lds + (size_t)kStage * 3 * 256 * 4;  // at most 48 + 48 + 64 KiB
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)one);
    kern<<<1 + wc.blocks, 256, one, L.stream>>>(L.nodes, rays, n_rays, hits, L.tune.traverse_mode, L.n_nodes, stack_words,
                                                offsets, scratch_pos, active, n_active, segs, capacity, L.state, L.cfg, wc);
    if (active_order_ws && L.tune.query_order != 0)
      return order_active_list(L, rays, n_rays, active, n_active, L.tune.query_order, active_order_ws);
    return check_launch("traverse");
  }
  if (n_rays > 0) {
    auto kern = L.cfg.inside_reverse ? (in_lds ? k_traverse_count<true, true> : k_traverse_count<true, false>)
                                     : (in_lds ? k_traverse_count<false, true> : k_traverse_count<false, false>);
    if (in_lds) (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    kern<<<grid + wc.blocks, 256, lds, L.stream>>>(L.nodes, rays, n_rays, scratch_counts, hits, segs ? staging : nullptr,
                                                   L.tune.traverse_mode, order ? order->perm : nullptr, L.n_nodes,
                                                   stack_words, L.cfg, wc);
  }
  const uint32_t n_tiles = n_rays > 0 ? (n_rays + kScanTile - 1) / kScanTile : 1;
  const int scanned = n_tiles > kScanDirectTiles ? 1 : 0;
  if (active && n_rays <= kScanSmall) {
    k_scan2_small<<<1, 1024, 0, L.stream>>>(scratch_counts, n_rays, order ? order->perm : nullptr, offsets, scratch_pos,
                                            n_active, capacity, L.state);
  } else if (active) {
    // offsets and the active-list positions in one set of scan launches
    k_scan2_tiles<<<n_tiles, 256, 0, L.stream>>>(scratch_counts, n_rays, order ? order->perm : nullptr, offsets,
                                                 scratch_pos, scratch_sums, scratch_sums2);
    if (scanned) k_scan2_sums<<<2, 1024, 0, L.stream>>>(scratch_sums, scratch_sums2, n_tiles);
    k_scan2_add<<<n_tiles, 256, 0, L.stream>>>(offsets, scratch_pos, n_rays, scratch_sums, scratch_sums2, scanned,
                                               n_active, capacity, L.state);
  } else {
    k_scan_tiles<<<n_tiles, 256, 0, L.stream>>>(scratch_counts, n_rays, offsets, scratch_sums);
    if (scanned) k_scan_sums<<<1, 1024, 0, L.stream>>>(scratch_sums, n_tiles, scratch_sums + n_tiles);
    k_scan_add<<<n_tiles, 256, 0, L.stream>>>(offsets, n_rays, scratch_sums, scanned, capacity, L.state);
  }
  if (segs && n_rays > 0)
    (L.cfg.inside_reverse ? k_traverse_compact<true> : k_traverse_compact<false>)<<<grid, 256, stack_lds(L),
                                                                                     L.stream>>>(
        L.nodes, rays, n_rays, offsets, staging, segs, capacity, L.tune.traverse_mode, order ? order->inv : nullptr,
        active ? scratch_pos : nullptr, active);
  if (active_order_ws && active && n_rays > 0 && L.tune.query_order != 0) {
    nbvh_status s = order_active_list(L, rays, n_rays, active, n_active, L.tune.query_order, active_order_ws);
    if (s != NBVH_OK) return s;
  }
  return check_launch("traverse");
}

}  // namespace nbvh
