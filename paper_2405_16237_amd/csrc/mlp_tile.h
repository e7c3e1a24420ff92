// MLP layers on one tile of M rows held in LDS, on the CDNA4 matrix cores.
//
// A layer computes out[m][n] = sum_k act[m][k] * W[n][k] (no bias). It is
// issued as the transposed product out^T = W x act^T: the A fragment is 16
// rows of W by 32 (FP32: 16) columns, read from copies in fragment order or
// from the row-major parameters themselves (FP32, or their BF16 shadow); the B
// fragment is the same columns of 16 activation rows, from LDS. The 16x16 accumulator tile of a lane then holds 4 consecutive
// output features of one row, handed to the epilogue (ReLU + store, mask +
// store, raw store).
//
// What bounds a layer here is the weights' way from L2 (a tile of 64 rows uses
// each once): row-major rows took a request slot of the L1 for every lane, and
// each group of products waited for its own loads. In fragment order a load is
// one contiguous kilobyte, and a fragment's registers are loaded again as soon
// as its products are issued, across column tiles and the layers' barriers.
// Bounce-ray query, MLP 256-4x256-8: 4.46 -> 3.84 ms; 1920x1080 query, MLP
// 256-4x128-5: 2.39 -> 2.30 ms. FP32, and BF16 outside queries, read the
// parameters: the caller may have written them, so a copy has to be made in
// every call. A query's traversal makes it on the side (10^6 camera rays, these
// two networks: 940 and 1,111 us with it, 1,092 and 1,205 from the parameters);
// a forward pass would need a launch more for what it gains (30,000 segments:
// 114 and 157 us, 118 and 158 from the parameters), a training step gains nothing.
//
// BF16: v_mfma_f32_16x16x32_bf16, activations rounded to bf16 between layers.
// FP8: 16x16x32 E4M3. FP32: v_mfma_f32_16x16x4_f32. FP32 accumulation.
#pragma once
#include "nbvh_internal.h"

namespace nbvh {

// FP8 E4M3 (OCP) activation byte
struct fp8e4 {
  uint8_t v;
};

template <typename AT>
struct Pad;
template <>
struct Pad<fp8e4> {
  static constexpr int v = 16;  // bytes: rows start 4 banks apart
  static constexpr int kstep = 32;
};
template <>
struct Pad<bf16> {
  static constexpr int v = 8;  // 16 bytes per row: rows start 4 banks apart
  static constexpr int kstep = 32;
};
template <>
struct Pad<float> {
  static constexpr int v = 4;
  static constexpr int kstep = 16;
};

__device__ inline bf16x8 zero_bf16x8() {
  bf16x8 z;
#pragma unroll
  for (int i = 0; i < 8; ++i) z[i] = (bf16)0.0f;
  return z;
}

template <typename AT>
struct Mma;
template <>
struct Mma<bf16> {
  typedef bf16x8 Frag;
  static constexpr int fk = 32;  // columns of a fragment
  __device__ static Frag zero() { return zero_bf16x8(); }
  __device__ static f32x4 mul(const Frag& a, const Frag& b, f32x4 acc) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0);
  }
};
template <>
struct Mma<fp8e4> {
  typedef long Frag;
  static constexpr int fk = 32;
  __device__ static Frag zero() { return 0l; }
  __device__ static f32x4 mul(const Frag& a, const Frag& b, f32x4 acc) {
    return __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(a, b, acc, 0, 0, 0);
  }
};
template <>
struct Mma<float> {
  typedef f32x4 Frag;
  static constexpr int fk = 16;
  __device__ static Frag zero() { return f32x4{0.f, 0.f, 0.f, 0.f}; }
  __device__ static f32x4 mul(const Frag& a, const Frag& b, f32x4 acc) {
#pragma unroll
    for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[i], acc, 0, 0, 0);
    return acc;
  }
};

// Where a wave finds four consecutive fragments of a row tile: the lane's byte
// offset into the weights and which of the four is the layer's last.
struct FragRun {
  uint32_t off;
  int last;
};

// A layer's weights: N rows (output features) of K columns, K a multiple of a
// fragment's. All layers are read from one base and 32-bit offsets: a pointer of
// its own for each kept so many scalar registers that the query moved them out
// and in (69 in the frame query's kernel, 54 now).
template <typename AT, bool ORDERED>
struct LayerW {
  static constexpr int FK = Mma<AT>::fk, E = FK / 4;
  static constexpr int stride = ORDERED ? 64 * E * (int)sizeof(AT) : FK * (int)sizeof(AT);  // between fragments
  const AT* p;   // the first layer's, in fragment order if ORDERED, else row-major
  uint32_t off;  // bytes from there to this layer's
  int K, N;
  __device__ int tiles() const { return (N + 15) >> 4; }
  __device__ FragRun run(int nt, int kf) const {
    const int lane = threadIdx.x & 63, nkf = K / FK;
    FragRun r;
    r.last = nkf - 1 - kf;
    if constexpr (ORDERED) {
      r.off = off + (uint32_t)(nt * nkf + kf) * stride + (uint32_t)lane * (E * (int)sizeof(AT));
    } else {
      const int n = min(nt * 16 + (lane & 15), N - 1);  // rows past the last repeat it: outputs nobody reads
      r.off = off + (uint32_t)(n * K + E * (lane >> 4)) * (uint32_t)sizeof(AT) + (uint32_t)kf * stride;
    }
    return r;
  }
  __device__ typename Mma<AT>::Frag load(const FragRun& r, int i) const {
    return *(const typename Mma<AT>::Frag NBVH_GLOBAL*)((const char NBVH_GLOBAL*)p + (r.off + (uint32_t)(i * stride)));
  }
};

// The four fragments a wave multiplies next.
template <typename AT>
struct Group {
  typename Mma<AT>::Frag a[4];
};

// the wave's first group of a layer, as far as it has one
template <typename AT, bool ORDERED>
__device__ inline Group<AT> first_group(const LayerW<AT, ORDERED>& w) {
  Group<AT> g;
  const int wave = wave_id();
  if (wave < w.tiles()) {
    const FragRun r = w.run(wave, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (i <= r.last) g.a[i] = w.load(r, i);
  }
  return g;
}

// out^T tile loop. Epi(m, col, f32x4) receives rows m, columns col..col+3. `g`
// holds the wave's first group on entry and, given `next`, that layer's on
// return. A fragment's registers are loaded again as soon as its products are
// issued, so the next group (of this column tile, the next one or the next
// layer) travels meanwhile with no copies, which would wait for it. Fragments
// past a layer's last are neither loaded nor multiplied: with 64 columns, two of
// a group's four (10^6 camera rays, MLP 64-3x64-5: 480 us with all loaded, 463).
template <int M, int NWAVES, typename AT, bool ORDERED, typename Epi>
__device__ inline void gemm_tile(const AT* act_in, int ld_in, const LayerW<AT, ORDERED>& w, Group<AT>& g, Epi epi,
                                 const LayerW<AT, ORDERED>* next = nullptr) {
  typedef typename Mma<AT>::Frag Frag;
  constexpr int FK = Mma<AT>::fk, E = FK / 4, MT = M / 16;
  const int lane = threadIdx.x & 63, wave = wave_id();
  const int r16 = lane & 15, q = lane >> 4;
  const int n_tiles = w.tiles(), nkf = w.K / FK;
  const AT* arow = act_in + (size_t)r16 * ld_in + E * q;
  const bool more = next && wave < next->tiles();
  for (int nt = wave; nt < n_tiles; nt += NWAVES) {
    f32x4 acc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int kf = 0; kf < nkf; kf += 4) {
      const bool here = kf + 4 < nkf || nt + NWAVES < n_tiles;
      FragRun r{0u, -1};
      if (here) r = kf + 4 < nkf ? w.run(nt, kf + 4) : w.run(nt + NWAVES, 0);
      else if (more) r = next->run(wave, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (i == 0 || kf + i < nkf) {
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) {
            const Frag b = lds_load<Frag>(arow + (size_t)mt * 16 * ld_in + (kf + i) * FK);
            acc[mt] = Mma<AT>::mul(g.a[i], b, acc[mt]);
          }
        }
        if (i <= r.last) g.a[i] = w.load(r, i);
      }
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) epi(mt * 16 + r16, nt * 16 + 4 * q, acc[mt]);
  }
  if (wave >= n_tiles && more) {
    const FragRun r = next->run(wave, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (i <= r.last) g.a[i] = w.load(r, i);
  }
}

// Quantise to FP8 E4M3 with saturation at +-448 (the format's largest value).
__device__ inline uint32_t pack_fp8x4(float a, float b, float c, float d) {
  a = fminf(fmaxf(a, -448.0f), 448.0f);
  b = fminf(fmaxf(b, -448.0f), 448.0f);
  c = fminf(fmaxf(c, -448.0f), 448.0f);
  d = fminf(fmaxf(d, -448.0f), 448.0f);
  int w = __builtin_amdgcn_cvt_pk_fp8_f32(a, b, 0, false);
  w = __builtin_amdgcn_cvt_pk_fp8_f32(c, d, w, true);
  return (uint32_t)w;
}

// four consecutive activations of an LDS tile row
template <typename AT>
__device__ inline void store4(AT* dst, f32x4 v) {
  if constexpr (sizeof(AT) == 2) {
    bf16x4 b;
#pragma unroll
    for (int i = 0; i < 4; ++i) b[i] = (bf16)v[i];
    lds_store<bf16x4>(dst, b);
  } else {
    lds_store<f32x4>(dst, v);
  }
}

// What a query's tiles and the other calls' forward tiles read: copies in
// fragment order (E4M3 from the calibration, a query's BF16 ones made by its
// traversal, see order_weights) or the parameters and their BF16 shadow.
template <typename AT>
constexpr bool kOrderedQuery = sizeof(AT) < 4;
template <typename AT>
constexpr bool kOrderedForward = sizeof(AT) == 1;

// weights of layer k; base: the first layer's
template <bool ORDERED, typename AT>
__device__ inline LayerW<AT, ORDERED> forward_layer(const DevCfg& c, const AT* base, int k) {
  const uint64_t off = ORDERED ? c.wf_off[k] : c.w_off[k] - c.w_off[0];
  return LayerW<AT, ORDERED>{base, (uint32_t)off * (uint32_t)sizeof(AT), c.fan_in[k], c.fan_out[k]};
}

// Full forward of the tile: act0 holds the encoded input [M][n_in]; hidden
// layers ping-pong between act0 and act1; z receives [M][kOutPad] fp32.
// keep(k, m, col, relu_vals) sees every hidden output (k = layer index). `g`
// holds the wave's first weight group of layer 0. FP8: act0 holds the input
// quantised with the activation scale sa[0], each hidden output is
// dequantised, ReLU'd and requantised with sa[k + 1] (scales: sw[kMaxLayers],
// then sa[kMaxLayers]).
template <int M, int NWAVES, bool ORDERED, typename AT, typename Keep>
__device__ inline void mlp_forward_tile_keep(const DevCfg& c, const AT* Wbase, const float* scales, AT* act0, int ld0,
                                             AT* act1, int ld1, float* z, int ldz, Group<AT>& g, Keep keep) {
  AT* cur = act0;
  int ldc = ld0;
  AT* nxt = act1;
  int ldn = ld1;
  for (int k = 0; k <= c.hidden; ++k) {
    const bool last = (k == c.hidden);
    const auto w = forward_layer<ORDERED>(c, Wbase, k);
    const float dq = sizeof(AT) == 1 ? 1.0f / (scales[k] * scales[kMaxLayers + k]) : 1.0f;  // 1 / (sw_k * sa_k)
    if (last) {
      gemm_tile<M, NWAVES, AT>(cur, ldc, w, g, [&](int m, int col, f32x4 v) {
        if constexpr (sizeof(AT) == 1) v = v * dq;
        lds_store<f32x4>(z + (size_t)m * ldz + col, v);
      });
    } else {
      const auto wn = forward_layer<ORDERED>(c, Wbase, k + 1);
      const float qn = sizeof(AT) == 1 ? scales[kMaxLayers + k + 1] : 1.0f;
      gemm_tile<M, NWAVES, AT>(
          cur, ldc, w, g,
          [&](int m, int col, f32x4 v) {
            if constexpr (sizeof(AT) == 1) {
#pragma unroll
              for (int i = 0; i < 4; ++i) v[i] = fmaxf(v[i] * dq, 0.0f) * qn;
              lds_store<uint32_t>(nxt + (size_t)m * ldn + col, pack_fp8x4(v[0], v[1], v[2], v[3]));
            } else {
#pragma unroll
              for (int i = 0; i < 4; ++i) v[i] = fmaxf(v[i], 0.0f);
              store4<AT>(nxt + (size_t)m * ldn + col, v);
            }
            keep(k, m, col, v);
          },
          &wn);
    }
    __syncthreads();
    AT* t = cur;
    cur = nxt;
    nxt = t;
    int tl = ldc;
    ldc = ldn;
    ldn = tl;
  }
}

template <int M, int NWAVES, bool ORDERED, typename AT>
__device__ inline void mlp_forward_tile(const DevCfg& c, const AT* Wbase, const float* scales, AT* act0, int ld0, AT* act1,
                                        int ld1, float* z, int ldz, Group<AT>& g) {
  mlp_forward_tile_keep<M, NWAVES, ORDERED, AT>(c, Wbase, scales, act0, ld0, act1, ld1, z, ldz, g, [](int, int, int, f32x4) {});
}

}  // namespace nbvh
