// Encoding of a tile of segments into the LDS activation tile: lanes are
// segments (slots), so the 64 lookups of one wave instruction hit one level
// and neighbouring segments share cache lines; waves stride over the
// (sample, level) pairs.
#pragma once
#include "mlp_tile.h"
#include "nbvh_internal.h"

namespace nbvh {

template <typename AT, int F>
__device__ inline void store_features(AT* dst, const float v[F], float qscale = 1.0f) {
  if constexpr (sizeof(AT) == 1) {
    const uint32_t w = pack_fp8x4(v[0] * qscale, v[1] * qscale, F == 4 ? v[2 % F] * qscale : 0.0f,
                                  F == 4 ? v[3 % F] * qscale : 0.0f);
    if constexpr (F == 2)
      *(uint16_t*)dst = (uint16_t)w;
    else
      *(uint32_t*)dst = w;
  } else if constexpr (sizeof(AT) == 2) {
    // round to nearest even on the hardware converter (one instruction per pair)
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    if constexpr (F == 2) {
      *(bf16x2*)dst = bf16x2{(bf16)v[0], (bf16)v[1]};
    } else {
      *(bf16x4*)dst = bf16x4{(bf16)v[0], (bf16)v[1], (bf16)v[2], (bf16)v[3]};
    }
  } else {
    if constexpr (F == 2)
      *(float2*)dst = make_float2(v[0], v[1]);
    else
      *(float4*)dst = make_float4(v[0], v[1], v[2], v[3]);
  }
}

// Raw table entry (F features) as loaded: packed bf16 or fp32 words.
template <int F, bool LP>
struct RawEntry;
template <>
struct RawEntry<2, true> {
  typedef uint32_t T;
};
template <>
struct RawEntry<4, true> {
  typedef uint2 T;
};
template <>
struct RawEntry<2, false> {
  typedef float2 T;
};
template <>
struct RawEntry<4, false> {
  typedef float4 T;
};

template <int F, bool LP>
__device__ inline typename RawEntry<F, LP>::T load_raw(const void* table, uint32_t byte_off) {
  typedef typename RawEntry<F, LP>::T T;
  // 32-bit byte offset from a uniform base: one VGPR per address (a level is
  // below 4 GiB); the pointer is a global one, so the load is a global (not a
  // flat) load whichever other loads sit beside it
  typedef uint32_t W __attribute__((ext_vector_type(sizeof(T) / 4)));
  const W w = *(const W __attribute__((address_space(1)))*)((const char __attribute__((address_space(1)))*)table +
                                                             byte_off);
  T r;
  __builtin_memcpy(&r, &w, sizeof(T));
  return r;
}

template <int F, bool LP>
__device__ inline void unpack_raw(const typename RawEntry<F, LP>::T& r, float v[F]) {
  if constexpr (LP) {
    if constexpr (F == 2) {
      v[0] = bf16_bits_to_f32(r & 0xffffu);
      v[1] = bf16_bits_to_f32(r >> 16);
    } else {
      v[0] = bf16_bits_to_f32(r.x & 0xffffu);
      v[1] = bf16_bits_to_f32(r.x >> 16);
      v[2] = bf16_bits_to_f32(r.y & 0xffffu);
      v[3] = bf16_bits_to_f32(r.y >> 16);
    }
  } else {
    if constexpr (F == 2) {
      v[0] = r.x;
      v[1] = r.y;
    } else {
      v[0] = r.x;
      v[1] = r.y;
      v[2] = r.z;
      v[3] = r.w;
    }
  }
}

// The same entry from the workgroup's LDS copy of the table's leading levels.
template <int F, bool LP>
__device__ inline typename RawEntry<F, LP>::T load_raw_lds(const unsigned char* ltab, uint32_t byte_off) {
  typedef typename RawEntry<F, LP>::T T;
  typedef uint32_t W __attribute__((ext_vector_type(sizeof(T) / 4)));
  const W w = *(const W __attribute__((address_space(3)))*)((const unsigned char __attribute__((address_space(3)))*)ltab +
                                                             byte_off);
  T r;
  __builtin_memcpy(&r, &w, sizeof(T));
  return r;
}

// Two adjacent table entries (an x-neighbour pair) as loaded.
template <int F, bool LP>
struct RawPair;
template <>
struct RawPair<2, true> {
  typedef uint2 T;  // 2 entries x 2 bf16
};
template <>
struct RawPair<4, true> {
  typedef uint4 T;  // 2 entries x 4 bf16
};
template <>
struct RawPair<2, false> {
  typedef float4 T;  // 2 entries x 2 fp32
};

template <int F, bool LP>
__device__ inline typename RawPair<F, LP>::T load_pair(const void* table, uint32_t byte_off) {
  typedef typename RawPair<F, LP>::T T;
  return *(const T*)((const char*)table + byte_off);
}

// entry 0 / 1 of a pair, as a raw entry
template <int F, bool LP>
__device__ inline typename RawEntry<F, LP>::T pair_half(const typename RawPair<F, LP>::T& p, bool second) {
  if constexpr (LP && F == 2) return second ? p.y : p.x;
  else if constexpr (LP && F == 4) return second ? uint2{p.z, p.w} : uint2{p.x, p.y};
  else return second ? float2{p.z, p.w} : float2{p.x, p.y};
}

// Partner lanes. The vector L1 merges two lanes of a 4-byte load into one
// request only where they name the same 64-byte line and sit 4, 8 or 12 lanes
// apart in a row of 16 (measured, cycles of a wave's load: every lane on its
// own line 64, lanes l and l + 1 on one line 64, lanes l and l + 8 on one line
// 33, random lines 35). So the two lanes that fetch the x-neighbours of a cell,
// which lie in one line but for every 16th x, are l and l ^ 8. Every function
// here is called by all lanes of the wave.
struct Partner {
  __device__ static bool lower() { return (threadIdx.x & 8) == 0; }
  __device__ static uint32_t swap(uint32_t v) {
    return __builtin_amdgcn_update_dpp(0u, v, 0x128, 0xf, 0xf, false);  // row_ror:8
  }
  // lower lanes keep `own`, upper lanes (banks 2 and 3 of a row) take their partner's `theirs`
  __device__ static uint32_t upper_takes(uint32_t own, uint32_t theirs) {
    return __builtin_amdgcn_update_dpp(own, theirs, 0x128, 0xf, 0xc, false);
  }
  __device__ static uint32_t lower_takes(uint32_t own, uint32_t theirs) {
    return __builtin_amdgcn_update_dpp(own, theirs, 0x128, 0xf, 0x3, false);
  }
};

// Bytes of the second activation tile and the logits of a forward tile, which
// hold the sample positions while the tile is encoded.
template <typename AT>
__host__ __device__ inline size_t tile_mid_bytes(int width, int n_samples) {
  const size_t mid = (size_t)64 * (width + Pad<AT>::v) * sizeof(AT) + (size_t)64 * kOutPad * 4;
  const size_t pos = (size_t)64 * n_samples * 12;
  return mid > pos ? mid : pos;
}

// Whether a tile's sample positions are computed once, into LDS, rather than
// by every wave for its own levels. With 4-byte entries the encode is short of
// vector issue (the frame's query spent 58 % of its cycles issuing), which this
// relieves; with wider ones it waits for table lines, and the extra barrier
// costs more (1 % of a bounce-ray query).
template <int F, bool LP>
constexpr bool kTilePositions = F * (LP ? 2 : 4) == 4;

// Unit-cube positions of the 64 segments' samples whose (o, t0) / (d, t1) sit
// in sA / sB: pos[(s * 3 + axis) * 64 + slot]. Ends with a barrier.
__device__ inline void sample_tile(const DevCfg& c, const float4* sA, const float4* sB, float* pos) {
  for (int e = threadIdx.x; e < c.n_samples * 64; e += blockDim.x) {
    const int s = e >> 6, m = e & 63;
    const float4 a = sA[m], b = sB[m];
    const float o[3] = {a.x, a.y, a.z}, d[3] = {b.x, b.y, b.z};
    float x[3];
    sample_position(c, o, d, a.w, b.w, s, x);
#pragma unroll
    for (int k = 0; k < 3; ++k) lds_store<float>(pos + (s * 3 + k) * 64 + m, x[k]);
  }
  __syncthreads();
}

// Encode the 64 segments whose (o, t0) / (d, t1) sit in sA / sB into act0. With
// kTilePositions, `pos` (LDS, 768 bytes a sample) holds the positions meanwhile.
// Called by the whole workgroup after a barrier.
// Wave w owns levels w, w + NWAVES, ... and walks them U at a time; for each
// group of levels it takes the samples in ray order, issuing the gathers of
// all U levels before consuming any. Consecutive samples of a segment often
// fall into the same cell at the coarser levels: such a lane keeps the
// corner values it already holds and is masked out of the gathers.
// Levels below lds_levels are gathered from ltab, the workgroup's LDS copy of
// the table's leading levels (not with PAIRS).
// With PAIRS, corners are fetched as x-neighbour pairs: on dense levels
// (x, x+1) are adjacent entries; on hashed levels they are the two halves of
// an aligned pair whenever x is even (the hash keeps x's low bit), so one
// load serves both and lanes with odd x add one masked load.
template <typename AT, int F, bool LP, int NWAVES, int UNROLL = 0, int GATHER = 0>
__device__ inline void encode_tile(const DevCfg& c, const void* table, const float4* sA, const float4* sB, float* pos,
                                   const int* s_valid, AT* act0, int ld0, float qscale = 1.0f, const unsigned char* ltab = nullptr,
                                   int lds_levels = 0) {
  typedef typename RawEntry<F, LP>::T Raw;
  constexpr uint32_t EB = sizeof(Raw);  // bytes of an entry
  constexpr bool kPairs = GATHER == 1 && !(F == 4 && !LP);  // a 32-byte fp32 pair has no single load
  constexpr bool kLds = GATHER == 2;
  constexpr bool kPartner = !kPairs && !kLds && EB == 4;
  constexpr int U = UNROLL > 0 ? UNROLL : 2;
  const int lane = threadIdx.x & 63, wave = wave_id();
  const int L = c.n_levels, S = c.n_samples;
  const uint32_t hmask = ((1u << c.log2_T) - 1u) * EB;  // over byte offsets
  const bool valid = s_valid[lane] != 0;
  float4 a, b;
  if constexpr (kTilePositions<F, LP>) {
    sample_tile(c, sA, sB, pos);
  } else {
    a = sA[lane];
    b = sB[lane];
  }
  for (int lg = wave; lg < L; lg += NWAVES * U) {
    Raw raw[U][8];
    int pcx[U], pcy[U], pcz[U];
    bool act[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      act[u] = lg + u * NWAVES < L;
      pcx[u] = pcy[u] = pcz[u] = -1;
    }
    for (int s = 0; s < S; ++s) {
      float x[3];
      if constexpr (kTilePositions<F, LP>) {
#pragma unroll
        for (int k = 0; k < 3; ++k) x[k] = lds_load<float>(pos + (s * 3 + k) * 64 + lane);
      } else {
        const float o[3] = {a.x, a.y, a.z}, d[3] = {b.x, b.y, b.z};
        sample_position(c, o, d, a.w, b.w, s, x);
      }
      float wx[U], wy[U], wz[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        // a group's missing levels are skipped (eight levels on eight waves have
        // one a wave: 10^6 camera rays, small network, 465 -> 439 us)
        if (!act[u]) continue;
        const int l = lg + u * NWAVES;
        const int N = c.level_res[l];
        const bool dense = (c.dense_mask >> l) & 1u;
        int cx, cy, cz;
        cell_weight(x[0], N, cx, wx[u]);
        cell_weight(x[1], N, cy, wy[u]);
        cell_weight(x[2], N, cz, wz[u]);
        const bool need = valid && (cx != pcx[u] || cy != pcy[u] || cz != pcz[u]);
        pcx[u] = cx;
        pcy[u] = cy;
        pcz[u] = cz;
        // Byte offsets, from the level's start, of the cell's corners (lower
        // x, upper x) at the four (y, z). Dense levels index
        // x + (N+1)(y + (N+1) z). Hashed ones XOR the per-axis products, the
        // upper y and z products being the lower ones plus the prime; at most
        // 24 bits of a hash are used, so 24-bit products (full rate) do.
        uint32_t i0[4], i1[4];
        if (dense) {
          const uint32_t r1 = ((uint32_t)N + 1u) * EB, r2 = r1 * ((uint32_t)N + 1u);
          const uint32_t e = (uint32_t)cx * EB + __umul24((uint32_t)cy, r1) + __umul24((uint32_t)cz, r2);  // N < 256
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            i0[j] = e + ((j & 1) ? r1 : 0u) + ((j & 2) ? r2 : 0u);
            i1[j] = i0[j] + EB;
          }
        } else {
          const uint32_t hy = __umul24((uint32_t)cy, kPrimeY & 0xffffffu), hz = __umul24((uint32_t)cz, kPrimeZ & 0xffffffu);
          const uint32_t hy0 = (hy * EB) & hmask, hy1 = ((hy + (kPrimeY & 0xffffffu)) * EB) & hmask;
          const uint32_t hz0 = (hz * EB) & hmask, hz1 = ((hz + (kPrimeZ & 0xffffffu)) * EB) & hmask;
          const uint32_t x0 = ((uint32_t)cx * EB) & hmask, x1 = ((uint32_t)cx * EB + EB) & hmask;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const uint32_t h = ((j & 1) ? hy1 : hy0) ^ ((j & 2) ? hz1 : hz0);
            i0[j] = x0 ^ h;
            i1[j] = x1 ^ h;
          }
        }
        const char* lt = (const char*)table + (size_t)c.level_off[l] * (LP ? 2 : 4);  // uniform
        if constexpr (kPairs) {
          if (need) {
            const bool even = dense || (cx & 1) == 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              const uint32_t at = dense ? i0[j] : i0[j] & ~EB;
              const auto p = load_pair<F, LP>(lt, at);
              raw[u][2 * j] = pair_half<F, LP>(p, at != i0[j]);
              raw[u][2 * j + 1] = even ? pair_half<F, LP>(p, at == i0[j]) : load_raw<F, LP>(lt, i1[j]);
            }
          }
        } else if constexpr (kPartner) {
          // first load: the lower lane's cell, its lower x by the lower lane
          // and its upper x by the partner; second load: the upper lane's
          const bool theirs = Partner::swap(need ? 1u : 0u) != 0u;
          const bool n_lo = Partner::lower() ? need : theirs, n_up = Partner::lower() ? theirs : need;
          uint32_t a_lo[4], a_up[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            a_lo[j] = Partner::upper_takes(i0[j], i1[j]);
            a_up[j] = Partner::lower_takes(i1[j], i0[j]);
          }
          if (n_lo) {
#pragma unroll
            for (int j = 0; j < 4; ++j) raw[u][j] = load_raw<F, LP>(lt, a_lo[j]);
          }
          if (n_up) {
#pragma unroll
            for (int j = 0; j < 4; ++j) raw[u][4 + j] = load_raw<F, LP>(lt, a_up[j]);
          }
        } else if (kLds && l < lds_levels) {  // wave-uniform
          const unsigned char* ll = ltab + (size_t)c.level_off[l] * (LP ? 2 : 4);
          if (need) {
#pragma unroll
            for (int k = 0; k < 8; ++k) raw[u][k] = load_raw_lds<F, LP>(ll, (k & 1) ? i1[k >> 1] : i0[k >> 1]);
          }
        } else if (need) {
#pragma unroll
          for (int k = 0; k < 8; ++k) raw[u][k] = load_raw<F, LP>(lt, (k & 1) ? i1[k >> 1] : i0[k >> 1]);
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (!act[u]) continue;
        float out[F];
#pragma unroll
        for (int f = 0; f < F; ++f) out[f] = 0.0f;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const float w = ((k & 1) ? wx[u] : 1.0f - wx[u]) * (((k >> 1) & 1) ? wy[u] : 1.0f - wy[u]) *
                          (((k >> 2) & 1) ? wz[u] : 1.0f - wz[u]);
          float v[F];
          if constexpr (kPartner) {
            // corner (lower x): the lower lane loaded its own first; the
            // upper lane's lies with its partner. Corner (upper x): mirrored
            const int j = k >> 1;
            unpack_raw<F, LP>((k & 1) ? Partner::lower_takes(raw[u][4 + j], raw[u][j])
                                      : Partner::upper_takes(raw[u][j], raw[u][4 + j]), v);
          } else {
            unpack_raw<F, LP>(raw[u][k], v);
          }
#pragma unroll
          for (int f = 0; f < F; ++f) out[f] = __builtin_fmaf(w, v[f], out[f]);
        }
#pragma unroll
        for (int f = 0; f < F; ++f) out[f] = valid ? out[f] : 0.0f;
        const int col = s * L * F + (lg + u * NWAVES) * F;
        store_features<AT, F>(act0 + (size_t)lane * ld0 + col, out, qscale);
      }
    }
  }
}

// Encode of a tile of few rows (16 or 32): the 64 lanes take several samples of
// each row at once, so a wave's chain of gathers is 64 / ROWS times shorter
// than encode_tile's; no use is made of samples that share a cell. Rows from
// n_rows on are left as they are.
template <typename AT, int F, bool LP, int NWAVES, int ROWS>
__device__ inline void encode_rows(const DevCfg& c, const void* table, const float4* sA, const float4* sB, int n_rows,
                                   AT* act0, int ld0, float qscale) {
  constexpr int P = 64 / ROWS;  // samples side by side
  const int lane = threadIdx.x & 63, row = lane % ROWS, sub = lane / ROWS;
  const float4 a = sA[row], b = sB[row];
  const float o[3] = {a.x, a.y, a.z}, d[3] = {b.x, b.y, b.z};
  const int L = c.n_levels, S = c.n_samples, tasks = L * ((S + P - 1) / P);
#pragma unroll 4
  for (int q = wave_id(); q < tasks; q += NWAVES) {
    const int l = q % L, s = P * (q / L) + sub;  // the level is uniform over the wave
    if (s < S && row < n_rows) {
      float x[3], v[F];
      sample_position(c, o, d, a.w, b.w, s, x);
      interp_level<F, LP>(c, table, l, x, v);
      store_features<AT, F>(act0 + (size_t)row * ld0 + s * L * F + l * F, v, qscale);
    }
  }
}

}  // namespace nbvh
