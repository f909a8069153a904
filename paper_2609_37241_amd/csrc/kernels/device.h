// Device-side building blocks shared by the standalone kernels and the fused
// decode-chain kernel: 16-byte packed element access, wavefront / workgroup
// reductions, and the per-role bodies. A role body is the same inlined code
// in both places, so the fused chain computes exactly what the three
// separate launches compute.
//
// Layout conventions: a workgroup has 256 work-items (4 wavefronts of 64),
// or 1024 for the longest norm rows (kWideLanes). A "vector" is 16 bytes: 4
// float32 or 8 bfloat16 elements, loaded and stored with one
// global_load/store_dwordx4 per lane.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../kernargs.h"

namespace tri {
namespace dev {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

constexpr int kF32 = 0, kBF16 = 1;
constexpr int kThreads = 256;

template <int DT>
struct Elt;

template <>
struct Elt<kF32> {
  static constexpr int V = 4;
  static constexpr int ES = 4;
  __device__ static inline void unpack(const u32x4 &p, float *f) {
#pragma unroll
    for (int i = 0; i < 4; ++i) f[i] = __uint_as_float(p[i]);
  }
  __device__ static inline u32x4 pack(const float *f) {
    u32x4 p;
#pragma unroll
    for (int i = 0; i < 4; ++i) p[i] = __float_as_uint(f[i]);
    return p;
  }
  __device__ static inline float ld(const void *b, int64_t i) {
    return static_cast<const float *>(b)[i];
  }
  __device__ static inline void st(void *b, int64_t i, float v) { static_cast<float *>(b)[i] = v; }
  __device__ static inline float round(float v) { return v; }
};

template <>
struct Elt<kBF16> {
  static constexpr int V = 8;
  static constexpr int ES = 2;
  // bf16 -> f32 is exact: the bf16 bits are the upper half of the f32 bits.
  __device__ static inline void unpack(const u32x4 &p, float *f) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      f[2 * j] = __uint_as_float(p[j] << 16);
      f[2 * j + 1] = __uint_as_float(p[j] & 0xFFFF0000u);
    }
  }
  // f32 -> bf16 round-to-nearest-even, two at a time (v_cvt_pk_bf16_f32).
  __device__ static inline uint32_t pack2(float a, float b) {
    const f32x2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
  }
  __device__ static inline u32x4 pack(const float *f) {
    u32x4 p;
#pragma unroll
    for (int j = 0; j < 4; ++j) p[j] = pack2(f[2 * j], f[2 * j + 1]);
    return p;
  }
  __device__ static inline float ld(const void *b, int64_t i) {
    return __uint_as_float(uint32_t(static_cast<const uint16_t *>(b)[i]) << 16);
  }
  __device__ static inline void st(void *b, int64_t i, float v) {
    static_cast<uint16_t *>(b)[i] = uint16_t(pack2(v, 0.0f) & 0xFFFFu);
  }
  __device__ static inline float round(float v) {
    return __uint_as_float(pack2(v, 0.0f) << 16);
  }
};

// 16-byte global access; NT marks streaming data (nontemporal: the line is
// not kept in the caches for reuse), used where the working set is far larger
// than the caches.
template <bool NT>
__device__ inline u32x4 ld16(const u32x4 *p) {
  if constexpr (NT)
    return __builtin_nontemporal_load(p);
  else
    return *p;
}

template <bool NT>
__device__ inline void st16(u32x4 *p, const u32x4 &v) {
  if constexpr (NT)
    __builtin_nontemporal_store(v, p);
  else
    *p = v;
}

// 16-byte access at element alignment, for tensors whose rows start anywhere:
// gfx950 global memory takes a 16-byte access at any element address as one
// instruction. A wavefront's 1 KiB then touches nine 128-byte lines instead
// of eight: measured 0.94-0.99 of the aligned rate (a 2-read, 1-write stream
// of 1.2 GB, one element off: 5.72 against 5.98 TB/s).
template <int DT>
struct AnyVec;
template <>
struct AnyVec<kF32> {
  typedef u32x4 type __attribute__((aligned(4)));
};
template <>
struct AnyVec<kBF16> {
  typedef u32x4 type __attribute__((aligned(2)));
};
template <int DT, bool NT>
__device__ inline u32x4 ld_any(const void *p) {
  typedef const typename AnyVec<DT>::type *ptr;
  if constexpr (NT)
    return __builtin_nontemporal_load(static_cast<ptr>(p));
  else
    return *static_cast<ptr>(p);
}
template <int DT, bool NT>
__device__ inline void st_any(void *p, const u32x4 &v) {
  typedef typename AnyVec<DT>::type *ptr;
  if constexpr (NT)
    __builtin_nontemporal_store(v, static_cast<ptr>(p));
  else
    *static_cast<ptr>(p) = v;
}

// ---- reductions ----------------------------------------------------------------
// DPP move within a row of 16 lanes (every source lane is in range for the
// controls used here, so no lane reads an out-of-row value).
template <int CTRL>
__device__ inline float dpp_mov(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}

// Sum over the 64 lanes of a wavefront (all lanes active). Within each row of
// 16 lanes: exchange with lane^1 and lane^2 (quad permutes), then with the
// mirrored lane in each half row and in the row, so every lane holds its
// row's sum; the four row sums are read from lanes 0, 16, 32, 48 and added in
// a fixed order. Every lane returns the same, bitwise equal total.
__device__ inline float wave_sum(float v) {
  v += dpp_mov<0xB1>(v);    // quad_perm [1,0,3,2]
  v += dpp_mov<0x4E>(v);    // quad_perm [2,3,0,1]
  v += dpp_mov<0x141>(v);   // row_half_mirror
  v += dpp_mov<0x140>(v);   // row_mirror
  const int b = __float_as_int(v);
  const float r0 = __int_as_float(__builtin_amdgcn_readlane(b, 0));
  const float r1 = __int_as_float(__builtin_amdgcn_readlane(b, 16));
  const float r2 = __int_as_float(__builtin_amdgcn_readlane(b, 32));
  const float r3 = __int_as_float(__builtin_amdgcn_readlane(b, 48));
  return (r0 + r1) + (r2 + r3);
}

// The same in float64 (long rows and rows of any alignment): a double moves
// between lanes as its two halves.
template <int CTRL>
__device__ inline double dpp_mov(double v) {
  const u32x2 b = __builtin_bit_cast(u32x2, v);
  u32x2 r;
  r[0] = __builtin_amdgcn_update_dpp(0, b[0], CTRL, 0xF, 0xF, false);
  r[1] = __builtin_amdgcn_update_dpp(0, b[1], CTRL, 0xF, 0xF, false);
  return __builtin_bit_cast(double, r);
}
__device__ inline double read_lane(double v, int lane) {
  const u32x2 b = __builtin_bit_cast(u32x2, v);
  u32x2 r;
  r[0] = __builtin_amdgcn_readlane(b[0], lane);
  r[1] = __builtin_amdgcn_readlane(b[1], lane);
  return __builtin_bit_cast(double, r);
}
__device__ inline double wave_sum(double v) {
  v += dpp_mov<0xB1>(v);
  v += dpp_mov<0x4E>(v);
  v += dpp_mov<0x141>(v);
  v += dpp_mov<0x140>(v);
  return (read_lane(v, 0) + read_lane(v, 16)) + (read_lane(v, 32) + read_lane(v, 48));
}

// Sum over aligned groups of n consecutive lanes (n a power of two, at most
// 64, the same for the whole wavefront); every lane of a group returns the
// same, bitwise equal sum. Lanes of one group must be active together.
template <typename T>
__device__ inline T group_sum(T v, int n) {
  if (n >= 2) v += dpp_mov<0xB1>(v);    // lane ^ 1
  if (n >= 4) v += dpp_mov<0x4E>(v);    // lane ^ 2
  if (n >= 8) v += dpp_mov<0x141>(v);   // the other quad of the half row
  if (n >= 16) v += dpp_mov<0x140>(v);  // the other half row
  if (n >= 32) v += __shfl_xor(v, 16, 64);
  if (n >= 64) v += __shfl_xor(v, 32, 64);
  return v;
}

// Sum over the NW wavefronts of a workgroup (256 work-items by default);
// `red` is NW words of LDS. The wavefront sums are added in a fixed order.
template <int NW = 4, typename T>
__device__ inline T block_sum(T v, T *red) {
  v = wave_sum(v);
  const int wid = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) red[wid] = v;
  __syncthreads();
  T s;
  if constexpr (NW == 4) {
    s = (red[0] + red[1]) + (red[2] + red[3]);
  } else {
    s = red[0];
#pragma unroll
    for (int i = 1; i < NW; ++i) s += red[i];
  }
  __syncthreads();
  return s;
}

// The same for the last sum a workgroup makes with `red` (it is not free again
// afterwards): one barrier.
template <int WAVES = 4, typename T>
__device__ inline T block_sum_once(T v, T *red) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  if constexpr (WAVES == 4)
    return (red[0] + red[1]) + (red[2] + red[3]);
  else   // each partial sum in 64 / WAVES lanes: the total that often, exactly
    return wave_sum(red[threadIdx.x & (WAVES - 1)]) * T(WAVES / 64.0);
}

// acc + the squares of a vector's N floats in float64. The products are exact
// in float64, so the fused form rounds as a product and a sum do; two chains
// of them run side by side.
template <int N>
__device__ inline void add_squares(double *acc, const float *f) {
#pragma unroll
  for (int e = 0; e < N; ++e) acc[e & 1] = __builtin_fma(double(f[e]), double(f[e]), acc[e & 1]);
}

// RN_f32(1 / sqrt(m)) for m = ss / H + eps: the hardware's reciprocal square
// root and two Newton steps (v_rsq_f64 is good to 2^-24; a step squares that
// and takes half as much again: one step alone would leave 2^-47) instead of a
// division, a square root and another division, about 100 dependent float64
// instructions between a row's sum and its first store. Before the rounding to
// float32 the error is at most 2.5 * 2^-53, as theirs: 1 / H, its product with
// ss and the last step's product and sum. 0 and infinity, where a step has
// 0 * infinity in it, keep the first value.
__device__ inline float inv_rms(double ss, double rcp_h, float eps) {
  const double m = __builtin_fma(ss, rcp_h, double(eps));
  const double y = __builtin_amdgcn_rsq(m);
  double r = y;
#pragma unroll
  for (int i = 0; i < 2; ++i) r = __builtin_fma(0.5 * r, __builtin_fma(-m * r, r, 1.0), r);
  return float(__builtin_isfinite(r) ? r : y);
}

// ---- RMSNorm / residual RMSNorm --------------------------------------------------
// One row held in registers: lane `lane` of LANES owns vectors lane + LANES*k,
// k < NV. With RES, h = RN(x + r) is written to res_out and normalised.
// LANES = 64: one wavefront per row, no barrier. LANES = 256 or kWideLanes:
// one workgroup of that many work-items.
// Without LATE (decode sizes) the weight vectors are requested together with the
// row, so the row costs one memory round trip; with it (streaming sizes) they
// are loaded after the reduction to keep fewer registers live.
template <int DT, int NV, bool RES, int LANES, bool NT, bool LATE = NT>
__device__ __forceinline__ void rn_row_regs(const RnArgs &a, int64_t row, int lane, float *red) {
  using E = Elt<DT>;
  constexpr int V = E::V;
  const int nvec = a.H / V;
  const u32x4 *xr = reinterpret_cast<const u32x4 *>(static_cast<const char *>(a.x) +
                                                     row * a.x_rs * E::ES);
  const u32x4 *wr = static_cast<const u32x4 *>(a.w);
  u32x4 xv[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int vi = lane + LANES * k;
    xv[k] = vi < nvec ? ld16<NT>(xr + vi) : u32x4{0, 0, 0, 0};
  }
  u32x4 rv[RES ? NV : 1];
  if constexpr (RES) {
    const u32x4 *rr = reinterpret_cast<const u32x4 *>(static_cast<const char *>(a.res) +
                                                       row * a.res_rs * E::ES);
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const int vi = lane + LANES * k;
      rv[k] = vi < nvec ? ld16<NT>(rr + vi) : u32x4{0, 0, 0, 0};
    }
  }
  u32x4 wv[LATE ? 1 : NV];
  if constexpr (!LATE) {
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const int vi = lane + LANES * k;
      wv[k] = vi < nvec ? wr[vi] : u32x4{0, 0, 0, 0};
    }
  }
  if constexpr (RES) {
    u32x4 *orow = reinterpret_cast<u32x4 *>(static_cast<char *>(a.res_out) + row * a.ro_rs * E::ES);
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      float f[V], g[V];
      E::unpack(xv[k], f);
      E::unpack(rv[k], g);
#pragma unroll
      for (int e = 0; e < V; ++e) f[e] += g[e];
      xv[k] = E::pack(f);
      const int vi = lane + LANES * k;
      if (vi < nvec) orow[vi] = xv[k];
    }
  }
  float ss = 0.0f;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    float f[V];
    E::unpack(xv[k], f);
#pragma unroll
    for (int e = 0; e < V; ++e) ss = __builtin_fmaf(f[e], f[e], ss);
  }
  if constexpr (LANES == 64)
    ss = wave_sum(ss);
  else if constexpr (LANES == kThreads)
    ss = block_sum_once(ss, red);
  else
    ss = block_sum<LANES / 64>(ss, red);
  const float inv = rsqrtf(ss / float(a.H) + a.eps);
  u32x4 *yr = reinterpret_cast<u32x4 *>(static_cast<char *>(a.y) + row * a.y_rs * E::ES);
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int vi = lane + LANES * k;
    if (vi < nvec) {
      float f[V], w[V];
      E::unpack(xv[k], f);
      if constexpr (LATE)
        E::unpack(wr[vi], w);
      else
        E::unpack(wv[k], w);
#pragma unroll
      for (int e = 0; e < V; ++e) f[e] = (f[e] * inv) * w[e];
      yr[vi] = E::pack(f);
    }
  }
}

// Workgroup `blk` of the one-wavefront-per-row layout: rows 4*blk .. 4*blk+3.
template <int DT, int NV, bool RES, bool NT>
__device__ __forceinline__ void rn_wave_block(const RnArgs &a, int64_t blk) {
  const int64_t row = blk * 4 + (threadIdx.x >> 6);
  if (row >= a.T) return;
  rn_row_regs<DT, NV, RES, 64, NT>(a, row, threadIdx.x & 63, nullptr);
}

// ---- split rows -------------------------------------------------------------------
// A row of nvec vectors is split over S = ceil(nvec / kSplitSpan)
// consecutive workgroups (workgroup b: row b / S, slice b % S, up to
// kSplitVecs vectors per work-item). Each holds its slice in registers,
// reduces its partial sum of squares, publishes it in the row's slot of the
// scratch buffer and waits until all S slots of the row are full; every
// workgroup of the row then adds the S partials in the same order (one
// wavefront, lanes 0..S-1), so all of them normalise with the same total.
// The row is read once and written once: nothing is re-read.
//
// Slots carry their own "full" bit, so the exchange needs no memory fence:
// a slot is one relaxed device-scope 64-bit atomic, and nothing else is
// communicated. The row's last reader (a per-row counter reaching S)
// clears the row's slots and counter, so the scratch is all zero again when
// the kernel ends, ready for the next call on the stream. No counter is
// shared between rows: atomics on one address serialise, and a ticket or
// completion counter for the whole grid measured 5-20x slower.
//
// The wait relies on the S workgroups of a row being resident together:
// they are consecutive in dispatch order, so once the earlier ones run the
// later ones are next in line (S <= 64, far below the workgroups the GPU
// holds). As a guard against anything else occupying the GPU indefinitely,
// the wait is bounded (kSplitSpinMax polls, several hundred milliseconds):
// a row whose partials do not all arrive is written as NaN and sets the
// sticky failure flag in header word 0, after which every call on that
// scratch writes NaN rows instead of trusting the exchange. A failure is
// therefore loud and never silent.
constexpr int kSplitSpinMax = 1 << 18;
constexpr uint64_t kSlotFull = uint64_t(1) << 63;

template <int DT, bool RES, bool NT>
__device__ __forceinline__ void rn_split_row(const RnArgs &a, uint64_t *scratch, float *red,
                                             float &total) {
  using E = Elt<DT>;
  constexpr int V = E::V;
  constexpr int NB = kSplitVecs;
  const int nvec = a.H / V;
  const int S = (nvec + kSplitSpan - 1) / kSplitSpan;
  // both divisions in 32 bits, as the row's first load waits for them (bf16
  // residual rows: 8 x 40960 6.68 against 6.98 us, 200 x 131,072 48.4 against 48.9)
  const uint32_t r32 = blockIdx.x / uint32_t(S);
  const int64_t row = r32;
  const int s = int(blockIdx.x - r32 * uint32_t(S));
  uint64_t *slots = scratch + kSplitHeaderWords + row * S;
  uint64_t *count = scratch + kSplitHeaderWords + a.T * S + row;
  // equal slices (whole wavefronts of vectors), so that no workgroup of the
  // row only waits for the others (bf16 residual rows of 49,408, whose fourth
  // slice of 2048 vectors would hold 32: 84.2 against 90.1 us at 1061 rows)
  const int span = int(uint32_t(nvec + S - 1) / uint32_t(S) + 63) & ~63;
  const int v0 = s * span + int(threadIdx.x);
  const int vend = (s + 1) * span < nvec ? (s + 1) * span : nvec;
  const u32x4 *xr = reinterpret_cast<const u32x4 *>(static_cast<const char *>(a.x) +
                                                     row * a.x_rs * E::ES);
  const u32x4 *wr = static_cast<const u32x4 *>(a.w);
  u32x4 xv[NB], wv[NB];
#pragma unroll
  for (int k = 0; k < NB; ++k) {
    const int vi = v0 + 256 * k;
    xv[k] = vi < vend ? ld16<NT>(xr + vi) : u32x4{0, 0, 0, 0};
  }
  if constexpr (RES) {
    const u32x4 *rr = reinterpret_cast<const u32x4 *>(static_cast<const char *>(a.res) +
                                                       row * a.res_rs * E::ES);
    u32x4 *orow = reinterpret_cast<u32x4 *>(static_cast<char *>(a.res_out) + row * a.ro_rs * E::ES);
    u32x4 rv[NB];
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      const int vi = v0 + 256 * k;
      rv[k] = vi < vend ? ld16<NT>(rr + vi) : u32x4{0, 0, 0, 0};
    }
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      float f[V], g[V];
      E::unpack(xv[k], f);
      E::unpack(rv[k], g);
#pragma unroll
      for (int e = 0; e < V; ++e) f[e] += g[e];
      xv[k] = E::pack(f);
      const int vi = v0 + 256 * k;
      if (vi < vend) orow[vi] = xv[k];
    }
  }
#pragma unroll
  for (int k = 0; k < NB; ++k) {
    const int vi = v0 + 256 * k;
    wv[k] = vi < vend ? wr[vi] : u32x4{0, 0, 0, 0};
  }
  float ss = 0.0f;
#pragma unroll
  for (int k = 0; k < NB; ++k) {
    float f[V];
    E::unpack(xv[k], f);
#pragma unroll
    for (int e = 0; e < V; ++e) ss = __builtin_fmaf(f[e], f[e], ss);
  }
  ss = block_sum(ss, red);
  if (threadIdx.x < 64) {   // one whole wavefront: the exchange
    const int lane = int(threadIdx.x);
    float sum = __builtin_nanf("");
    if (scratch[0] == 0) {
      if (lane == 0)
        __hip_atomic_store(&slots[s], kSlotFull | __float_as_uint(ss), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
      bool have = lane >= S;
      float part = 0.0f;
      bool late = false;
      for (int it = 0;; ++it) {
        if (!have) {
          const uint64_t w = __hip_atomic_load(&slots[lane], __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
          if (w & kSlotFull) {
            have = true;
            part = __uint_as_float(uint32_t(w));
          }
        }
        if (__all(have)) break;
        if (it >= kSplitSpinMax) {
          late = true;
          break;
        }
        __builtin_amdgcn_s_sleep(1);
      }
      sum = wave_sum(part);
      if (lane == 0) {
        if (late) {
          sum = __builtin_nanf("");
          __hip_atomic_store(&scratch[0], uint64_t(1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        const uint64_t c = __hip_atomic_fetch_add(count, uint64_t(1), __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT);
        if (c == uint64_t(S) - 1) {   // the row's last reader: clear for the next call
          for (int j = 0; j < S; ++j)
            __hip_atomic_store(&slots[j], uint64_t(0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          __hip_atomic_store(count, uint64_t(0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
    }
    if (lane == 0) total = sum;
  }
  __syncthreads();
  const float inv = rsqrtf(total / float(a.H) + a.eps);
  u32x4 *yr = reinterpret_cast<u32x4 *>(static_cast<char *>(a.y) + row * a.y_rs * E::ES);
#pragma unroll
  for (int k = 0; k < NB; ++k) {
    const int vi = v0 + 256 * k;
    if (vi < vend) {
      float f[V], w[V];
      E::unpack(xv[k], f);
      E::unpack(wv[k], w);
#pragma unroll
      for (int e = 0; e < V; ++e) f[e] = (f[e] * inv) * w[e];
      yr[vi] = E::pack(f);
    }
  }
}

// Vectors a work-item keeps in flight in the long-row kernels' streaming
// passes (one 16-byte load each, all issued before any is used).
constexpr int kRnBatch = 8;

// Long rows: two passes over global memory with float64 accumulation (each
// thread sums up to H/256 elements, so a float32 running sum would lose
// accuracy at the largest H). Vector form (16-byte aligned rows). Both passes
// keep kRnBatch vectors per work-item in flight; pass 2 re-reads x (or h from
// res_out: the thread's own writes).
template <int DT, bool RES>
__device__ __forceinline__ void rn_loop_row(const RnArgs &a, int64_t row, double *red) {
  using E = Elt<DT>;
  constexpr int V = E::V;
  constexpr int B = kRnBatch;
  const int nvec = a.H / V;
  const u32x4 *xr = reinterpret_cast<const u32x4 *>(static_cast<const char *>(a.x) +
                                                     row * a.x_rs * E::ES);
  const u32x4 *src = xr;
  double ss = 0.0;
  if constexpr (RES) {
    const u32x4 *rr = reinterpret_cast<const u32x4 *>(static_cast<const char *>(a.res) +
                                                       row * a.res_rs * E::ES);
    u32x4 *orow = reinterpret_cast<u32x4 *>(static_cast<char *>(a.res_out) + row * a.ro_rs * E::ES);
    for (int base = threadIdx.x; base < nvec; base += kThreads * B) {
      u32x4 xv[B], rv[B];
#pragma unroll
      for (int k = 0; k < B; ++k) {
        const int vi = base + k * kThreads;
        if (vi < nvec) {
          xv[k] = xr[vi];
          rv[k] = rr[vi];
        }
      }
#pragma unroll
      for (int k = 0; k < B; ++k) {
        const int vi = base + k * kThreads;
        if (vi < nvec) {
          float f[V], g[V];
          E::unpack(xv[k], f);
          E::unpack(rv[k], g);
#pragma unroll
          for (int e = 0; e < V; ++e) f[e] += g[e];
          const u32x4 h = E::pack(f);
          orow[vi] = h;
          E::unpack(h, f);
#pragma unroll
          for (int e = 0; e < V; ++e) ss += double(f[e]) * double(f[e]);
        }
      }
    }
    src = orow;
  } else {
    for (int base = threadIdx.x; base < nvec; base += kThreads * B) {
      u32x4 xv[B];
#pragma unroll
      for (int k = 0; k < B; ++k) {
        const int vi = base + k * kThreads;
        if (vi < nvec) xv[k] = xr[vi];
      }
#pragma unroll
      for (int k = 0; k < B; ++k) {
        const int vi = base + k * kThreads;
        if (vi < nvec) {
          float f[V];
          E::unpack(xv[k], f);
#pragma unroll
          for (int e = 0; e < V; ++e) ss += double(f[e]) * double(f[e]);
        }
      }
    }
  }
  ss = block_sum(ss, red);
  const float inv = float(1.0 / sqrt(ss / double(a.H) + double(a.eps)));
  const u32x4 *wr = static_cast<const u32x4 *>(a.w);
  u32x4 *yr = reinterpret_cast<u32x4 *>(static_cast<char *>(a.y) + row * a.y_rs * E::ES);
  for (int base = threadIdx.x; base < nvec; base += kThreads * B) {
    u32x4 hv[B], wv[B];
#pragma unroll
    for (int k = 0; k < B; ++k) {
      const int vi = base + k * kThreads;
      if (vi < nvec) {
        hv[k] = src[vi];
        wv[k] = wr[vi];
      }
    }
#pragma unroll
    for (int k = 0; k < B; ++k) {
      const int vi = base + k * kThreads;
      if (vi < nvec) {
        float f[V], w[V];
        E::unpack(hv[k], f);
        E::unpack(wv[k], w);
#pragma unroll
        for (int e = 0; e < V; ++e) f[e] = (f[e] * inv) * w[e];
        yr[vi] = E::pack(f);
      }
    }
  }
}

// A row of any length that starts at any element, held by one workgroup
// (LANES = 256) or one wavefront (LANES = 64, no barrier): lane t owns vectors
// t, t + LANES, ... (NV of them) and, past the last whole vector, element
// nvec * V + t. The row is read once; the sum is
// float64, as in the two-pass form. Up to two vectors per work-item the
// weights are requested with the row (one memory round trip). Beyond that
// the residual and, after the reduction, the weights are taken two or four
// vectors at a time: the lane then stays within 64 registers, so that eight
// workgroups fit on a compute unit and their rows' loads, reductions and
// stores overlap.
template <int DT, int NV, bool RES, int LANES, bool NT>
__device__ __forceinline__ void rn_any_regs(const RnArgs &a, int64_t row, double *red) {
  using E = Elt<DT>;
  using vec = typename AnyVec<DT>::type;
  constexpr int V = E::V;
  constexpr bool W0 = NV <= 2;
  constexpr int B = NV < 4 ? NV : (NV == 8 ? 2 : 4);   // residual vectors at a time
  constexpr int C = NV < 4 ? NV : 4;                    // weight vectors at a time
  const int nvec = a.H / V;
  const int tid = int(threadIdx.x) & (LANES - 1);
  const int te = nvec * V + tid;
  const bool tail = te < a.H;
  const vec *xr = reinterpret_cast<const vec *>(static_cast<const char *>(a.x) +
                                                row * a.x_rs * E::ES);
  const vec *wr = static_cast<const vec *>(a.w);
  u32x4 xv[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int vi = tid + LANES * k;
    xv[k] = vi < nvec ? ld_any<DT, NT>(xr + vi) : u32x4{0, 0, 0, 0};
  }
  float xt = tail ? E::ld(xr, te) : 0.0f;
  double rcp_h = 1.0 / double(a.H);   // while the row is under way
  asm volatile("" : "+v"(rcp_h));
  u32x4 wv[W0 ? NV : 1];
  if constexpr (RES) {
    const vec *rr = reinterpret_cast<const vec *>(static_cast<const char *>(a.res) +
                                                  row * a.res_rs * E::ES);
    vec *orow = reinterpret_cast<vec *>(static_cast<char *>(a.res_out) + row * a.ro_rs * E::ES);
    const float rt = tail ? E::ld(rr, te) : 0.0f;
#pragma unroll
    for (int k0 = 0; k0 < NV; k0 += B) {
      u32x4 rv[B];
#pragma unroll
      for (int k = 0; k < B; ++k) {
        const int vi = tid + LANES * (k0 + k);
        rv[k] = vi < nvec ? ld_any<DT, NT>(rr + vi) : u32x4{0, 0, 0, 0};
      }
      if constexpr (W0) {
#pragma unroll
        for (int k = 0; k < NV; ++k) {
          const int vi = tid + LANES * k;
          wv[k] = vi < nvec ? u32x4(wr[vi]) : u32x4{0, 0, 0, 0};
        }
      }
#pragma unroll
      for (int k = 0; k < B; ++k) {
        float f[V], g[V];
        E::unpack(xv[k0 + k], f);
        E::unpack(rv[k], g);
#pragma unroll
        for (int e = 0; e < V; ++e) f[e] += g[e];
        xv[k0 + k] = E::pack(f);
        const int vi = tid + LANES * (k0 + k);
        if (vi < nvec) orow[vi] = xv[k0 + k];
      }
      if constexpr (NV > B) asm volatile("" ::: "memory");   // the next ones after these
    }
    if (tail) {
      xt = E::round(xt + rt);
      E::st(orow, te, xt);
    }
  } else if constexpr (W0) {
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const int vi = tid + LANES * k;
      wv[k] = vi < nvec ? u32x4(wr[vi]) : u32x4{0, 0, 0, 0};
    }
  }
  const float wt = tail ? E::ld(a.w, te) : 0.0f;
  double acc[2] = {double(xt) * double(xt), 0.0};
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    float f[V];
    E::unpack(xv[k], f);
    add_squares<V>(acc, f);
    // the output pass unpacks again: the floats are not kept
    if constexpr (!W0) asm volatile("" : "+v"(xv[k]));
  }
  double ss = acc[0] + acc[1];
  if constexpr (LANES == 64)
    ss = wave_sum(ss);
  else
    ss = block_sum_once<LANES / 64>(ss, red);
  const float inv = inv_rms(ss, rcp_h, a.eps);
  vec *yr = reinterpret_cast<vec *>(static_cast<char *>(a.y) + row * a.y_rs * E::ES);
  if (tail) E::st(yr, te, (xt * inv) * wt);
#pragma unroll
  for (int k0 = 0; k0 < NV; k0 += C) {
    if constexpr (!W0) {
#pragma unroll
      for (int k = 0; k < C; ++k) {
        const int vi = tid + LANES * (k0 + k);
        if (vi < nvec) {
          float f[V], w[V];
          E::unpack(xv[k0 + k], f);
          E::unpack(u32x4(wr[vi]), w);
#pragma unroll
          for (int e = 0; e < V; ++e) f[e] = (f[e] * inv) * w[e];
          yr[vi] = E::pack(f);
        }
      }
      asm volatile("" ::: "memory");
    } else {
#pragma unroll
      for (int k = 0; k < NV; ++k) {
        const int vi = tid + LANES * k;
        if (vi < nvec) {
          float f[V], w[V];
          E::unpack(xv[k], f);
          E::unpack(wv[k], w);
#pragma unroll
          for (int e = 0; e < V; ++e) f[e] = (f[e] * inv) * w[e];
          yr[vi] = E::pack(f);
        }
      }
    }
  }
}

// A row of more than 8 LANES vectors that starts at any element: the first
// four vectors per work-item are held as in rn_any_regs, the rest are read
// (residual_out: written) in pass 1 and read again in pass 2, B at a time.
// Holding eight vectors, or taking four at a time, needs more than the 64
// registers that let two such workgroups share a compute unit. Bound by
// memory and, for a few rows, by the round trips of the passes: bf16 plain
// rows 607 x 86272 63.7 us against 71.9 in two passes by 256 work-items and
// 68.5 by 1024, f32 2 x 37001 6.3 against 9.7 and 7.4 us.
template <int DT, bool RES, int LANES, bool NT>
__device__ __forceinline__ void rn_any_long(const RnArgs &a, int64_t row, double *red) {
  using E = Elt<DT>;
  using vec = typename AnyVec<DT>::type;
  constexpr int V = E::V, NV = 4, B = 2;
  const int nvec = a.H / V;
  const int tid = int(threadIdx.x);
  const int te = nvec * V + tid;
  const bool tail = te < a.H;
  const vec *xr = reinterpret_cast<const vec *>(static_cast<const char *>(a.x) +
                                                row * a.x_rs * E::ES);
  const vec *rr = reinterpret_cast<const vec *>(static_cast<const char *>(a.res) +
                                                row * a.res_rs * E::ES);
  vec *orow = reinterpret_cast<vec *>(static_cast<char *>(a.res_out) + row * a.ro_rs * E::ES);
  u32x4 xv[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) xv[k] = ld_any<DT, NT>(xr + tid + LANES * k);
  double acc[2] = {0.0, 0.0};
  float xt = 0.0f;
  if (tail) {
    xt = E::ld(xr, te);
    if constexpr (RES) {
      xt = E::round(xt + E::ld(rr, te));
      E::st(orow, te, xt);
    }
    acc[0] = double(xt) * double(xt);
  }
  // h of vector vi from x and its residual, stored; its squares added
  auto take = [&](u32x4 &x, const u32x4 &r, int vi) {
    float f[V], g[V];
    E::unpack(x, f);
    if constexpr (RES) {
      E::unpack(r, g);
#pragma unroll
      for (int e = 0; e < V; ++e) f[e] += g[e];
      x = E::pack(f);
      orow[vi] = x;
      E::unpack(x, f);
    }
    add_squares<V>(acc, f);
  };
#pragma unroll
  for (int k0 = 0; k0 < NV; k0 += B) {
    u32x4 rv[B];
#pragma unroll
    for (int k = 0; k < B; ++k)
      if constexpr (RES) rv[k] = ld_any<DT, NT>(rr + tid + LANES * (k0 + k));
#pragma unroll
    for (int k = 0; k < B; ++k) {
      take(xv[k0 + k], rv[k], tid + LANES * (k0 + k));
      asm volatile("" : "+v"(xv[k0 + k]));   // the output pass unpacks again
    }
    if constexpr (RES) asm volatile("" ::: "memory");
  }
  for (int base = NV * LANES + tid; base < nvec; base += LANES * B) {
    u32x4 sv[B], rv[B];
#pragma unroll
    for (int k = 0; k < B; ++k) {
      const int vi = base + k * LANES;
      if (vi < nvec) {
        sv[k] = ld_any<DT, NT>(xr + vi);
        if constexpr (RES) rv[k] = ld_any<DT, NT>(rr + vi);
      }
    }
#pragma unroll
    for (int k = 0; k < B; ++k) {
      const int vi = base + k * LANES;
      if (vi < nvec) take(sv[k], rv[k], vi);
    }
  }
  const double rcp_h = 1.0 / double(a.H);
  const float inv = inv_rms(block_sum_once<LANES / 64>(acc[0] + acc[1], red), rcp_h, a.eps);
  const vec *wr = static_cast<const vec *>(a.w);
  const vec *src = RES ? orow : xr;
  vec *yr = reinterpret_cast<vec *>(static_cast<char *>(a.y) + row * a.y_rs * E::ES);
  if (tail) E::st(yr, te, (xt * inv) * E::ld(a.w, te));
  auto put = [&](const u32x4 &h, const u32x4 &wv, int vi) {
    float f[V], w[V];
    E::unpack(h, f);
    E::unpack(wv, w);
#pragma unroll
    for (int e = 0; e < V; ++e) f[e] = (f[e] * inv) * w[e];
    yr[vi] = E::pack(f);
  };
  for (int base = NV * LANES + tid; base < nvec; base += LANES * B) {
    u32x4 sv[B], wv[B];
#pragma unroll
    for (int k = 0; k < B; ++k) {
      const int vi = base + k * LANES;
      if (vi < nvec) {
        sv[k] = src[vi];
        wv[k] = wr[vi];
      }
    }
#pragma unroll
    for (int k = 0; k < B; ++k) {
      const int vi = base + k * LANES;
      if (vi < nvec) put(sv[k], wv[k], vi);
    }
  }
#pragma unroll
  for (int k0 = 0; k0 < NV; k0 += B) {
#pragma unroll
    for (int k = 0; k < B; ++k) {
      const int vi = tid + LANES * (k0 + k);
      put(xv[k0 + k], u32x4(wr[vi]), vi);
    }
    asm volatile("" ::: "memory");
  }
}

// Rows that are not 16-byte aligned or not whole vectors; the launch has a
// workgroup per row. In registers (the fewest that hold the row) up to 2048
// vectors on 256 work-items and 8192 on 1024, two passes beyond. Rows of up to
// 256 vectors take one wavefront each, four to a workgroup, once there are more
// rows than workgroups fit on the chip (eight per compute unit): all rows then
// run at once and no lane waits at a barrier; with fewer rows a workgroup per
// row has them done sooner. (The launch's other workgroups have no row and end.)
//
// Bound by memory: bf16 residual rows of 1536 x 4097 take 10.1 us (5.0 TB/s),
// against 15.7 us for element-wise accesses in two passes (10.7 us where a
// lane of up to 94 registers left five workgroups to a compute unit);
// 512 x 4096 one element off a 16-byte boundary 5.4 against 12.4 us; plain
// rows of 6198 x 1139 8.3 against 15.3 us (9.3 us with a workgroup per row and
// the library's float64 division and square root). Rows of more than 2048
// vectors on 256 work-items passed twice over memory with too few loads in
// flight: bf16 plain rows of 52,352 went from 12.5 to 7.3 us (21 of them) and
// from 33.6 to 28.3 us (607), residual ones from 14.8 to 11.9 and 66.8 to 55.0.
// Below 2048 vectors 1024 work-items gain nothing.
template <int DT, bool RES, bool NT>
__device__ __forceinline__ void rn_any_row(const RnArgs &a, int64_t row, double *red) {
  const int nvec = a.H / Elt<DT>::V;
  if (nvec <= 256 && a.T > kAnyBlockRows) {
    row = row * 4 + (threadIdx.x >> 6);
    if (row >= a.T) return;
    if (nvec <= 64)
      rn_any_regs<DT, 1, RES, 64, NT>(a, row, red);
    else if (nvec <= 128)
      rn_any_regs<DT, 2, RES, 64, NT>(a, row, red);
    else
      rn_any_regs<DT, 4, RES, 64, NT>(a, row, red);
  } else if (nvec <= kThreads)
    rn_any_regs<DT, 1, RES, kThreads, NT>(a, row, red);
  else if (nvec <= 2 * kThreads)
    rn_any_regs<DT, 2, RES, kThreads, NT>(a, row, red);
  else if (nvec <= 4 * kThreads)
    rn_any_regs<DT, 4, RES, kThreads, NT>(a, row, red);
  else if (nvec <= kAnyBlockVecs)
    rn_any_regs<DT, 8, RES, kThreads, NT>(a, row, red);
  else if (nvec <= 4 * kWideLanes)
    rn_any_regs<DT, 4, RES, kWideLanes, NT>(a, row, red);
  else if (nvec <= 8 * kWideLanes)
    rn_any_regs<DT, 8, RES, kWideLanes, NT>(a, row, red);
  else
    rn_any_long<DT, RES, kWideLanes, NT>(a, row, red);
}

// ---- RoPE ---------------------------------------------------------------------
// Angles: theta = float(pos) * inv_i (one float32 product; int64 positions
// convert with one rounding) and cos / sin of it, or cos / sin read from the
// caller's cache row min(max(pos, 0), cs_len - 1). They are computed once per
// (token, pair) into LDS; every head of the token reuses them.
__device__ __forceinline__ int64_t rope_pos(const RopeArgs &a, int64_t t) {
  return (a.mode & kRopePos64) ? static_cast<const int64_t *>(a.pos)[t]
                               : int64_t(static_cast<const int32_t *>(a.pos)[t]);
}

__device__ __forceinline__ void rope_cos_sin(const RopeArgs &a, int64_t t, int i, float &c,
                                             float &s) {
  const int64_t p = rope_pos(a, t);
  if (a.mode & kRopeCache) {
    const int64_t r = p < 0 ? 0 : (p >= a.cs_len ? a.cs_len - 1 : p);
    const float *row = a.cos_sin + r * a.rd;
    c = row[i];
    s = row[(a.rd >> 1) + i];
  } else {
    sincosf(float(p) * a.inv_freq[i], &s, &c);
  }
}

// The rotation of a pair (x, y) by (c, s): x c - y s and y c + x s, each one
// fused multiply-add on a rounded product (device code is compiled without
// contraction, so these are the only fused operations and their rounding
// does not depend on the surrounding code).
__device__ __forceinline__ float rot_a(float x, float y, float c, float s) {
  return __builtin_fmaf(x, c, -(y * s));
}
__device__ __forceinline__ float rot_b(float x, float y, float c, float s) {
  return __builtin_fmaf(y, c, x * s);
}

// Heads hg, hg + hstep, ... of ntok tokens from t on (all Q and K heads of the
// first token, then of the second, ...) by the group of cpb lanes of which
// this lane is number `chunk` (see rope_vec_block). With one token (MULTI
// false) it is the same for the whole workgroup, so its row addresses and its
// position are scalar work and a lane adds one 32-bit offset. PF heads are
// requested at a time, the first ones before the angle math and the barrier,
// with the angle operands ahead of them.
//
// Bound by latency at decode sizes: with 64-bit addresses per head and four
// heads requested where a group has one, some 250 instructions preceded the
// last load. 8 one-token chains 18.9 -> 16.9 us, 32 captured 8-token chains
// 96.9 -> 90.0 us, the 512-token GQA chain 12.3 -> 11.8 us. Two heads at a time
// beyond decode sizes: four cost 107 instead of 69 registers a lane. With the
// QK norm one: two cost 90-110 instead of 75-83, and at decode sizes a group
// has one (eight 48-token chains 33.7 -> 32.7 us; 2048 tokens alone
// 9.98 -> 9.61 us, 8192 tokens after a flush 0.74 -> 0.765 of 8 TB/s); the
// streaming form, which has wavefronts enough to cover their latency, asks for
// the weights after the reduction: 61 registers and eight wavefronts per SIMD
// instead of 75 and six. Several tokens are spread over all groups: with the second token's heads left to
// the first one's groups, four 308-token chains of 16 heads took 24.6 us, now
// 23.5, and 8192 tokens of 9 heads with their norm and SwiGLU 130.4, now 122.7.
template <int DT, bool NT, int PF, bool QKN, bool INTER, bool MULTI>
__device__ __forceinline__ void rope_tokens_block(const RopeArgs &a, int64_t t, int ntok, int chunk,
                                                  int cpb, int hg, int hstep, float *lds) {
  using E = Elt<DT>;
  constexpr int V = E::V;
  const int P2 = a.rd >> 1;
  const int nh = a.nq + a.nk;
  const int off2 = P2 * E::ES;
  const int tid = int(threadIdx.x);
  float *cs = lds, *sn = lds + kRopeTokensMax * 256;

  const int n = MULTI ? ntok * nh : nh;         // heads of the workgroup
  const int na = MULTI ? ntok * P2 : P2;        // angles
  const int ia = MULTI ? tid & (P2 - 1) : tid;  // P2 is a power of two
  const bool ang = tid < na;
  float c = 1.0f, s = 0.0f, p = 0.0f;
  if (ang) {
    const int64_t pos = rope_pos(a, MULTI ? t + (tid >> __builtin_ctz(unsigned(P2))) : t);
    if (a.mode & kRopeCache) {
      const int64_t r = pos < 0 ? 0 : (pos >= a.cs_len ? a.cs_len - 1 : pos);
      const float *row = a.cos_sin + r * a.rd;
      c = row[ia];
      s = row[P2 + ia];
    } else {
      p = (a.mode & kRopePos64) ? float(pos) : float(int32_t(pos));
      c = a.inv_freq[ia];
    }
  }

  // Q heads 0 .. nq - 1, K heads nq .. nh - 1 at one stride from kb
  char *qb = static_cast<char *>(a.q) + t * a.q_ts * E::ES;
  char *kb = static_cast<char *>(a.k) + (t * a.k_ts - int64_t(a.nq) * a.hd) * E::ES;
  const uint32_t hbytes = uint32_t(a.hd * E::ES), cbytes = uint32_t(chunk) * 16u;
  // the i-th head of the workgroup: its token and number
  auto token_of = [&](int i) { return MULTI ? int(uint32_t(i) / uint32_t(nh)) : 0; };
  auto head = [&](int tt, int h) {
    char *b = (h < a.nq ? qb : kb) + (uint32_t(h) * hbytes + cbytes);
    if constexpr (MULTI) b += int64_t(tt) * (h < a.nq ? a.q_ts : a.k_ts) * E::ES;
    return b;
  };
  u32x4 x1[PF], x2[PF], w1[QKN ? PF : 1], w2[QKN ? PF : 1];
  auto weights = [&](int j, int h) {   // the head's chunk of the Q or K weights
    const char *w = static_cast<const char *>(h < a.nq ? a.qw : a.kw) + cbytes;
    w1[j] = *reinterpret_cast<const u32x4 *>(w);
    if constexpr (!INTER) w2[j] = *reinterpret_cast<const u32x4 *>(w + off2);
  };
  auto gather = [&](int h0) {
#pragma unroll
    for (int j = 0; j < PF; ++j) {
      const int i = h0 + j * hstep;
      if (i < n) {
        const int tt = token_of(i);
        const char *b = head(tt, i - tt * nh);
        x1[j] = ld16<NT>(reinterpret_cast<const u32x4 *>(b));
        if constexpr (!INTER) x2[j] = ld16<NT>(reinterpret_cast<const u32x4 *>(b + off2));
        if constexpr (QKN && !NT) weights(j, i - tt * nh);
      }
    }
  };
  gather(hg);

  if (ang) {
    if (!(a.mode & kRopeCache)) {
      const float inv = c;
      sincosf(p * inv, &s, &c);
    }
    cs[tid] = c;
    sn[tid] = s;
  }
  if constexpr (MULTI) {
    for (int e = tid + kThreads; e < na; e += kThreads) {
      rope_cos_sin(a, t + (e >> __builtin_ctz(unsigned(P2))), e & (P2 - 1), c, s);
      cs[e] = c;
      sn[e] = s;
    }
  }
  __syncthreads();

  for (int h0 = hg; h0 < n;) {
#pragma unroll
    for (int j = 0; j < PF; ++j) {
      const int i = h0 + j * hstep;
      if (i >= n) continue;   // uniform over the lanes of a head group
      const int tt = token_of(i), h = i - tt * nh;
      float f1[V], f2[V];
      E::unpack(x1[j], f1);
      if constexpr (!INTER) E::unpack(x2[j], f2);
      if constexpr (QKN) {
        float ss = 0.0f;
#pragma unroll
        for (int e = 0; e < V; ++e) ss = __builtin_fmaf(f1[e], f1[e], ss);
        if constexpr (!INTER) {
#pragma unroll
          for (int e = 0; e < V; ++e) ss = __builtin_fmaf(f2[e], f2[e], ss);
        }
        ss = group_sum(ss, cpb);
        const float inv = rsqrtf(ss / float(a.hd) + a.eps);
        if constexpr (NT) weights(j, h);
        float w[V];
        E::unpack(w1[j], w);
#pragma unroll
        for (int e = 0; e < V; ++e) f1[e] = (f1[e] * inv) * w[e];
        if constexpr (!INTER) {
          E::unpack(w2[j], w);
#pragma unroll
          for (int e = 0; e < V; ++e) f2[e] = (f2[e] * inv) * w[e];
        }
      }
      char *b = head(tt, h);
      if constexpr (INTER) {
        const int base = tt * P2 + ((chunk * V) >> 1);
        float o[V];
#pragma unroll
        for (int e = 0; e < V; e += 2) {
          const float ce = cs[base + (e >> 1)], se = sn[base + (e >> 1)];
          o[e] = rot_a(f1[e], f1[e + 1], ce, se);
          o[e + 1] = rot_b(f1[e], f1[e + 1], ce, se);
        }
        st16<NT>(reinterpret_cast<u32x4 *>(b), E::pack(o));
      } else {
        const int base = tt * P2 + chunk * V;
        float o1[V], o2[V];
#pragma unroll
        for (int e = 0; e < V; ++e) {
          const float ce = cs[base + e], se = sn[base + e];
          o1[e] = rot_a(f1[e], f2[e], ce, se);
          o2[e] = rot_b(f1[e], f2[e], ce, se);
        }
        st16<NT>(reinterpret_cast<u32x4 *>(b), E::pack(o1));
        st16<NT>(reinterpret_cast<u32x4 *>(b + off2), E::pack(o2));
      }
    }
    h0 += PF * hstep;
    if (h0 < n) gather(h0);
  }
}

// tpb tokens per workgroup (mode bits 16..23, at most kRopeTokensMax; `lds`
// holds 2 * 256 * kRopeTokensMax floats); with one token per workgroup a
// token's heads may instead be split round-robin over S = slices workgroups
// (mode bits 8..15: workgroup blk takes token blk / S and heads s, s + S,
// s + 2S, ... with s = blk % S). P2 = rd/2 angle
// pairs per token (a power of two). Rotate-half (INTER false): each half of the rotated span is
// cpb = P2/V 16-byte vectors and a work-item holds chunk c of both halves;
// GPT-J pairs (INTER true): the span is cpb = rd/V vectors of V/2 adjacent
// pairs each and a work-item holds one. Work-item `tid` owns chunk tid % cpb
// of heads tid / cpb, tid / cpb + 256 / cpb, ... of the block's tokens,
// numbered through. A group's heads are processed PF at a time (one where the
// workgroup has no more heads than groups, as the slices and the tokens of a
// workgroup are chosen for) with all loads issued before any use, and the
// first batch is requested before the angle math and the barrier, so at
// decode sizes the block costs one memory round trip. Elements past rd are
// not touched.
//
// QKN (requires rd == hd): each head is first RMS-normalised over its hd
// elements with the Q or K head-norm weight. The cpb work-items of a head
// hold the whole head in registers, so the sum of squares is a reduction
// over cpb adjacent lanes and the head is read and written once. Whether an
// item is valid depends only on the work-item's head group, so the lanes of
// a group skip or process an item together and every lane a reduction reads
// from is active. cpb <= 64 (the policy guarantees it).
template <int DT, bool NT, int PF = 2, bool QKN = false, bool INTER = false>
__device__ __forceinline__ void rope_vec_block(const RopeArgs &a, int64_t blk, float *lds) {
  constexpr int V = Elt<DT>::V;
  const int cpb = (INTER ? a.rd : a.rd >> 1) / V;
  const int shift = __builtin_ctz(unsigned(cpb));
  const int chunk = threadIdx.x & (cpb - 1);
  const int nh = a.nq + a.nk;
  const int tb = int((a.mode >> kRopeTokensShift) & 0xFFu);
  const int tpb = tb < 1 ? 1 : (tb > kRopeTokensMax ? kRopeTokensMax : tb);
  const int g = int(threadIdx.x >> shift), ng = kThreads >> shift;
  if (tpb == 1) {
    const int sb = int((a.mode >> kRopeSliceShift) & 0xFFu);
    const int S = sb > 1 ? sb : 1;
    const int64_t t = S > 1 ? blk / S : blk;
    const int hg = int(blk - t * S) + S * g, hstep = S * ng;
    if (PF > 1 && hstep >= nh)
      rope_tokens_block<DT, NT, 1, QKN, INTER, false>(a, t, 1, chunk, cpb, hg, hstep, lds);
    else
      rope_tokens_block<DT, NT, PF, QKN, INTER, false>(a, t, 1, chunk, cpb, hg, hstep, lds);
  } else {
    const int64_t t = blk * tpb;
    const int64_t left = a.T - t;
    const int ntok = left < tpb ? int(left) : tpb;
    if (PF > 1 && ng >= tpb * nh)
      rope_tokens_block<DT, NT, 1, QKN, INTER, true>(a, t, ntok, chunk, cpb, g, ng, lds);
    else
      rope_tokens_block<DT, NT, PF, QKN, INTER, true>(a, t, ntok, chunk, cpb, g, ng, lds);
  }
}

// m elements (whole vectors: m >= V) at element e of a head that starts at any
// element; zeros past them.
template <int DT>
__device__ __forceinline__ u32x4 ld_part(const char *head, int e, int m) {
  using E = Elt<DT>;
  const char *p = head + e * E::ES;
  if (m >= E::V) return *reinterpret_cast<const typename AnyVec<DT>::type *>(p);
  float f[E::V];
#pragma unroll
  for (int i = 0; i < E::V; ++i) f[i] = i < m ? E::ld(p, i) : 0.0f;
  return E::pack(f);   // exact: the floats came from elements
}
template <int DT>
__device__ __forceinline__ void st_part(char *head, int e, int m, const float *f) {
  using E = Elt<DT>;
  char *p = head + e * E::ES;
  if (m >= E::V) {
    *reinterpret_cast<typename AnyVec<DT>::type *>(p) = E::pack(f);
  } else {
#pragma unroll
    for (int i = 0; i < E::V - 1; ++i)
      if (i < m) E::st(p, i, f[i]);
  }
}

// Any alignment, head size and variant: one token per workgroup, `lds` holds
// 2 * 256 floats (cos, sin). As in rope_vec_block a group of lanes takes a
// head, one chunk of V elements each (of both halves, rotate-half; of V / 2
// adjacent pairs, INTER), but the chunks of a head need not be a power of
// two, whole or aligned: a group is the next power of two of lanes, of which
// the last ones may have no chunk, the last chunk may be short, and accesses
// are element-aligned. PF heads per group are requested before the angle
// math and the barrier.
//
// QKN: the group sums the squares of its head, so a group is at most 64
// lanes; chunks beyond that (float32, INTER, more than 256 elements) and the
// elements past rd, which are normalised only, are read again after the sum.
// A group has lanes enough for eight chunks of those each: with the lanes of
// the rotated chunks only, one lane would take a head of 512 with rd = 8 alone.
// A lane's squares go to four float32 chains, and the lanes' sums join in
// float64: no further from the exact sum than a wavefront per head, whose
// lanes hold at most eight squares each (rms of the relative error of heads
// of 64-512: 0.42-0.57 of 2^-24 against 0.63-0.72; one float32 chain and a
// float32 group sum had 0.70-0.80, 2.7 at 512 with rd = 64 and 17 with rd = 8).
// That costs 2048 tokens of 40 heads of 96 0.2 us of 9.2 (bf16).
//
// Bound by memory latency and the lanes that a group leaves idle: 2048
// tokens of 64 heads of 96 (bf16, six of eight lanes) take 9.7 us (5.3 TB/s),
// against 14.8 us with one element pair per work-item and a division each;
// 512 tokens of 64 heads of 128 one element off a 16-byte boundary 4.8 us,
// against 7.9 us. Held to 64 registers for eight workgroups per compute unit it
// spills and takes 15.3 us.
template <int DT, bool QKN, bool INTER, int PF = 2>
__device__ __forceinline__ void rope_any_block(const RopeArgs &a, int64_t t, float *lds) {
  using E = Elt<DT>;
  constexpr int V = E::V;
  const int P2 = a.rd >> 1;
  const int span = INTER ? a.rd : P2;
  const int pass = QKN ? a.hd - a.rd : 0;
  int cpb = (span + V - 1) / V;
  if (QKN && pass > 8 * V * cpb) cpb = (pass + 8 * V - 1) / (8 * V);
  int lg = cpb > 1 ? 32 - __builtin_clz(unsigned(cpb - 1)) : 0;
  if (QKN && lg > 6) lg = 6;
  const int G = 1 << lg;
  const int lane = int(threadIdx.x) & (G - 1);
  const int hg = int(threadIdx.x) >> lg, hstep = kThreads >> lg;
  const int nh = a.nq + a.nk;
  const int e0 = lane * V;
  const int m = span - e0;               // elements of this lane's chunk (idle: <= 0)
  float *cs = lds, *sn = lds + 256;

  // the angle operands of pair threadIdx.x, ahead of the heads
  const bool ang = int(threadIdx.x) < P2;
  float c = 1.0f, s = 0.0f;
  int64_t pos = 0;
  if (ang) {
    pos = rope_pos(a, t);
    if (a.mode & kRopeCache) {
      const int64_t r = pos < 0 ? 0 : (pos >= a.cs_len ? a.cs_len - 1 : pos);
      const float *row = a.cos_sin + r * a.rd;
      c = row[threadIdx.x];
      s = row[P2 + threadIdx.x];
    } else {
      c = a.inv_freq[threadIdx.x];
    }
  }

  // one token: scalar row addresses and a 32-bit offset per head
  char *qb = static_cast<char *>(a.q) + t * a.q_ts * E::ES;
  char *kb = static_cast<char *>(a.k) + (t * a.k_ts - int64_t(a.nq) * a.hd) * E::ES;
  const uint32_t hbytes = uint32_t(a.hd * E::ES);
  auto head = [&](int h) { return (h < a.nq ? qb : kb) + uint32_t(h) * hbytes; };
  auto weights = [&](int h) { return static_cast<const char *>(h < a.nq ? a.qw : a.kw); };

  u32x4 x1[PF], x2[PF], w1[QKN ? PF : 1], w2[QKN ? PF : 1];
  auto gather = [&](int h) {
#pragma unroll
    for (int j = 0; j < PF; ++j) {
      x1[j] = x2[j] = u32x4{0, 0, 0, 0};
      if (m > 0 && h + j * hstep < nh) {
        const char *b = head(h + j * hstep);
        x1[j] = ld_part<DT>(b, e0, m);
        if constexpr (!INTER) x2[j] = ld_part<DT>(b, P2 + e0, m);
        if constexpr (QKN) {
          const char *w = weights(h + j * hstep);
          w1[j] = ld_part<DT>(w, e0, m);
          if constexpr (!INTER) w2[j] = ld_part<DT>(w, P2 + e0, m);
        }
      }
    }
  };
  gather(hg);

  if (ang) {
    if (!(a.mode & kRopeCache)) {
      const float inv = c;
      sincosf(float(pos) * inv, &s, &c);
    }
    cs[threadIdx.x] = c;
    sn[threadIdx.x] = s;
  }
  __syncthreads();

  // normalise (QKN) and rotate the chunk at element e of the span
  auto rotate = [&](char *b, int e, int n, float *f1, float *f2, float inv, const u32x4 &h1,
                    const u32x4 &h2) {
    if constexpr (QKN) {
      float w[V];
      E::unpack(h1, w);
#pragma unroll
      for (int i = 0; i < V; ++i) f1[i] = (f1[i] * inv) * w[i];
      if constexpr (!INTER) {
        E::unpack(h2, w);
#pragma unroll
        for (int i = 0; i < V; ++i) f2[i] = (f2[i] * inv) * w[i];
      }
    }
    float o1[V], o2[V];
    if constexpr (INTER) {
#pragma unroll
      for (int i = 0; i < V; i += 2) {
        const float ci = cs[(e + i) >> 1], si = sn[(e + i) >> 1];
        o1[i] = rot_a(f1[i], f1[i + 1], ci, si);
        o1[i + 1] = rot_b(f1[i], f1[i + 1], ci, si);
      }
      st_part<DT>(b, e, n, o1);
    } else {
#pragma unroll
      for (int i = 0; i < V; ++i) {
        const float ci = cs[e + i], si = sn[e + i];
        o1[i] = rot_a(f1[i], f2[i], ci, si);
        o2[i] = rot_b(f1[i], f2[i], ci, si);
      }
      st_part<DT>(b, e, n, o1);
      st_part<DT>(b, P2 + e, n, o2);
    }
  };

  for (int h0 = hg; h0 < nh; h0 += PF * hstep) {
    if (h0 != hg) gather(h0);
#pragma unroll
    for (int j = 0; j < PF; ++j) {
      const int h = h0 + j * hstep;
      if (h >= nh) continue;              // uniform over a group
      char *b = head(h);
      float f1[V], f2[V];
      E::unpack(x1[j], f1);
      E::unpack(x2[j], f2);
      float inv = 1.0f;
      const char *hw = nullptr;
      if constexpr (QKN) {
        hw = weights(h);
        float sq[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        auto squares = [&](const float *f) {
#pragma unroll
          for (int i = 0; i < V; ++i) sq[i & 3] = __builtin_fmaf(f[i], f[i], sq[i & 3]);
        };
        squares(f1);
        if constexpr (!INTER) squares(f2);
        auto add = [&](int e, int n) {
          float f[V];
          E::unpack(ld_part<DT>(b, e, n), f);
          squares(f);
        };
        if constexpr (INTER)
          for (int e = e0 + G * V; e < span; e += G * V) add(e, span - e);
        for (int e = e0; e < pass; e += G * V) add(a.rd + e, pass - e);
        const double ss = group_sum(double((sq[0] + sq[1]) + (sq[2] + sq[3])), G);
        inv = rsqrtf(float(ss) / float(a.hd) + a.eps);
      }
      if (m > 0) {
        rotate(b, e0, m, f1, f2, inv, w1[QKN ? j : 0], w2[QKN ? j : 0]);
      }
      if constexpr (QKN) {
        if constexpr (INTER) {
          for (int e = e0 + G * V; e < span; e += G * V) {
            const u32x4 w = ld_part<DT>(hw, e, span - e);
            E::unpack(ld_part<DT>(b, e, span - e), f1);
            rotate(b, e, span - e, f1, f2, inv, w, w);
          }
        }
        for (int e = e0; e < pass; e += G * V) {
          float w[V];
          E::unpack(ld_part<DT>(b, a.rd + e, pass - e), f1);
          E::unpack(ld_part<DT>(hw, a.rd + e, pass - e), w);
#pragma unroll
          for (int i = 0; i < V; ++i) f1[i] = (f1[i] * inv) * w[i];
          st_part<DT>(b, a.rd + e, pass - e, f1);
        }
      }
    }
  }
}

// ---- SwiGLU ----------------------------------------------------------------------
// silu(g) = g / (1 + exp(-g)), evaluated as g * rcp(1 + exp(-g)) with the
// hardware reciprocal (v_rcp_f32, 1 ulp): the correctly rounded float32
// division costs about ten vector instructions per element, which made the
// streaming SwiGLU and silu kernels bound by vector ALU throughput rather
// than by HBM. Below g = -80, 1 + exp(g) is 1 in float32 and silu(g) is
// g * exp(g); that form keeps the tail where exp(-g) overflows (from
// g = -88.7 on) and would flush the product to zero although the value is
// still a normal float32 down to about g = -91.5. At g = -inf the tail gives
// -inf * 0 = NaN, as -inf / (1 + inf) does.
//
// exp(-g) itself is 2^th * 2^tl with th = RN(-g * hi), tl = the rest of
// -g * log2(e) (an fma recovers the product's rounding error, lo carries
// log2(e) - hi), and 2^tl = 1 + tl ln 2 to first order (|tl| < 2^-17): the
// hardware exp2 (v_exp_f32, 1 ulp) and four more instructions instead of
// the library expf's range reduction. The relative error of silu stays
// below 2.4e-7 for |g| <= 80 (checked against the float64 value over
// 3 million arguments, as expf's form gives 1.9e-7). g is capped at 100 for
// the exponent (exp(-100) is far below float32's resolution next to 1), which
// keeps th and tl finite at g = +inf, where silu is +inf; v_med3_f32 caps
// without the quieting instruction that fminf takes first.
__device__ __forceinline__ float silu_main(float g) {
  constexpr float kLog2eHi = 1.44269502162933349609375f;   // RN_f32(log2 e)
  constexpr float kLog2eLo = 1.925963e-08f;                // log2 e - kLog2eHi
  constexpr float kLn2 = 0.693147180559945309f;
  const float ng = -__builtin_amdgcn_fmed3f(g, -3.402823466e+38f, 100.0f);
  const float th = ng * kLog2eHi;
  const float tl = __builtin_fmaf(ng, kLog2eHi, -th) + ng * kLog2eLo;
  const float e = __builtin_amdgcn_exp2f(th);
  return g * __builtin_amdgcn_rcpf(1.0f + __builtin_fmaf(e * tl, kLn2, e));
}

// silu of N elements in place. The tail is recomputed only where an element
// is in it (the sign and magnitude of the most negative one, as the largest
// unsigned bit pattern: one instruction for two elements), once for all N: a
// test and branch per element kept the elements' exp2 and rcp from
// overlapping, which at decode sizes, where SwiGLU's one wavefront per SIMD
// runs its instructions back to back, is on the chain's critical path (32
// captured 8-token chains 99.4 -> 96.9 us, 8 one-token chains 19.2 -> 18.9 us;
// silu of bf16 1024 x 4096 from Python 4.67 -> 4.48 us).
template <int N>
__device__ __forceinline__ void silu_all(float *g) {
  constexpr uint32_t kTail = 0xC2A00000u;   // the bits of -80
  float r[N];
  uint32_t low = 0;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    r[i] = silu_main(g[i]);
    const uint32_t b = __float_as_uint(g[i]);
    low = b > low ? b : low;
  }
  if (__builtin_expect(low > kTail, 0)) {
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (g[i] < -80.0f) r[i] = g[i] * expf(g[i]);
  }
#pragma unroll
  for (int i = 0; i < N; ++i) g[i] = r[i];
}

__device__ __forceinline__ float silu(float g) {
  silu_all<1>(&g);
  return g;
}

__device__ __forceinline__ float silu_mul(float g, float u) {
  return silu(g) * u;
}

// Flat contiguous [T*I]: workgroup `blk` of `nblk` handles U vectors per
// work-item per step; workgroup 0 also does the < V element tail.
template <int DT, int U, bool NT>
__device__ __forceinline__ void sw_flat_part(const SwArgs &a, int64_t blk, int64_t nblk) {
  using E = Elt<DT>;
  constexpr int V = E::V;
  const u32x4 *g = static_cast<const u32x4 *>(a.gate);
  const u32x4 *u = static_cast<const u32x4 *>(a.up);
  u32x4 *o = static_cast<u32x4 *>(a.out);
  const int64_t nvec = a.nvec;
  const int64_t step = nblk * kThreads * U;
  for (int64_t base = blk * kThreads * U + threadIdx.x; base < nvec; base += step) {
    u32x4 gv[U], uv[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int64_t idx = base + int64_t(k) * kThreads;
      if (idx < nvec) {
        gv[k] = ld16<NT>(g + idx);
        uv[k] = ld16<NT>(u + idx);
      }
    }
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int64_t idx = base + int64_t(k) * kThreads;
      if (idx < nvec) {
        float fg[V], fu[V];
        E::unpack(gv[k], fg);
        E::unpack(uv[k], fu);
        silu_all<V>(fg);
#pragma unroll
        for (int e = 0; e < V; ++e) fg[e] *= fu[e];
        st16<NT>(o + idx, E::pack(fg));
      }
    }
  }
  if (blk == 0) {
    const int64_t i = nvec * V + threadIdx.x;
    if (i < a.n) E::st(a.out, i, silu_mul(E::ld(a.gate, i), E::ld(a.up, i)));
  }
}

// Row-wise passes over [T, W]: a row is ceil(W / V) slots of V elements (the
// last one shorter when W is no whole number of vectors), and the slots of
// all rows are numbered through, so every lane of a workgroup has one
// whatever the row length. Rows that follow each other without a gap are one
// row of T * W elements. A work-item finds its row by one division, of 32
// bits unless there are more slots than that (a 64-bit division is about a
// hundred instructions, as much as the rest of a SwiGLU vector).
struct Slots {
  int64_t T, W, per_row, total;
};
template <int V>
__device__ __forceinline__ Slots make_slots(int64_t T, int64_t W, bool contiguous) {
  Slots s;
  s.T = contiguous ? 1 : T;
  s.W = contiguous ? T * W : W;
  s.per_row = (s.W + V - 1) / V;
  s.total = s.T * s.per_row;
  return s;
}
// Row and first element of slot `i`.
template <int V>
__device__ __forceinline__ void slot_at(const Slots &s, int64_t i, int64_t &row, int64_t &e0) {
  if (s.T == 1) {
    row = 0;
    e0 = i * V;
  } else if (s.total <= int64_t(0xFFFFFFFFu)) {
    const uint32_t r = uint32_t(i) / uint32_t(s.per_row);
    row = r;
    e0 = int64_t(uint32_t(i) - r * uint32_t(s.per_row)) * V;
  } else {
    row = i / s.per_row;
    e0 = (i - row * s.per_row) * V;
  }
}

// 16-byte access at element e of a row: aligned, or at any element (ANY).
template <int DT, bool ANY, bool NT>
__device__ __forceinline__ u32x4 ld_slot(const void *row, int64_t e) {
  const char *p = static_cast<const char *>(row) + e * Elt<DT>::ES;
  if constexpr (ANY)
    return ld_any<DT, NT>(p);
  else
    return ld16<NT>(reinterpret_cast<const u32x4 *>(p));
}
template <int DT, bool ANY, bool NT>
__device__ __forceinline__ void st_slot(void *row, int64_t e, const u32x4 &v) {
  char *p = static_cast<char *>(row) + e * Elt<DT>::ES;
  if constexpr (ANY)
    st_any<DT, NT>(p, v);
  else
    st16<NT>(reinterpret_cast<u32x4 *>(p), v);
}

// Rows with padded strides: aligned and whole vectors long, or of any start
// and length (ANY).
template <int DT, bool ANY, bool NT>
__device__ __forceinline__ void sw_slots(const SwArgs &a, int64_t blk, int64_t nblk) {
  using E = Elt<DT>;
  constexpr int V = E::V;
  const Slots sl = make_slots<V>(a.T, a.I, ANY && a.g_rs == a.I && a.u_rs == a.I && a.o_rs == a.I);
  for (int64_t i = blk * kThreads + threadIdx.x; i < sl.total; i += nblk * kThreads) {
    int64_t row, e0;
    slot_at<V>(sl, i, row, e0);
    const char *g = static_cast<const char *>(a.gate) + row * a.g_rs * E::ES;
    const char *u = static_cast<const char *>(a.up) + row * a.u_rs * E::ES;
    char *o = static_cast<char *>(a.out) + row * a.o_rs * E::ES;
    float fg[V], fu[V];
    if (!ANY || e0 + V <= sl.W) {
      const u32x4 gv = ld_slot<DT, ANY, NT>(g, e0), uv = ld_slot<DT, ANY, NT>(u, e0);
      E::unpack(gv, fg);
      E::unpack(uv, fu);
      silu_all<V>(fg);
#pragma unroll
      for (int e = 0; e < V; ++e) fg[e] *= fu[e];
      st_slot<DT, ANY, NT>(o, e0, E::pack(fg));
    } else {
      const int m = int(sl.W - e0);   // 1 .. V - 1
#pragma unroll
      for (int e = 0; e < V - 1; ++e) {
        fg[e] = e < m ? E::ld(g, e0 + e) : 0.0f;
        fu[e] = e < m ? E::ld(u, e0 + e) : 0.0f;
      }
#pragma unroll
      for (int e = 0; e < V - 1; ++e)
        if (e < m) E::st(o, e0 + e, silu_mul(fg[e], fu[e]));
    }
  }
}

// As the flat form, calls that move more than the last-level cache stream
// nontemporally (a 2-read, 1-write stream of 1.2 GB over three buffer sets:
// 6.52 against 5.98 TB/s). Bound by memory: bf16 4096 x 14336 on the halves
// of a fused buffer 55.8 us (6.3 TB/s), against 61.0 us cached with a 64-bit
// division per 256-vector piece of a row; 512 x 11008 one element off a
// 16-byte boundary 6.5 against 13.6 us element by element.
template <int DT, bool ANY>
__device__ __forceinline__ void sw_rows_part(const SwArgs &a, int64_t blk, int64_t nblk) {
  if (3 * a.n * Elt<DT>::ES > int64_t(kStreamBytes))
    sw_slots<DT, ANY, true>(a, blk, nblk);
  else
    sw_slots<DT, ANY, false>(a, blk, nblk);
}

// ---- element-wise ops (silu, add, masked_fill) and embedding -------------------------
constexpr int kOpSilu = 8, kOpAdd = 9, kOpMaskedFill = 10;   // the ABI's op ids

// One element of an element-wise op on float values (masked_fill works on
// bit patterns instead, see below).
template <int OP>
__device__ __forceinline__ float elt_value(float a, float b) {
  if constexpr (OP == kOpAdd)
    return a + b;
  else
    return silu(a);
}

// masked_fill on one 16-byte vector: element e takes `fill` (the fill
// value's bit pattern) where mask byte e is nonzero, else keeps its bits.
template <int DT>
__device__ __forceinline__ u32x4 mask_select(u32x4 x, uint64_t m, uint32_t fill) {
  u32x4 o;
  if constexpr (DT == kF32) {
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = ((m >> (8 * e)) & 0xFF) ? fill : x[e];
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t lo = ((m >> (16 * j)) & 0xFF) ? fill : (x[j] & 0xFFFFu);
      const uint32_t hi = ((m >> (16 * j + 8)) & 0xFF) ? fill : (x[j] >> 16);
      o[j] = lo | (hi << 16);
    }
  }
  return o;
}

template <int DT>
__device__ __forceinline__ uint32_t fill_bits(float value) {
  if constexpr (DT == kF32)
    return __float_as_uint(value);
  else
    return Elt<kBF16>::pack2(value, 0.0f) & 0xFFFFu;   // round to nearest even
}

// The V mask bytes of elements e .. e + V - 1 of a row starting at `m`, as
// one load (aligned to V, or at any byte with ANY).
template <int DT, bool ANY>
__device__ __forceinline__ uint64_t mask_bytes(const uint8_t *m, int64_t e) {
  typedef uint32_t u32b __attribute__((aligned(1)));
  typedef uint64_t u64b __attribute__((aligned(1)));
  if constexpr (DT == kF32)
    return ANY ? *reinterpret_cast<const u32b *>(m + e)
               : *reinterpret_cast<const uint32_t *>(m + e);
  else
    return ANY ? *reinterpret_cast<const u64b *>(m + e)
               : *reinterpret_cast<const uint64_t *>(m + e);
}

// The V elements x at element e of a row of an element-wise op; b is the
// second operand's or the mask's row.
template <int DT, int OP, bool ANY, bool NT>
__device__ __forceinline__ u32x4 elt_vector(u32x4 x, const void *b, int64_t e, uint32_t fill) {
  using E = Elt<DT>;
  constexpr int V = E::V;
  if constexpr (OP == kOpMaskedFill) {
    return mask_select<DT>(x, mask_bytes<DT, ANY>(static_cast<const uint8_t *>(b), e), fill);
  } else {
    float fa[V], fb[V];
    E::unpack(x, fa);
    if constexpr (OP == kOpAdd) {
      E::unpack(ld_slot<DT, ANY, NT>(b, e), fb);
#pragma unroll
      for (int i = 0; i < V; ++i) fa[i] += fb[i];
    } else {
      silu_all<V>(fa);
    }
    return E::pack(fa);
  }
}

// Element e of a row (masked_fill copies bit patterns).
template <int DT, int OP>
__device__ __forceinline__ void elt_element(const void *x, const void *b, void *o, int64_t e,
                                            uint32_t fill) {
  using E = Elt<DT>;
  if constexpr (OP == kOpMaskedFill) {
    const bool set = static_cast<const uint8_t *>(b)[e] != 0;
    if constexpr (DT == kF32)
      static_cast<uint32_t *>(o)[e] = set ? fill : static_cast<const uint32_t *>(x)[e];
    else
      static_cast<uint16_t *>(o)[e] = set ? uint16_t(fill) : static_cast<const uint16_t *>(x)[e];
  } else {
    E::st(o, e, elt_value<OP>(E::ld(x, e), OP == kOpAdd ? E::ld(b, e) : 0.0f));
  }
}

// Flat contiguous [T*W]: U vectors per work-item per step (all loads
// issued before any use); workgroup 0 also does the < V element tail.
template <int DT, int OP, bool NT, int U = 1>
__device__ __forceinline__ void elt_flat_part(const EltArgs &a, int64_t blk, int64_t nblk) {
  using E = Elt<DT>;
  constexpr int V = E::V;
  const u32x4 *x = static_cast<const u32x4 *>(a.a);
  u32x4 *o = static_cast<u32x4 *>(a.out);
  const uint32_t fill = fill_bits<DT>(a.value);
  const int64_t step = nblk * kThreads * U;
  for (int64_t base = blk * kThreads * U + threadIdx.x; base < a.nvec; base += step) {
    u32x4 xv[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int64_t i = base + int64_t(k) * kThreads;
      if (i < a.nvec) xv[k] = ld16<NT>(x + i);
    }
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int64_t i = base + int64_t(k) * kThreads;
      if (i < a.nvec) o[i] = elt_vector<DT, OP, false, NT>(xv[k], a.b, i * V, fill);
    }
  }
  if (blk == 0) {
    const int64_t i = a.nvec * V + threadIdx.x;
    if (i < a.n) elt_element<DT, OP>(a.a, a.b, a.out, i, fill);
  }
}

// Element-wise calls that move more than the 256 MiB last-level cache read
// nontemporally and write through it. bf16 add of 4096 x 12288, three buffer
// sets in turn: 45.3 us, against 53.5 cached and 47.9 nontemporal both ways;
// after a flush of the cache, where it takes the writes, 16384 x 8192: add
// 120.7, masked_fill 99.6, silu 78.4 us, against 133.0 / 105.9 / 79.8 cached
// and 136.9 / 111.4 / 86.9 nontemporal both ways.
template <int DT, int OP>
__device__ __forceinline__ bool elt_streams(const EltArgs &a) {
  return (OP == kOpAdd ? 3 : 2) * a.T * a.W * Elt<DT>::ES > int64_t(kCacheBytes);
}

// Rows with padded strides: aligned and whole vectors long, or of any start
// and length (ANY). Bound by memory: masked_fill of bf16 8008 x 1001 takes
// 7.6 us (5.3 TB/s, a contiguous Python call), against 19.7 us element by
// element with a 64-bit division each.
template <int DT, int OP, bool ANY, bool NT>
__device__ __forceinline__ void elt_slots(const EltArgs &a, int64_t blk, int64_t nblk) {
  using E = Elt<DT>;
  constexpr int V = E::V;
  constexpr int BS = OP == kOpMaskedFill ? 1 : E::ES;
  const uint32_t fill = fill_bits<DT>(a.value);
  const Slots sl = make_slots<V>(a.T, a.W, ANY && a.a_rs == a.W && a.b_rs == a.W && a.o_rs == a.W);
  for (int64_t i = blk * kThreads + threadIdx.x; i < sl.total; i += nblk * kThreads) {
    int64_t row, e0;
    slot_at<V>(sl, i, row, e0);
    const char *x = static_cast<const char *>(a.a) + row * a.a_rs * E::ES;
    const char *b = static_cast<const char *>(a.b) + row * a.b_rs * BS;
    char *o = static_cast<char *>(a.out) + row * a.o_rs * E::ES;
    if (!ANY || e0 + V <= sl.W) {
      const u32x4 xv = ld_slot<DT, ANY, NT>(x, e0);
      st_slot<DT, ANY, false>(o, e0, elt_vector<DT, OP, ANY, NT>(xv, b, e0, fill));
    } else {
      const int m = int(sl.W - e0);   // 1 .. V - 1
#pragma unroll
      for (int e = 0; e < V - 1; ++e)
        if (e < m) elt_element<DT, OP>(x, b, o, e0 + e, fill);
    }
  }
}

template <int DT, int OP, bool ANY>
__device__ __forceinline__ void elt_rows_part(const EltArgs &a, int64_t blk, int64_t nblk) {
  if (elt_streams<DT, OP>(a))
    elt_slots<DT, OP, ANY, true>(a, blk, nblk);
  else
    elt_slots<DT, OP, ANY, false>(a, blk, nblk);
}

// Embedding rows: a work-item copies slots of V elements of output rows (the
// slots of all rows numbered through) from table row ids[t] when it is in
// [0, n_rows), else writes zeros. Aligned rows of whole vectors, or rows of
// any start and length (ANY). A workgroup takes kEmbSlots * 256 consecutive
// slots; a lane's ids and then its table vectors are requested together.
// Bound by the gather and the output's writes: bf16 8192 rows of 4096 from a
// 32,000-row table 22.1-22.7 us, float32 8192 x 5120 65.6 us, against 23.0 and
// 66.6 us with a workgroup per row; 4096 x 5000 one element
// off a 16-byte boundary 14.7 against 26 us element by element.
template <int DT, bool ANY, bool NT>
__device__ __forceinline__ void emb_slots(const EmbArgs &a, uint32_t nblk) {
  using E = Elt<DT>;
  constexpr int V = E::V, B = kEmbSlots;
  const Slots sl = make_slots<V>(a.T, a.H, false);
  constexpr int step = kThreads;
  for (int64_t i0 = int64_t(blockIdx.x) * (B * step) + threadIdx.x; i0 < sl.total;
       i0 += int64_t(nblk) * (B * step)) {
    int64_t t[B], e0[B], id[B];
    bool ok[B];
#pragma unroll
    for (int k = 0; k < B; ++k) {
      ok[k] = false;
      if (i0 + k * step < sl.total) {
        slot_at<V>(sl, i0 + k * step, t[k], e0[k]);
        id[k] = a.ids64 ? static_cast<const int64_t *>(a.ids)[t[k]]
                        : int64_t(static_cast<const int32_t *>(a.ids)[t[k]]);
      }
    }
    u32x4 v[B];
#pragma unroll
    for (int k = 0; k < B; ++k) {
      v[k] = u32x4{0u, 0u, 0u, 0u};
      if (i0 + k * step < sl.total) {
        ok[k] = id[k] >= 0 && id[k] < a.n_rows;
        if (ok[k] && (!ANY || e0[k] + V <= sl.W))
          v[k] = ld_slot<DT, ANY, false>(
              static_cast<const char *>(a.table) + id[k] * a.t_rs * E::ES, e0[k]);
      }
    }
#pragma unroll
    for (int k = 0; k < B; ++k) {
      if (i0 + k * step >= sl.total) continue;
      char *dst = static_cast<char *>(a.out) + t[k] * a.o_rs * E::ES;
      if (!ANY || e0[k] + V <= sl.W) {
        st_slot<DT, ANY, NT>(dst, e0[k], v[k]);
      } else {
        const char *src = static_cast<const char *>(a.table) + (ok[k] ? id[k] : 0) * a.t_rs * E::ES;
        for (int64_t e = e0[k]; e < sl.W; ++e) {   // 1 .. V - 1 elements
          if constexpr (DT == kF32)
            reinterpret_cast<uint32_t *>(dst)[e] =
                ok[k] ? reinterpret_cast<const uint32_t *>(src)[e] : 0u;
          else
            reinterpret_cast<uint16_t *>(dst)[e] =
                ok[k] ? reinterpret_cast<const uint16_t *>(src)[e] : uint16_t(0);
        }
      }
    }
  }
}

// Outputs larger than the last-level cache are written nontemporally (float32
// rows of 8192 after a flush of the cache: 16384 of them 161 against 168 us,
// 32768 306 against 348 us). Smaller ones the cache takes: 8192 rows of 4096
// bf16 24.9 against 26.8 us, with a norm that reads them 45.2 against 48.2 us
// (back to back, where older outputs have to leave it first, 22.1-22.7 against
// 21.1 us). Nontemporal loads of the table, whose rows repeat, took 24.5 us.
template <int DT, bool VEC>
__device__ __forceinline__ void emb_rows(const EmbArgs &a, uint32_t nblk) {
  if (a.T * a.H * Elt<DT>::ES > int64_t(kEmbStreamBytes))
    emb_slots<DT, !VEC, true>(a, nblk);
  else
    emb_slots<DT, !VEC, false>(a, nblk);
}

// ---- kernel bodies -----------------------------------------------------------------
// One body per kernel family, called by the precompiled kernels and by the
// runtime-compiled specializations; a specialization passes arguments whose
// shape fields are compile-time constants.
template <int DT, int NV, bool RES>
__device__ __forceinline__ void body_rn_wave(const RnArgs &a) {
  rn_wave_block<DT, NV, RES, false>(a, blockIdx.x);
}

// Residual rows of calls that move more than kStreamBytes are read
// nontemporally and written through the last-level cache (bf16 8192 x 8192,
// three buffer sets in turn: 91.2 against 91.9 us cached; after a flush of the
// cache 0.827 against 0.821 of 8 TB/s. Nontemporal stores too: 88.0 us, but
// 0.73 after a flush, as the cache then takes none of the writes). Plain rows
// gained nothing at any size (256-512 MiB: 46.3-46.0 and 98.5-100.2 us). With
// eight or more vectors a work-item, whose registers leave two to four
// wavefronts per SIMD either way, the weights are requested with the row: asked
// for after the reduction nothing covers them (float32 2048 x 16384 after a
// flush 83.6 against 93.7 us, 86.7 cached; back to back 83.8 against 91.9 and
// 103.3; bf16 2730 x 24,576 84.8 against 92.8 and 86.4, 84.8 against 92.4 and 101.5).
template <int DT, int NB, bool RES>
__device__ __forceinline__ void body_rn_block(const RnArgs &a) {
  __shared__ float red[4];
  if constexpr (RES) {
    if (4 * a.T * a.H * Elt<DT>::ES > int64_t(kStreamBytes)) {
      rn_row_regs<DT, NB, RES, 256, true, (NB < 8)>(a, blockIdx.x, threadIdx.x, red);
      return;
    }
  }
  rn_row_regs<DT, NB, RES, 256, false>(a, blockIdx.x, threadIdx.x, red);
}

template <int DT, bool RES>
__device__ __forceinline__ void body_rn_loop(const RnArgs &a) {
  __shared__ double red[4];
  rn_loop_row<DT, RES>(a, blockIdx.x, red);
}

// Plain RMSNorm of a row held by a 1024-work-item workgroup, 8 vectors per
// lane: the row is kept packed across the reduction and the weights are
// requested only after it, in two halves, so a lane holds at most 8 + 4
// vectors and two workgroups fit on a CU (61 VGPRs, 8 waves per SIMD,
// against 122 with the weights requested with the row and the row kept
// unpacked: one workgroup per CU, whose loads then never overlap another
// row's stores). Same arithmetic in the same order as rn_row_regs.
template <int DT>
__device__ __forceinline__ void rn_row_wide_plain(const RnArgs &a, int64_t row, int lane,
                                                  float *red) {
  using E = Elt<DT>;
  constexpr int V = E::V;
  constexpr int NV = 8, L = kWideLanes, HALF = NV / 2;
  const int nvec = a.H / V;
  // uniform row bases and 32-bit per-lane byte offsets, so that every
  // access is a scalar base plus one offset register
  const char *xb = static_cast<const char *>(a.x) + row * a.x_rs * E::ES;
  const char *wb = static_cast<const char *>(a.w);
  char *yb = static_cast<char *>(a.y) + row * a.y_rs * E::ES;
  const uint32_t off0 = uint32_t(lane) * 16u;
  // Loads past the row's end read its last vector instead (no branch, no
  // saved lane masks) and are zeroed.
  const uint32_t last = uint32_t(nvec - 1) * 16u;
  u32x4 xv[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const uint32_t off = off0 + uint32_t(k) * (L * 16u);
    const u32x4 v = *reinterpret_cast<const u32x4 *>(xb + (off < last ? off : last));
    xv[k] = off <= last ? v : u32x4{0, 0, 0, 0};
  }
  float ss = 0.0f;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    float f[V];
    E::unpack(xv[k], f);
#pragma unroll
    for (int e = 0; e < V; ++e) ss = __builtin_fmaf(f[e], f[e], ss);
  }
  // the unpacked floats are not kept for the output pass: it unpacks again
#pragma unroll
  for (int k = 0; k < NV; ++k) asm volatile("" : "+v"(xv[k]));
  // The 16 wavefront sums: each lane takes one of them (every one four
  // times over the wavefront), so the combine holds one value per lane
  // rather than all 16 next to the row; the wavefront total is exactly four
  // times the row's and is the same bits in every lane.
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  static_assert(L / 64 == 16, "one partial per lane of a 16-lane group");
  ss = wave_sum(red[threadIdx.x & 15]) * 0.25f;
  const float inv = rsqrtf(ss / float(a.H) + a.eps);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    u32x4 wv[HALF];
#pragma unroll
    for (int k = 0; k < HALF; ++k) {
      const uint32_t off = off0 + uint32_t(h * HALF + k) * (L * 16u);
      wv[k] = *reinterpret_cast<const u32x4 *>(wb + (off < last ? off : last));
    }
#pragma unroll
    for (int k = 0; k < HALF; ++k) {
      const int j = h * HALF + k;
      if (off0 + uint32_t(j) * (L * 16u) <= last) {
        // one 32-bit word at a time: few temporaries live at once
        u32x4 yv;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          if constexpr (DT == kBF16) {
            const float x0 = __uint_as_float(xv[j][d] << 16), x1 = __uint_as_float(xv[j][d] & 0xFFFF0000u);
            const float w0 = __uint_as_float(wv[k][d] << 16), w1 = __uint_as_float(wv[k][d] & 0xFFFF0000u);
            yv[d] = E::pack2((x0 * inv) * w0, (x1 * inv) * w1);
          } else {
            yv[d] = __float_as_uint((__uint_as_float(xv[j][d]) * inv) * __uint_as_float(wv[k][d]));
          }
        }
        *reinterpret_cast<u32x4 *>(yb + off0 + uint32_t(j) * (L * 16u)) = yv;
      }
    }
    // the second half's weights are requested after the first half's stores
    asm volatile("" ::: "memory");
  }
}

// Buffer access to one row: the row's uniform base with its byte length as
// the range. A load past the range returns zeros and a store past it is
// dropped, so a row of any length up to 8 * kWideLanes vectors needs no
// branch, and each access is the descriptor plus one per-lane offset.
// Descriptor word 3: data format 32 bits (nonzero, as untyped loads need),
// no swizzle, no index stride.
constexpr int kRowRsrcWord3 = 0x00020000;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const void *base, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, bytes, kRowRsrcWord3);
}

__device__ __forceinline__ void wide_load(__amdgpu_buffer_rsrc_t r, uint32_t off0, u32x4 *xv) {
#pragma unroll
  for (int k = 0; k < 8; ++k)
    xv[k] = __builtin_amdgcn_raw_buffer_load_b128(r, off0 + uint32_t(k) * (kWideLanes * 16u), 0, 0);
}

// One row of the pipelined plain form, held packed in xv (zeros past the
// row's end); the lane's weight vectors are in wl. Same arithmetic in the
// same order as rn_row_wide_plain, so both give the same bits.
template <int DT>
__device__ __forceinline__ void wide_norm_store(const RnArgs &a, u32x4 *xv, const u32x4 *wl,
                                                __amdgpu_buffer_rsrc_t yr, uint32_t off0,
                                                float *red) {
  using E = Elt<DT>;
  constexpr int V = E::V;
  float ss = 0.0f;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    float f[V];
    E::unpack(xv[k], f);
#pragma unroll
    for (int e = 0; e < V; ++e) ss = __builtin_fmaf(f[e], f[e], ss);
  }
  // the output pass unpacks again: the floats are not kept
#pragma unroll
  for (int k = 0; k < 8; ++k) asm volatile("" : "+v"(xv[k]));
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  ss = wave_sum(red[threadIdx.x & 15]) * 0.25f;
  const float inv = rsqrtf(ss / float(a.H) + a.eps);
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const u32x4 w = wl[j * kWideLanes + threadIdx.x];
    u32x4 yv;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      if constexpr (DT == kBF16) {
        const float x0 = __uint_as_float(xv[j][d] << 16), x1 = __uint_as_float(xv[j][d] & 0xFFFF0000u);
        const float w0 = __uint_as_float(w[d] << 16), w1 = __uint_as_float(w[d] & 0xFFFF0000u);
        yv[d] = E::pack2((x0 * inv) * w0, (x1 * inv) * w1);
      } else {
        yv[d] = __float_as_uint((__uint_as_float(xv[j][d]) * inv) * __uint_as_float(w[d]));
      }
    }
    __builtin_amdgcn_raw_buffer_store_b128(yv, yr, off0 + uint32_t(j) * (kWideLanes * 16u), 0, 0);
  }
}

// Plain RMSNorm when a workgroup has several rows: workgroup b takes rows
// b, b + nblk, ... and requests each next row before the current row's
// reduction, so one row's loads overlap the previous row's stores on the
// same CU (one row per workgroup, the loads of every workgroup on the chip
// start together and then their stores, at bf16 rows of 57,344 measured
// 0.85 of a copy of the same bytes, against 0.90 with this loop). Two row
// buffers used in turn, so no register copy makes the next row's loads
// complete early; the weights wait in LDS (each lane reads back only the
// vectors it wrote: no barrier), which keeps the lane at 8 + 8 vectors
// (121 VGPRs; holding the weights in registers spills). The partial sums
// alternate between two LDS rows, so one barrier per row suffices.
template <int DT>
__device__ __forceinline__ void rn_rows_wide_plain(const RnArgs &a, uint32_t nblk, u32x4 *wl,
                                                   float (*red)[kWideLanes / 64]) {
  using E = Elt<DT>;
  const uint32_t off0 = uint32_t(threadIdx.x) * 16u;
  const int rowb = (a.H / E::V) * 16;
  const char *xbase = static_cast<const char *>(a.x);
  char *ybase = static_cast<char *>(a.y);
  const int64_t xs = a.x_rs * E::ES, ys = a.y_rs * E::ES;
  int64_t row = blockIdx.x;
  u32x4 ra[8], rb[8];
  wide_load(row_rsrc(a.w, rowb), off0, ra);
#pragma unroll
  for (int k = 0; k < 8; ++k) wl[k * kWideLanes + threadIdx.x] = ra[k];
  wide_load(row_rsrc(xbase + row * xs, rowb), off0, ra);
  for (;;) {
    if (row + nblk >= a.T) {
      wide_norm_store<DT>(a, ra, wl, row_rsrc(ybase + row * ys, rowb), off0, red[0]);
      return;
    }
    wide_load(row_rsrc(xbase + (row + nblk) * xs, rowb), off0, rb);
    wide_norm_store<DT>(a, ra, wl, row_rsrc(ybase + row * ys, rowb), off0, red[0]);
    row += nblk;
    if (row + nblk >= a.T) {
      wide_norm_store<DT>(a, rb, wl, row_rsrc(ybase + row * ys, rowb), off0, red[1]);
      return;
    }
    wide_load(row_rsrc(xbase + (row + nblk) * xs, rowb), off0, ra);
    wide_norm_store<DT>(a, rb, wl, row_rsrc(ybase + row * ys, rowb), off0, red[1]);
    row += nblk;
  }
}

// Rows of 4097..8192 vectors on 1024-work-item workgroups, up to 8 vectors
// per lane held in registers (all loads issued up front). The residual form
// takes one row per workgroup (grid T) and requests the weights with the
// row (measured 1 % faster for it; a loop over rows measured 4-35 % slower).
// The plain form is launched on at most kWideGrid workgroups: with one row
// each, rn_row_wide_plain; with more, rn_rows_wide_plain.
template <int DT, bool RES>
__device__ __forceinline__ void body_rn_wide(const RnArgs &a, uint32_t nblk = gridDim.x) {
  if constexpr (RES) {
    __shared__ float red[kWideLanes / 64];
    rn_row_regs<DT, 8, RES, kWideLanes, false>(a, blockIdx.x, threadIdx.x, red);
  } else {
    __shared__ float red[2][kWideLanes / 64];
    __shared__ u32x4 wl[8 * kWideLanes];
    if (a.T <= int64_t(nblk)) {
      if (int64_t(blockIdx.x) < a.T) rn_row_wide_plain<DT>(a, blockIdx.x, threadIdx.x, red[0]);
    } else {
      rn_rows_wide_plain<DT>(a, nblk, wl, red);
    }
  }
}

// Rows of more than 4096 vectors over several workgroups (rn_split_row);
// residual calls that move more than kStreamBytes read nontemporally (1061
// rows of 49,408 bf16: 81.1 against 84.2 us, 700 of 131,072: 133.1 against
// 135.2 us; 2048 of 65,536 after a flush of the cache 0.80 against 0.757 of
// 8 TB/s, and 0.73 with nontemporal stores).
template <int DT, bool RES>
__device__ __forceinline__ void body_rn_split(const RnSplitArgs &a) {
  __shared__ float red[4];
  __shared__ float total;
  if (RES && 4 * a.rn.T * a.rn.H * Elt<DT>::ES > int64_t(kStreamBytes))
    rn_split_row<DT, RES, RES>(a.rn, a.scratch, red, total);
  else
    rn_split_row<DT, RES, false>(a.rn, a.scratch, red, total);
}

// Residual calls that move more than kStreamBytes read nontemporally (f32
// 295 x 88763 131.3 against 135.1 us; 2560 x 10240 77.8 against 78.2 us).
template <int DT, bool RES>
__device__ __forceinline__ void body_rn_scalar(const RnArgs &a) {
  __shared__ double red[kWideLanes / 64];
  if (RES && 4 * a.T * a.H * Elt<DT>::ES > int64_t(kStreamBytes))
    rn_any_row<DT, RES, RES>(a, blockIdx.x, red);
  else
    rn_any_row<DT, RES, false>(a, blockIdx.x, red);
}

// QKN: per-head RMSNorm of Q and K before the rotation; INTER: GPT-J pairs.
template <int DT, bool QKN, bool INTER>
__device__ __forceinline__ void body_rope_vec(const RopeArgs &a) {
  __shared__ float lds[2 * 256 * kRopeTokensMax];
  rope_vec_block<DT, false, QKN ? 1 : 2, QKN, INTER>(a, blockIdx.x, lds);
}

template <int DT, bool QKN>
__device__ __forceinline__ void body_rope_scalar(const RopeArgs &a) {
  __shared__ float lds[2 * 256];
  if (a.mode & kRopeInterleaved)
    rope_any_block<DT, QKN, true>(a, blockIdx.x, lds);
  else
    rope_any_block<DT, QKN, false>(a, blockIdx.x, lds);
}

// The bodies that stride over the grid take the launch's workgroup count:
// gridDim.x, or a resident block's count in a launch without kernel
// arguments (which must not read gridDim: that would give it implicit
// kernel arguments again).
template <int DT, int U, bool NT>
__device__ __forceinline__ void body_sw_flat(const SwArgs &a, uint32_t nblk = gridDim.x) {
  sw_flat_part<DT, U, NT>(a, blockIdx.x, nblk);
}

template <int DT>
__device__ __forceinline__ void body_sw_rows(const SwArgs &a, uint32_t nblk = gridDim.x) {
  sw_rows_part<DT, false>(a, blockIdx.x, nblk);
}

template <int DT>
__device__ __forceinline__ void body_sw_scalar(const SwArgs &a, uint32_t nblk = gridDim.x) {
  sw_rows_part<DT, true>(a, blockIdx.x, nblk);
}

// U vectors per work-item, nontemporal when the call streams (elt_streams).
template <int DT, int OP, int U>
__device__ __forceinline__ void body_elt_flat(const EltArgs &a, uint32_t nblk = gridDim.x) {
  if (elt_streams<DT, OP>(a))
    elt_flat_part<DT, OP, true, U>(a, blockIdx.x, nblk);
  else
    elt_flat_part<DT, OP, false, U>(a, blockIdx.x, nblk);
}

template <int DT, int OP>
__device__ __forceinline__ void body_elt_rows(const EltArgs &a, uint32_t nblk = gridDim.x) {
  elt_rows_part<DT, OP, false>(a, blockIdx.x, nblk);
}

template <int DT, int OP>
__device__ __forceinline__ void body_elt_scalar(const EltArgs &a, uint32_t nblk = gridDim.x) {
  elt_rows_part<DT, OP, true>(a, blockIdx.x, nblk);
}

template <int DT, bool VEC>
__device__ __forceinline__ void body_emb(const EmbArgs &a, uint32_t nblk = gridDim.x) {
  emb_rows<DT, VEC>(a, nblk);
}

template <int DT, bool WAVE, int N, bool NT>
__device__ __forceinline__ void chain_norm_role(const ChainArgs &a, uint32_t blk) {
  if constexpr (WAVE) {
    rn_wave_block<DT, N, true, NT>(a.rn, blk);
  } else {
    __shared__ float red[4];
    rn_row_regs<DT, N, true, 256, NT>(a.rn, blk, threadIdx.x, red);
  }
}

// The fused decode chain: workgroups take the residual-RMSNorm, RoPE-QK and
// SwiGLU roles by blockIdx range. Norm role: one wavefront per row with N
// vectors per lane (WAVE) or one workgroup per row with N per work-item;
// RoPE role: one token, one head slice of a token, or up to four tokens per
// workgroup, as the argument block's mode says (QK norm first when QKN,
// GPT-J pairs when INTER); SwiGLU role: one vector per work-item,
// nontemporal when NT (calls that stream more than the last-level cache).
//
// Role order by blockIdx: norm rows, RoPE tokens, then SwiGLU. At decode
// sizes the norm and RoPE roles take about as long as SwiGLU but have far
// fewer workgroups, so dispatching them first shortens the critical path
// (2.75 vs 3.1 us device time at 1 token); at 8192 tokens this order with a
// one-vector nontemporal SwiGLU role measured 331.5 us, against 344-349 us
// for SwiGLU first or with two / four vectors per work-item.
//
// In the streaming form (NT: calls that move more than the last-level
// cache) the RoPE role also streams nontemporally and the norm role reads so
// (365.7 against 371.3 us at 8192 tokens, hidden 8192, three buffer sets in
// turn; with its stores nontemporal too 360 us, but after a flush of the cache
// 0.83 instead of 0.846 of 8 TB/s), and the RoPE role keeps one head per lane group in flight instead of
// two (as with the QK norm at any size): more registers per lane cap the whole fused kernel below the 8
// wavefronts per SIMD that SwiGLU alone runs (with four heads and 77
// registers, 357 against 346.5 us at 8192 tokens).
//
// `nblk` is the launch's workgroup count (gridDim.x, or the resident block's
// count in a launch without kernel arguments, which must not read gridDim:
// that would give the kernel implicit arguments again).
template <int DT, bool WAVE, int N, bool NT, bool QKN, bool INTER>
__device__ __forceinline__ void body_chain(const ChainArgs &a, uint32_t nblk) {
  __shared__ float lds[2 * 256 * kRopeTokensMax];
  const uint32_t b = blockIdx.x;
  const uint32_t R = a.rn_blocks, P = a.rope_blocks, S = nblk - R - P;
  if (b < R) {
    chain_norm_role<DT, WAVE, N, NT>(a, b);
  } else if (b < R + P) {
    rope_vec_block<DT, NT, NT || QKN ? 1 : 2, QKN, INTER>(a.rope, b - R, lds);
  } else {
    sw_flat_part<DT, 1, NT>(a.sw, b - R - P, S);
  }
}

// The slot of a launch without kernel arguments. The workgroup's LDS
// allocation is readable in the LDS_ALLOC hardware register (bits 12..20,
// in 256-byte units; the hardware allocates whole kLdsGranule-byte
// granules): less the granules of the kernel's static LDS, it is the slot
// the host encoded as slot * kLdsGranule bytes of dynamic LDS. Reading a
// register costs no memory access, unlike the dispatch packet.
__device__ __forceinline__ uint32_t resident_slot() {
  const uint32_t units = __builtin_amdgcn_s_getreg((8 << 11) | (12 << 6) | 6);
  return units / (kLdsGranule / 256) -
         (__builtin_amdgcn_groupstaticsize() + kLdsGranule - 1) / kLdsGranule;
}

template <typename P>
__device__ __forceinline__ P *in_global(P *p) {
  typedef __attribute__((address_space(1))) P *gptr;
  gptr g;
  // an empty move the compiler cannot look through: the result is a
  // global-address-space pointer, so no cast pair folds back to flat
  asm("" : "=s"(g) : "0"((gptr)p));
  return (P *)g;
}

// Pointers read from memory could point anywhere; these are global memory,
// as kernel-argument pointers are taken to be (global, not flat, loads and
// stores).
__device__ __forceinline__ void to_global(RnArgs &a) {
  a.x = in_global(a.x);
  a.res = in_global(a.res);
  a.w = in_global(a.w);
  a.y = in_global(a.y);
  a.res_out = in_global(a.res_out);
}
__device__ __forceinline__ void to_global(RnSplitArgs &a) {
  to_global(a.rn);
  a.scratch = in_global(a.scratch);
}
__device__ __forceinline__ void to_global(RopeArgs &a) {
  a.q = in_global(a.q);
  a.k = in_global(a.k);
  a.pos = in_global(a.pos);
  a.inv_freq = in_global(a.inv_freq);
  a.qw = in_global(a.qw);
  a.kw = in_global(a.kw);
  a.cos_sin = in_global(a.cos_sin);
}
__device__ __forceinline__ void to_global(SwArgs &a) {
  a.gate = in_global(a.gate);
  a.up = in_global(a.up);
  a.out = in_global(a.out);
}
__device__ __forceinline__ void to_global(EltArgs &a) {
  a.a = in_global(a.a);
  a.b = in_global(a.b);
  a.out = in_global(a.out);
}
__device__ __forceinline__ void to_global(EmbArgs &a) {
  a.table = in_global(a.table);
  a.ids = in_global(a.ids);
  a.out = in_global(a.out);
}
__device__ __forceinline__ void to_global(ChainArgs &a) {
  to_global(a.rn);
  to_global(a.rope);
  to_global(a.sw);
}

// An argument struct from constant memory, every word requested before any is
// waited for. Loaded where they are used, the words cost one round trip of a
// scalar load (200-300 ns: a kernel starts with a cold scalar cache) per
// branch that precedes their use; an opaque use of all of them here keeps the
// compiler from moving a load back behind a branch. Back to back, the fused
// 1-token chain from resident blocks went from 2.61 to 2.40 us a launch, the
// captured 8-token chain from 3.29 to 3.11 us. `extra` is the pair of words
// at dword E of the block, requested with them.
typedef __attribute__((address_space(4))) const uint32_t cu32;
template <typename V>
struct __attribute__((packed, aligned(4))) Words {   // as argument words lie
  V v;
};
template <typename V>
__device__ __forceinline__ V ld_const(cu32 *w) {
  return reinterpret_cast<__attribute__((address_space(4))) const Words<V> *>(w)->v;
}
template <int E, class A>
__device__ __forceinline__ u32x2 load_args(cu32 *w, A &a) {
  constexpr int N = sizeof(A) / 4;
  static_assert(sizeof(A) % 8 == 0 && (N < 32 || N == 72), "argument struct sizes");
  asm volatile("" : "+s"(w));   // one base address for all the loads
  u32x2 extra = {0u, 0u};
  if constexpr (E >= 0) extra = ld_const<u32x2>(w + E);
  uint32_t words[N];
  if constexpr (N == 72) {
    u32x16 c0 = ld_const<u32x16>(w), c1 = ld_const<u32x16>(w + 16),
           c2 = ld_const<u32x16>(w + 32), c3 = ld_const<u32x16>(w + 48);
    u32x8 c4 = ld_const<u32x8>(w + 64);
    asm volatile("" : "+s"(c0), "+s"(c1), "+s"(c2), "+s"(c3), "+s"(c4), "+s"(extra));
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      words[i] = c0[i];
      words[16 + i] = c1[i];
      words[32 + i] = c2[i];
      words[48 + i] = c3[i];
      if (i < 8) words[64 + i] = c4[i];
    }
  } else {
    constexpr int o4 = 16 + (N & 8), o2 = o4 + (N & 4);
    u32x16 c0 = ld_const<u32x16>(w);
    u32x8 c1 = {};
    u32x4 c2 = {};
    u32x2 c3 = {};
    if constexpr (N & 8) c1 = ld_const<u32x8>(w + 16);
    if constexpr (N & 4) c2 = ld_const<u32x4>(w + o4);
    if constexpr (N & 2) c3 = ld_const<u32x2>(w + o2);
    asm volatile("" : "+s"(c0), "+s"(extra));
    if constexpr (N & 8) asm volatile("" : "+s"(c1));
    if constexpr (N & 4) asm volatile("" : "+s"(c2));
    if constexpr (N & 2) asm volatile("" : "+s"(c3));
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      words[i] = c0[i];
      if ((N & 8) && i < 8) words[16 + i] = c1[i];
      if ((N & 4) && i < 4) words[o4 + i] = c2[i];
      if ((N & 2) && i < 2) words[o2 + i] = c3[i];
    }
  }
  __builtin_memcpy(&a, words, sizeof a);
  to_global(a);
  return extra;
}

// The fused chain's kernel arguments (its role's words are otherwise requested
// only after the role is known).
__device__ __forceinline__ void chain_args(ChainArgs &a, uint32_t &grid) {
  grid = gridDim.x;
  (void)load_args<-1>((cu32 *)__builtin_amdgcn_kernarg_segment_ptr(), a);
  asm volatile("" : "+s"(grid));
}

// The argument block of a launch without kernel arguments: slot
// resident_slot() of `table` (this device's table of the kernel's family and
// dtype, read as constant memory: the host writes a slot only while no
// launch can read it). False for an index beyond the table or an unwritten
// slot: the launch then runs nothing. The block is requested together with
// its tag, from the table's last slot when the index is beyond it.
template <class A>
__device__ __forceinline__ bool resident_args(const ResidentBlock *table, A &a, uint32_t &grid) {
  const uint32_t s = resident_slot();
  const uint32_t at = s < kResidentSlots ? s : kResidentSlots - 1;
  static_assert(__builtin_offsetof(ResidentBlock, tag) ==
                    __builtin_offsetof(ResidentBlock, grid) + 4, "grid and tag side by side");
  const u32x2 gt = load_args<__builtin_offsetof(ResidentBlock, grid) / 4>((cu32 *)(table + at), a);
  grid = gt[0];
  return s < kResidentSlots && gt[1] == kResidentTag + s;
}

}  // namespace dev
}  // namespace tri
