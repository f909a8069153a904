// The fused decode-chain kernel (f32): one launch whose workgroups take the
// residual-RMSNorm, RoPE-QK and SwiGLU roles by blockIdx range. Instantiated
// for every (norm role variant, SwiGLU role) the install policy can pick, in
// two forms: with the argument block as the kernel argument, and without
// kernel arguments, reading the block from this device's resident table.
#include "../internal.h"
#include "device.h"

namespace tri {
using namespace dev;

// RNV: RN_WAVE_1/2 (one wavefront per row) or RN_BLOCK_1..16 (one
// workgroup per row); SWV: SW_FLAT or SW_FLAT_NT; QKN: QK norm before the
// rotation; INTER: GPT-J pairs.
//
// Eight wavefronts per SIMD hide the most memory latency in the streaming
// forms. With the QK norm they are held to that (no spills; 61 registers a lane
// in bf16, 58 in float32), and the compiler loads their arguments where they are
// used, as in bf16 with a workgroup per norm row: chain_args has all of them in
// scalar registers at once, 105, which leaves seven wavefronts. After a flush
// of the cache, against chain_args: bf16 8192 tokens of 72 heads 341.0 and 344.3
// us, of 9 heads 111.8 and 113.0; 72 heads with the QK norm (then six wavefronts)
// 345.2 and 347.7. The other streaming forms gain more from the one round trip
// of chain_args (back to back, bf16 rows of 512 elements 114.8 against 117.5 us,
// float32 rows of 4096 162.0 against 163.6).
template <int DT, int RNV, int SWV, bool QKN, bool INTER>
__global__ __launch_bounds__(256, QKN && SWV == SW_FLAT_NT && RNV <= RN_BLOCK_4 ? 8 : 1)
void k_chain(ChainArgs a) {
  constexpr bool wave = RNV <= RN_WAVE_2;
  constexpr int n = wave ? 1 << (RNV - RN_WAVE_1) : 1 << (RNV - RN_BLOCK_1);
  constexpr bool nt = SWV == SW_FLAT_NT;
  if constexpr (nt && (QKN || (DT == kBF16 && !wave))) {
    body_chain<DT, wave, n, nt, QKN, INTER>(a, gridDim.x);
  } else {
    ChainArgs c;
    uint32_t g;
    chain_args(c, g);
    body_chain<DT, wave, n, nt, QKN, INTER>(c, g);
  }
}

// Resident argument blocks of this dtype's fused chain: one table per GPU,
// zero at load (every tag unset). In host code the name stands for a
// host-side shadow, not for device memory: the host writes the table through
// its device address, never through the name. Not static: the address of an
// internal symbol would be loaded from the code object's offset table, a
// round trip before the block's own.
__device__ __align__(256) ResidentBlock resident_chain_f32[kResidentSlots];

template <int DT, int RNV, int SWV, bool QKN, bool INTER>
__global__ __launch_bounds__(256, QKN && SWV == SW_FLAT_NT && RNV <= RN_BLOCK_4 ? 6 : 1)
void k_chain_res() {
  constexpr bool wave = RNV <= RN_WAVE_2;
  constexpr int n = wave ? 1 << (RNV - RN_WAVE_1) : 1 << (RNV - RN_BLOCK_1);
  ChainArgs a;
  uint32_t g;
  if (resident_args(resident_chain_f32, a, g))
    body_chain<DT, wave, n, SWV == SW_FLAT_NT, QKN, INTER>(a, g);
}

namespace {
template <bool RES, int RNV, bool QKN, bool INTER>
const void *chain_pick_sw(bool nt) {
  if constexpr (RES)
    return nt ? reinterpret_cast<const void *>(&k_chain_res<kF32, RNV, SW_FLAT_NT, QKN, INTER>)
              : reinterpret_cast<const void *>(&k_chain_res<kF32, RNV, SW_FLAT, QKN, INTER>);
  else
    return nt ? reinterpret_cast<const void *>(&k_chain<kF32, RNV, SW_FLAT_NT, QKN, INTER>)
              : reinterpret_cast<const void *>(&k_chain<kF32, RNV, SW_FLAT, QKN, INTER>);
}

template <bool RES, int RNV>
const void *chain_pick_rn(int32_t rope_bits, bool nt) {
  switch (rope_bits) {
    case 0: return chain_pick_sw<RES, RNV, false, false>(nt);
    case 1: return chain_pick_sw<RES, RNV, true, false>(nt);
    case 2: return chain_pick_sw<RES, RNV, false, true>(nt);
    default: return chain_pick_sw<RES, RNV, true, true>(nt);
  }
}

template <bool RES>
const void *chain_pick(int32_t sub) {
  const bool nt = sub & 1;
  const int32_t rb = (sub >> 1) & 3;   // bit 0: QK norm, bit 1: GPT-J pairs
  switch (RN_WAVE_1 + (sub >> 3)) {
    case RN_WAVE_1: return chain_pick_rn<RES, RN_WAVE_1>(rb, nt);
    case RN_WAVE_2: return chain_pick_rn<RES, RN_WAVE_2>(rb, nt);
    case RN_BLOCK_1: return chain_pick_rn<RES, RN_BLOCK_1>(rb, nt);
    case RN_BLOCK_2: return chain_pick_rn<RES, RN_BLOCK_2>(rb, nt);
    case RN_BLOCK_4: return chain_pick_rn<RES, RN_BLOCK_4>(rb, nt);
    case RN_BLOCK_8: return chain_pick_rn<RES, RN_BLOCK_8>(rb, nt);
    case RN_BLOCK_16: return chain_pick_rn<RES, RN_BLOCK_16>(rb, nt);
    default: return nullptr;
  }
}
}  // namespace

// sub = (norm role - RN_WAVE_1) * 8 + 4 * (GPT-J pairs) + 2 * (QK norm)
//       + (SwiGLU role streams nontemporally).
const void *chain_kernel_f32(int32_t sub) { return chain_pick<false>(sub); }
const void *chain_kernel_resident_f32(int32_t sub) { return chain_pick<true>(sub); }

// Host shadow of this dtype's resident table.
const void *resident_symbol_chain_f32() {
  return reinterpret_cast<const void *>(&resident_chain_f32);
}

}  // namespace tri
