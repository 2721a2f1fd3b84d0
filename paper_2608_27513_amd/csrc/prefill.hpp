// Launch parameters shared by the two prefill kernels (prefill.hip,
// prefill_chunk.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace damp {

struct PrefillParams {
  uint8_t* layer_base;
  uint64_t slot_stride;
  uint64_t tile_stride;
  const int32_t* slot_idx;
  const uint16_t* q;  // [B, t_pitch, HK, D]
  const uint16_t* k;
  const uint16_t* v;  // [B, t_pitch, HV, D]
  const uint16_t* g;  // [B, t_pitch, HV] or [B, t_pitch, HV, D]
  const uint16_t* beta;  // [B, t_pitch, HV]
  const uint8_t* perm;
  void* o;  // [B, T, HV, D], or NULL: no outputs
  float scale;
  int32_t T;        // tokens run by this launch
  int32_t t_pitch;  // tokens per request in the input arrays
  int32_t t0;       // first input token of this launch
  int32_t num_slots;
  int32_t HK;
  int32_t HV;
  int32_t k_hi;
  int32_t o_bf16;
  int32_t had;
};

// The d = 128 kernel of prefill_chunk.hip for a layout codec (internal.hpp).
void launch_prefill_chunk128(int codec, bool kda, const PrefillParams& p, int B,
                             hipStream_t stream);

}  // namespace damp
