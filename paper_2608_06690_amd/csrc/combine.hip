// K4 - combine: out[t] = sum_{j<k} gate[t,j] * y_perm[token_row[t,j]] (+ y_shared[t]).
//
// One workgroup per token; each thread owns 8 consecutive bf16 (or 4 fp32) columns,
// loaded as 16-byte vectors, so every y_perm row is read with full coalescing. The
// sum runs in fp32 in slot order j = 0..k-1 and is rounded once, which makes the
// output bitwise deterministic (no atomics). Slots with token_row = -1 (an invalid
// expert id upstream) contribute nothing.
//
// In a layer forward an extra first block may run the audit reduce: it needs only the expert
// FFN's counters, so it finishes beside the combine instead of after it (3 to 11 us of a launch of
// its own). The caller decides where that pays.
#include "audit_block.h"

namespace pmpe {
namespace {

constexpr int CB_THREADS = 256;

// KC > 0: top-k fixed at compile time, so the k row loads of a token are issued
// together (rows and gates first, then every slot's 16-byte vector) before the sum;
// KC == 0: any k, one slot at a time. Both add the slots in the same order.
// AUDIT: block 0 reduces the audit, block t + 1 combines token t.
template <int KC, bool AUDIT>
__device__ __forceinline__ void combine_bf16(const CombineArgs& a, const AuditArgs& aud) {
  if (AUDIT && blockIdx.x == 0) {
    audit_block<CB_THREADS / 64>(aud);
    return;
  }
  const int t = AUDIT ? blockIdx.x - 1 : blockIdx.x;
  const int H = a.H;
  const uint16_t* yp = (const uint16_t*)a.y_perm;
  const uint16_t* ysh = (const uint16_t*)a.y_shared;
  uint16_t* out = (uint16_t*)a.out;
  int rows[KC > 0 ? KC : 1];
  float gs[KC > 0 ? KC : 1];
  if constexpr (KC > 0) {
#pragma unroll
    for (int j = 0; j < KC; ++j) {
      rows[j] = a.token_row[(size_t)t * KC + j];
      gs[j] = a.gate[(size_t)t * KC + j];
    }
  }
  for (int c = threadIdx.x * 8; c < H; c += CB_THREADS * 8) {
    float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if constexpr (KC > 0) {
      u32x4 v[KC];
#pragma unroll
      for (int j = 0; j < KC; ++j)  // a slot without a row (-1) loads row 0 and is skipped
        v[j] = *(const u32x4*)(yp + (size_t)(rows[j] < 0 ? 0 : rows[j]) * H + c);
#pragma unroll
      for (int j = 0; j < KC; ++j) {
        if (rows[j] < 0) continue;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          acc[2 * q] += gs[j] * bf16_to_f32(v[j][q] & 0xFFFFu);
          acc[2 * q + 1] += gs[j] * bf16_to_f32(v[j][q] >> 16);
        }
      }
    } else {
      for (int j = 0; j < a.k; ++j) {
        const int row = a.token_row[(size_t)t * a.k + j];
        if (row < 0) continue;
        const float g = a.gate[(size_t)t * a.k + j];
        const u32x4 v = *(const u32x4*)(yp + (size_t)row * H + c);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          acc[2 * q] += g * bf16_to_f32(v[q] & 0xFFFFu);
          acc[2 * q + 1] += g * bf16_to_f32(v[q] >> 16);
        }
      }
    }
    if (ysh) {
      const u32x4 v = *(const u32x4*)(ysh + (size_t)t * H + c);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        acc[2 * q] += bf16_to_f32(v[q] & 0xFFFFu);
        acc[2 * q + 1] += bf16_to_f32(v[q] >> 16);
      }
    }
    u32x4 o;
#pragma unroll
    for (int q = 0; q < 4; ++q) o[q] = pack_bf16x2(acc[2 * q], acc[2 * q + 1]);
    *(u32x4*)(out + (size_t)t * H + c) = o;
  }
}

template <bool AUDIT>
__device__ __forceinline__ void combine_f32(const CombineArgs& a, const AuditArgs& aud) {
  if (AUDIT && blockIdx.x == 0) {
    audit_block<CB_THREADS / 64>(aud);
    return;
  }
  const int t = AUDIT ? blockIdx.x - 1 : blockIdx.x;
  const int H = a.H;
  const float* yp = (const float*)a.y_perm;
  const float* ysh = (const float*)a.y_shared;
  float* out = (float*)a.out;
  for (int c = threadIdx.x * 4; c < H; c += CB_THREADS * 4) {
    float4 acc = make_float4(0, 0, 0, 0);
    for (int j = 0; j < a.k; ++j) {
      const int row = a.token_row[(size_t)t * a.k + j];
      if (row < 0) continue;
      const float g = a.gate[(size_t)t * a.k + j];
      const float4 v = *(const float4*)(yp + (size_t)row * H + c);
      acc.x += g * v.x;
      acc.y += g * v.y;
      acc.z += g * v.z;
      acc.w += g * v.w;
    }
    if (ysh) {
      const float4 v = *(const float4*)(ysh + (size_t)t * H + c);
      acc.x += v.x;
      acc.y += v.y;
      acc.z += v.z;
      acc.w += v.w;
    }
    *(float4*)(out + (size_t)t * H + c) = acc;
  }
}

// (a combine without the audit carries none of it: with the choice at run time it took up to 6 %
// more at narrow rows)
template <int KC>
__global__ __launch_bounds__(CB_THREADS) void combine_bf16_kernel(CombineArgs a) { combine_bf16<KC, false>(a, AuditArgs{}); }
template <int KC>
__global__ __launch_bounds__(CB_THREADS) void combine_bf16_audit_kernel(CombineArgs a, AuditArgs aud) { combine_bf16<KC, true>(a, aud); }
__global__ __launch_bounds__(CB_THREADS) void combine_f32_kernel(CombineArgs a) { combine_f32<false>(a, AuditArgs{}); }
__global__ __launch_bounds__(CB_THREADS) void combine_f32_audit_kernel(CombineArgs a, AuditArgs aud) { combine_f32<true>(a, aud); }

template <int KC>
void launch_bf16(const CombineArgs& a, hipStream_t s, const AuditArgs* audit) {
  if (audit)
    hipLaunchKernelGGL(combine_bf16_audit_kernel<KC>, dim3((unsigned)a.T + 1), dim3(CB_THREADS), 0, s, a, *audit);
  else
    hipLaunchKernelGGL(combine_bf16_kernel<KC>, dim3(a.T), dim3(CB_THREADS), 0, s, a);
}

}  // namespace

hipError_t launch_combine(const CombineArgs& a, hipStream_t s, const AuditArgs* audit) {
  if (a.act_bf16) {
    switch (a.k) {
      case 2: launch_bf16<2>(a, s, audit); break;
      case 6: launch_bf16<6>(a, s, audit); break;
      case 8: launch_bf16<8>(a, s, audit); break;
      default: launch_bf16<0>(a, s, audit); break;
    }
  } else if (audit) {
    hipLaunchKernelGGL(combine_f32_audit_kernel, dim3((unsigned)a.T + 1), dim3(CB_THREADS), 0, s, a, *audit);
  } else {
    hipLaunchKernelGGL(combine_f32_kernel, dim3(a.T), dim3(CB_THREADS), 0, s, a);
  }
  return hipGetLastError();
}

}  // namespace pmpe
