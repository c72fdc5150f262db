// The audit reduce by one workgroup, shared by pmpe_audit's kernel and by the combine kernel
// (whose extra block runs it beside the combine of the same layer forward).
//
// Each request gets the sum of its tokens' executed-private-row counts (64-bit integer sums,
// order independent) and its deny violations (tokens with allow == 0 and a nonzero count); a
// fixed-order reduction over the waves gives the total. All outputs are overwritten.
#pragma once
#include "pmpe_internal.h"

namespace pmpe {

// G requests of one wave at a time, the loads of their first 64 tokens issued together.
template <int G>
__device__ __forceinline__ void audit_requests(const AuditArgs& a, int r0, unsigned long long& wtot,
                                               unsigned int& wviol) {
  const int lane = threadIdx.x & 63;
  int lo[G], hi[G];
  uint32_t cnt[G], alw[G];
#pragma unroll
  for (int i = 0; i < G; ++i) {
    const int r = min(r0 + i, a.R - 1);
    lo[i] = min(max(a.req_offset[r], 0), a.T);
    hi[i] = min(max(a.req_offset[r + 1], lo[i]), a.T);
  }
#pragma unroll
  for (int i = 0; i < G; ++i) {
    const int t = min(lo[i] + lane, a.T - 1);  // past the request: read, not counted
    cnt[i] = a.rows[t];
    alw[i] = a.allow[t];
  }
  unsigned long long sum[G];
  unsigned int viol[G];
#pragma unroll
  for (int i = 0; i < G; ++i) {
    const bool in = lo[i] + lane < hi[i];
    sum[i] = in ? cnt[i] : 0;
    viol[i] = (in && alw[i] == 0 && cnt[i] > 0) ? 1u : 0u;
#pragma unroll 8
    for (int t = lo[i] + 64 + lane; t < hi[i]; t += 64) {  // unrolled: several loads in flight per lane
      const uint32_t v = a.rows[t];
      sum[i] += v;
      viol[i] += (a.allow[t] == 0 && v > 0) ? 1u : 0u;
    }
  }
  for (int off = 32; off > 0; off >>= 1) {
#pragma unroll
    for (int i = 0; i < G; ++i) {
      sum[i] += __shfl_xor(sum[i], off, 64);
      viol[i] += __shfl_xor(viol[i], off, 64);
    }
  }
#pragma unroll
  for (int i = 0; i < G; ++i) {
    if (r0 + i >= a.R) break;  // (the last request again: not counted)
    if (lane == 0) a.req_rows[r0 + i] = sum[i];
    wtot += sum[i];
    wviol += viol[i];
  }
}

// Every thread of a workgroup of WAVES waves. Short requests: one lane per request. Else one
// wave per request, or per four of them when every wave has several.
template <int WAVES>
__device__ __forceinline__ void audit_block(const AuditArgs& a) {
  __shared__ unsigned long long s_tot[WAVES];
  __shared__ unsigned int s_viol[WAVES];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  unsigned long long wtot = 0;
  unsigned int wviol = 0;
  // One lane per request where the requests are short: on average up to 16 tokens with at
  // least 256 of them, up to 4 with more than 16 (200 requests of one token: 15.1 -> 4.5 us;
  // 37 requests of 30 tokens stay with the waves, 4.8 us).
  if (a.T == 0 || a.T <= (int64_t)a.R * (a.R >= 256 ? 16 : a.R > 16 ? 4 : 0)) {
    for (int r = threadIdx.x; r < a.R; r += 64 * WAVES) {
      const int lo = min(max(a.req_offset[r], 0), a.T);
      const int hi = min(max(a.req_offset[r + 1], lo), a.T);
      unsigned long long sum = 0;
      for (int t = lo; t < hi; ++t) {
        const uint32_t v = a.rows[t];
        sum += v;
        wviol += (a.allow[t] == 0 && v > 0) ? 1u : 0u;
      }
      a.req_rows[r] = sum;
      wtot += sum;
    }
    for (int off = 32; off > 0; off >>= 1) {
      wtot += __shfl_xor(wtot, off, 64);
      wviol += __shfl_xor(wviol, off, 64);
    }
  } else if (a.R > 2 * WAVES) {
    for (int r = wave * 4; r < a.R; r += WAVES * 4) audit_requests<4>(a, r, wtot, wviol);
  } else {
    for (int r = wave; r < a.R; r += WAVES) audit_requests<1>(a, r, wtot, wviol);
  }
  if (lane == 0) {
    s_tot[wave] = wtot;
    s_viol[wave] = wviol;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long tot = 0;
    unsigned int viol = 0;
    for (int w = 0; w < WAVES; ++w) {
      tot += s_tot[w];
      viol += s_viol[w];
    }
    *a.total = tot;
    *a.violations = viol;
  }
}

}  // namespace pmpe
