// The audit reduce by one workgroup, shared by pmpe_audit's kernel and by the combine kernel
// (whose extra block runs it beside the combine of the same layer forward).
//
// Each request gets the sum of its tokens' executed-private-row counts (64-bit integer sums,
// order independent) and its deny violations (tokens with allow == 0 and a nonzero count); a
// fixed-order reduction over the waves gives the total. All outputs are overwritten.
#pragma once
#include "pmpe_internal.h"

namespace pmpe {

// Tokens [lo, hi) of request r, clamped to [0, T).
__device__ __forceinline__ void audit_span(const AuditArgs& a, int r, int& lo, int& hi) {
  lo = min(max(a.req_offset[r], 0), a.T);
  hi = min(max(a.req_offset[r + 1], lo), a.T);
}

// This lane's share of a wave's walk: the tokens t0, t0 + 64, ... below hi, U loads of each array
// in flight (past the end the last token is read again and not counted).
template <int U>
__device__ __forceinline__ void audit_tokens(const AuditArgs& a, int t0, int hi, unsigned long long& sum,
                                             unsigned int& viol) {
  for (int t = t0; t < hi; t += 64 * U) {
    uint32_t cnt[U], alw[U];
#pragma unroll
    for (int i = 0; i < U; ++i) {
      const int ti = min(t + i * 64, hi - 1);
      cnt[i] = a.rows[ti];
      alw[i] = a.allow[ti];
    }
#pragma unroll
    for (int i = 0; i < U; ++i) {
      const bool in = t + i * 64 < hi;
      sum += in ? cnt[i] : 0;
      viol += (in && alw[i] == 0 && cnt[i] > 0) ? 1u : 0u;
    }
  }
}

// One wave: request r of tokens [lo, hi) (the same in every lane, like what is added to the totals).
__device__ __forceinline__ void audit_request(const AuditArgs& a, int r, int lo, int hi, unsigned long long& wtot, unsigned int& wviol) {
  const int lane = threadIdx.x & 63;
  unsigned long long sum = 0;
  unsigned int viol = 0;
  if (hi - lo <= 64)
    audit_tokens<1>(a, lo + lane, hi, sum, viol);
  else if (hi - lo <= 256)
    audit_tokens<4>(a, lo + lane, hi, sum, viol);
  else
    audit_tokens<8>(a, lo + lane, hi, sum, viol);
  for (int off = 32; off > 0; off >>= 1) {
    sum += __shfl_xor(sum, off, 64);
    viol += __shfl_xor(viol, off, 64);
  }
  if (lane == 0) a.req_rows[r] = sum;
  wtot += sum;
  wviol += viol;
}

// The same for requests r0 .. r0 + 3 (T > 0, r0 < R), the loads of their first 64 tokens together.
__device__ __forceinline__ void audit_4_requests(const AuditArgs& a, int r0, unsigned long long& wtot, unsigned int& wviol) {
  constexpr int G = 4;
  const int lane = threadIdx.x & 63;
  int lo[G], hi[G];
  uint32_t cnt[G], alw[G];
  unsigned long long sum[G];
  unsigned int viol = 0;
#pragma unroll
  for (int i = 0; i < G; ++i) {
    audit_span(a, min(r0 + i, a.R - 1), lo[i], hi[i]);
    if (r0 + i >= a.R) hi[i] = lo[i];
  }
#pragma unroll
  for (int i = 0; i < G; ++i) {
    const int t = min(lo[i] + lane, a.T - 1);  // past the request: read, not counted
    cnt[i] = a.rows[t];
    alw[i] = a.allow[t];
  }
#pragma unroll
  for (int i = 0; i < G; ++i) {
    const bool in = lo[i] + lane < hi[i];
    sum[i] = in ? cnt[i] : 0;
    viol += (in && alw[i] == 0 && cnt[i] > 0) ? 1u : 0u;
    audit_tokens<4>(a, lo[i] + 64 + lane, hi[i], sum[i], viol);
  }
  for (int off = 32; off > 0; off >>= 1) {
#pragma unroll
    for (int i = 0; i < G; ++i) sum[i] += __shfl_xor(sum[i], off, 64);
    viol += __shfl_xor(viol, off, 64);
  }
#pragma unroll
  for (int i = 0; i < G; ++i) {
    if (lane == 0 && r0 + i < a.R) a.req_rows[r0 + i] = sum[i];
    wtot += sum[i];
  }
  wviol += viol;
}

// Every thread of a workgroup of WAVES waves. Up to 16 requests are walked by a wave each, and more
// of them where they are long on average (more than 4 tokens for up to 64 requests, 16 for up to
// 256, 64 for more: fewer than 16 waves with lanes at work would walk the longer ones in turn). Else
// a wave takes 64 requests at a time: those of up to 16 tokens (64 where it has many of 17 to 64) are
// walked by one lane each, all at once, and longer ones by the whole wave, one after the other. A
// token of a lane costs about 0.08 us, a request of a wave up to 0.8 us, both latency.
// (A rule on the mean length alone gave a long request among short ones to a lane: 200 requests of
// one token and one of 500 took 46 us, now 4; a list of the long ones for all waves costs every
// batch two block barriers, 10,000 requests of 1.6 tokens 14 us, now 9.)
template <int WAVES>
__device__ __forceinline__ void audit_block(const AuditArgs& a) {
  __shared__ unsigned long long s_tot[WAVES];
  __shared__ unsigned int s_viol[WAVES];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  unsigned long long wtot = 0;  // of the wave
  unsigned int wviol = 0;
  if (a.R <= 16 || a.T > (int64_t)a.R * (a.R <= 64 ? 4 : a.R <= 256 ? 16 : 64)) {
    if (WAVES < 16 && a.R > 2 * WAVES && a.T <= 128 * a.R) {  // many short ones for few waves
      for (int r = 4 * wave; r < a.R; r += 4 * WAVES) audit_4_requests(a, r, wtot, wviol);
    } else {
      for (int r = wave; r < a.R; r += WAVES) {
        int lo, hi;
        audit_span(a, r, lo, hi);
        audit_request(a, r, lo, hi, wtot, wviol);
      }
    }
  } else {
    unsigned long long ltot = 0;  // this lane's requests
    unsigned int lviol = 0;
    for (int r0 = wave * 64; r0 < a.R; r0 += 64 * WAVES) {
      const int r = r0 + lane;
      int lo = 0, hi = 0;
      if (r < a.R) audit_span(a, r, lo, hi);
      const int len = hi - lo;
      int limit = 16;
      uint64_t longer = __ballot(len > 16);
      if (longer != 0) {
        const uint64_t over64 = __ballot(len > 64);
        if (__popcll(longer) - __popcll(over64) > 5) {
          limit = 64;
          longer = over64;
        }
      }
      if (r < a.R && len <= limit) {
        unsigned long long sum = 0;
        for (int t = lo; t < hi; ++t) {
          const uint32_t v = a.rows[t];
          sum += v;
          lviol += (a.allow[t] == 0 && v > 0) ? 1u : 0u;
        }
        a.req_rows[r] = sum;
        ltot += sum;
      }
      for (; longer != 0; longer &= longer - 1) {
        const int i = __builtin_ctzll(longer);
        audit_request(a, r0 + i, __builtin_amdgcn_readlane(lo, i), __builtin_amdgcn_readlane(hi, i), wtot, wviol);
      }
    }
    for (int off = 32; off > 0; off >>= 1) {
      ltot += __shfl_xor(ltot, off, 64);
      lviol += __shfl_xor(lviol, off, 64);
    }
    wtot += ltot;
    wviol += lviol;
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
