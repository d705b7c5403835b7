// Aggregation (FaaSMoE Sec. 3 and Sec. 4.2: the orchestrator aggregates what the expert blocks
// return).  out[t,:] = sum_j topk_w[t,j] * Yp[row_of_pair[t*K+j],:] + sigmoid(sg[t]) * S[t,:],
// where S may come as the separate outputs of the shared experts (n_parts tensors [T,H], added in
// fp32 in ascending order before the gate is applied).
//
// A gather, not a scatter: one workgroup per token reads its K expert rows (and the shared
// row) with 16-byte loads, accumulates in fp32 in slot order j = 0..K-1 and rounds once to
// bf16.  No atomics, so the result does not depend on which block produced a row or when.
#include "common.h"

namespace moe {

constexpr int COMBINE_KMAX = 16;

// <x[t,:], wgate>: one wave per token, fp32.
__device__ __forceinline__ float gate_dot(const bf16_t* __restrict__ x, const bf16_t* __restrict__ wgate, int t, int H, int lane) {
  float a = 0.0f;
  for (int c = lane; c < H / 8; c += 64) {
    const uint4 v = reinterpret_cast<const uint4*>(x + (size_t)t * H)[c];
    const uint4 g = reinterpret_cast<const uint4*>(wgate)[c];
    a = __builtin_fmaf(bf16_lo(v.x), bf16_lo(g.x), a); a = __builtin_fmaf(bf16_hi(v.x), bf16_hi(g.x), a);
    a = __builtin_fmaf(bf16_lo(v.y), bf16_lo(g.y), a); a = __builtin_fmaf(bf16_hi(v.y), bf16_hi(g.y), a);
    a = __builtin_fmaf(bf16_lo(v.z), bf16_lo(g.z), a); a = __builtin_fmaf(bf16_hi(v.z), bf16_hi(g.z), a);
    a = __builtin_fmaf(bf16_lo(v.w), bf16_lo(g.w), a); a = __builtin_fmaf(bf16_hi(v.w), bf16_hi(g.w), a);
  }
  return wave_sum(a);
}
// u = x + y of eight columns; 1 / sqrt(mean(u^2) + eps) of a row from its 256 threads' sums of squares; u * scale in bf16.
__device__ __forceinline__ void residual(uint4 a, uint4 b, float (&u)[8]) {
  u[0] = bf16_lo(a.x) + bf16_lo(b.x); u[1] = bf16_hi(a.x) + bf16_hi(b.x);
  u[2] = bf16_lo(a.y) + bf16_lo(b.y); u[3] = bf16_hi(a.y) + bf16_hi(b.y);
  u[4] = bf16_lo(a.z) + bf16_lo(b.z); u[5] = bf16_hi(a.z) + bf16_hi(b.z);
  u[6] = bf16_lo(a.w) + bf16_lo(b.w); u[7] = bf16_hi(a.w) + bf16_hi(b.w);
}
__device__ __forceinline__ float row_scale(float ss, int H, float eps) {
  __shared__ float s_part[4];
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = ss;
  __syncthreads();
  const float total = (s_part[0] + s_part[1]) + (s_part[2] + s_part[3]);
  return 1.0f / sqrtf(total / (float)H + eps);
}
__device__ __forceinline__ uint4 scaled(const float (&u)[8], float scale) {
  return uint4{pack_bf16x2(u[0] * scale, u[1] * scale), pack_bf16x2(u[2] * scale, u[3] * scale),
               pack_bf16x2(u[4] * scale, u[5] * scale), pack_bf16x2(u[6] * scale, u[7] * scale)};
}

// What the aggregation may do besides, where a launch of its own costs more than the work: FORM & 1: the gate logit is
// formed from x and wgate (nullptr: it is in sg) and left in sg; FORM & 2: the shared expert's down projection arrives as
// fp32 parts, which are added in ascending order and rounded to S (a few tokens); FORM & 4: the residual step behind the
// layer, next = bf16(u / sqrt(mean(u^2) + eps)) with u = x + out as residual_norm_kernel forms it, from the values at
// hand.  2048 tokens of H 2048: aggregation, gate logits and residual step 9.7 + 4.8 + 6.2 us in three launches, 16.9 in one.
struct CombineExtra { const float* part; int parts; const bf16_t* x; const bf16_t* wgate; bf16_t* S; float* sg; float eps; bf16_t* next; };

template <int FORM>
__global__ __launch_bounds__(256) void combine_kernel(const bf16_t* __restrict__ Yp,
                                                      const int32_t* __restrict__ row_of_pair,
                                                      const float* __restrict__ topk_w,
                                                      const bf16_t* __restrict__ S, int n_parts, long part_stride,
                                                      const float* __restrict__ sg, int H, int K,
                                                      bf16_t* __restrict__ out, CombineExtra form) {
  const int t = blockIdx.x;
  __shared__ int s_row[COMBINE_KMAX];
  __shared__ float s_w[COMBINE_KMAX];
  if (threadIdx.x < K) {
    s_row[threadIdx.x] = row_of_pair[(size_t)t * K + threadIdx.x];
    s_w[threadIdx.x] = topk_w[(size_t)t * K + threadIdx.x];
  }
  __shared__ float s_gate;
  if ((FORM & 1) && threadIdx.x < 64) {
    const int lane = threadIdx.x;
    const float logit = form.wgate != nullptr ? gate_dot(form.x, form.wgate, t, H, lane) : form.sg[t];
    if (lane == 0) {
      s_gate = logit;
      if (form.wgate != nullptr) form.sg[t] = logit;
    }
  }
  __syncthreads();
  float gate = 0.0f;
  if (FORM & 1) gate = 1.0f / (1.0f + expf(-s_gate));
  else if (S != nullptr) gate = 1.0f / (1.0f + expf(-sg[t]));

  float u[4][8];      // (FORM & 4: x + out of this thread's columns; H <= 8192)
  float ss = 0.0f;
  auto columns = [&](int c, float (&uc)[8]) {
    float acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = 0.0f;
    // the shared row and four expert rows at a time are requested before any of them is used
    // (the sum still takes the rows in slot order)
    uint4 vs = {0u, 0u, 0u, 0u};
    if (FORM & 2) {
      const long row = (long)t * H + 8 * c;
      float v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = form.part[row + i];
      for (int p = 1; p < form.parts; ++p) {
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] += form.part[row + (long)p * part_stride + i];
      }
      vs = uint4{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7])};
      *reinterpret_cast<uint4*>(form.S + row) = vs;
    } else if (S != nullptr) {
      vs = reinterpret_cast<const uint4*>(S + (size_t)t * H)[c];
    }
    float sh[8];
    if (n_parts > 1) {   // the shared experts' outputs come as separate tensors: summed first, in order
      sh[0] = bf16_lo(vs.x); sh[1] = bf16_hi(vs.x); sh[2] = bf16_lo(vs.y); sh[3] = bf16_hi(vs.y);
      sh[4] = bf16_lo(vs.z); sh[5] = bf16_hi(vs.z); sh[6] = bf16_lo(vs.w); sh[7] = bf16_hi(vs.w);
      for (int p = 1; p < n_parts; ++p) {
        const uint4 v = reinterpret_cast<const uint4*>(S + (size_t)p * part_stride + (size_t)t * H)[c];
        sh[0] += bf16_lo(v.x); sh[1] += bf16_hi(v.x); sh[2] += bf16_lo(v.y); sh[3] += bf16_hi(v.y);
        sh[4] += bf16_lo(v.z); sh[5] += bf16_hi(v.z); sh[6] += bf16_lo(v.w); sh[7] += bf16_hi(v.w);
      }
    }
    for (int j0 = 0; j0 < K; j0 += 4) {
      uint4 vv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (j0 + u < K) vv[u] = reinterpret_cast<const uint4*>(Yp + (size_t)s_row[j0 + u] * H)[c];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (j0 + u < K) {
          const uint4 v = vv[u];
          const float wj = s_w[j0 + u];
          acc[0] = __builtin_fmaf(wj, bf16_lo(v.x), acc[0]); acc[1] = __builtin_fmaf(wj, bf16_hi(v.x), acc[1]);
          acc[2] = __builtin_fmaf(wj, bf16_lo(v.y), acc[2]); acc[3] = __builtin_fmaf(wj, bf16_hi(v.y), acc[3]);
          acc[4] = __builtin_fmaf(wj, bf16_lo(v.z), acc[4]); acc[5] = __builtin_fmaf(wj, bf16_hi(v.z), acc[5]);
          acc[6] = __builtin_fmaf(wj, bf16_lo(v.w), acc[6]); acc[7] = __builtin_fmaf(wj, bf16_hi(v.w), acc[7]);
        }
      }
    }
    if (!(FORM & 2) && S != nullptr && n_parts > 1) {
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] = __builtin_fmaf(gate, sh[i], acc[i]);
    } else if ((FORM & 2) || S != nullptr) {
      const uint4 v = vs;
      acc[0] = __builtin_fmaf(gate, bf16_lo(v.x), acc[0]); acc[1] = __builtin_fmaf(gate, bf16_hi(v.x), acc[1]);
      acc[2] = __builtin_fmaf(gate, bf16_lo(v.y), acc[2]); acc[3] = __builtin_fmaf(gate, bf16_hi(v.y), acc[3]);
      acc[4] = __builtin_fmaf(gate, bf16_lo(v.z), acc[4]); acc[5] = __builtin_fmaf(gate, bf16_hi(v.z), acc[5]);
      acc[6] = __builtin_fmaf(gate, bf16_lo(v.w), acc[6]); acc[7] = __builtin_fmaf(gate, bf16_hi(v.w), acc[7]);
    }
    uint4 o;
    o.x = pack_bf16x2(acc[0], acc[1]);
    o.y = pack_bf16x2(acc[2], acc[3]);
    o.z = pack_bf16x2(acc[4], acc[5]);
    o.w = pack_bf16x2(acc[6], acc[7]);
    reinterpret_cast<uint4*>(out + (size_t)t * H)[c] = o;
    if (FORM & 4) {
      const uint4 xv = reinterpret_cast<const uint4*>(form.x + (size_t)t * H)[c];
      residual(xv, o, uc);
#pragma unroll
      for (int i = 0; i < 8; ++i) ss = __builtin_fmaf(uc[i], uc[i], ss);
    }
  };
  if constexpr ((FORM & 4) != 0) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (threadIdx.x + 256 * r < H / 8) columns(threadIdx.x + 256 * r, u[r]);
    const float scale = row_scale(ss, H, form.eps);
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (threadIdx.x + 256 * r < H / 8) reinterpret_cast<uint4*>(form.next + (size_t)t * H)[threadIdx.x + 256 * r] = scaled(u[r], scale);
  } else {
    for (int c = threadIdx.x; c < H / 8; c += 256) columns(c, u[0]);
  }
}

__global__ __launch_bounds__(256) void gate_dot_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ wgate,
                                                       int T, int H, float* __restrict__ sg) {
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= T) return;
  const float logit = gate_dot(x, wgate, t, H, threadIdx.x & 63);
  if ((threadIdx.x & 63) == 0) sg[t] = logit;
}

// Second kernel of a down projection whose K was cut: the fp32 parts are added in ascending order and rounded
// once to bf16.  The workgroups past the sums form the gate logits (wgate may be nullptr), which depend on
// neither and would otherwise be one more launch of their own (about 4 us behind each K-cut shared expert).
__global__ __launch_bounds__(256) void sum_parts_kernel(const float* __restrict__ part, int parts, long n4, bf16_t* __restrict__ C,
                                                        int sum_groups, const bf16_t* __restrict__ x,
                                                        const bf16_t* __restrict__ wgate, int T, int H,
                                                        float* __restrict__ sg) {
  if ((int)blockIdx.x >= sum_groups) {
    const int t = ((int)blockIdx.x - sum_groups) * 4 + (threadIdx.x >> 6);
    if (t >= T) return;
    const float logit = gate_dot(x, wgate, t, H, threadIdx.x & 63);
    if ((threadIdx.x & 63) == 0) sg[t] = logit;
    return;
  }
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= n4) return;
  const float4* p = reinterpret_cast<const float4*>(part);
  float4 s = p[i];
  for (int k = 1; k < parts; ++k) {
    const float4 v = p[i + (long)k * n4];
    s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
  }
  uint2 o;
  o.x = pack_bf16x2(s.x, s.y);
  o.y = pack_bf16x2(s.z, s.w);
  reinterpret_cast<uint2*>(C)[i] = o;
}

// out[t,:] = bf16( u / sqrt(mean_h(u^2) + eps) ),  u = x[t,:] + y[t,:] in fp32: the step between two
// MoE layers when layers are chained without attention.  One workgroup per token; the row stays in
// registers between the two passes (H <= 8192).
__global__ __launch_bounds__(256) void residual_norm_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ y,
                                                            int H, float eps, bf16_t* __restrict__ out) {
  const int t = blockIdx.x;
  float u[4][8];
  float ss = 0.0f;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int c = threadIdx.x + 256 * r;
    if (c < H / 8) {
      residual(reinterpret_cast<const uint4*>(x + (size_t)t * H)[c], reinterpret_cast<const uint4*>(y + (size_t)t * H)[c], u[r]);
#pragma unroll
      for (int i = 0; i < 8; ++i) ss = __builtin_fmaf(u[r][i], u[r][i], ss);
    }
  }
  const float scale = row_scale(ss, H, eps);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int c = threadIdx.x + 256 * r;
    if (c < H / 8) reinterpret_cast<uint4*>(out + (size_t)t * H)[c] = scaled(u[r], scale);
  }
}

int launch_residual_norm(const void* x, const void* y, int T, int H, float eps, void* out, hipStream_t st) {
  if (T == 0) return 0;
  hipLaunchKernelGGL(residual_norm_kernel, dim3(T), dim3(256), 0, st, (const bf16_t*)x, (const bf16_t*)y, H, eps,
                     (bf16_t*)out);
  return hipGetLastError() == hipSuccess ? 0 : -4;
}

template <int FORM>
static int launch_combine_t(const void* Yp, const int32_t* row_of_pair, const float* w, const void* S, int n_parts, const float* sg,
                            int T, int H, int K, void* out, const CombineExtra& form, hipStream_t st) {
  if (T == 0) return 0;
  hipLaunchKernelGGL(combine_kernel<FORM>, dim3(T), dim3(256), 0, st, (const bf16_t*)Yp, row_of_pair, w, (const bf16_t*)S, n_parts,
                     (long)T * H, sg, H, K, (bf16_t*)out, form);
  return hipGetLastError() == hipSuccess ? 0 : -4;
}

int launch_combine(const void* Yp, const int32_t* row_of_pair, const float* w, const void* S, int n_parts,
                   const float* sg, int T, int H, int K, void* out, hipStream_t st) {
  return launch_combine_t<0>(Yp, row_of_pair, w, S, n_parts, sg, T, H, K, out, CombineExtra{}, st);
}

int launch_combine_layer(const void* Yp, const int32_t* row_of_pair, const float* w, const float* part, int parts,
                         const void* x, const void* wgate, void* S, float* sg, int T, int H, int K, void* out, float eps,
                         void* next, hipStream_t st) {
  const CombineExtra form{part, parts, (const bf16_t*)x, (const bf16_t*)wgate, (bf16_t*)S, sg, eps, (bf16_t*)next};
  const int what = (wgate != nullptr || part != nullptr ? 1 : 0) + (part != nullptr ? 2 : 0) + (next != nullptr ? 4 : 0);
  const void* S_in = part != nullptr ? nullptr : S;
  switch (what) {
    case 0: return launch_combine_t<0>(Yp, row_of_pair, w, S_in, 1, sg, T, H, K, out, form, st);
    case 1: return launch_combine_t<1>(Yp, row_of_pair, w, S_in, 1, sg, T, H, K, out, form, st);
    case 3: return launch_combine_t<3>(Yp, row_of_pair, w, S_in, 1, sg, T, H, K, out, form, st);
    case 4: return launch_combine_t<4>(Yp, row_of_pair, w, S_in, 1, sg, T, H, K, out, form, st);
    case 5: return launch_combine_t<5>(Yp, row_of_pair, w, S_in, 1, sg, T, H, K, out, form, st);
    default: return launch_combine_t<7>(Yp, row_of_pair, w, S_in, 1, sg, T, H, K, out, form, st);
  }
}

int launch_sum_parts(const float* part, int parts, int T, int H, void* C, const void* x, const void* wgate, float* sg,
                     hipStream_t st) {
  const long n4 = (long)T * H / 4;
  const int sums = (int)((n4 + 255) / 256), gates = wgate != nullptr ? (T + 3) / 4 : 0;
  hipLaunchKernelGGL(sum_parts_kernel, dim3(sums + gates), dim3(256), 0, st, part, parts, n4, (bf16_t*)C, sums, (const bf16_t*)x,
                     (const bf16_t*)wgate, T, H, sg);
  return hipGetLastError() == hipSuccess ? 0 : -4;
}

int launch_gate_dot(const void* x, const void* wgate, int T, int H, float* sg, hipStream_t st) {
  if (T == 0) return 0;
  hipLaunchKernelGGL(gate_dot_kernel, dim3((T + 3) / 4), dim3(256), 0, st, (const bf16_t*)x, (const bf16_t*)wgate,
                     T, H, sg);
  return hipGetLastError() == hipSuccess ? 0 : -4;
}

}  // namespace moe
