// FOP cross-attention of a few rows with its projections folded into the keys and values.
//
// An adapter computes x += tanh(alpha) W_o softmax((W_q y) K^T scale) V.  K and V (the FOP
// tokens') do not depend on x, so per head KW = K W_q (n_fop x w) and VW = V W_o^T (w x
// n_fop) are formed once per step for every adapter layer, in one launch off the layers'
// chain, and a layer is left with the scores y KW^T and their softmax (one launch), P VW and
// the residual/norm kernel, over nq n_fop rows of weights instead of 2 nq hd.
//
// Precision: KW is rounded to bf16 once, as q is otherwise.  VW and P are held as two bf16
// parts (value, remainder): otherwise it is the attention rows that are rounded, after the
// softmax has averaged the tokens; rounding every token's VW instead leaves its error where
// the tokens' values cancel, and the same error in all Euler steps of a chunk.  Errors of
// velocities and chunks against 64 bits, folded over unfolded, 60 inputs: one part each
// +0.7 +-0.2 % (2 layers of 1024), +0.4 +-0.1 (6 layers, 4 envs), +1.9 +-0.3 (chunk, 4 layers of
// 1024), +4.1 +-0.9 (chunk, 4 layers of 512); two parts -1.3, -1.5, -0.5 and -1.9 %.  What the
// remainders cost a step, us: 18 layers of 1024, one env 979 -> 980, 6 layers, 4 envs 488 -> 493,
// 6 layers of 512, one env 226 -> 229.
#include "kernels.h"

namespace ravel {

bool adapter_fold_ok(int w, int nq, int hd, int n_fop) {
  return w % 128 == 0 && w <= 1024 && hd % 32 == 0 && hd <= 256 && n_fop >= 1 && n_fop <= 32 && nq * n_fop <= 128;
}

// What bf16(x) leaves of x; 0 where that is not finite.
RAVEL_DEV float remainder_of(float x) {
  const float h = bf16_to_f32(f32_to_bf16(x));
  return fabsf(h) < INFINITY ? x - h : 0.f;
}

// KW[e][a][h F + f][n] = sum_d K[f][d] W_q[h hd + d][n], VW[e][a][n][h F + f] = sum_d V[f][d]
// W_o[n][h hd + d].  A wave owns 16 columns n of one head: its weights' rows (W_q transposed,
// W_o) are read once, all at a time; bound by the weights' bytes (8.4 MB per adapter at
// width 1024, 8 heads of 256).  FR: 16-row fragments of the n_fop tokens.
template <int FR>
__global__ __launch_bounds__(256) void adapter_fold_kernel(AdapterArgs a) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, grp = lane >> 4;
  const int h = blockIdx.y, side = blockIdx.z & 1, ad = (blockIdx.z >> 1) % a.n_ad, e = (blockIdx.z >> 1) / a.n_ad;
  const int qd = a.nq * a.hd, kvd = a.nkv * a.hd, ld = a.n_ad * 2 * kvd, g = h / (a.nq / a.nkv);
  const int n0 = blockIdx.x * 64 + wave * 16, steps = a.hd / 32;
  const bf16_t* wr = (side ? a.wo : a.wqT) + ((size_t)ad * a.w + n0 + l16) * qd + h * a.hd + grp * 8;
  const bf16_t* kr = a.kva + (size_t)e * a.F * ld + ad * 2 * kvd + side * kvd + g * a.hd + grp * 8;
  bf16x8_t wf[8], kf[8][FR];
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const int o = min(s, steps - 1) * 32;
    wf[s] = *(const bf16x8_t*)(wr + o);
#pragma unroll
    for (int f = 0; f < FR; ++f) kf[s][f] = *(const bf16x8_t*)(kr + (size_t)min(f * 16 + l16, a.F - 1) * ld + o);
  }
  __builtin_amdgcn_sched_barrier(0);
  f32x4_t acc[FR];
#pragma unroll
  for (int f = 0; f < FR; ++f) acc[f] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const size_t ea = (size_t)e * a.n_ad + ad;
  if (side == 0) {
#pragma unroll
    for (int s = 0; s < 8; ++s)
      if (s < steps)
#pragma unroll
        for (int f = 0; f < FR; ++f) acc[f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[s], kf[s][f], acc[f], 0, 0, 0);
    // acc[f][r]: column n0 + 4 grp + r of token 16 f + l16
#pragma unroll
    for (int f = 0; f < FR; ++f) {
      const int t = f * 16 + l16;
      if (t >= a.F) continue;
      const u32x2_t v = {pack_bf16x2(acc[f][0], acc[f][1]), pack_bf16x2(acc[f][2], acc[f][3])};
      *(u32x2_t*)(a.kw + (ea * a.Jp + h * a.F + t) * a.w + n0 + grp * 4) = v;
    }
  } else {
#pragma unroll
    for (int s = 0; s < 8; ++s)
      if (s < steps)
#pragma unroll
        for (int f = 0; f < FR; ++f) acc[f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[s][f], wf[s], acc[f], 0, 0, 0);
    // acc[f][r]: token 16 f + 4 grp + r, column n0 + l16
    bf16_t* vr = a.vw + (ea * a.w + n0 + l16) * 2 * a.Jp + h * a.F;
    const bool quads = a.F % 4 == 0;  // 8-byte stores: 27 -> 24 us (9 adapters of 1024, one env), 32 -> 28 (4 envs, 3 adapters)
#pragma unroll
    for (int f = 0; f < FR; ++f) {
      const int t = f * 16 + grp * 4;
      if (quads) {
        if (t >= a.F) continue;
        *(u32x2_t*)(vr + t) = u32x2_t{pack_bf16x2(acc[f][0], acc[f][1]), pack_bf16x2(acc[f][2], acc[f][3])};
        *(u32x2_t*)(vr + a.Jp + t) = u32x2_t{pack_bf16x2(remainder_of(acc[f][0]), remainder_of(acc[f][1])),
                                             pack_bf16x2(remainder_of(acc[f][2]), remainder_of(acc[f][3]))};
        continue;
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (t + r >= a.F) continue;
        vr[t + r] = f32_to_bf16(acc[f][r]);
        vr[a.Jp + t + r] = f32_to_bf16(remainder_of(acc[f][r]));
      }
    }
  }
}

// P[row][h F + f] = softmax_f(y[row] . KW[h F + f] scale): 16 rows of one env and one head per
// block, four waves adding quarters of K through LDS, 16 threads per row for the softmax.
template <int FR>
__global__ __launch_bounds__(256) void adapter_scores_kernel(AdapterArgs a) {
  __shared__ __attribute__((aligned(16))) float part[4][16][FR * 16 + 4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, grp = lane >> 4;
  const int i0 = blockIdx.x * 16, h = blockIdx.y, e = blockIdx.z, steps = a.w / 128;
  const int k0 = wave * (a.w / 4) + grp * 8;
  const bf16_t* py = a.y + ((size_t)e * a.H + min(i0 + l16, a.H - 1)) * a.w + k0;
  const bf16_t* pw = a.kw + (((size_t)e * a.n_ad + a.ad) * a.Jp + h * a.F) * a.w + k0;
  bf16x8_t yf[8], wf[8][FR];
#pragma unroll
  for (int s = 0; s < 8; ++s) {  // w <= 1024: at most 8 steps
    const int o = min(s, steps - 1) * 32;
    yf[s] = *(const bf16x8_t*)(py + o);
#pragma unroll
    for (int f = 0; f < FR; ++f) wf[s][f] = *(const bf16x8_t*)(pw + (size_t)min(f * 16 + l16, a.F - 1) * a.w + o);
  }
  __builtin_amdgcn_sched_barrier(0);
  f32x4_t acc[FR];
#pragma unroll
  for (int f = 0; f < FR; ++f) acc[f] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < 8; ++s)
    if (s < steps)
#pragma unroll
      for (int f = 0; f < FR; ++f) acc[f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[s][f], yf[s], acc[f], 0, 0, 0);
#pragma unroll
  for (int f = 0; f < FR; ++f) *(f32x4_t*)&part[wave][l16][f * 16 + grp * 4] = acc[f];
  __syncthreads();
  const int i = tid >> 4, c = tid & 15;
  float s[FR], m = -INFINITY, sum = 0.f;
#pragma unroll
  for (int f = 0; f < FR; ++f) {
    const int t = f * 16 + c;
    s[f] = ((part[0][i][t] + part[1][i][t]) + (part[2][i][t] + part[3][i][t])) * (a.scale * 1.4426950408889634f);
    if (t >= a.F) s[f] = -INFINITY;
    m = fmaxf(m, s[f]);
  }
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
#pragma unroll
  for (int f = 0; f < FR; ++f) {
    s[f] = __builtin_amdgcn_exp2f(s[f] - m);
    sum += s[f];
  }
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
  if (i0 + i >= a.H) return;
  bf16_t* pr = a.p + ((size_t)e * a.H + i0 + i) * 2 * a.Jp + h * a.F;
#pragma unroll
  for (int f = 0; f < FR; ++f) {
    if (f * 16 + c >= a.F) continue;
    const float p = s[f] / sum;
    pr[f * 16 + c] = f32_to_bf16(p);
    pr[a.Jp + f * 16 + c] = f32_to_bf16(remainder_of(p));
  }
}

// out = P VW^T (fp32 rows; the residual kernel adds them and normalises), the product of the two
// remainders left out: 16 rows of one env and 64 columns per block, 16 columns per wave.  A
// block that owned whole rows, norm included, pulled 256 KB through one CU: 18.8 us, against
// 3.5 and 3.4 for the two (one part each).
__global__ __launch_bounds__(256) void adapter_out_kernel(AdapterArgs a, float* __restrict__ out) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, grp = lane >> 4;
  const int i0 = blockIdx.x * 16, n0 = blockIdx.y * 64 + wave * 16, e = blockIdx.z, steps = a.Jp / 32;
  const size_t row = (size_t)e * a.H + min(i0 + l16, a.H - 1);
  const bf16_t* pp = a.p + row * 2 * a.Jp + grp * 8;
  const bf16_t* pv = a.vw + (((size_t)e * a.n_ad + a.ad) * a.w + n0 + l16) * 2 * a.Jp + grp * 8;
  bf16x8_t pf[4][2], vf[4][2];
#pragma unroll
  for (int s = 0; s < 4; ++s) {  // nq n_fop <= 128: at most 4 steps
    const int o = min(s, steps - 1) * 32;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      pf[s][q] = *(const bf16x8_t*)(pp + q * a.Jp + o);
      vf[s][q] = *(const bf16x8_t*)(pv + q * a.Jp + o);
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  f32x4_t acc = {0.f, 0.f, 0.f, 0.f}, rem = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < 4; ++s)
    if (s < steps) {
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[s][0], pf[s][0], acc, 0, 0, 0);
      rem = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[s][1], pf[s][0], rem, 0, 0, 0);
      rem = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[s][0], pf[s][1], rem, 0, 0, 0);
    }
#pragma unroll
  for (int r = 0; r < 4; ++r) acc[r] += rem[r];
  if (i0 + l16 < a.H) *(f32x4_t*)(out + row * a.w + n0 + grp * 4) = acc;
}

static bool args_ok(const AdapterArgs& a) {
  return adapter_fold_ok(a.w, a.nq, a.hd, a.F) && a.nkv >= 1 && a.nq % a.nkv == 0 && a.Jp % 32 == 0 && a.Jp <= 128 &&
         a.Jp >= a.nq * a.F && a.B >= 1 && a.H >= 1 && a.n_ad >= 1 && a.ad >= 0 && a.ad < a.n_ad;
}

hipError_t launch_adapter_fold(const AdapterArgs& a, hipStream_t s) {
  if (!args_ok(a) || !a.kva || !a.wqT || !a.wo || !a.kw || !a.vw) return hipErrorInvalidValue;
  const dim3 grid(a.w / 64, a.nq, a.B * a.n_ad * 2);
  hipLaunchKernelGGL((a.F <= 16 ? adapter_fold_kernel<1> : adapter_fold_kernel<2>), grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_adapter_scores(const AdapterArgs& a, hipStream_t s) {
  if (!args_ok(a) || !a.y || !a.kw || !a.p) return hipErrorInvalidValue;
  const dim3 grid((a.H + 15) / 16, a.nq, a.B);
  hipLaunchKernelGGL((a.F <= 16 ? adapter_scores_kernel<1> : adapter_scores_kernel<2>), grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_adapter_out(const AdapterArgs& a, float* out, hipStream_t s) {
  if (!args_ok(a) || !a.p || !a.vw || !out) return hipErrorInvalidValue;
  hipLaunchKernelGGL(adapter_out_kernel, dim3((a.H + 15) / 16, a.w / 64, a.B), dim3(256), 0, s, a, out);
  return hipGetLastError();
}

// dst[c][r] = src[r][c] of an R x C matrix (weights, at model creation)
__global__ void transpose_bf16_kernel(const bf16_t* __restrict__ src, int R, int C, bf16_t* __restrict__ dst) {
  __shared__ bf16_t tile[32][34];
  const int c0 = blockIdx.x * 32, r0 = blockIdx.y * 32, tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int i = ty; i < 32; i += 8)
    if (r0 + i < R && c0 + tx < C) tile[i][tx] = src[(size_t)(r0 + i) * C + c0 + tx];
  __syncthreads();
  for (int i = ty; i < 32; i += 8)
    if (c0 + i < C && r0 + tx < R) dst[(size_t)(c0 + i) * R + r0 + tx] = tile[tx][i];
}

hipError_t launch_transpose_bf16(const bf16_t* src, int R, int C, bf16_t* dst, hipStream_t s) {
  hipLaunchKernelGGL(transpose_bf16_kernel, dim3((C + 31) / 32, (R + 31) / 32), dim3(256), 0, s, src, R, C, dst);
  return hipGetLastError();
}

}  // namespace ravel
