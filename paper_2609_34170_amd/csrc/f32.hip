// fp32 models: GEMM and attention on the fp32 matrix instruction
// (v_mfma_f32_16x16x4_f32, IEEE fp32 products and sums).  Operands go straight from
// global memory to registers: a lane's float4 holds four k of one row, and step j of the
// instruction takes component j, so lane group g supplies k = 4 g + j -- the same
// assignment on both operands, which leaves the sum over k complete.  The waves of a
// block split K (the keys) and are added (merged) through LDS in fixed order.
// These models are small and their calls a chain of short launches, each bound by the
// latency of its loads: one thread per output with a serial K loop took 17 us at 8 rows,
// K = 128 and 64 us at 64 rows, N = K = 512.
#include <algorithm>

#include "gemm_epilogue.h"

namespace ravel {

namespace {

RAVEL_DEV f32x4_t mfma_f32(float a, float b, f32x4_t c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

template <bool VEC>
RAVEL_DEV f32x4_t load_k4(const float* row, int k, int kend) {
  f32x4_t v = {0.f, 0.f, 0.f, 0.f};
  if constexpr (VEC) {
    if (k < kend) v = *(const f32x4_t*)(row + k);  // K a multiple of 4
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (k + i < kend) v[i] = row[k + i];
  }
  return v;
}

RAVEL_DEV void epi_f32(const GemmArgs& a, int m, int n, float v) {
  switch (a.mode) {
    case EPI_F32: epi1<EPI_F32, float>(a, m, n, v); break;
    case EPI_T: epi1<EPI_T, float>(a, m, n, v); break;
    case EPI_RESID: epi1<EPI_RESID, float>(a, m, n, v); break;
    case EPI_RESID_TANH: epi1<EPI_RESID_TANH, float>(a, m, n, v); break;
    case EPI_GELU_T: epi1<EPI_GELU_T, float>(a, m, n, v); break;
    case EPI_SILU_T: epi1<EPI_SILU_T, float>(a, m, n, v); break;
    default: break;
  }
}

// Block: 16 MT rows x 16 NC columns, NW waves each over a K range of whole 16s.
template <int MT, int NC, int NW, bool VEC>
__global__ __launch_bounds__(64 * NW) void gemm_f32_kernel(GemmArgs a) {
  constexpr int U = MT * NC >= 8 ? 2 : 4;  // steps of 16 k whose loads are in flight together
  constexpr int FR = MT * NC;
  __shared__ __attribute__((aligned(16))) float red[NW][FR][64][4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, grp = lane >> 4;
  const int n0 = blockIdx.x * 16 * NC, m0 = blockIdx.y * 16 * MT;
  if (a.m_rows) a.M = min(a.M, *a.m_rows);
  if (m0 >= a.M) return;
  const int kq = ((a.K + NW - 1) / NW + 15) / 16 * 16;
  const int kb = wave * kq, ke = min(a.K, kb + kq);
  const float* ar[MT];
  const float* br[NC];
  // rows past M and columns past N repeat the last one: computed, never stored
#pragma unroll
  for (int i = 0; i < MT; ++i) ar[i] = (const float*)a.A + (size_t)min(m0 + i * 16 + l16, a.M - 1) * a.lda;
#pragma unroll
  for (int j = 0; j < NC; ++j) br[j] = (const float*)a.B + (size_t)min(n0 + j * 16 + l16, a.N - 1) * a.ldb;
  f32x4_t acc[NC][MT];
#pragma unroll
  for (int j = 0; j < NC; ++j)
#pragma unroll
    for (int i = 0; i < MT; ++i) acc[j][i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  for (int k0 = kb; k0 < ke; k0 += 16 * U) {
    f32x4_t wf[U][NC], xf[U][MT];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = k0 + u * 16 + grp * 4;
#pragma unroll
      for (int j = 0; j < NC; ++j) wf[u][j] = load_k4<VEC>(br[j], k, ke);
#pragma unroll
      for (int i = 0; i < MT; ++i) xf[u][i] = load_k4<VEC>(ar[i], k, ke);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int j = 0; j < NC; ++j)
#pragma unroll
          for (int i = 0; i < MT; ++i) acc[j][i] = mfma_f32(wf[u][j][r], xf[u][i][r], acc[j][i]);
  }
#pragma unroll
  for (int j = 0; j < NC; ++j)
#pragma unroll
    for (int i = 0; i < MT; ++i) *(f32x4_t*)&red[wave][j * MT + i][lane][0] = acc[j][i];
  __syncthreads();
  const auto sum = [&](int fr, int ln) {
    f32x4_t s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const f32x4_t v = *(const f32x4_t*)&red[w][fr][ln][0];
#pragma unroll
      for (int r = 0; r < 4; ++r) s[r] += v[r];
    }
    return s;
  };
  // item = fragment (j * MT + i) x lane: row i*16 + (lane & 15), columns j*16 + 4*(lane >> 4) .. +3
  for (int item = tid; item < FR * 64; item += 64 * NW) {
    const int fr = item >> 6, ln = item & 63, j = fr / MT, i = fr % MT;
    const int m = m0 + i * 16 + (ln & 15), n = n0 + j * 16 + (ln >> 4) * 4;
    if (m >= a.M) continue;
    const f32x4_t s = sum(fr, ln);
    if (a.mode == EPI_GEGLU) {
      if constexpr (NC % 2 == 0) {  // even column blocks are gates, the next one their ups
        if ((j & 1) || n >= a.N) continue;
        const f32x4_t u = sum(fr + MT, ln);
        float* o = (float*)a.out_t + (size_t)m * a.ldo_t + ((n0 + j * 16) >> 1) + (ln >> 4) * 4;
#pragma unroll
        for (int r = 0; r < 4; ++r) o[r] = gelu_tanh_f(s[r]) * u[r];
      }
      continue;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (n + r < a.N) epi_f32(a, m, n + r, s[r]);
  }
}

template <int MT, int NC, int NW>
hipError_t launch_f32_tile(const GemmArgs& a, hipStream_t s) {
  const dim3 grid((a.N + 16 * NC - 1) / (16 * NC), (a.M + 16 * MT - 1) / (16 * MT));
  const bool vec = a.K % 4 == 0 && a.lda % 4 == 0 && a.ldb % 4 == 0 && ((uintptr_t)a.A | (uintptr_t)a.B) % 16 == 0;
  if (vec)
    hipLaunchKernelGGL((gemm_f32_kernel<MT, NC, NW, true>), grid, dim3(64 * NW), 0, s, a);
  else
    hipLaunchKernelGGL((gemm_f32_kernel<MT, NC, NW, false>), grid, dim3(64 * NW), 0, s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm_f32(const GemmArgs& a, hipStream_t s) {
  if (a.M < 1 || a.N < 1 || a.K < 1 || (a.mode == EPI_GEGLU && a.N % 32)) return hipErrorInvalidValue;
  // the largest tile that still gives a block per CU; smaller ones re-read the operands
  // more but the caches hold them
  const auto blocks = [&](int bm, int bn) { return (long long)((a.M + bm - 1) / bm) * ((a.N + bn - 1) / bn); };
  if (blocks(64, 64) >= 256) return launch_f32_tile<4, 4, 4>(a, s);
  if (blocks(32, 32) >= 256) return launch_f32_tile<2, 2, 4>(a, s);
  if (a.mode == EPI_GEGLU) return launch_f32_tile<1, 2, 8>(a, s);
  return launch_f32_tile<1, 1, 8>(a, s);
}

// ---------------------------------------------------------------------------
// Attention: one block per (16 rows of a KV head's queries, KV head, env); row =
// h * Hq + query over the group's heads.  Wave w takes the 16-key blocks w, w + NW, ...
// S^T = K Q^T leaves each lane four keys of one row; P^T is the second product's B
// operand as it stands (step j: key 4 g + j), and V's rows its A operand, read in
// 64-byte pieces.  NF = hd / 16.
// ---------------------------------------------------------------------------
namespace {

template <int NF>
__global__ __launch_bounds__(256) void attn_f32_kernel(AttnArgs a, int chunks) {
  constexpr int HD = NF * 16, NW = 4;
  __shared__ __attribute__((aligned(16))) float so[NW][16][HD + 4];
  __shared__ float sml[NW][16][2];
  const int chunk = blockIdx.x % chunks, g = (blockIdx.x / chunks) % a.nkv, e = blockIdx.x / (chunks * a.nkv);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, grp = lane >> 4;
  const int G = a.nq / a.nkv, R = G * a.Hq;
  const int row = chunk * 16 + l16;
  const int slot = a.slot ? a.slot[e] : 0;
  const float* pk = (const float*)a.pk + slot * a.p_slot_stride + e * a.p_env_stride + g * HD;
  const float* pv = (const float*)a.pv + slot * a.p_slot_stride + e * a.p_env_stride + g * HD;
  const float* sk = (const float*)a.sk + (long long)e * a.S * a.s_ld + g * HD;
  const float* sv = (const float*)a.sv + (long long)e * a.S * a.s_ld + g * HD;
  const auto key_row = [&](const float* p, const float* s, int k) {
    return k < a.P ? p + (long long)k * a.p_ld : s + (long long)(k - a.P) * a.s_ld;
  };
  f32x4_t q[NF], o[NF];
  {
    const int r = min(row, R - 1);  // rows past the group are computed and never stored
    const float* qr = (const float*)a.q + (size_t)(e * a.Hq + r % a.Hq) * a.ldq + (g * G + r / a.Hq) * HD + grp * 4;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      q[f] = *(const f32x4_t*)(qr + f * 16);
      o[f] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
  }
  float m = -INFINITY, l = 0.f;
  const int nkeys = a.P + a.S;
  for (int k0 = wave * 16; k0 < nkeys; k0 += NW * 16) {
    const float* kr = key_row(pk, sk, min(k0 + l16, nkeys - 1)) + grp * 4;
    f32x4_t kf[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) kf[f] = *(const f32x4_t*)(kr + f * 16);
    const float* vr[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) vr[j] = key_row(pv, sv, min(k0 + grp * 4 + j, nkeys - 1)) + l16;
    f32x4_t s[2] = {f32x4_t{0.f, 0.f, 0.f, 0.f}, f32x4_t{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
      for (int r = 0; r < 4; ++r) s[r & 1] = mfma_f32(kf[f][r], q[f][r], s[r & 1]);
    // s[.][r]: key k0 + 4 grp + r of this lane's row
    float x[4], mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      x[r] = k0 + grp * 4 + r < nkeys ? (s[0][r] + s[1][r]) * a.scale : -INFINITY;
      mx = fmaxf(mx, x[r]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float mnew = fmaxf(m, mx);
    // without a finite score so far (keys whose products overflow): probabilities 0
    const float mref = mnew == -INFINITY ? 0.f : mnew;
    const float corr = expf(m - mref);
    float p[4], ps = 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      p[r] = expf(x[r] - mref);
      ps += p[r];
    }
    ps += __shfl_xor(ps, 16, 64);
    ps += __shfl_xor(ps, 32, 64);
    l = l * corr + ps;
    m = mnew;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
#pragma unroll
      for (int r = 0; r < 4; ++r) o[f][r] *= corr;
#pragma unroll
      for (int j = 0; j < 4; ++j) o[f] = mfma_f32(vr[j][f * 16], p[j], o[f]);
    }
  }
  // o[f][r]: dim f*16 + 4 grp + r of row l16
#pragma unroll
  for (int f = 0; f < NF; ++f) *(f32x4_t*)&so[wave][l16][f * 16 + grp * 4] = o[f];
  if (grp == 0) {
    sml[wave][l16][0] = m;
    sml[wave][l16][1] = l;
  }
  __syncthreads();
  for (int i = tid; i < 16 * HD; i += 256) {
    const int r = i / HD, d = i % HD, rr = chunk * 16 + r;
    if (rr >= R) break;
    float mm = sml[0][r][0];
#pragma unroll
    for (int w = 1; w < NW; ++w) mm = fmaxf(mm, sml[w][r][0]);
    float num = 0.f, den = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float wt = expf(sml[w][r][0] - mm);  // a wave without keys: 2^-inf = 0
      num += wt * so[w][r][d];
      den += wt * sml[w][r][1];
    }
    ((float*)a.out)[(size_t)(e * a.Hq + rr % a.Hq) * a.ldo + (g * G + rr / a.Hq) * HD + d] = num / den;
  }
}

template <int NF>
hipError_t launch_f32_hd(const AttnArgs& a, hipStream_t s) {
  const int chunks = (a.nq / a.nkv * a.Hq + 15) / 16;
  hipLaunchKernelGGL((attn_f32_kernel<NF>), dim3(chunks * a.nkv * a.B), dim3(256), 0, s, a, chunks);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_attn_f32(const AttnArgs& a, hipStream_t s) {
  if (a.hd > 256 || a.hd < 32 || a.hd % 32 || a.nkv < 1 || a.nq % a.nkv || a.P + a.S < 1 || a.ldq % 4 || a.p_ld % 4 ||
      a.s_ld % 4)
    return hipErrorInvalidValue;
  switch (a.hd / 32) {
    case 1: return launch_f32_hd<2>(a, s);
    case 2: return launch_f32_hd<4>(a, s);
    case 3: return launch_f32_hd<6>(a, s);
    case 4: return launch_f32_hd<8>(a, s);
    case 5: return launch_f32_hd<10>(a, s);
    case 6: return launch_f32_hd<12>(a, s);
    case 7: return launch_f32_hd<14>(a, s);
    default: return launch_f32_hd<16>(a, s);
  }
}

}  // namespace ravel
