// Epilogues and tile orders shared by the GEMM kernels.
#pragma once

#include "kernels.h"

namespace ravel {

// Epilogues.  Every MFMA result fragment here holds 4 consecutive output columns
// n .. n+3 of one row m per lane; epilogues are specialised by mode so that the
// fully unrolled fragment loops stay small (a large inlined switch there makes
// the compiler keep the accumulators in scratch memory).
template <int MODE, typename T>
RAVEL_DEV void epi1(const GemmArgs& a, int m, int n, float acc) {
  const float b = a.bias ? a.bias[n] : 0.0f;
  if constexpr (MODE == EPI_F32) {
    a.out_f[(size_t)m * a.ldo_f + n] = acc + b;
  } else if constexpr (MODE == EPI_T) {
    ((T*)a.out_t)[(size_t)m * a.ldo_t + n] = act<T>::from_f(acc + b);
  } else if constexpr (MODE == EPI_RESID) {
    const size_t gm = a.gate_rows ? (size_t)a.gate_rows[m] : (size_t)m;
    const float g = a.gate ? a.gate[gm * a.ldg + n] : 1.0f;
    float* o = a.out_f + (size_t)m * a.ldo_f + n;
    *o = *o + g * acc;
  } else if constexpr (MODE == EPI_RESID_TANH) {
    float* o = a.out_f + (size_t)m * a.ldo_f + n;
    *o = *o + tanhf(*a.gate_scalar) * acc;
  } else if constexpr (MODE == EPI_GELU_T) {
    ((T*)a.out_t)[(size_t)m * a.ldo_t + n] = act<T>::from_f(gelu_tanh_f(acc + b));
  } else if constexpr (MODE == EPI_SILU_T) {
    ((T*)a.out_t)[(size_t)m * a.ldo_t + n] = act<T>::from_f(silu_f(acc + b));
  }
}

// Whether the 4-column vector path applies to this launch (row strides aligned).
RAVEL_DEV bool epi_vec_ok(const GemmArgs& a) {
  switch (a.mode) {
    case EPI_F32: return (a.ldo_f % 4) == 0;
    case EPI_RESID: return (a.ldo_f % 4) == 0 && (!a.gate || (a.ldg % 4) == 0);
    case EPI_RESID_TANH: return (a.ldo_f % 4) == 0;
    case EPI_T:
    case EPI_GELU_T:
    case EPI_SILU_T: return (a.ldo_t % 4) == 0;
    default: return true;
  }
}

RAVEL_DEV void store_bf16x4(bf16_t* p, float v0, float v1, float v2, float v3) {
  u32x2_t w;
  w[0] = (uint32_t)f32_to_bf16(v0) | ((uint32_t)f32_to_bf16(v1) << 16);
  w[1] = (uint32_t)f32_to_bf16(v2) | ((uint32_t)f32_to_bf16(v3) << 16);
  *(u32x2_t*)p = w;
}

// bf16 activations; fp32 outputs are written as float4.
template <int MODE>
RAVEL_DEV void epi4(const GemmArgs& a, int m, int n, f32x4_t v, bool vec) {
  if (!(vec && n + 4 <= a.N)) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (n + r < a.N) epi1<MODE, bf16_t>(a, m, n + r, v[r]);
    return;
  }
  f32x4_t b = {0.f, 0.f, 0.f, 0.f};
  if (a.bias) b = *(const f32x4_t*)(a.bias + n);
  if constexpr (MODE == EPI_F32) {
    *(f32x4_t*)(a.out_f + (size_t)m * a.ldo_f + n) = f32x4_t{v[0] + b[0], v[1] + b[1], v[2] + b[2], v[3] + b[3]};
  } else if constexpr (MODE == EPI_T) {
    store_bf16x4((bf16_t*)a.out_t + (size_t)m * a.ldo_t + n, v[0] + b[0], v[1] + b[1], v[2] + b[2], v[3] + b[3]);
  } else if constexpr (MODE == EPI_RESID || MODE == EPI_RESID_TANH) {
    f32x4_t g = {1.f, 1.f, 1.f, 1.f};
    if constexpr (MODE == EPI_RESID_TANH) {
      const float t = tanhf(*a.gate_scalar);
      g = f32x4_t{t, t, t, t};
    } else {
      if (a.gate) g = *(const f32x4_t*)(a.gate + (a.gate_rows ? (size_t)a.gate_rows[m] : (size_t)m) * a.ldg + n);
    }
    f32x4_t* o = (f32x4_t*)(a.out_f + (size_t)m * a.ldo_f + n);
    f32x4_t x = *o;
    x[0] = x[0] + g[0] * v[0];
    x[1] = x[1] + g[1] * v[1];
    x[2] = x[2] + g[2] * v[2];
    x[3] = x[3] + g[3] * v[3];
    *o = x;
  } else if constexpr (MODE == EPI_GELU_T) {
    store_bf16x4((bf16_t*)a.out_t + (size_t)m * a.ldo_t + n, gelu_tanh_f(v[0] + b[0]), gelu_tanh_f(v[1] + b[1]),
                 gelu_tanh_f(v[2] + b[2]), gelu_tanh_f(v[3] + b[3]));
  } else if constexpr (MODE == EPI_SILU_T) {
    store_bf16x4((bf16_t*)a.out_t + (size_t)m * a.ldo_t + n, silu_f(v[0] + b[0]), silu_f(v[1] + b[1]),
                 silu_f(v[2] + b[2]), silu_f(v[3] + b[3]));
  }
}

// Gated GeLU of a gate fragment g and its up fragment u: columns f .. f+3 of row m.
RAVEL_DEV void epi_geglu4(const GemmArgs& a, int m, int f, f32x4_t g, f32x4_t u) {
  store_bf16x4((bf16_t*)a.out_t + (size_t)m * a.ldo_t + f, gelu_tanh_f(g[0]) * u[0], gelu_tanh_f(g[1]) * u[1],
               gelu_tanh_f(g[2]) * u[2], gelu_tanh_f(g[3]) * u[3]);
}

// Apply the epilogue to an NI x NJ grid of fragments: fragment (i, j) holds
// rows m0 + 16 i + l16 and columns n0 + 16 j + 4 grp .. +3.
template <int MODE, int NI, int NJ>
RAVEL_DEV void epi_frags(const GemmArgs& a, const f32x4_t (&acc)[NI][NJ], int m0, int n0, int l16, int grp) {
  const bool vec = epi_vec_ok(a);
  if constexpr (MODE == EPI_GEGLU) {
    if constexpr (NJ % 2 == 0) {
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; j += 2) {
          const int m = m0 + i * 16 + l16;
          const int ng = n0 + j * 16;  // gate block start (multiple of 32)
          if (m < a.M && ng < a.N) epi_geglu4(a, m, (ng >> 5) * 16 + grp * 4, acc[i][j], acc[i][j + 1]);
        }
    }
  } else {
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int m = m0 + i * 16 + l16, n = n0 + j * 16 + grp * 4;
        if (m < a.M && n < a.N) epi4<MODE>(a, m, n, acc[i][j], vec);
      }
  }
}

template <int NI, int NJ>
RAVEL_DEV void epilogue(const GemmArgs& a, const f32x4_t (&acc)[NI][NJ], int m0, int n0, int l16, int grp) {
  switch (a.mode) {
    case EPI_F32: epi_frags<EPI_F32>(a, acc, m0, n0, l16, grp); break;
    case EPI_T: epi_frags<EPI_T>(a, acc, m0, n0, l16, grp); break;
    case EPI_RESID: epi_frags<EPI_RESID>(a, acc, m0, n0, l16, grp); break;
    case EPI_RESID_TANH: epi_frags<EPI_RESID_TANH>(a, acc, m0, n0, l16, grp); break;
    case EPI_GEGLU: epi_frags<EPI_GEGLU>(a, acc, m0, n0, l16, grp); break;
    case EPI_GELU_T: epi_frags<EPI_GELU_T>(a, acc, m0, n0, l16, grp); break;
    case EPI_SILU_T: epi_frags<EPI_SILU_T>(a, acc, m0, n0, l16, grp); break;
    default: break;
  }
}

// Blocks are dispatched round-robin over the 8 XCDs (block b runs on XCD b % 8),
// each with its own L2.  Give every XCD a contiguous range of row-major tiles so
// that the tiles sharing an activation row panel share one L2.
RAVEL_DEV int xcd_tile(int b, int T) {
  const int x = b & 7, local = b >> 3;
  const int q = T >> 3, r = T & 7;  // XCD x owns q + (x < r) tiles
  const int start = x * q + (x < r ? x : r);
  return start + local;
}
// Row and column of tile t of a tiles_m x tiles_n grid ordered in groups of up to 8
// column tiles, row-major inside a group: an XCD's contiguous range of t covers a
// compact rectangle (about 8 x 8 tiles), so its L2 holds the activation row panels and
// the weight column panels it reads instead of every column panel of a wide output.
RAVEL_DEV void tile_rc(int t, int tiles_m, int tiles_n, int& r, int& c) {
  constexpr int GN = 8;
  const int g = t / (tiles_m * GN);
  const int gw = min(GN, tiles_n - g * GN);
  const int ti = t - g * tiles_m * GN;
  r = ti / gw;
  c = g * GN + ti % gw;
}

// Row tile, column tile and K range of work item t (tiles_m * tiles_n * ksplit of them).
// With few row tiles the weights are most of the bytes: the row tiles that share a
// weight panel are neighbours, so one XCD's L2 fetches the panel once.  With many,
// tile_rc's rectangles.
RAVEL_DEV void item_rcz(int t, int tiles_m, int tiles_n, int ksplit, int& r, int& c, int& z) {
  if (tiles_m <= 8) {
    r = t % tiles_m;
    const int q = t / tiles_m;
    z = q % ksplit;
    c = q / ksplit;
  } else {
    const int tiles = tiles_m * tiles_n;
    z = t / tiles;
    tile_rc(t - z * tiles, tiles_m, tiles_n, r, c);
  }
}

}  // namespace ravel
