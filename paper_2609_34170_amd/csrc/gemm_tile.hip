// Launches of the LDS-tiled bf16 GEMM: which tile, how many K ranges.
#include "gemm_tile.h"

namespace ravel {

namespace {
struct TileShape {
  int bm, bn;
};
constexpr TileShape kTiles[] = {{128, 128}, {128, 64}, {64, 64}, {64, 32}, {32, 64}, {32, 32}};
enum { T128x128, T128x64, T64x64, T64x32, T32x64, T32x32 };
constexpr int kTargetItems = 224;  // close to one item per CU

int items_of(int t, int M, int N) {
  return ((M + kTiles[t].bm - 1) / kTiles[t].bm) * ((N + kTiles[t].bn - 1) / kTiles[t].bn);
}
}  // namespace

// (EPI_RESID is what residual GEMMs wider than kResidNormMaxW take: 800 rows x 5120, K = 5120
// 99 us, on register-staged tiles 899.)
bool tile_ok(const GemmArgs& a) {
  return a.M > 0 && a.N > 0 && a.K > 0 && a.K % 64 == 0 && a.lda % 8 == 0 && a.ldb % 8 == 0 &&
         ((uintptr_t)a.A % 16) == 0 && ((uintptr_t)a.B % 16) == 0 && (a.mode != EPI_GEGLU || a.N % 32 == 0) &&
         (a.mode != EPI_PART || a.N % 4 == 0);
}

// The largest tile that still gives about one item per CU: a larger tile moves fewer
// bytes per product (each CU pulls 50-130 GB/s from the L2s, which is what bounds few
// rows), a smaller one fills the chip.  K is split (EPI_PART only: the sums of the ranges
// are added by the residual kernel that follows) as far as the partial sums stay small
// against the weights: 8 ranges for up to 128 rows, 4 up to 256 (512 where K >= 4096),
// 2 up to 2048.  The ranges are whole K tiles, the last what is left (K = 6976 = 109 tiles at
// 4 layers of width 192, 16 rows: 235 us a step with one range, 157 with 8).  Measured per
// launch in a chain (us, one CU-filling choice against the next larger tile), weights from
// HBM: M = 50, N = 2560, K = 1024 6.0 (32x32) against 7.9 (64x64); M = 200, N = 8192 10.3
// (128x64) / 12.9 (128x128, half the CUs); M = 1200 31 (128x128) / 35 (64x64); with the
// residual kernel M = 200, N = 1024, K = 4096 11.8 (64x64, 4 ranges) / 16 (2 ranges); M =
// 1200 27.7 (2 ranges) / 30 (one).
TilePlan plan_tile(int M, int N, int K, int mode) {
  const int ks_max = mode != EPI_PART ? 1 : M <= 128 ? 8 : (M <= 256 || (M <= 512 && K >= 4096)) ? 4 : M <= 2048 ? 2 : 1;
  const auto chunk = [&](int ks) { return (K / 64 + ks - 1) / ks * 64; };
  TilePlan p{};
  for (int t = T128x128; t <= T32x32; ++t) {
    if (t == T32x64 && mode != EPI_GEGLU) continue;  // a gate block and its up block need 32 columns per wave
    if (t == T32x32 && mode == EPI_GEGLU) break;
    if (M <= 32 && kTiles[t].bm > 32 && mode != EPI_GEGLU) continue;  // 32 rows: half of a 64-row tile would be padding
    if (M <= 64 && kTiles[t].bm > 64) continue;
    int ks = 1;
    const auto enough = [&](int n) {
      // 128x128: two blocks share a CU; one and a bit (257 .. 399 items) leaves half the chip waiting
      return t == T128x128 ? n >= 400 || (n >= kTargetItems && n <= 256) : n >= kTargetItems;
    };
    const int tiles = items_of(t, M, N);
    // (whole K tiles a range, the last range what is left)
    while (!enough(tiles * ks) && ks * 2 <= ks_max && K / (ks * 2) >= 256 && (ks * 2 - 1) * chunk(ks * 2) < K) ks *= 2;
    p.tile = t;
    p.ksplit = ks;
    p.items = tiles * ks;
    if (enough(p.items)) break;
  }
  p.kchunk = chunk(p.ksplit);
  p.bm = kTiles[p.tile].bm;
  p.bn = kTiles[p.tile].bn;
  return p;
}

template <int MODE>
static hipError_t launch_mode(const GemmArgs& a, const TilePlan& p, hipStream_t s) {
  // stages by how many blocks share a CU's 160 KB: deeper where one or two do
  switch (p.tile) {
    case T128x128:
      return p.items <= 256 ? launch_tile_mode<128, 128, 2, 2, 3, MODE>(a, s)
                            : launch_tile_mode<128, 128, 2, 2, 2, MODE>(a, s);
    case T128x64: return launch_tile_mode<128, 64, 2, 2, 3, MODE>(a, s);
    case T64x64:
      return p.items <= 512 ? launch_tile_mode<64, 64, 2, 2, 4, MODE>(a, s)
                            : launch_tile_mode<64, 64, 2, 2, 3, MODE>(a, s);
    case T64x32: return launch_tile_mode<64, 32, 4, 1, 5, MODE>(a, s);
    case T32x64: return launch_tile_mode<32, 64, 2, 2, 5, MODE>(a, s);
    default:
      if constexpr (MODE != EPI_GEGLU) return launch_tile_mode<32, 32, 2, 2, 6, MODE>(a, s);
      return hipErrorInvalidValue;
  }
}

hipError_t launch_gemm_tile(GemmArgs a, const TilePlan& p, hipStream_t s) {
  if (!tile_ok(a) || p.kchunk % 64 || p.ksplit * p.kchunk < a.K || (p.ksplit - 1) * p.kchunk >= a.K || (p.ksplit > 1 && a.mode != EPI_PART))
    return hipErrorInvalidValue;
  a.ksplit = p.ksplit;
  a.kchunk = p.kchunk;
  if (a.m_rows) {
    // the distinct modulation rows (a device count) times many columns: a fixed grid of
    // two blocks per CU walks the live items, so each weight panel is fetched once per
    // row tile and XCD and dead row tiles cost nothing.  Tiles of 128 columns read fewer bytes
    // per product, and eight waves (two blocks: four per SIMD) hide each other's waits;
    // where one row of them would leave CUs idle, of 64 columns.  us, 128 / 64 columns, by
    // live rows: 112640 x 1024 50 rows 62 / 66, 250 111 / 136, 500 206 / 249; 28672 x 2048 100 rows
    // 46 / 41, 200 51 / 62, 300 80 / 87; 38912 x 1024 150 rows 47 / 42, 250 53 / 52, 500 75 / 94;
    // 19456 x 512 48 rows 12.8 / 11.9, 160 17.6 / 19.9.
    if (a.mode != EPI_F32 || a.ksplit != 1) return hipErrorInvalidValue;
    const bool wide = items_of(T128x128, 1, a.N) >= kTargetItems;
    const int items = items_of(wide ? T128x128 : T128x64, a.M, a.N);
    const dim3 grid(items < 512 ? items : 512);
    if (wide)
      hipLaunchKernelGGL((gemm_tile_kernel<128, 128, 4, 2, 2, EPI_F32, true>), grid, dim3(512), 0, s, a);
    else
      hipLaunchKernelGGL((gemm_tile_kernel<128, 64, 2, 2, 3, EPI_F32, true>), grid, dim3(256), 0, s, a);
    return hipGetLastError();
  }
  switch (a.mode) {
    case EPI_F32: return launch_mode<EPI_F32>(a, p, s);
    case EPI_T: return launch_mode<EPI_T>(a, p, s);
    case EPI_RESID: return launch_mode<EPI_RESID>(a, p, s);
    case EPI_RESID_TANH: return launch_mode<EPI_RESID_TANH>(a, p, s);
    case EPI_GEGLU: return launch_mode<EPI_GEGLU>(a, p, s);
    case EPI_GELU_T: return launch_mode<EPI_GELU_T>(a, p, s);
    case EPI_SILU_T: return launch_mode<EPI_SILU_T>(a, p, s);
    case EPI_PART: return launch_mode<EPI_PART>(a, p, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace ravel
