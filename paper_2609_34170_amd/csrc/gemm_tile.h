// Tiled bf16 GEMM, K tiles loaded straight into LDS (global_load_lds, 16 bytes per
// lane: no register staging and no LDS store instructions).  STAGES LDS buffers; tile
// kt + STAGES - 1 is in flight while tile kt is multiplied.  Rows are 64 bf16 (128
// bytes, unpadded); the 16-byte chunk c of row r sits at chunk position
// c ^ ((r >> 1) & 7), so the 16 rows read by one fragment load hit 16 distinct bank
// groups.  Loads clamp rows to the matrix (rows / columns past M / N only feed outputs
// that are never written); K and the K range must be multiples of 64.  The fragment
// reads are inline asm with an explicit LDS wait: as plain loads the compiler would
// wait for every global->LDS load in flight (including later stages) before each of
// them, and __syncthreads() would wait for them too, so the K loop uses s_barrier after
// an explicit wait for this wave's loads of the current tile.
#pragma once

#include "gemm_epilogue.h"

namespace ravel {

typedef __attribute__((address_space(3))) void lds_void_t;
typedef const __attribute__((address_space(1))) void gmem_void_t;

// wait until at most N of this wave's vector memory operations are outstanding
// (gfx9 s_waitcnt immediate; expcnt and lgkmcnt not waited for)
template <int N>
RAVEL_DEV void wait_vm() {
  __builtin_amdgcn_s_waitcnt((unsigned)((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8)));
}
// at most LATER tiles of L loads each outstanding, for a run-time LATER <= MAX
template <int L, int MAX>
RAVEL_DEV void wait_tiles(int later) {
  if constexpr (MAX == 0) {
    wait_vm<0>();
  } else {
    if (later >= MAX)
      wait_vm<MAX * L>();
    else
      wait_tiles<L, MAX - 1>(later);
  }
}

// MODE: the epilogue, fixed at compile time (a run-time switch over the modes makes
// the compiler keep the accumulators in scratch memory).  EPI_PART stores the K range's
// sums as they are; every other mode takes the whole K.
// ROWS: the row count is known on the device only (*a.m_rows): a fixed grid walks the
// items of the live row tiles.
template <int BM, int BN, int WM, int WN, int STAGES, int MODE, bool ROWS = false>
__global__ __launch_bounds__(64 * WM * WN) void gemm_tile_kernel(GemmArgs a) {
  constexpr int NW = WM * WN;
  constexpr int BK = 64;
  constexpr int TM = BM / (16 * WM), TN = BN / (16 * WN);
  constexpr int LA = BM / 8 / NW, LB = BN / 8 / NW;  // 1 KB (8-row) segments per wave per tile
  static_assert(LA >= 1 && LB >= 1 && (BM / 8) % NW == 0 && (BN / 8) % NW == 0, "segments per wave");
  static_assert(MODE != EPI_GEGLU || TN % 2 == 0, "a gate block and its up block in one wave");
  constexpr int AHEAD = STAGES - 1;
  static_assert(AHEAD >= 1 && (AHEAD - 1) * (LA + LB) <= 63, "stages");
  __shared__ __attribute__((aligned(1024))) bf16_t As[STAGES][BM * BK];
  __shared__ __attribute__((aligned(1024))) bf16_t Bs[STAGES][BN * BK];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, grp = lane >> 4;
  const int wm = wave / WN, wn = wave % WN;
  if constexpr (ROWS) a.M = min(a.M, *a.m_rows);
  const int tiles_n = (a.N + BN - 1) / BN, tiles_m = (a.M + BM - 1) / BM;
  const int items = tiles_m * tiles_n * a.ksplit;
  const bf16_t* __restrict__ A = (const bf16_t*)a.A;
  const bf16_t* __restrict__ B = (const bf16_t*)a.B;
  const int srow = lane >> 3, spos = lane & 7;  // lane -> (row in segment, chunk position)
  auto frag = [&](const bf16_t* base, int row, int c) -> bf16x8_t {
    const unsigned addr =
        (unsigned)(size_t)(const __attribute__((address_space(3))) bf16_t*)(&base[row * BK + ((c ^ ((row >> 1) & 7)) * 8)]);
    bf16x8_t v;
    asm volatile("ds_read_b128 %0, %1" : "=v"(v) : "v"(addr));
    return v;
  };

  for (int item = blockIdx.x; item < items; item += gridDim.x) {  // once, or (ROWS) several times
    int tr, tc, z;
    item_rcz(xcd_tile(item, items), tiles_m, tiles_n, a.ksplit, tr, tc, z);
    const int m0 = tr * BM, n0 = tc * BN;
    const int kbeg = z * a.kchunk;
    const int nk = (min(a.K, kbeg + a.kchunk) - kbeg) / BK;
    const bf16_t* pa[LA];
    const bf16_t* pb[LB];
#pragma unroll
    for (int i = 0; i < LA; ++i) {
      const int row = (wave * LA + i) * 8 + srow;
      pa[i] = A + (size_t)min(m0 + row, a.M - 1) * a.lda + kbeg + (spos ^ ((row >> 1) & 7)) * 8;
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
      const int row = (wave * LB + i) * 8 + srow;
      pb[i] = B + (size_t)min(n0 + row, a.N - 1) * a.ldb + kbeg + (spos ^ ((row >> 1) & 7)) * 8;
    }
    auto issue = [&](int kt, int st) {
#pragma unroll
      for (int i = 0; i < LB; ++i)
        __builtin_amdgcn_global_load_lds((gmem_void_t*)(pb[i] + kt * BK), (lds_void_t*)&Bs[st][(wave * LB + i) * 512], 16,
                                         0, 0);
#pragma unroll
      for (int i = 0; i < LA; ++i)
        __builtin_amdgcn_global_load_lds((gmem_void_t*)(pa[i] + kt * BK), (lds_void_t*)&As[st][(wave * LA + i) * 512], 16,
                                         0, 0);
    };
    f32x4_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < AHEAD; ++t)
      if (t < nk) issue(t, t);
    int st = 0;
    for (int kt = 0; kt < nk; ++kt) {
      // this wave's loads of tile kt are complete once at most the later tiles'
      // loads are outstanding (vector memory operations complete in order)
      wait_tiles<LA + LB, AHEAD - 1>(min(AHEAD - 1, nk - 1 - kt));
      __builtin_amdgcn_s_barrier();  // every wave's part of tile kt is in LDS; tile kt-1's buffer is free
      if (kt + AHEAD < nk) issue(kt + AHEAD, st == 0 ? STAGES - 1 : st - 1);
      const bf16_t* as = As[st];
      const bf16_t* bs = Bs[st];
      if (++st == STAGES) st = 0;
#pragma unroll
      for (int ks = 0; ks < BK / 32; ++ks) {
        bf16x8_t af[TM], bfr[TN];
#pragma unroll
        for (int i = 0; i < TM; ++i) af[i] = frag(as, wm * (BM / WM) + i * 16 + l16, ks * 4 + grp);
#pragma unroll
        for (int j = 0; j < TN; ++j) bfr[j] = frag(bs, wn * (BN / WN) + j * 16 + l16, ks * 4 + grp);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int i = 0; i < TM; ++i) asm volatile("" : "+v"(af[i]));
#pragma unroll
        for (int j = 0; j < TN; ++j) asm volatile("" : "+v"(bfr[j]));
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[j], af[i], acc[i][j], 0, 0, 0);
      }
    }
    // acc[i][j][r] = C[m0 + wm*(BM/WM) + i*16 + l16][n0 + wn*(BN/WN) + j*16 + grp*4 + r]
    // (the weights are the MFMA's A operand, so each lane owns 4 consecutive columns)
    const int mw = m0 + wm * (BM / WM), nw = n0 + wn * (BN / WN);
    if constexpr (MODE == EPI_PART) {
      float* out = a.partial + (size_t)z * a.M * a.N;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const int m = mw + i * 16 + l16, n = nw + j * 16 + grp * 4;
          if (m < a.M && n < a.N) *(f32x4_t*)(out + (size_t)m * a.N + n) = acc[i][j];
        }
    } else {
      epi_frags<MODE>(a, acc, mw, nw, l16, grp);
    }
    if constexpr (!ROWS) return;
    // every wave's LDS reads of this item completed before its MFMAs; the next item's
    // loads may overwrite the stages once all waves are here
    __syncthreads();
  }
}

template <int BM, int BN, int WM, int WN, int STAGES, int MODE>
hipError_t launch_tile_mode(const GemmArgs& a, hipStream_t s) {
  const int items = ((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN) * a.ksplit;
  hipLaunchKernelGGL((gemm_tile_kernel<BM, BN, WM, WN, STAGES, MODE>), dim3(items), dim3(64 * WM * WN), 0, s, a);
  return hipGetLastError();
}

}  // namespace ravel
