// Attention of the buffer tokens over [prefix tokens ; buffer tokens] (and of
// the FOP adapters over FOP tokens), bidirectional, grouped-query heads.
//
// bf16 path (MFMA, wave64): one block per (key range, row chunk of a KV head's
// queries, KV head, env).  Key/value tiles are staged in LDS as they lie in memory and
// shared by the waves.  Scores are computed transposed, S^T = K Q^T, so that each lane of a
// score wave owns one query and the online softmax statistics stay in its registers; P^T goes
// through LDS to the output waves, in the shape of the second MFMA's operand (O^T += V^T P^T).
// With several key ranges, each block writes (m, l, unnormalised O) and a second kernel
// adds the ranges in fixed order.
#include <algorithm>

#include "kernels.h"

namespace ravel {

static constexpr float kLog2e = 1.4426950408889634f;

// ---------------------------------------------------------------------------
// Grouped-query attention.  The G = nq/nkv query heads that share one K/V head are
// flattened with the queries into one row space of G*Hq rows (row = h*Hq + query), cut
// into chunks of 16 NB rows (64 or 128).  A block of 2 NB waves owns one chunk of one
// (env, KV head) and walks the key tiles (TK keys).  The first NB waves ("score waves")
// compute the scores and probabilities of 16 rows each over all keys of tile t (so the
// softmax statistics never leave a wave) and put P^T in LDS in the shape of the second
// product's B operand; the others ("output waves") meanwhile compute O^T of tile t - 1,
// each for a quarter of the head's dims over 64 rows (a value fragment feeds four MFMAs).
// One barrier per tile, and each SIMD has both kinds of work to choose from.  One wave after
// the other through scores, softmax and output is a chain of ~2400 cycles per 32 keys at
// 256 dims whatever the memory does (measured with 7 blocks as with 168), and
// a wave that keeps all dims of its rows needs a body of 1000 instructions a tile, which a
// short launch walks cold (9.7 us for a single tile of 16 keys, 6.5 split by dims).
//
// K and V tiles go straight from global memory to LDS (16 bytes per lane, rows kept
// whole, their 16-byte chunks XOR-swizzled by row so that a fragment's 16 rows hit
// distinct banks), three buffers each: two tiles are in flight while one is computed on
// (one in flight costs a round trip of 0.6 us per tile, as long as the computation).  V's
// fragments are read transposed (ds_read_b64_tr_b16: 16 lanes fetch 4 keys x 16 dims and
// each receives one dim's 4 keys).  LDS accesses are inline asm with explicit waits: as
// plain loads and stores the compiler would wait for every global->LDS load in flight
// before each of them.
//
// Key tiles: the prefix rows padded to whole tiles, then the buffer's own rows, so that
// every tile reads one part from one uniform base.  Rows past a part's end repeat its
// last row (finite values) and are masked out of the softmax.
//
// Softmax rescaling is lazy: the running maximum m of a row only moves when a
// tile raises it by more than kLazy (log2 units), so between moves exp2(s - m)
// <= 2^kLazy and the O rescale is skipped unless one of the row block's rows moved (a
// flag and the factors go through LDS with P).  The result is the same softmax;
// only the reference point of the bf16-rounded probabilities differs.
//
// SPLIT: the tiles are cut into a.nsplit ranges (a.keys_per_split keys: whole tiles),
// for launches whose (row chunk, KV head, env) blocks alone leave CUs idle.
// ---------------------------------------------------------------------------
static constexpr float kLazy = 8.f;

typedef __attribute__((address_space(3))) void lds_void_t;
typedef const __attribute__((address_space(1))) void gmem_void_t;

RAVEL_DEV unsigned lds_addr(const void* p) {
  return (unsigned)(size_t)(const __attribute__((address_space(3))) char*)p;
}
template <int OFF>
RAVEL_DEV bf16x8_t lds_read_b128(unsigned addr) {
  bf16x8_t v;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
  return v;
}
template <int OFF>
RAVEL_DEV u32x2_t lds_read_tr(unsigned addr) {
  u32x2_t v;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
  return v;
}
// at most N LDS reads outstanding (they complete in order)
template <int N>
RAVEL_DEV void lds_wait() {
  asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(N) : "memory");
}
template <class V>
RAVEL_DEV void lds_ready(V& v) {  // a value whose read the last lds_wait covered: not used before here
  asm volatile("" : "+v"(v));
}

RAVEL_DEV void lds_write_b128(unsigned addr, u32x4_t v) {
  asm volatile("ds_write_b128 %0, %1" ::"v"(addr), "v"(v) : "memory");
}
RAVEL_DEV void lds_write_b32(unsigned addr, uint32_t v) {
  asm volatile("ds_write_b32 %0, %1" ::"v"(addr), "v"(v) : "memory");
}
RAVEL_DEV float lds_read_f32(unsigned addr) {  // waits
  float v;
  asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(v) : "v"(addr) : "memory");
  return v;
}

// at most N vector memory operations and no LDS operation outstanding (gfx9 encoding)
template <int N>
RAVEL_DEV void wait_vm_lds0() {
  __builtin_amdgcn_s_waitcnt((unsigned)((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4)));
}

template <int HD, int TK, int NB, bool SPLIT>
__global__ __launch_bounds__(NB * 128) void attn_gqa_kernel(AttnArgs a, int chunks) {
  constexpr int NW = 2 * NB;
  constexpr int KS = HD / 32;                 // k-steps of the score MFMA
  constexpr int DT = HD / 16;                 // 16-dim tiles of O^T
  constexpr int DW = DT >= 4 ? DT / 4 : 1;    // of them per output wave (HD = 32: two waves have one)
  constexpr int NS = TK / 16;                 // 16-key sub-tiles
  constexpr int NH = TK / 32;                 // 32-key steps of the second product
  constexpr int RB = HD * 2;                  // bytes of a row
  constexpr int CH = HD / 8;                  // 16-byte chunks of a row
  constexpr int TB = TK * RB;                 // bytes of a K (or V) tile
  constexpr int RP = RB >= 256 ? 1 : 256 / RB;  // rows per 256 bytes (all banks)
  constexpr int XK = (CH < 16 ? CH : 16) - 1;   // swizzle mask (chunks)
  constexpr int SEG = TB / 1024;                // 1 KB loads of a tile, spread over the waves
  constexpr int LPW = SEG > NW ? SEG / NW : 1;  // of them per wave (the first SEG waves where SEG < NW)
  constexpr int PD = KS < 8 / NS ? KS : 8 / NS;  // k-steps whose key fragments are in flight
  static_assert(TB % 1024 == 0 && NS <= 4 && (SEG % NW == 0 || SEG < NW) && (NB == 4 || NB == 8), "tile");
  __shared__ __attribute__((aligned(1024))) char ks_s[3][TB];
  __shared__ __attribute__((aligned(1024))) char vs_s[3][TB];
  __shared__ __attribute__((aligned(1024))) char pbuf[2][NB][NH][1024];
  __shared__ __attribute__((aligned(16))) float corr_s[2][NB][16];  // O's rescale factors; at the end 1 / l
  __shared__ __attribute__((aligned(16))) uint32_t flag_s[2][NB];

  // blocks that share an (env, KV head) sit on one XCD (dispatch is round-robin
  // over the 8 XCDs), so the group's K/V is fetched into one L2 only
  const int total = gridDim.x;
  const int L = blockIdx.x;
  const int w = (total % 8 == 0) ? (L % 8) * (total / 8) + L / 8 : L;
  const int chunk = w % chunks;
  const int split = SPLIT ? (w / chunks) % a.nsplit : 0;
  const int eg = SPLIT ? w / (chunks * a.nsplit) : w / chunks;
  const int g = eg % a.nkv;
  const int e = eg / a.nkv;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, grp = lane >> 4;
  const int G = a.nq / a.nkv;
  const int R = G * a.Hq;
  const int row0 = chunk * NB * 16;
  const bool score = wave < NB;
  // score wave: its row block; output wave: its quarter of the dims, its four row blocks from b0
  const int sub = score ? wave : wave & 3, b0 = score ? 0 : (wave - NB) & ~3;
  const int nb = min(score ? NB : 4, (R - row0 - b0 * 16 + 15) >> 4);  // row blocks with rows
  const bool work = score ? sub < nb : sub * DW < DT && nb > 0;

  const bf16_t* q = (const bf16_t*)a.q;
  const int slot = a.slot ? a.slot[e] : 0;
  const bf16_t* pk = (const bf16_t*)a.pk + slot * a.p_slot_stride + e * a.p_env_stride + g * HD;
  const bf16_t* pv = (const bf16_t*)a.pv + slot * a.p_slot_stride + e * a.p_env_stride + g * HD;
  const bf16_t* sk = (const bf16_t*)a.sk + (long long)e * a.S * a.s_ld + g * HD;
  const bf16_t* sv = (const bf16_t*)a.sv + (long long)e * a.S * a.s_ld + g * HD;

  const int ptiles = (a.P + TK - 1) / TK, ntiles = ptiles + (a.S + TK - 1) / TK;
  const int tbeg = SPLIT ? split * (a.keys_per_split / TK) : 0;
  const int tend = SPLIT ? min(ntiles, tbeg + a.keys_per_split / TK) : ntiles;

  // tile t of K (rot = 1) or V (rot = 2: its swizzle keeps chunk pairs together)
  auto issue = [&](const bf16_t* pre_base, const bf16_t* self_base, int rot, int t, char* dst) {
    const bool pre = t < ptiles;  // uniform
    const int r0 = (pre ? t : t - ptiles) * TK;
    const int last = (pre ? a.P : a.S) - 1;
    const long long ld = pre ? a.p_ld : a.s_ld;
    const bf16_t* base = pre ? pre_base : self_base;
#pragma unroll
    for (int i = 0; i < LPW; ++i) {
      const int seg = wave + i * NW;
      if (SEG < NW && seg >= SEG) break;
      const int p = seg * 64 + lane;  // 16-byte position in the tile
      const int r = p / CH, pos = p % CH;
      const int c = pos ^ ((rot * (r / RP)) & XK);
      __builtin_amdgcn_global_load_lds((gmem_void_t*)(base + min(r0 + r, last) * ld + c * 8),
                                       (lds_void_t*)(dst + seg * 1024), 16, 0, 0);
    }
  };
  issue(pk, sk, 1, tbeg, ks_s[0]);
  if (tbeg + 1 < tend) issue(pk, sk, 1, tbeg + 1, ks_s[1]);
  issue(pv, sv, 2, tbeg, vs_s[0]);

  const unsigned corr0 = lds_addr(&corr_s[0][0][0]), flag0 = lds_addr(&flag_s[0][0]);
  const unsigned p0 = lds_addr(&pbuf[0][0][0][0]), k0 = lds_addr(&ks_s[0][0]), v0 = lds_addr(&vs_s[0][0]);
  // K of tile t and V of tile t - 1 have landed (this wave's part: at most K of t + 1 and V
  // of t are outstanding), this wave's LDS writes are done; after the barrier everyone's
  // are, and the buffers of K of t - 1 and V of t - 2 are free.  nx: (t - tbeg + 2) mod 3.
  auto next = [&](int t, int nx) {
    const int later = (t + 1 < tend ? 1 : 0) + (t < tend ? 1 : 0);
    if (later == 2)
      wait_vm_lds0<2 * LPW>();
    else if (later == 1)
      wait_vm_lds0<LPW>();
    else
      wait_vm_lds0<0>();
    __builtin_amdgcn_s_barrier();
    if (t + 2 < tend) issue(pk, sk, 1, t + 2, ks_s[nx]);
    if (t + 1 < tend) issue(pv, sv, 2, t + 1, vs_s[nx == 0 ? 2 : nx - 1]);
  };

  if (score) {
    // rows past the group are clamped to a real row, computed and never used
    const int row = row0 + sub * 16 + l16;
    bf16x8_t qf[KS];
    {
      const int r = min(row, R - 1);
      const bf16_t* qr = q + (size_t)(e * a.Hq + r % a.Hq) * a.ldq + (g * G + r / a.Hq) * HD + grp * 8;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) qf[ks] = *(const bf16x8_t*)(qr + ks * 32);
    }
    float mrow = -INFINITY, lrow = 0.f;
    const float sl2 = a.scale * kLog2e;
    // fragment addresses inside a tile; k-step ks is XORed in (the swizzle only flips chunk bits)
    const unsigned ka0 = l16 * RB + ((grp ^ ((l16 / RP) & XK)) << 4);
    for (int t = tbeg, nx = 2; t <= tend; ++t, nx = nx == 2 ? 0 : nx + 1) {
      next(t, nx);
      const int buf = (t - tbeg) & 1;
      if (t == tend) break;
      if (!work) continue;
      const unsigned kt = k0 + (nx == 2 ? 0 : nx + 1) * TB + ka0;
      // S^T[key][row]; PD k-steps' fragments in flight
      bf16x8_t kf[PD][NS];
      auto read_k = [&](bf16x8_t(&f)[NS], int ks) {
        const unsigned ad = kt ^ (ks << 6);
#pragma unroll
        for (int u = 0; u < NS; ++u) {
          if (u == 0) f[u] = lds_read_b128<0>(ad);
          if (u == 1) f[u] = lds_read_b128<16 * RB>(ad);
          if (u == 2) f[u] = lds_read_b128<32 * RB>(ad);
          if (u == 3) f[u] = lds_read_b128<48 * RB>(ad);
        }
      };
#pragma unroll
      for (int ks = 0; ks < PD; ++ks) read_k(kf[ks], ks);
      f32x4_t s[NS];
#pragma unroll
      for (int u = 0; u < NS; ++u) s[u] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        // reads issued after this step's
        constexpr int M = PD - 1;
        const int later = KS - 1 - ks < M ? KS - 1 - ks : M;
        if (later == 0) lds_wait<0>();
        if (later == 1) lds_wait<NS>();
        if (later == 2) lds_wait<2 * NS>();
        if (later == 3) lds_wait<3 * NS>();
#pragma unroll
        for (int u = 0; u < NS; ++u) lds_ready(kf[ks % PD][u]);
#pragma unroll
        for (int u = 0; u < NS; ++u)
          s[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[ks % PD][u], qf[ks], s[u], 0, 0, 0);
        if (ks + PD < KS) read_k(kf[ks % PD], ks + PD);
      }
      // valid keys of the tile (uniform): the last tile of each part is ragged
      const int nvalid = t < ptiles ? a.P - t * TK : a.S - (t - ptiles) * TK;
      float x[4 * NS];
#pragma unroll
      for (int u = 0; u < NS; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r) x[4 * u + r] = s[u][r] * sl2;
      if (nvalid < TK) {
#pragma unroll
        for (int u = 0; u < NS; ++u)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (u * 16 + grp * 4 + r >= nvalid) x[4 * u + r] = -INFINITY;
      }
      float lmx = x[0];
#pragma unroll
      for (int r = 1; r < 4 * NS; ++r) lmx = fmaxf(lmx, x[r]);
      const bool move = __any(lmx > mrow + kLazy);
      if (move) {
        float mx = fmaxf(lmx, __shfl_xor(lmx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float mnew = mx > mrow + kLazy ? mx : mrow;
        const float corr = mrow == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mrow - mnew);
        mrow = mnew;
        lrow *= corr;
        if (grp == 0) lds_write_b32(corr0 + ((buf * NB + sub) * 16 + l16) * 4, __float_as_uint(corr));
      }
      if (lane == 0) lds_write_b32(flag0 + (buf * NB + sub) * 4, move ? 1u : 0u);
      // a row without a finite score so far (keys whose products overflow): probabilities 0
      const float mref = mrow == -INFINITY ? 0.f : mrow;
#pragma unroll
      for (int r = 0; r < 4 * NS; ++r) x[r] = __builtin_amdgcn_exp2f(x[r] - mref);
#pragma unroll
      for (int h = 0; h < NH; ++h) {
        lrow += ((x[8 * h] + x[8 * h + 1]) + (x[8 * h + 2] + x[8 * h + 3])) +
                ((x[8 * h + 4] + x[8 * h + 5]) + (x[8 * h + 6] + x[8 * h + 7]));
        // P^T as the B operand, one per 32 keys: slot jj of group grp is key
        // 32 h + (jj < 4 ? 4 grp + jj : 16 + 4 grp + jj - 4)
        const u32x4_t pw = {pack_bf16x2(x[8 * h], x[8 * h + 1]), pack_bf16x2(x[8 * h + 2], x[8 * h + 3]),
                            pack_bf16x2(x[8 * h + 4], x[8 * h + 5]), pack_bf16x2(x[8 * h + 6], x[8 * h + 7])};
        lds_write_b128(p0 + ((buf * NB + sub) * NH + h) * 1024 + lane * 16, pw);
      }
    }
    lrow += __shfl_xor(lrow, 16, 64);
    lrow += __shfl_xor(lrow, 32, 64);
    if constexpr (SPLIT) {
      if (grp == 0 && row < R) {
        const size_t prow = (size_t)split * a.B * a.Hq + (size_t)e * a.Hq + row % a.Hq;
        float* ml = a.part_ml + (prow * a.nq + g * G + row / a.Hq) * 2;
        ml[0] = mrow;
        ml[1] = lrow;
      }
    } else {
      // the last tile's factors are read in the other buffer of corr_s
      if (work && grp == 0) corr_s[(tend - tbeg) & 1][sub][l16] = 1.f / lrow;
      __syncthreads();
    }
    return;
  }

  f32x4_t o[4][DW];
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int d = 0; d < DW; ++d) o[b][d] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const int vr = grp * 4 + (l16 >> 2);
  const unsigned va0 = vr * RB + ((((l16 & 3) >> 1) ^ ((2 * (vr / RP)) & XK)) << 4) + (l16 & 1) * 8;
  next(tbeg, 2);
  for (int t = tbeg, nx = 0; t < tend; ++t, nx = nx == 2 ? 0 : nx + 1) {
    next(t + 1, nx);
    if (!work) continue;
    const int buf = (t - tbeg) & 1;
    const unsigned vt = v0 + nx * TB + va0;
    u32x4_t fl = __builtin_bit_cast(u32x4_t, lds_read_b128<0>(flag0 + (buf * NB + b0) * 4));
    bf16x8_t pf[4][NH];
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int h = 0; h < NH; ++h) pf[b][h] = lds_read_b128<0>(p0 + ((buf * NB + b0 + b) * NH + h) * 1024 + lane * 16);
    u32x2_t vf[DW][NS];
#pragma unroll
    for (int d = 0; d < DW; ++d) {
      const unsigned ad = vt ^ ((sub * DW + d) << 5);
#pragma unroll
      for (int u = 0; u < NS; ++u) {
        if (u == 0) vf[d][u] = lds_read_tr<0>(ad);
        if (u == 1) vf[d][u] = lds_read_tr<16 * RB>(ad);
        if (u == 2) vf[d][u] = lds_read_tr<32 * RB>(ad);
        if (u == 3) vf[d][u] = lds_read_tr<48 * RB>(ad);
      }
    }
    lds_wait<0>();
    lds_ready(fl);
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int h = 0; h < NH; ++h) lds_ready(pf[b][h]);
#pragma unroll
    for (int d = 0; d < DW; ++d)
#pragma unroll
      for (int u = 0; u < NS; ++u) lds_ready(vf[d][u]);
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      if (b >= nb) break;  // uniform
      if (__builtin_amdgcn_readfirstlane(fl[b])) {
        const float corr = lds_read_f32(corr0 + ((buf * NB + b0 + b) * 16 + l16) * 4);
#pragma unroll
        for (int d = 0; d < DW; ++d)
#pragma unroll
          for (int r = 0; r < 4; ++r) o[b][d][r] *= corr;
      }
#pragma unroll
      for (int d = 0; d < DW; ++d)
#pragma unroll
        for (int h = 0; h < NH; ++h) {
          const u32x4_t vv = {vf[d][2 * h][0], vf[d][2 * h][1], vf[d][2 * h + 1][0], vf[d][2 * h + 1][1]};
          o[b][d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, vv), pf[b][h], o[b][d], 0, 0, 0);
        }
    }
  }
  if constexpr (!SPLIT) __syncthreads();
  if (!work) return;

  // o[b][d][r] = O^T[dim (sub DW + d) 16 + 4 grp + r][row0 + 16 (b0 + b) + l16]
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const int row = row0 + (b0 + b) * 16 + l16;
    if (row >= R) break;
    const int h = row / a.Hq, query = row % a.Hq;
    const int d0 = sub * DW * 16 + grp * 4;
    if constexpr (SPLIT) {
      const size_t prow = (size_t)split * a.B * a.Hq + (size_t)e * a.Hq + query;
      float* po = a.part_o + (prow * a.nq + g * G + h) * HD + d0;
#pragma unroll
      for (int d = 0; d < DW; ++d) *(f32x4_t*)(po + d * 16) = o[b][d];
    } else {
      const float inv = corr_s[(tend - tbeg) & 1][b0 + b][l16];
      bf16_t* orow = (bf16_t*)a.out + (size_t)(e * a.Hq + query) * a.ldo + (g * G + h) * HD + d0;
#pragma unroll
      for (int d = 0; d < DW; ++d) {
        u32x2_t wv;
        wv[0] = pack_bf16x2(o[b][d][0] * inv, o[b][d][1] * inv);
        wv[1] = pack_bf16x2(o[b][d][2] * inv, o[b][d][3] * inv);
        *(u32x2_t*)(orow + d * 16) = wv;
      }
    }
  }
}

// out = sum_s 2^(m_s - m) O_s / sum_s 2^(m_s - m) l_s over the (at most NS) key ranges s, in
// range order, four dims per thread.  Every range's loads are in flight together: the
// launch is one round trip to memory long.
template <int NS>
__global__ __launch_bounds__(256) void attn_combine_kernel(const float* __restrict__ part_o,
                                                           const float* __restrict__ part_ml, int nsplit, int rows,
                                                           int nq, int hd, bf16_t* __restrict__ out, int ldo) {
  const int qd = nq * hd;
  const long long i = ((long long)blockIdx.x * 256 + threadIdx.x) * 4;
  if (i >= (long long)rows * qd) return;
  const int row = (int)(i / qd), c = (int)(i % qd), h = c / hd;
  float2 ml[NS];
  f32x4_t o[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const size_t pr = (size_t)min(s, nsplit - 1) * rows + row;
    ml[s] = *(const float2*)(part_ml + (pr * nq + h) * 2);
    o[s] = *(const f32x4_t*)(part_o + pr * qd + c);
  }
  __builtin_amdgcn_sched_barrier(0);  // without it the compiler sinks the loads to their uses
  float mx = ml[0].x;  // -infinity for a range without a finite score: weight 0
#pragma unroll
  for (int s = 1; s < NS; ++s) mx = fmaxf(mx, ml[s].x);
  f32x4_t num = {0.f, 0.f, 0.f, 0.f};
  float den = 0.f;
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const float wt = s < nsplit ? __builtin_amdgcn_exp2f(ml[s].x - mx) : 0.f;
    den += wt * ml[s].y;
#pragma unroll
    for (int k = 0; k < 4; ++k) num[k] += wt * o[s][k];
  }
  const float inv = 1.f / den;
  const u32x2_t wv = {pack_bf16x2(num[0] * inv, num[1] * inv), pack_bf16x2(num[2] * inv, num[3] * inv)};
  *(u32x2_t*)(out + (size_t)row * ldo + c) = wv;
}

namespace {
constexpr int tile_keys(int hd) { return hd <= 128 ? 64 : 32; }
int blocks_of(const AttnArgs& a, int rows) { return (a.nq / a.nkv * a.Hq + rows - 1) / rows * a.nkv * a.B; }
// 128-row chunks (each key tile fetched half as often) once they alone fill most of the chip
bool wide(const AttnArgs& a) { return a.nsplit == 1 && a.nq / a.nkv * a.Hq > 64 && blocks_of(a, 128) >= 160; }
}  // namespace

// Key ranges: with fewer than ~160 blocks the chip idles, so the tiles are cut into as many
// ranges as give at most 256 blocks (one per CU: three tiles' buffers take most of its
// LDS), at least 64 keys each and at most 16 (a range costs its partial sums a write and a
// read: 4 bytes per query and dim).  At 866 keys x 256 dims (us, ranges added up): 7 blocks
// 14 with 14 ranges, 34 without; 168 blocks 29 without, 52 with 2.
void plan_attn(AttnArgs& a) {
  a.nsplit = 1;
  const int TK = tile_keys(a.hd);
  const int tiles = (a.P + TK - 1) / TK + (a.S + TK - 1) / TK;
  a.keys_per_split = tiles * TK;
  const int blocks = blocks_of(a, 64);
  // up to 8 tiles in a row (0.4-0.8 us each) cost less than the partial sums and their launch
  if (blocks >= 160 || tiles < 8) return;
  const int ns = std::min({256 / blocks, tiles / (64 / TK), 16});
  if (ns < 2) return;
  const int tps = (tiles + ns - 1) / ns;
  a.nsplit = (tiles + tps - 1) / tps;
  a.keys_per_split = tps * TK;
}

template <int HD>
static hipError_t launch_gqa(const AttnArgs& a, hipStream_t s) {
  constexpr int TK = tile_keys(HD);
  const int R = a.nq / a.nkv * a.Hq, chunks = (R + 63) / 64;
  if (a.nsplit > 1) {
    if (a.keys_per_split % TK || a.nsplit > 16 || !a.part_o || !a.part_ml) return hipErrorInvalidValue;
    hipLaunchKernelGGL((attn_gqa_kernel<HD, TK, 4, true>), dim3(blocks_of(a, 64) * a.nsplit), dim3(512), 0, s, a, chunks);
    const long long n = (long long)a.B * a.Hq * a.nq * HD / 4;
    const auto combine = a.nsplit <= 4 ? attn_combine_kernel<4> : a.nsplit <= 8 ? attn_combine_kernel<8> : attn_combine_kernel<16>;
    hipLaunchKernelGGL(combine, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a.part_o, a.part_ml, a.nsplit,
                       a.B * a.Hq, a.nq, HD, (bf16_t*)a.out, a.ldo);
  } else if (wide(a)) {
    hipLaunchKernelGGL((attn_gqa_kernel<HD, TK, 8, false>), dim3(blocks_of(a, 128)), dim3(1024), 0, s, a, (R + 127) / 128);
  } else {
    hipLaunchKernelGGL((attn_gqa_kernel<HD, TK, 4, false>), dim3(blocks_of(a, 64)), dim3(512), 0, s, a, chunks);
  }
  return hipGetLastError();
}

hipError_t launch_attn_bf16(const AttnArgs& a, hipStream_t s) {
  if ((a.Hq + 15) / 16 > 8 || a.nkv < 1 || a.nq % a.nkv || a.P + a.S < 1 || a.nsplit < 1) return hipErrorInvalidValue;
  switch (a.hd) {
    case 32: return launch_gqa<32>(a, s);
    case 64: return launch_gqa<64>(a, s);
    case 128: return launch_gqa<128>(a, s);
    case 256: return launch_gqa<256>(a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace ravel
