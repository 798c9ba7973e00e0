// Matrix products of launches with many rows (batched sentences times block
// positions, teacher-forced rows, batched encoder rows) and the vocabulary
// projection of some tens of rows, on MFMA without LDS staging.
//
// Y[r][n] = sum_k X[r][k] * W[n][k] (+ the epilogues of k_gemm).  Both operands
// are read in the MFMA feed order (a wave-wide load is 1 KB contiguous: the 16
// bytes every lane feeds to one matrix instruction), X also row-major, straight
// into registers; a wave owns FM x FN subtiles of 16 x 16 and keeps D steps of
// its FM + FN operand words in flight.
//
// KW > 1 (decoder and encoder products): the KW waves of a tile each take one
// of the KW ranges of K that the row-streaming kernel's waves take, so no wave
// waits for another inside the loop (no barrier per stage, as an LDS-staged
// tile has); their sums meet in LDS and are added in range order by threads
// that each finish eight consecutive columns of a row (16-byte residual loads
// and stores).  KW = 1 (vocabulary): a wave takes all of K.
//
// Same arithmetic as the row-streaming kernel, element for element: a range
// accumulates from zero in increasing k, ranges are added in order, and the
// epilogues evaluate the same expressions.  A row's values depend neither on
// the kernel, nor on the tile slot, nor on the other rows of the call.
//
// Bound: a wave moves FM + FN KB through the vector cache for FM * FN matrix
// instructions, 64 bytes a cycle against 16 cycles each on four units: 50% of
// the matrix peak at 64 x 64 per wave, 33% at 32 x 64.
//
// Workgroups are laid out for the eight XCDs (each with its own L2): the tiles
// are ordered with row blocks fastest and cut into eight contiguous chunks,
// chunk x going to the workgroups that the dispatcher places on XCD x (linear
// workgroup id = x mod 8), so the row blocks that share a weight tile read it
// from one L2.
//
// Rows at or above the device row count are not stored; a workgroup whose rows
// all lie there returns at once.
#include <algorithm>
#include <cstring>
#include <type_traits>

#include "common.h"
#include "epilogue.h"
#include "kernels.h"
#include "mma.h"

namespace pdec {

namespace {

constexpr int kBufferWord3 = 0x00020000;   // raw buffer resource: 32-bit data format, no swizzle, no index
constexpr int kPartPad = 4;                // floats of padding per row of the partial tiles (conflict-free writes)

template <typename WT> __device__ __forceinline__ typename Mma<WT>::frag feed_load(__amdgpu_buffer_rsrc_t r,
                                                                                   uint32_t off, uint32_t soff) {
  return __builtin_bit_cast(typename Mma<WT>::frag, __builtin_amdgcn_raw_buffer_load_b128(r, off, soff, 0));
}

}  // namespace

template <typename WT, int EPI, int FM, int FN, int KW, int WM, int WN, int D>
__global__ __launch_bounds__(64 * KW * WM * WN) void k_gemm_feed(GemmArgs a, int n_rb, int n_tiles) {
  if constexpr (EPI == EPI_QKV) layer_select(a, blockIdx.y);
  using MM = Mma<WT>;
  using frag = typename MM::frag;
  constexpr int KS = MM::KS, EPL = MM::EPL;
  constexpr int ES = static_cast<int>(sizeof(WT));
  constexpr int NT = 64 * KW * WM * WN;
  constexpr int BM = 16 * FM * WM, BN = 16 * FN * WN;
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int kw = wave % KW, wmn = wave / KW, wm = wmn / WN, wn = wmn % WN;
  const int lr = lane & 15, lg = lane >> 4;

  // XCD-aware tile order (see the header comment)
  constexpr bool VOCAB = EPI == EPI_ARGMAX || EPI == EPI_LOGITS;
  const int L = VOCAB ? min(static_cast<int>(blockIdx.x + (blockIdx.z << kTilesXBits)), n_tiles - 1) : blockIdx.x;
  const int xcd = L & 7, q8 = n_tiles >> 3, rem = n_tiles & 7;
  const int tile = xcd * q8 + min(xcd, rem) + (L >> 3);
  const int cb = tile / n_rb, rb = tile - cb * n_rb;
  const int m0 = rb * BM, n0 = cb * BN;
  const int R_max = a.n_rows, K = a.K, N = a.N;
  const int n_steps = K / KS;
  const int s_begin = KW > 1 ? (n_steps * kw) / KW : 0;
  const int n = (KW > 1 ? (n_steps * (kw + 1)) / KW : n_steps) - s_begin;   // steps of this wave

  // Operand words: the tile's first row and column in the buffers' base (64
  // bits: rows and weights of any size), a fixed byte offset per lane and
  // subtile, and the step's offset in a scalar register (subtiles past the last
  // repeat it; every read lies inside its buffer)
  const char* wf = static_cast<const char*>(EPI == EPI_QKV && a.n_layers > 1 ? a.w : a.wp);
  const size_t tile_bytes = static_cast<size_t>(16) * K * ES;      // 16 rows or columns in feed order
  const int rt0 = m0 / 16, ct0 = n0 / 16;
  const int rts = min(BM / 16, (R_max + 15) / 16 - rt0), cts = min(BN / 16, (N + 15) / 16 - ct0);
  const int rows = min(BM, R_max - m0);
  const char* x0 = static_cast<const char*>(a.x) + (a.x_feed ? rt0 * tile_bytes : static_cast<size_t>(m0) * a.ldx * ES);
  const uint32_t x_bytes = a.x_feed ? rts * static_cast<uint32_t>(tile_bytes) : static_cast<uint32_t>(rows) * a.ldx * ES;
  const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(x0), static_cast<short>(0),
                                                                      static_cast<int>(x_bytes), kBufferWord3);
  const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<char*>(wf + ct0 * tile_bytes), static_cast<short>(0), static_cast<int>(cts * static_cast<uint32_t>(tile_bytes)),
      kBufferWord3);
  const uint32_t x_step = a.x_feed ? kWave * 16 : KS * ES;
  uint32_t oa[FM], ob[FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
    oa[i] = a.x_feed ? (static_cast<uint32_t>(min(wm * FM + i, rts - 1)) * n_steps * kWave + lane) * 16
                     : (static_cast<uint32_t>(min(16 * (wm * FM + i) + lr, rows - 1)) * a.ldx + EPL * lg) * ES;
#pragma unroll
  for (int j = 0; j < FN; ++j) ob[j] = (static_cast<uint32_t>(min(wn * FN + j, cts - 1)) * n_steps * kWave + lane) * 16;
  frag fa[D][FM], fb[D][FN];
  auto load_step = [&](int u, int s) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < FN; ++j) fb[u][j] = feed_load<WT>(wr, ob[j], static_cast<uint32_t>(s_begin + s) * (kWave * 16));
#pragma unroll
    for (int i = 0; i < FM; ++i) fa[u][i] = feed_load<WT>(xr, oa[i], static_cast<uint32_t>(s_begin + s) * x_step);
  };
#pragma unroll
  for (int u = 0; u < D; ++u) load_step(u, max(min(u, n - 1), 0));
  const int R = a.n_rows_dev ? *a.n_rows_dev : a.n_rows;
  if (m0 >= R) return;                                   // workgroup-uniform

  floatx4_t acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  auto step = [&](int u) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) acc[i][j] = MM::step(fa[u][i], fb[u][j], acc[i][j]);
  };
  int s0 = 0;
  for (; s0 + D < n; s0 += D) {
#pragma unroll
    for (int u = 0; u < D; ++u) {
      step(u);
      load_step(u, min(s0 + u + D, n - 1));
    }
  }
#pragma unroll
  for (int u = 0; u < D; ++u)
    if (s0 + u < n) step(u);                              // the last steps: their loads have all been issued

  if constexpr (KW > 1) {
    // partial tiles through LDS; each thread finishes eight consecutive columns of a row
    extern __shared__ __align__(16) unsigned char s_dyn[];
    float* part = reinterpret_cast<float*>(s_dyn);        // [KW][BM][BN + kPartPad]
    constexpr int LD = BN + kPartPad;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          part[(kw * BM + (wm * FM + i) * 16 + 4 * lg + e) * LD + (wn * FN + j) * 16 + lr] = acc[i][j][e];
    __syncthreads();
    constexpr int ITEMS = BM * BN / 8;
#pragma unroll
    for (int it0 = 0; it0 < ITEMS; it0 += NT) {
      const int it = it0 + tid;
      const int tr = it / (BN / 8), tc = (it - tr * (BN / 8)) * 8;
      const int row = m0 + tr, col = n0 + tc;
      if (it >= ITEMS || row >= R || col >= N) continue;
      float bias_v[8], v[8];
      load_n<WT, 8>(static_cast<const WT*>(a.bias), col, bias_v);
      float rv[8];
      if constexpr (EPI == EPI_RESID) load_n<WT, 8>(static_cast<const WT*>(a.resid), static_cast<size_t>(row) * a.ldr + col, rv);
      int sent = 0, pos = 0;
      if constexpr (EPI == EPI_QKV) row_place(a.rows, row, sent, pos);
      const float* p = part + tr * LD + tc;
#pragma unroll
      for (int e = 0; e < 8; e += 4) {
        floatx4_t t = *reinterpret_cast<const floatx4_t*>(p + e);
#pragma unroll
        for (int w = 1; w < KW; ++w) t = t + *reinterpret_cast<const floatx4_t*>(p + w * BM * LD + e);   // range order
#pragma unroll
        for (int i = 0; i < 4; ++i) v[e + i] = t[i];
      }
      finish8<WT, EPI>(a, row, col, v, bias_v, rv, sent, pos);
    }
  } else {
    // lane holds C[4 lg + e][lr] of each subtile
    float bias_v[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j)
      bias_v[j] = Elt<WT>::load(static_cast<const WT*>(a.bias), min(n0 + (wn * FN + j) * 16 + lr, N - 1));
    if constexpr (EPI == EPI_LOGITS) {
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int row = m0 + (wm * FM + i) * 16 + 4 * lg + e;
          if (row >= R) continue;
          float* out = a.out_f32 + static_cast<size_t>(row) * a.ldo;
#pragma unroll
          for (int j = 0; j < FN; ++j) {
            const int col = n0 + (wn * FN + j) * 16 + lr;
            if (col < N) out[col] = fmaf(a.logit_scale, acc[i][j][e], bias_v[j]);
          }
        }
    } else {
      static_assert(EPI == EPI_ARGMAX, "whole-K waves serve the vocabulary projection");
      __shared__ uint32_t s_key[WN][BM];
      __shared__ uint32_t s_idx[WN][BM];
      __shared__ float2 s_lse[WN][BM];
      const bool want_lse = a.part_lse != nullptr;
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          uint32_t bk = 0u, bi = 0x7fffffffu, nf = 0u;
          float lm = -INFINITY, ls = 0.f;
#pragma unroll
          for (int j = 0; j < FN; ++j) {
            const int col = n0 + (wn * FN + j) * 16 + lr;
            const float logit = fmaf(a.logit_scale, acc[i][j][e], bias_v[j]);   // s * (h . E[col]) + bias[col]
            if (col < N) {
              if (!isfinite(logit)) nf = 1u;
              else {
                best_take(bk, bi, float_key(logit), static_cast<uint32_t>(col));
                if (want_lse) lse_take(lm, ls, logit);
              }
            }
          }
          group16_best(bk, bi);
          nf = group16_or(nf);
          if (want_lse) group16_lse(lm, ls);
          if (lr == 0) {
            const int rl = (wm * FM + i) * 16 + 4 * lg + e;
            s_key[wn][rl] = bk;
            s_idx[wn][rl] = bi | (nf << 31);
            if (want_lse) s_lse[wn][rl] = make_float2(lm, ls);
          }
        }
      __syncthreads();
      for (int t = tid; t < BM; t += NT) {
        if (m0 + t >= R) break;
        uint32_t kk = s_key[0][t], ii = s_idx[0][t] & 0x7fffffffu, ff = s_idx[0][t] >> 31;
#pragma unroll
        for (int w = 1; w < WN; ++w) {
          best_take(kk, ii, s_key[w][t], s_idx[w][t] & 0x7fffffffu);
          ff |= s_idx[w][t] >> 31;
        }
        a.partials[static_cast<size_t>(m0 + t) * a.part_ld + cb] = make_uint2(kk, ii | (ff << 31));
        if (want_lse) {
          float m = s_lse[0][t].x, sm = s_lse[0][t].y;
#pragma unroll
          for (int w = 1; w < WN; ++w) lse_merge(m, sm, s_lse[w][t].x, s_lse[w][t].y);   // wave order
          a.part_lse[static_cast<size_t>(m0 + t) * a.part_ld + cb] = make_float2(m, sm);
        }
      }
    }
  }
}

namespace {

// Tile configurations of the products: subtiles per wave (K split over the waves).
enum ProductCfg { P_32x32 = 0, P_32x64, P_64x64, P_COUNT };

template <typename WT, int EPI, int FM, int FN, int KW, int WM, int WN, int D>
hipError_t launch_shape(const GemmArgs& a, hipStream_t s, bool init) {
  constexpr int BM = 16 * FM * WM, BN = 16 * FN * WN;
  constexpr size_t lds = KW > 1 ? static_cast<size_t>(KW) * BM * (BN + kPartPad) * sizeof(float) : 0;
  const int n_rb = (a.n_rows + BM - 1) / BM;
  const int n_tiles = n_rb * ((a.N + BN - 1) / BN);
  const dim3 grid = EPI == EPI_ARGMAX || EPI == EPI_LOGITS
                        ? vocab_tile_grid(n_tiles)
                        : dim3(n_tiles, EPI == EPI_QKV && a.n_layers > 1 ? a.n_layers : 1);
  auto kernel = &k_gemm_feed<WT, EPI, FM, FN, KW, WM, WN, D>;
  if (init) {          // gfx950 has 160 KB of LDS per CU
    if (lds <= 65536) return hipSuccess;
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                               static_cast<int>(lds));
  }
  hipLaunchKernelGGL(kernel, grid, dim3(64 * KW * WM * WN), lds, s, a, n_rb, n_tiles);
  return hipGetLastError();
}

template <typename WT, int EPI, int KW>
hipError_t launch_product(const GemmArgs& a, int cfg, hipStream_t s, bool init) {
  switch (cfg) {
    case P_32x32: return launch_shape<WT, EPI, 2, 2, KW, 1, 1, 4>(a, s, init);
    case P_32x64: return launch_shape<WT, EPI, 2, 4, KW, 1, 1, 4>(a, s, init);
    case P_64x64: return launch_shape<WT, EPI, 4, 4, KW, 1, 1, 2>(a, s, init);
    default: return hipErrorInvalidValue;
  }
}

// The vocabulary: 16 x 64, 32 x 128 or 32 x 256 tiles, four waves side by side.
template <typename WT, int EPI> hipError_t launch_vocab(const GemmArgs& a, int bn, hipStream_t s) {
  if (bn == 64) return launch_shape<WT, EPI, 1, 1, 1, 1, 4, 8>(a, s, false);
  if (bn == 128) return launch_shape<WT, EPI, 2, 2, 1, 1, 4, 4>(a, s, false);
  if constexpr (std::is_same<WT, bf16_t>::value)
    if (bn == 256) return launch_shape<WT, EPI, 2, 4, 1, 1, 4, 4>(a, s, false);
  return hipErrorInvalidValue;
}

template <typename WT> hipError_t launch_vocab_w(int epi, const GemmArgs& a, int bn, hipStream_t s) {
  return epi == EPI_ARGMAX ? launch_vocab<WT, EPI_ARGMAX>(a, bn, s) : launch_vocab<WT, EPI_LOGITS>(a, bn, s);
}

template <typename WT>
hipError_t launch_w(int epi, int ksplit, int cfg, const GemmArgs& a, hipStream_t s, bool init) {
  switch (epi) {
    case EPI_F32: return ksplit == 8 ? launch_product<WT, EPI_F32, 8>(a, cfg, s, init) : launch_product<WT, EPI_F32, 4>(a, cfg, s, init);
    case EPI_ACT: return ksplit == 8 ? launch_product<WT, EPI_ACT, 8>(a, cfg, s, init) : launch_product<WT, EPI_ACT, 4>(a, cfg, s, init);
    case EPI_RESID: return ksplit == 8 ? launch_product<WT, EPI_RESID, 8>(a, cfg, s, init) : launch_product<WT, EPI_RESID, 4>(a, cfg, s, init);
    case EPI_QKV: return ksplit == 8 ? launch_product<WT, EPI_QKV, 8>(a, cfg, s, init) : launch_product<WT, EPI_QKV, 4>(a, cfg, s, init);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

// The configurations whose partial tiles exceed 64 KB of LDS are allowed it here, once.
hipError_t gemm_feed_init() {
  GemmArgs a;
  memset(&a, 0, sizeof(a));
  for (int epi : {EPI_F32, EPI_ACT, EPI_RESID, EPI_QKV})
    for (int ksplit : {4, 8})
      for (int cfg = 0; cfg < P_COUNT; ++cfg) {
        hipError_t e = launch_w<bf16_t>(epi, ksplit, cfg, a, nullptr, true);
        if (e == hipSuccess) e = launch_w<float>(epi, ksplit, cfg, a, nullptr, true);
        if (e != hipSuccess) return e;
      }
  return hipSuccess;
}

// The largest tile that still gives `least` workgroups: a larger one reads less
// through the cache, a smaller one leaves fewer CUs with an extra tile.
// bf16, bound by the cache: 192 of them, measured against 256 / 512: batch-8
// scoring of the large model 3391 against 3466 / 3712 us, MT-base batch 16 1192
// against 1245 / 1267 (160 and 224 as 192).  float32, bound by the matrix units, so
// an even spread counts: 1024, against 256 / 512: MT-base batch-16 scoring 1974
// against 2113 / 2025 us, batch 4 1086 / 1108 / 1087, batch 40 6472 / 6577 / 6602.
static int gemm_feed_cfg(int dtype, int N, int rows) {
  const auto wgs = [&](int bm, int bn) { return ((rows + bm - 1) / bm) * ((N + bn - 1) / bn); };
  const int least = dtype == DT_BF16 ? 192 : 1024;
  if (wgs(64, 64) >= least) return P_64x64;
  if (wgs(32, 64) >= least) return P_32x64;
  return P_32x32;
}

hipError_t launch_vocab_feed(int dtype, int epi, int bn, const GemmArgs& a, hipStream_t s) {
  if (a.n_rows <= 0) return hipSuccess;
  const int ks = dtype == DT_BF16 ? Mma<bf16_t>::KS : Mma<float>::KS;
  if (epi != EPI_ARGMAX && epi != EPI_LOGITS) return hipErrorInvalidValue;
  if (a.K % ks != 0 || a.x_f32 || a.wp == nullptr || !tile_offsets_fit(dtype, a)) return hipErrorInvalidValue;
  return dtype == DT_BF16 ? launch_vocab_w<bf16_t>(epi, a, bn, s) : launch_vocab_w<float>(epi, a, bn, s);
}

hipError_t launch_gemm_feed(int dtype, int epi, int ksplit, const GemmArgs& a, hipStream_t s) {
  if (a.n_rows <= 0) return hipSuccess;
  const int ks = dtype == DT_BF16 ? Mma<bf16_t>::KS : Mma<float>::KS;
  if (a.K % ks != 0 || a.N % 16 != 0 || a.x_f32 || ksplit != (a.K >= 2048 ? 8 : 4)) return hipErrorInvalidValue;
  if (!tile_offsets_fit(dtype, a)) return hipErrorInvalidValue;
  if (a.out_feed && (epi != EPI_ACT || a.N % 32 != 0)) return hipErrorInvalidValue;
  if (epi == EPI_QKV && a.n_layers > 1 ? !a.lw_feed : a.wp == nullptr) return hipErrorInvalidValue;
  const int cfg = gemm_feed_cfg(dtype, a.N, a.n_rows);
  return dtype == DT_BF16 ? launch_w<bf16_t>(epi, ksplit, cfg, a, s, false)
                          : launch_w<float>(epi, ksplit, cfg, a, s, false);
}

}  // namespace pdec
