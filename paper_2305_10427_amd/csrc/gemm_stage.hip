// The vocabulary projection of many rows (batched sentences times block
// positions, teacher-forced rows) and the layers' bf16 products of a thousand
// rows or more, on MFMA with both operands staged through LDS by direct loads.
//
// Y[r][n] = sum_k X[r][k] * W[n][k] with the epilogues of k_gemm, the vocabulary
// as the fused argmax (EPI_ARGMAX) or stored (EPI_LOGITS).  X and W are in the
// MFMA feed order, so a stage of one MFMA step is BM / 16 + BN / 16 blocks of 1 KB: each block is one
// wave-wide 16-byte load that lands in LDS without passing through registers,
// and one conflict-free wave-wide LDS read per use.  A wave owns FM x FN
// subtiles of 16 x 16.
//
// Bound and split: read straight into registers (k_gemm_feed) a 64 x 64 wave
// tile moves 8 KB through the 64-byte-a-cycle vector cache per 16 matrix
// instructions, half of the matrix rate at best; staged through registers
// (row-major tiles, the kernel this one replaces) the LDS stores took the
// issue slots and a 256-column tile did not fit.  Here a block comes through
// the cache once per workgroup and the waves' reads go to LDS (128 bytes a
// cycle): 64 x 128 per wave of a 128 x 256 tile needs 48 + 24 KB of LDS traffic
// per 512 matrix cycles.  NS stages are in the ring; the fragments of stage
// s + 1 are read while stage s is multiplied, and stage s + NS is requested as
// soon as the barrier says that every wave has read stage s: one barrier per
// stage, and several workgroups per CU to fill the gaps.
// 250,027 x 1024, argmax of 64 / 128 / 256 / 512 / 1024 / 2048 rows: 101 / 145 /
// 252 / 481 / 940 / 1811 us -> 92 / 95 / 154 / 275 / 508 / 913 us (1148 TFLOP/s);
// logits of 952 / 4160 rows 989 / 4131 -> 715 / 2796 us (4.2 GB stored).
//
// Same arithmetic as the row-streaming kernels, element for element: K is cut
// into their KR ranges of MFMA steps (one for the vocabulary), a range
// accumulates from zero in increasing k, range sums are added in range order,
// and the epilogues evaluate the same expressions.  A row's values depend
// neither on the kernel, nor on the tile slot, nor on the other rows of the call.
//
// Products: 64 x 128 tiles of four 32 x 64 waves (two sets of sums for the
// ranges leave no room for more at four waves per SIMD), three workgroups per
// CU.  us against k_gemm_feed: 2048 x 1024 x 4096 (rows, K, N; GELU) 40.9 -> 33.5,
// 4160 rows 97 -> 62; 4160 x 4096 x 1024 91 -> 64; 4000 x 512 x 2048 27.3 -> 23.6.
//
// Tile order for the eight XCDs as in k_gemm_feed (row blocks fastest, eight
// contiguous chunks).  Rows at or above the device row count are not stored; a
// workgroup whose rows all lie there returns at once.
#include <algorithm>
#include <cstring>

#include "common.h"
#include "epilogue.h"
#include "kernels.h"
#include "mma.h"

namespace pdec {

namespace {

typedef int i32x4_t __attribute__((ext_vector_type(4)));

constexpr int kBlock = kWave * 16;         // bytes of one operand block (16 rows or columns, one MFMA step)
constexpr int kOutPad = 4;                 // floats of padding per row of an output subtile in LDS

// Raw buffer resource of n bytes at p (32-bit data format, no swizzle, no index), wave-uniform.
__device__ __forceinline__ i32x4_t buffer_of(const char* p, uint32_t n) {
  const uint64_t u = reinterpret_cast<uint64_t>(p);
  return i32x4_t{__builtin_amdgcn_readfirstlane(static_cast<int>(u)),
                 __builtin_amdgcn_readfirstlane(static_cast<int>(u >> 32) & 0xffff),
                 __builtin_amdgcn_readfirstlane(static_cast<int>(n)), 0x00020000};
}

// 16 bytes per lane from r[voff + soff] to LDS lds + 16 lane (no register is
// written; completion is counted by vmcnt, waited for in stage_wait).
__device__ __forceinline__ void load_to_lds(i32x4_t r, uint32_t voff, uint32_t soff, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
               :: "s"(lds), "v"(voff), "s"(r), "s"(soff) : "memory", "m0");
}

// All but the N youngest loads of this wave have landed and its LDS reads are
// done; then the workgroup's barrier.
template <int N> __device__ __forceinline__ void stage_wait() {
  static_assert(N <= 63, "vmcnt");
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(N) : "memory");
}

// The same with `later` stages (at most MAX; wave-uniform) of LPS loads each left in flight.
template <int MAX, int LPS> __device__ __forceinline__ void stage_wait_for(int later) {
  if constexpr (MAX > 0) {
    if (later < MAX) return stage_wait_for<MAX - 1, LPS>(later);
  }
  stage_wait<MAX * LPS>();
}

}  // namespace

template <typename WT, int EPI, int FM, int FN, int WM, int WN, int KR, int NS>
__global__ __launch_bounds__(64 * WM * WN, 2) void k_gemm_stage(GemmArgs a, int n_rb, int n_tiles) {
  if constexpr (EPI == EPI_QKV) layer_select(a, blockIdx.y);
  using MM = Mma<WT>;
  using frag = typename MM::frag;
  constexpr int KS = MM::KS;
  constexpr int ES = static_cast<int>(sizeof(WT));
  constexpr int NW = WM * WN, NT = 64 * NW;
  constexpr int BM = 16 * FM * WM, BN = 16 * FN * WN;
  constexpr int TA = BM / 16, TB = BN / 16, NB = TA + TB;   // blocks of a stage
  static_assert(TA % NW == 0 && TB % NW == 0, "whole blocks per wave");
  constexpr int LA = TA / NW, LB = TB / NW, LPS = LA + LB;  // loads per wave and stage
  constexpr uint32_t STAGE = NB * kBlock;
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int wm = wave / WN, wn = wave % WN;
  const int lr = lane & 15, lg = lane >> 4;

  constexpr bool VOCAB = EPI == EPI_ARGMAX || EPI == EPI_LOGITS;
  const int L = VOCAB ? min(static_cast<int>(blockIdx.x + (blockIdx.z << kTilesXBits)), n_tiles - 1) : blockIdx.x;
  const int xcd = L & 7, q8 = n_tiles >> 3, rem = n_tiles & 7;
  const int tile = xcd * q8 + min(xcd, rem) + (L >> 3);
  const int cb = tile / n_rb, rb = tile - cb * n_rb;
  const int m0 = rb * BM, n0 = cb * BN;
  const int R_max = a.n_rows, K = a.K, N = a.N;
  const int R = a.n_rows_dev ? *a.n_rows_dev : a.n_rows;
  if (m0 >= R) return;                                   // workgroup-uniform
  const int n = K / KS;                                  // MFMA steps = stages

  // the tile's operand blocks: subtiles past the last repeat it (every read lies inside its buffer)
  const char* wf = static_cast<const char*>(EPI == EPI_QKV && a.n_layers > 1 ? a.w : a.wp);
  const size_t tile_bytes = static_cast<size_t>(16) * K * ES;
  const int rts = min(TA, (R_max + 15) / 16 - m0 / 16), cts = min(TB, (N + 15) / 16 - n0 / 16);
  const i32x4_t xr = buffer_of(static_cast<const char*>(a.x) + (m0 / 16) * tile_bytes,
                               rts * static_cast<uint32_t>(tile_bytes));
  const i32x4_t wr = buffer_of(wf + (n0 / 16) * tile_bytes, cts * static_cast<uint32_t>(tile_bytes));
  extern __shared__ __align__(16) unsigned char s_dyn[];
  const uint32_t lds0 = static_cast<uint32_t>(
      reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) unsigned char*)(s_dyn)));
  uint32_t ga[LA], gb[LB];                               // this wave's blocks: byte offsets of their first step
#pragma unroll
  for (int u = 0; u < LA; ++u) ga[u] = static_cast<uint32_t>(min(wave + NW * u, rts - 1)) * static_cast<uint32_t>(tile_bytes);
#pragma unroll
  for (int u = 0; u < LB; ++u) gb[u] = static_cast<uint32_t>(min(wave + NW * u, cts - 1)) * static_cast<uint32_t>(tile_bytes);
  const uint32_t voff = lane * 16;
  auto issue = [&](int s, uint32_t buf) __attribute__((always_inline)) {
    const uint32_t at = lds0 + buf + wave * kBlock, ks = static_cast<uint32_t>(s) * kBlock;
#pragma unroll
    for (int u = 0; u < LA; ++u) load_to_lds(xr, voff, ga[u] + ks, at + u * NW * kBlock);
#pragma unroll
    for (int u = 0; u < LB; ++u) load_to_lds(wr, voff, gb[u] + ks, at + (TA + u * NW) * kBlock);
  };
  struct Frags {
    frag a[FM], b[FN];
  };
  Frags f0, f1;
  const unsigned char* pa = s_dyn + wm * FM * kBlock + lane * 16;
  const unsigned char* pb = s_dyn + (TA + wn * FN) * kBlock + lane * 16;
  auto read = [&](Frags& f, uint32_t buf) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < FM; ++i) f.a[i] = *reinterpret_cast<const frag*>(pa + buf + i * kBlock);
#pragma unroll
    for (int j = 0; j < FN; ++j) f.b[j] = *reinterpret_cast<const frag*>(pb + buf + j * kBlock);
  };

  floatx4_t acc[FM][FN], tot[KR > 1 ? FM : 1][KR > 1 ? FN : 1];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  // ranges of K: w_cur is the one being accumulated, bnd the first step of the next
  int w_cur = 0;
  int bnd = KR > 1 ? n / KR : n + 1;
  auto fold = [&]() __attribute__((always_inline)) {
    if constexpr (KR > 1) {
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          tot[i][j] = w_cur == 0 ? acc[i][j] : tot[i][j] + acc[i][j];
          acc[i][j] = floatx4_t{0.f, 0.f, 0.f, 0.f};
        }
    }
    ++w_cur;
  };

#pragma unroll
  for (int s = 0; s < NS; ++s)
    if (s < n) issue(s, s * STAGE);
  stage_wait_for<NS - 1, LPS>(n - 1);
  read(f0, 0);
  uint32_t cur = 0;                                      // LDS offset of stage s
  auto range_edge = [&](int s) __attribute__((always_inline)) {
    if constexpr (KR > 1) {
      while (w_cur + 1 < KR && s == bnd) {
        fold();
        bnd = (n * (w_cur + 1)) / KR;
      }
    }
  };
  auto step_row = [&](const Frags& f, int i) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = MM::step(f.a[i], f.b[j], acc[i][j]);
  };
  // Stage s with every ring slot still to be refilled.  The requests and the
  // fragment reads are spread between the matrix instructions (a wave issues
  // in order: all of them up front leave its matrix unit idle meanwhile).
  auto iter = [&](int s, const Frags& f, Frags& fn) __attribute__((always_inline)) {
    const uint32_t nxt = cur == (NS - 1) * STAGE ? 0 : cur + STAGE;
    range_edge(s);
    stage_wait<(NS - 2) * LPS>();                        // stage s + 1 has landed, every wave has read stage s
    const uint32_t at = lds0 + cur + wave * kBlock, ks = static_cast<uint32_t>(s + NS) * kBlock;
#pragma unroll
    for (int i = 0; i < FM; ++i) {
#pragma unroll
      for (int u = (FM + FN) * i / FM; u < (FM + FN) * (i + 1) / FM; ++u) {
        if (u < FM) fn.a[u] = *reinterpret_cast<const frag*>(pa + nxt + u * kBlock);
        else fn.b[u - FM] = *reinterpret_cast<const frag*>(pb + nxt + (u - FM) * kBlock);
      }
#pragma unroll
      for (int u = LPS * i / FM; u < LPS * (i + 1) / FM; ++u) {
        if (u < LA) load_to_lds(xr, voff, ga[u] + ks, at + u * NW * kBlock);
        else load_to_lds(wr, voff, gb[u - LA] + ks, at + (TA + (u - LA) * NW) * kBlock);
      }
      step_row(f, i);
      __builtin_amdgcn_sched_barrier(0);
    }
    cur = nxt;
  };
  auto last = [&](int s, const Frags& f, Frags& fn) __attribute__((always_inline)) {
    const uint32_t nxt = cur == (NS - 1) * STAGE ? 0 : cur + STAGE;
    range_edge(s);
    if (s + 1 < n) {
      stage_wait_for<NS - 2, LPS>(n - 2 - s);
      if (s + NS < n) issue(s + NS, cur);
      read(fn, nxt);
    }
#pragma unroll
    for (int i = 0; i < FM; ++i) step_row(f, i);
    cur = nxt;
  };
  int s0 = 0;
  for (; s0 + 1 + NS < n; s0 += 2) {
    iter(s0, f0, f1);
    iter(s0 + 1, f1, f0);
  }
  for (; s0 + 1 < n; s0 += 2) {
    last(s0, f0, f1);
    last(s0 + 1, f1, f0);
  }
  if (s0 < n) last(s0, f0, f1);
  if constexpr (KR > 1)
    while (w_cur < KR) fold();                           // the last range, then any empty trailing ranges
  auto res = [&](int i, int j) __attribute__((always_inline)) -> const floatx4_t& {
    if constexpr (KR > 1) return tot[i][j];
    else return acc[i][j];
  };
  __syncthreads();                                       // the stages are dead: LDS holds outputs from here

  if constexpr (EPI == EPI_ARGMAX) {
    // lane holds C[4 lg + e][lr] of each subtile
    float bias_v[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j)
      bias_v[j] = Elt<WT>::load(static_cast<const WT*>(a.bias), min(n0 + (wn * FN + j) * 16 + lr, N - 1));
    uint32_t* s_key = reinterpret_cast<uint32_t*>(s_dyn);          // [WN][BM]
    uint32_t* s_idx = s_key + WN * BM;
    float2* s_lse = reinterpret_cast<float2*>(s_idx + WN * BM);
    const bool want_lse = a.part_lse != nullptr;
    // Whole column tiles without a log-sum-exp compare the logits as floats:
    // five instructions a logit.  A non-finite logit, or a best of zero (whose
    // sign the order keys tell apart), sends the wave's row group to the keys.
    const bool whole = n0 + BN <= N && !want_lse;
    const uint32_t c0 = static_cast<uint32_t>(n0 + wn * FN * 16 + lr);
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int rl = (wm * FM + i) * 16 + 4 * lg + e;
        uint32_t bk = 0u, bi = 0x7fffffffu, nf = 0u;
        float best = -INFINITY, chk = 0.f;
        int bj = 0;
        if (whole) {
#pragma unroll
          for (int j = 0; j < FN; ++j) {
            const float logit = fmaf(a.logit_scale, res(i, j)[e], bias_v[j]);   // s * (h . E[col]) + bias[col]
            chk = fmaf(logit, 0.f, chk);                 // NaN once a logit is not finite
            const bool t = logit > best;
            best = t ? logit : best;
            bj = t ? j : bj;
          }
        }
        if (whole && __builtin_amdgcn_ballot_w64(!(chk == 0.f) || best == 0.f) == 0) {
          const float mx = group16_max(best);
          bi = best == mx ? c0 + 16u * bj : 0x7fffffffu;
          bi = min(bi, dpp_u<kDppXor1>(bi));
          bi = min(bi, dpp_u<kDppXor2>(bi));
          bi = min(bi, dpp_u<kDppHalfMirror>(bi));
          bi = min(bi, dpp_u<kDppMirror>(bi));
          bk = float_key(mx);
        } else {
          float lm = -INFINITY, ls = 0.f;
#pragma unroll
          for (int j = 0; j < FN; ++j) {
            const uint32_t col = c0 + 16u * j;
            const float logit = fmaf(a.logit_scale, res(i, j)[e], bias_v[j]);
            if (col < static_cast<uint32_t>(N)) {
              if (!isfinite(logit)) nf = 1u;
              else {
                best_take(bk, bi, float_key(logit), col);
                if (want_lse) lse_take(lm, ls, logit);
              }
            }
          }
          group16_best(bk, bi);
          nf = group16_or(nf);
          if (want_lse) {
            group16_lse(lm, ls);
            if (lr == 0) s_lse[wn * BM + rl] = make_float2(lm, ls);
          }
        }
        if (lr == 0) {
          s_key[wn * BM + rl] = bk;
          s_idx[wn * BM + rl] = bi | (nf << 31);
        }
      }
    __syncthreads();
    for (int t = tid; t < BM; t += NT) {
      if (m0 + t >= R) break;
      uint32_t kk = s_key[t], ii = s_idx[t] & 0x7fffffffu, ff = s_idx[t] >> 31;
#pragma unroll
      for (int w = 1; w < WN; ++w) {
        best_take(kk, ii, s_key[w * BM + t], s_idx[w * BM + t] & 0x7fffffffu);
        ff |= s_idx[w * BM + t] >> 31;
      }
      a.partials[static_cast<size_t>(m0 + t) * a.part_ld + cb] = make_uint2(kk, ii | (ff << 31));
      if (want_lse) {
        float m = s_lse[t].x, sm = s_lse[t].y;
#pragma unroll
        for (int w = 1; w < WN; ++w) lse_merge(m, sm, s_lse[w * BM + t].x, s_lse[w * BM + t].y);   // wave order
        a.part_lse[static_cast<size_t>(m0 + t) * a.part_ld + cb] = make_float2(m, sm);
      }
    }
  } else {
    // 16 rows at a time through this wave's slice of LDS, so that a lane
    // stores consecutive columns of a row
    constexpr int LD = 16 * FN + kOutPad;
    float* part = reinterpret_cast<float*>(s_dyn) + wave * 16 * LD;
    const int nw = n0 + wn * FN * 16, mw = m0 + wm * FM * 16;
    auto to_lds = [&](int i) __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) part[(4 * lg + e) * LD + 16 * j + lr] = res(i, j)[e];
      wave_lds_sync();
    };
    if constexpr (EPI == EPI_LOGITS) {
      float bias_l[FN / 4];
#pragma unroll
      for (int u = 0; u < FN / 4; ++u)
        bias_l[u] = Elt<WT>::load(static_cast<const WT*>(a.bias), min(nw + 64 * u + lane, N - 1));
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        if (mw + 16 * i >= R) break;                     // wave-uniform
        to_lds(i);
        for (int r = 0; r < 16; ++r) {
          if (mw + 16 * i + r >= R) break;
          float* out = a.out_f32 + static_cast<size_t>(mw + 16 * i + r) * a.ldo + nw;
#pragma unroll
          for (int u = 0; u < FN / 4; ++u)
            if (nw + 64 * u + lane < N) out[64 * u + lane] = fmaf(a.logit_scale, part[r * LD + 64 * u + lane], bias_l[u]);
        }
        wave_lds_sync();                                 // the next subtile overwrites the slice
      }
    } else {
      // a lane finishes eight columns of PASS rows of each subtile; what it
      // reads for them from memory is requested first, for all of its rows
      constexpr int GR = 2 * FN, RP = kWave / GR, PASS = 16 / RP, RW = EPI == EPI_RESID ? ES / 2 : 0;
      const int tr0 = lane / GR, cl = lane % GR * 8, col = nw + cl;
      const int col_ok = min(col, N - 8);
      float bias8[8];
      load_n<WT, 8>(static_cast<const WT*>(a.bias), col_ok, bias8);
      u32x4_t rw[FM * PASS][RW > 0 ? RW : 1];
      int sent[EPI == EPI_QKV ? FM * PASS : 1], pos[EPI == EPI_QKV ? FM * PASS : 1];
      if constexpr (EPI == EPI_RESID || EPI == EPI_QKV) {
#pragma unroll
        for (int t = 0; t < FM * PASS; ++t) {
          const int row = min(mw + RP * t + tr0, R - 1);
          if constexpr (EPI == EPI_QKV) row_place(a.rows, row, sent[t], pos[t]);
#pragma unroll
          for (int x = 0; x < RW; ++x)
            rw[t][x] = reinterpret_cast<const u32x4_t*>(static_cast<const WT*>(a.resid) + static_cast<size_t>(row) * a.ldr + col_ok)[x];
        }
      }
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        if (mw + 16 * i >= R) break;                     // wave-uniform
        to_lds(i);
#pragma unroll
        for (int u = 0; u < PASS; ++u) {
          const int t = i * PASS + u, tr = u * RP + tr0, row = mw + 16 * i + tr;
          float v[8], rv[8];
          *reinterpret_cast<floatx4_t*>(v) = *reinterpret_cast<const floatx4_t*>(part + tr * LD + cl);
          *reinterpret_cast<floatx4_t*>(v + 4) = *reinterpret_cast<const floatx4_t*>(part + tr * LD + cl + 4);
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            if constexpr (RW == 1) rv[e] = __uint_as_float((e & 1) ? (rw[t][0][e >> 1] & 0xffff0000u) : (rw[t][0][e >> 1] << 16));
            else if constexpr (RW == 2) rv[e] = __uint_as_float(rw[t][e >> 2][e & 3]);
            else rv[e] = 0.f;
          }
          if (row < R && col < N)
            finish8<WT, EPI>(a, row, col, v, bias8, rv, EPI == EPI_QKV ? sent[t] : 0, EPI == EPI_QKV ? pos[t] : 0);
        }
        wave_lds_sync();                                 // the next subtile overwrites the slice
      }
    }
  }
}

namespace {

// Tiles (rows x columns of a workgroup) and ring depths.
enum StageCfg { S_NONE = -1, S_64x256 = 0, S_128x128, S_128x256, S_256x256, S_COUNT };   // vocabulary; products: 64 x 128

template <typename WT, int EPI, int FM, int FN, int WM, int WN, int KR, int NS>
hipError_t launch_shape(const GemmArgs& a, hipStream_t s, bool init) {
  constexpr int BM = 16 * FM * WM, BN = 16 * FN * WN, NW = WM * WN;
  constexpr size_t stages = static_cast<size_t>(NS) * (BM + BN) / 16 * kBlock;
  constexpr size_t outs = EPI == EPI_ARGMAX ? 16ull * WN * BM : 4ull * NW * 16 * (16 * FN + kOutPad);
  constexpr size_t lds = stages > outs ? stages : outs;
  static_assert(lds <= 160 * 1024, "LDS of a CU");
  const int n_rb = (a.n_rows + BM - 1) / BM;
  const int n_tiles = n_rb * ((a.N + BN - 1) / BN);
  const dim3 grid = EPI == EPI_ARGMAX || EPI == EPI_LOGITS
                        ? vocab_tile_grid(n_tiles)
                        : dim3(n_tiles, EPI == EPI_QKV && a.n_layers > 1 ? a.n_layers : 1);
  auto kernel = &k_gemm_stage<WT, EPI, FM, FN, WM, WN, KR, NS>;
  if (init) {          // gfx950 has 160 KB of LDS per CU
    if (lds <= 65536) return hipSuccess;
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                               static_cast<int>(lds));
  }
  hipLaunchKernelGGL(kernel, grid, dim3(64 * NW), lds, s, a, n_rb, n_tiles);
  return hipGetLastError();
}

template <typename WT, int EPI> hipError_t launch_cfg(const GemmArgs& a, int cfg, hipStream_t s, bool init) {
  if (cfg == S_128x256) return launch_shape<WT, EPI, 4, 8, 2, 2, 1, 3>(a, s, init);
  if constexpr (std::is_same<WT, bf16_t>::value) {
    if (cfg == S_64x256) return launch_shape<WT, EPI, 4, 4, 1, 4, 1, 4>(a, s, init);
    if (cfg == S_128x128) return launch_shape<WT, EPI, 4, 4, 2, 2, 1, 3>(a, s, init);
    if constexpr (EPI == EPI_LOGITS)
      if (cfg == S_256x256) return launch_shape<WT, EPI, 8, 4, 2, 4, 1, 4>(a, s, init);
  }
  return init ? hipSuccess : hipErrorInvalidValue;
}

template <typename WT> hipError_t launch_w(int epi, int cfg, const GemmArgs& a, hipStream_t s, bool init) {
  return epi == EPI_ARGMAX ? launch_cfg<WT, EPI_ARGMAX>(a, cfg, s, init) : launch_cfg<WT, EPI_LOGITS>(a, cfg, s, init);
}

template <int EPI> hipError_t launch_product(const GemmArgs& a, int ksplit, hipStream_t s) {   // 48 KB of LDS
  return ksplit == 8 ? launch_shape<bf16_t, EPI, 2, 4, 2, 2, 8, 4>(a, s, false)
                     : launch_shape<bf16_t, EPI, 2, 4, 2, 2, 4, 4>(a, s, false);
}

// Whether a bf16 product in feed order runs on 64 x 128 staged tiles: enough
// of them for the workgroups of a CU to cover each other's fixed parts (about
// 5 us a tile at 1.4 of them per CU), sooner where K is long.  us, k_gemm_feed
// against staged, by tiles: K = 1024: 256 tiles 11.2 / 11.6, 376 19.8 / 15.4, 480
// (GELU) 21.1 / 18.8, 576 22.2 / 19.7, 2112 97 / 62; K = 512: 256 8.8 / 10.8, 384
// 11.0 / 10.9, 512 14.5 / 13.4; K = 4096: 120 23.1 / 25.6, 192 30.3 / 27.3, 256
// 41.9 / 28.9; K = 2048: 128 13.1 / 16.6, 252 24.1 / 18.3.
bool stage_product(int dtype, const GemmArgs& a) {
  if (dtype != DT_BF16 || !a.x_feed) return false;
  const long long tiles = static_cast<long long>((a.n_rows + 63) / 64) * ((a.N + 127) / 128) * std::max(a.n_layers, 1);
  return tiles >= (a.K >= 2048 ? 192 : 360);
}

// Whether a narrow float32 product gives k_gemm_feed too few 32 x 32 tiles for the
// 256 CUs; k_gemm, with a workgroup per 16 x 16, is the faster one then.  us per
// iteration of three layers, k_gemm_feed / k_gemm below 96 tiles: d = 256, 224
// rows 173 / 159, 256 rows 164 / 152, 320 rows 172 / 162; d = 128, 256 rows 141 / 134,
// 448 rows 152 / 146, 576 rows 146 / 146, 768 rows (96 tiles in k_gemm too) 152 / 156.
// N = 512 with as few (160 rows of d = 512, six encoder layers): 304 / 315.
bool few_tiles(int dtype, const GemmArgs& a) {
  return dtype == DT_F32 && a.n_layers <= 1 && a.N <= 256 &&
         static_cast<long long>((a.n_rows + 31) / 32) * ((a.N + 31) / 32) < 96;
}

// The tile for a vocabulary projection of `rows` rows: the largest that leaves
// enough workgroups.  us measured with the weights out of the caches (argmax
// unless said; f: k_gemm_feed, s: staged, workgroups in brackets):
//
// f16x64 while there are few of them.  A larger tile is one long serial chain
// of products and epilogue on few CUs: float32 V = 1000, K = 64 / 512, any rows
// up to 256: 4.3 / 6 against f32x256 [4 to 32] 10 / 23; bf16 V = 7001, K = 640,
// 64 rows 7.1 [440], s64x256 [28] 17.5.  It gives way to f32x128 where its
// repeated operand reads cost more: bf16 K = 512 at 1500 (V = 8000, 192 rows
// 10.0 / 10.2; V = 20,000, 64 rows [1252] 9.3 / 10.9, 96 rows [1878] 11.9 / 10.6),
// K = 1024 at 750 (V = 8000, 96 rows 10.3 / 10.0; V = 32,000, 32 rows [1000] 15.2 /
// 14.9), float32 at 1850 (V = 4003, 384 rows [1512] 12.2 / 14.6, 512 [2016] 15.7 /
// 14.7; V = 58,101, 32 rows [1816] 24.3 / 26.1, 64 rows [3632] 41.1 / 39.1), and stored
// beyond 128 rows (V = 58,101: 48 / 96 / 128 / 256 rows 29.8 / 55.1 / 72.6 / 136, f32x128
// 39.9 / 64.4 / 73.9 / 134).
// f32x256 for the bf16 vocabularies that f32x128 would cut into more than 2560
// (K <= 512) or 6000 units of 16 x 64: V = 58,101, K = 512, 64 stored rows 14.3 / 15.6;
// K = 1024: V = 80,000, 64 rows [5000] 33.2 / 29.9, V = 250,027, 32 stored 101.7 / 104.0.
//
// Staged, bf16: s128x128 from 300 workgroups (K <= 512) or 240 on: K = 512, V = 8000:
// 512 rows [252] 17.3, f32x128 14.3, V = 20,000: 256 rows [314] 16.1 / 16.5, 384 rows
// [471] 16.6 / 22.3; K = 1024: V = 8000, 384 rows [189] 20.2 / 17.4, V = 32,000, 128 rows
// [250] 16.7 / 22.6.  Of few rows only: V = 58,101, K = 512, 160 rows f 28, s 30.
// s64x256 for 33 to 64 rows where it gives more than the 512 workgroups of one
// round: V = 250,027 90.1, s128x128 91.9; V = 80,000 [313] 37.0, f32x128 29.9.
// s128x256, K = 1024: from 1600 on (V = 250,027, 512 rows 252, s128x128 265; V = 80,000,
// 512 rows [1252] 87.7 / 77.7, 2048 rows [5008] 283 / 306), and where it takes one round
// and s128x128 (768 a round) two (V = 32,000, 512 rows [500] 31.8 / 35.1); stored logits
// from 900 on (V = 250,027, 256 rows 181 / 197; V = 80,000, 384 rows [939] 87 / 93, 256 rows
// [626] 56 / 47).  s256x256 for stored logits (fuller rows of 256 columns go out
// together) from 220 on: V = 58,101, K = 512, 512 rows [454] 48, s128x128 61; V = 32,000,
// 512 rows [250] 35 / 46; V = 8000, 1024 rows [128] 29 / 21.
// float32, bound by the matrix units: a CU takes 63 us per s128x256 tile of K = 512,
// 71 for as many outputs in f32x128, so s128x256 where at least 0.9 of its outputs on
// the busiest CU are real: V = 58,101, 1120 rows (0.97) 503 / 548, 1024 rows (0.89) 499 /
// 470, stored 503 / 501; V = 20,000, 2048 rows (0.98) 310 / 334, 1024 rows (0.81) 190 /
// 168.  Not with K <= 256, where its epilogue weighs more (V = 4003, K = 256, 2048 rows 51 / 43).
struct VocabTile {
  int cfg;   // staged, or S_NONE: k_gemm_feed
  int bn;    // columns of a workgroup
};

VocabTile vocab_tile(int dtype, int epi, int V, int K, int rows) {
  const auto wgs = [&](int bm, int bn) {
    return static_cast<long long>((rows + bm - 1) / bm) * ((V + bn - 1) / bn);
  };
  const bool store = epi == EPI_LOGITS, wide = K > 512;
  if (dtype == DT_F32) {
    const long long big = wgs(128, 256), full = (big + 255) / 256 * 256;
    if (K > 256 && big >= 240 && 10LL * rows * V >= 9 * full * (128 * 256)) return {S_128x256, 256};
    return {S_NONE, wgs(16, 64) <= 1850 || (store && rows <= 128) ? 64 : 128};
  }
  if (store && rows > 448 && wgs(256, 256) >= 220) return {S_256x256, 256};
  if (wide) {
    const long long big = wgs(128, 256);
    if (store ? rows > 128 && big >= 900 : rows > 256 && (big >= 1600 || (big <= 512 && wgs(128, 128) > 768)))
      return {S_128x256, 256};
    if (rows > 32 && rows <= 64 && wgs(64, 256) > 512) return {S_64x256, 256};
  }
  if (rows > (wide || store ? 64 : 160) && wgs(128, 128) >= (wide ? 240 : 300)) return {S_128x128, 128};
  const long long u = wgs(16, 64);
  return {S_NONE, u <= (wide ? 750 : 1500) ? 64 : u <= (wide ? 6000 : 2560) ? 128 : 256};
}

}  // namespace

// The configurations whose stages exceed 64 KB of LDS are allowed it here, once.
hipError_t gemm_stage_init() {
  GemmArgs a;
  memset(&a, 0, sizeof(a));
  for (int epi : {EPI_ARGMAX, EPI_LOGITS})
    for (int cfg = 0; cfg < S_COUNT; ++cfg) {
      hipError_t e = launch_w<bf16_t>(epi, cfg, a, nullptr, true);
      if (e == hipSuccess) e = launch_w<float>(epi, cfg, a, nullptr, true);
      if (e != hipSuccess) return e;
    }
  return hipSuccess;
}

int vocab_rows_parts(int dtype, int V, int K, int rows) {
  const int bn = vocab_tile(dtype, EPI_ARGMAX, V, K, rows).bn;
  return (V + bn - 1) / bn;
}

hipError_t launch_vocab_rows(int dtype, int epi, const GemmArgs& a, hipStream_t s) {
  if (a.n_rows <= 0) return hipSuccess;
  if (epi != EPI_ARGMAX && epi != EPI_LOGITS) return hipErrorInvalidValue;
  if (epi == EPI_ARGMAX && a.part_ld < vocab_rows_parts(dtype, a.N, a.K, a.n_rows)) return hipErrorInvalidValue;
  const VocabTile t = vocab_tile(dtype, epi, a.N, a.K, a.n_rows);
  if (t.cfg == S_NONE) return launch_vocab_feed(dtype, epi, t.bn, a, s);
  const int ks = dtype == DT_BF16 ? Mma<bf16_t>::KS : Mma<float>::KS;
  if (a.K % ks != 0 || a.x_f32 || !a.x_feed || a.wp == nullptr) return hipErrorInvalidValue;
  if (!tile_offsets_fit(dtype, a)) return hipErrorInvalidValue;
  return dtype == DT_BF16 ? launch_w<bf16_t>(epi, t.cfg, a, s, false) : launch_w<float>(epi, t.cfg, a, s, false);
}

hipError_t launch_product_rows(int dtype, int epi, int ksplit, const GemmArgs& a, hipStream_t s) {
  if (a.n_rows <= 0) return hipSuccess;
  if (few_tiles(dtype, a) || (a.n_layers <= 1 && !tile_offsets_fit(dtype, a)))
    return launch_gemm(dtype, PRO_NONE, epi, ksplit, a, s, nullptr, nullptr);
  if (!stage_product(dtype, a)) return launch_gemm_feed(dtype, epi, ksplit, a, s);
  if (a.K % Mma<bf16_t>::KS != 0 || a.x_f32 || ksplit != (a.K >= 2048 ? 8 : 4) || a.N % 16 != 0) return hipErrorInvalidValue;
  if (!tile_offsets_fit(dtype, a)) return hipErrorInvalidValue;
  if (a.out_feed && (epi != EPI_ACT || a.N % 32 != 0)) return hipErrorInvalidValue;
  if (epi == EPI_QKV && a.n_layers > 1 ? !a.lw_feed : a.wp == nullptr) return hipErrorInvalidValue;
  switch (epi) {
    case EPI_F32: return launch_product<EPI_F32>(a, ksplit, s);
    case EPI_ACT: return launch_product<EPI_ACT>(a, ksplit, s);
    case EPI_RESID: return launch_product<EPI_RESID>(a, ksplit, s);
    case EPI_QKV: return launch_product<EPI_QKV>(a, ksplit, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace pdec
