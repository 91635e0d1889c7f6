// Half-precision GEMMs with float32 accumulation on gfx950 MFMA, for the
// forward and backward passes of MPX's mixed-precision step (§2: forward and
// backward in half precision; the products accumulate in float32).
//
// One kernel template computes  C[m,n] = sum_k A(m,k) B(n,k)  where each
// operand is stored either with the reduction index contiguous ("k-major") or
// with the output index contiguous ("mn-major"):
//   forward  Y  = X W^T   : A = X  k-major,  B = W  k-major
//   backward dX = dY W    : A = dY k-major,  B = W  mn-major
//   backward dW = dY^T X  : A = dY mn-major, B = X  mn-major
// Tiles lie in LDS as they lie in memory; k-major fragments are read with
// ds_read_b128, mn-major ones with transposing reads.  The MFMA is
// v_mfma_f32_32x32x16_{f16,bf16}: lane l holds 8 k-values of row l%32 for A and
// of column l%32 for B; its operands are swapped, so the 16 accumulators of lane
// l are row l%32, columns 8*(i/4) + 4*(l/32) + i%4.
//
// Epilogue (all optional, in this order, each rounding once to half):
//   h = half(acc + bias[n]);  pre_out = h;  h = half(gelu(h));
//   h = half(h * gelu'(dact[m,n]));  h = half(h + resid[m,n]);  C = h
// or, for split-K, the float32 partial sums go to a workspace and a second
// kernel adds the partials in a fixed order and rounds once.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>
#include <utility>

#include "colsum.h"
#include "common.h"
#include "dma.h"
#include "mfma.h"

namespace mpx {

struct GemmArgs {
  const uint16_t* A;
  const uint16_t* B;
  uint16_t* C;
  float* ws;  // split-K partials [splits][M][N] (when splits > 1)
  int64_t M, N, K, lda, ldb, ldc;
  int64_t sA0, sA1, sB0, sB1, sC0, sC1, nb1;
  int32_t splits;
  int64_t k_split;  // reduction length per split (multiple of the k tile)
  const uint16_t* bias;
  const uint16_t* resid;
  int64_t ldr;
  uint16_t* pre;
  const uint16_t* dact;
  int32_t act;
  int32_t full_epi;  // set by the dispatcher: every epilogue operand is 16-byte aligned
  // if set, the number of non-finite half outputs C is added to *nonfinite
  // (split-K partials are counted by the reduction that rounds them instead)
  int32_t* nonfinite;
  // weight-gradient products (both operands mn-major) may also return the
  // bias gradient db[m] = half(sum_k A(m, k)), summed from the A fragments
  // the MFMAs read: set by the dispatcher only for the kernel variant that
  // does it.  Split-K calls write float32 partial sums dbp[M][splits * C] instead,
  // one per split and column of the output's C tile columns, which the split-K
  // reduction adds.
  uint16_t* db;
  float* dbp;
};

// Epilogue operations compiled into a kernel (a mask of these bits);
// EPI_GENERIC takes them from the call's arguments, the same arithmetic step
// for step.
enum : int { EPI_BIAS = 1, EPI_GELU = 2, EPI_DACT = 4, EPI_RESID = 8, EPI_GENERIC = -1 };

// 16 bytes at any 2-byte aligned address (one instruction: global accesses
// need no alignment on gfx950)
typedef u32x4 u32x4_any __attribute__((aligned(2)));

// Epilogue through LDS, for the transposed accumulator layout.  Step 1
// (accumulator layout: lane = one row, runs of 4 consecutive columns):
// h = half(acc + bias), written to the wave's own [WM][WN + 4] half region of
// the LDS the main loop no longer needs.  Step 2 (row layout: lane = 8
// consecutive columns of one row): the pre-activation store, GELU, GELU' of
// the previous layer and the residual add with 16-byte accesses, each store
// of a 64-wide wave tile writing 8 rows x 128 contiguous bytes.
// E: the epilogue operations, compiled in; EPI_GENERIC tests the call's
// arguments instead.  EDGE = false: the wave's whole tile lies inside the
// output and every operand is 16-byte aligned.  EDGE = true: rows from mv and
// columns from nv on lie outside (either may be <= 0) and no alignment is
// assumed; vectors inside the output keep the 16-byte accesses, only those
// that straddle its last column go one value at a time.  The loads have no
// conditions (rows and vectors outside load the last ones inside): with them forward
// 1792 x 528 x 192 with residual took 7.4 us, 128 x 904 x 128 with bias 4.7 and 256 x 392
// x 192 with GELU 6.4; now 6.2, 4.0 and 5.3.
// In float16 the compiler forms half(x sigma) and half(h gelu') with one
// instruction that rounds once or through float32, so GELU results of two tile shapes,
// or of whole and edge tiles, may differ in the last place.
// pf (nullable): the wave's GELU' or residual operand rows, already loaded
// in the row layout (16 bytes of row (lane >> 3) + 8 t per entry t).
// J0: first of the TN accumulator columns handled (of TNA).
template <int DT, int TM, int TN, int E, bool EDGE = false, int J0 = 0, int TNA = TN>
__device__ __forceinline__ void gemm_epilogue_lds(const GemmArgs& g, const f32x16 (&acc)[TM][TNA],
                                                  int64_t mw, int64_t nw, int lane, int64_t offC,
                                                  uint16_t* lds, const u32x4* pf = nullptr, int mv = 0,
                                                  int nv = 0) {
  constexpr int WN = 32 * TN, PITCH = WN + 4;  // a column of 32 rows spreads over all banks
  constexpr int LPR = WN / 8, RPT = 64 / LPR;  // lanes per row, rows per step
  using vec = std::conditional_t<EDGE, u32x4_any, u32x4>;
  if constexpr (EDGE) {
    if (mv <= 0 || nv <= 0) return;  // nothing of the wave's tile is in the output
  }
  const int hi = lane >> 5, r32 = lane & 31;
  const bool do_bias = E == EPI_GENERIC ? g.bias != nullptr : (E & EPI_BIAS) != 0;
  const bool do_pre = E == EPI_GENERIC ? g.pre != nullptr : (E & EPI_GELU) != 0;
  const bool do_gelu = E == EPI_GENERIC ? g.act == MPX_ACT_GELU_TANH : (E & EPI_GELU) != 0;
  const bool do_dact = E == EPI_GENERIC ? g.dact != nullptr : (E & EPI_DACT) != 0;
  const bool do_res = E == EPI_GENERIC ? g.resid != nullptr : (E & EPI_RESID) != 0;
  const bool do_count = E == EPI_GENERIC && g.nonfinite != nullptr;
  auto unpack = [](u32x2 w, float (&f)[4]) {
    f[0] = h2f<DT>((uint16_t)(w.x & 0xFFFFu));
    f[1] = h2f<DT>((uint16_t)(w.x >> 16));
    f[2] = h2f<DT>((uint16_t)(w.y & 0xFFFFu));
    f[3] = h2f<DT>((uint16_t)(w.y >> 16));
  };
  asm volatile("" ::: "memory");  // the wave's reads of its last 64 columns come first
  static_for<TN>([&](auto j) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int col = 32 * j + 8 * q + 4 * hi;
      float b[4] = {0.0f, 0.0f, 0.0f, 0.0f};
      if (do_bias) {
        if constexpr (EDGE) {  // no conditions: loads under one are waited for one by one
#pragma unroll
          for (int c = 0; c < 4; ++c) b[c] = h2f<DT>(g.bias[nw + min(col + c, nv - 1)]);
        } else {
          unpack(ld_u2(g.bias + nw + col), b);
        }
      }
      static_for<TM>([&](auto i) {
        const int row = 32 * i + r32;
        uint16_t h[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) h[c] = f2h<DT>(acc[i][J0 + j][4 * q + c] + b[c]);
        *reinterpret_cast<u32x2*>(lds + row * PITCH + col) =
            u32x2{h[0] | ((uint32_t)h[1] << 16), h[2] | ((uint32_t)h[3] << 16)};
      });
    }
  });
  const int c8 = 8 * (lane % LPR);
  const int64_t ldc = g.ldc;
  uint16_t* C = g.C + (offC + mw * ldc + nw);
  uint16_t* pre = do_pre ? g.pre + (mw * ldc + nw) : nullptr;
  const uint16_t* dact = do_dact ? g.dact + (mw * ldc + nw) : nullptr;
  const uint16_t* res = do_res ? g.resid + (mw * g.ldr + nw) : nullptr;
  auto h8 = [](u32x4 w, uint16_t (&h)[8]) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      h[2 * k] = (uint16_t)(w[k] & 0xFFFFu);
      h[2 * k + 1] = (uint16_t)(w[k] >> 16);
    }
  };
  auto p8 = [](const uint16_t (&h)[8]) {
    return u32x4{h[0] | ((uint32_t)h[1] << 16), h[2] | ((uint32_t)h[3] << 16),
                 h[4] | ((uint32_t)h[5] << 16), h[6] | ((uint32_t)h[7] << 16)};
  };
  using off_t = std::conditional_t<EDGE, int64_t, uint32_t>;
  // one row's 8 columns; nc of them exist (8 unless EDGE)
  const int nc = EDGE ? min(8, nv - c8) : 8;
  auto load8 = [&](const uint16_t* p, uint16_t (&h)[8]) {
    if (!EDGE || nc == 8) {
      h8(*reinterpret_cast<const vec*>(p), h);
    } else {
#pragma unroll
      for (int c = 0; c < 8; ++c) h[c] = c < nc ? p[c] : (uint16_t)0;
    }
  };
  auto store8 = [&](uint16_t* p, const uint16_t (&h)[8]) {
    if (!EDGE || nc == 8) {
      *reinterpret_cast<vec*>(p) = p8(h);
    } else {
#pragma unroll
      for (int c = 0; c < 8; ++c)
        if (c < nc) p[c] = h[c];
    }
  };
  // the GELU' or residual rows, all in flight before the first store (a load
  // behind a store that may alias it would wait for it: one memory latency
  // per step)
  constexpr int STEPS = 32 * TM / RPT;
  constexpr bool kOp = E != EPI_GENERIC && (E & (EPI_DACT | EPI_RESID)) != 0;
  u32x4 op[kOp ? STEPS : 1];
  if constexpr (kOp) {
    const uint16_t* src = (E & EPI_DACT) ? dact : res;
    const int64_t ld_op = (E & EPI_DACT) ? ldc : g.ldr;
#pragma unroll
    for (int t = 0; t < STEPS; ++t) {
      const int row = lane / LPR + RPT * t;
      if constexpr (EDGE) {
        if (nv >= 8)  // uniform: rows and vectors outside load the last ones inside
          op[t] = *reinterpret_cast<const vec*>(src + (min(row, mv - 1) * ld_op + min(c8, nv - 8)));
        else op[t] = u32x4{0u, 0u, 0u, 0u};
      } else {
        op[t] = pf ? pf[t] : *reinterpret_cast<const vec*>(src + (off_t)(row * ld_op + c8));
      }
    }
  }
  asm volatile("" ::: "memory");  // the lanes' writes to LDS come before the wave's reads
  auto operand8 = [&](int t, const uint16_t* p, uint16_t (&h)[8]) {
    if (kOp && nc == 8) h8(op[kOp ? t : 0], h);
    else load8(p, h);
  };
  int bad = 0;
  // edge tiles: GELU of every step ahead of the conditions around the stores, which
  // keep the steps apart.  half(x sigma) one value at a time, as behind them.  Not
  // the 16 steps of 256 x 256 tiles, which spill
  constexpr bool kAhead = EDGE && E != EPI_GENERIC && (E & EPI_GELU) != 0 && TM <= 2;
  u32x4 gel[kAhead ? STEPS : 1];
  if constexpr (kAhead) {
#pragma unroll
    for (int t = 0; t < STEPS; ++t) {
      const int row = lane / LPR + RPT * t;
      const u32x2 w0 = *reinterpret_cast<const u32x2*>(lds + row * PITCH + c8);
      const u32x2 w1 = *reinterpret_cast<const u32x2*>(lds + row * PITCH + c8 + 4);
      uint16_t h[8];
      h8(u32x4{w0.x, w0.y, w1.x, w1.y}, h);
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        h[c] = f2h<DT>(gelu_tanh(h2f<DT>(h[c])));
        asm volatile("" : "+v"(h[c]));
      }
      gel[t] = p8(h);
    }
  }
#pragma unroll
  for (int t = 0; t < STEPS; ++t) {
    const int row = lane / LPR + RPT * t;
    const u32x2 w0 = *reinterpret_cast<const u32x2*>(lds + row * PITCH + c8);
    const u32x2 w1 = *reinterpret_cast<const u32x2*>(lds + row * PITCH + c8 + 4);
    if constexpr (EDGE) {
      if (row >= mv || nc <= 0) continue;
    }
    uint16_t h[8];
    h8(u32x4{w0.x, w0.y, w1.x, w1.y}, h);
    const off_t off = (off_t)(row * ldc + c8);
    if (do_pre) store8(pre + off, h);
    if constexpr (kAhead) {
      h8(gel[t], h);
    } else if (do_gelu) {
#pragma unroll
      for (int c = 0; c < 8; ++c) h[c] = f2h<DT>(gelu_tanh(h2f<DT>(h[c])));
    }
    if (do_dact) {
      uint16_t da[8];
      operand8(t, dact + off, da);
#pragma unroll
      for (int c = 0; c < 8; ++c) h[c] = f2h<DT>(h2f<DT>(h[c]) * gelu_tanh_grad(h2f<DT>(da[c])));
    }
    if (do_res) {
      uint16_t rv[8];
      operand8(t, res + (off_t)(row * g.ldr + c8), rv);
#pragma unroll
      for (int c = 0; c < 8; ++c) h[c] = f2h<DT>(h2f<DT>(h[c]) + h2f<DT>(rv[c]));
    }
    if (do_count) {
      if (!EDGE || nc == 8) {  // no branch inside the store loop
        const u32x4 o = p8(h);
        bad += nonfinite2<DT>(o[0]) + nonfinite2<DT>(o[1]) + nonfinite2<DT>(o[2]) +
               nonfinite2<DT>(o[3]);
      } else {
#pragma unroll
        for (int c = 0; c < 8; ++c) bad += (c < nc && h_nonfinite<DT>(h[c])) ? 1 : 0;
      }
    }
    store8(C + off, h);
  }
  if (do_count) add_nonfinite(g.nonfinite, bad);
}

// Split-K: the wave's float32 sums (accumulators hold C^T blocks: lane l has
// row l % 32, columns 8 q + 4 (l / 32) + (0..3) for q = 0..3) go to the
// split's partial matrix in the workspace, 16 bytes at a time where its rows
// allow.
template <int TM, int TN>
__device__ __forceinline__ void gemm_partials(const GemmArgs& g, const f32x16 (&acc)[TM][TN], int64_t mw,
                                              int64_t nw, int lane, int split) {
  float* W = g.ws + (int64_t)split * g.M * g.N;
  const bool v16 = g.N % 4 == 0 && (reinterpret_cast<uintptr_t>(W) & 15u) == 0;
  static_for<TM>([&](auto i) {
    static_for<TN>([&](auto j) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int64_t m = mw + i * 32 + (lane & 31), n = nw + j * 32 + 8 * q + 4 * (lane >> 5);
        const f32x4 v = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
        if (m < g.M && n < g.N) {
          float* out = W + m * g.N + n;
          if (v16) *reinterpret_cast<f32x4*>(out) = v;  // N % 4 == 0: the 4 columns exist
          else
#pragma unroll
            for (int c = 0; c < 4; ++c)
              if (n + c < g.N) out[c] = v[c];
        }
      }
    });
  });
}

// ------------------------------------------------- direct-to-LDS kernel --
//
// The main loop of the kernel below moves operand tiles from global memory
// straight into LDS (global_load_lds_dwordx4: each lane's 16 bytes land at
// M0 + 16 * lane, so one wave instruction fills 1 KiB of LDS).  The compiler
// does not track these copies: an explicit vmcnt waits for a k tile, and one
// barrier makes it visible to every wave.
//
// LDS layouts (no padding: a copy fills 1 KiB contiguously, so bank
// conflicts are avoided by permuting 16-byte chunks instead):
//   k-major operand   [row][64 k], 128 B per row; chunk c of row r sits at
//                     position c ^ ((r >> 1) & 7).  The 16 lanes reading one
//                     ds_read_b128 phase (16 rows, one chunk) hit all 64 banks.
//   mn-major operand  [k][ROWS] (64 to 256 outputs, 8 to 32 chunks per k
//                     row), chunks permuted by dma_chunk.
//                     MFMA fragments are read with ds_read_b64_tr_b16, which
//                     transposes 16-bit elements across groups of 16 lanes, so
//                     the operand needs no transposition on the way in.
// Requirements of the copies (checked by the dispatcher; other operands go
// through StagedOperand): 16-byte aligned operands with leading dimensions and
// batch strides that are multiples of 8, and every split's k range a multiple
// of 64.  Rows past M or N read clamped (valid) addresses; their results are
// never stored.

// Position of 16-byte chunk c of row r (k-major: output row of 64 k; mn-major:
// k row of ROWS outputs) within the row in LDS; its own inverse.  An mn-major
// row of 64 (192) outputs spans half (one and a half times) the banks, so there
// rows 2 and 3 of each four move to the other half of each 128 bytes.
template <int ROWS, bool KMAJ>
__device__ __forceinline__ int dma_chunk(int r, int c) {
  if constexpr (KMAJ) return c ^ ((r >> 1) & 7);
  else if constexpr (ROWS % 128 == 64) return c ^ (4 * ((r >> 1) & 1));
  else return c ^ (4 * (r & 3));
}

// One operand of the direct-to-LDS kernel: ROWS output rows (of M or N) by
// 64 k per stage, copied by NWAVES waves, Q copies per wave.
template <int ROWS, bool KMAJ, int NWAVES>
struct DmaOperand {
  static constexpr int BLOCKS = ROWS / 8;  // 1 KiB copies per stage
  static constexpr int Q = BLOCKS / NWAVES;
  static_assert(BLOCKS % NWAVES == 0, "copies do not split evenly over the waves");
  static_assert(KMAJ || ROWS == 64 || ROWS == 128 || ROWS == 192 || ROWS == 256, "mn-major tile widths");
  uint32_t off[Q];  // per-lane byte offsets of the copies, relative to the tile base
  int64_t step;     // bytes from one k tile to the next

  // rv: valid rows (>= 1) of the tile; ld: leading dimension in elements
  __device__ __forceinline__ void init(int64_t ld, int rv, int wave, int lane) {
    if constexpr (KMAJ) {
      step = 128;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const int r = 8 * (wave + NWAVES * q) + (lane >> 3);
        const int c = dma_chunk<ROWS, true>(r, lane & 7);
        off[q] = (uint32_t)(min(r, rv - 1) * ld * 2 + c * 16);
      }
    } else {
      constexpr int CH = ROWS / 8;  // 16-byte chunks per k row
      step = 64 * ld * 2;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const int at = 64 * (wave + NWAVES * q) + lane;  // the tile's chunk this lane copies
        const int kr = at / CH;
        const int c = dma_chunk<ROWS, false>(kr, at % CH);
        off[q] = (uint32_t)(kr * ld * 2 + (8 * c < rv ? 16 * c : 0));
      }
    }
  }
  // copy the tile whose first element is at base into LDS at lds (both
  // wave-uniform; made explicitly scalar for the copy instruction)
  __device__ __forceinline__ void issue(const uint16_t* base, uint32_t lds, int wave) const {
    const uint64_t p = reinterpret_cast<uint64_t>(base);
    const uint64_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)p);
    const uint64_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(p >> 32));
    const void* sbase = reinterpret_cast<const void*>(lo | (hi << 32));
    const uint32_t slds = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds);
#pragma unroll
    for (int q = 0; q < Q; ++q)
      dma16(sbase, off[q], slds + 1024u * (uint32_t)(wave + NWAVES * q));
  }
};

// The same operand staged through registers, for operands the copies cannot
// take (rows that are not 16-byte aligned, a reduction that is not a multiple
// of 64): 16-byte loads at any alignment, written to the LDS positions the
// copies would have filled, so the fragment reads are the same.  Vectors that
// would reach past the end of their row (the last k of a k-major row, the
// last output of an mn-major one) are loaded ending at the row's last element
// and shifted down, with zeros behind: no access leaves the matrix.  Two k
// tiles are in flight (the register sets v[0] and v[1]).
// ANY: rows of fewer than 8 values (no whole vector fits) or strides past the
// 32-bit lane offsets: one value at a time with 64-bit addresses, clamped to the
// row's last value (no branch: one around the loads makes them wait) and packed
// when they are written.
// past: the loop's prefetch has run past the last k tile, and the loads are
// not used: every lane then reads its wave's first address, so they cost next to
// nothing.  Against packed one-value loads under a condition and the last tile
// loaded again: 12960 x 1905 x 6 bf16 dX 91 -> 40 us, forward 20172 x 1108 x 4 f16
// 83 -> 48, dW of 4504 rows 3 x 478 70 -> 29.
template <int ROWS, bool KMAJ, int NWAVES, bool ANY>
struct StagedOperand {
  static constexpr int BLOCKS = ROWS / 8, Q = BLOCKS / NWAVES;
  static_assert(BLOCKS % NWAVES == 0, "blocks do not split evenly over the waves");
  static constexpr int CH = KMAJ ? 8 : ROWS / 8;
  static constexpr int RSTEP = 64 / CH * NWAVES;  // rows from one vector of a lane to its next
  std::conditional_t<ANY, uint16_t[8], u32x4> v[2][Q];
  uint32_t off[Q];  // lane offsets (bytes) from 8 elements before the tile's first
  int64_t ld;
  int c8;       // first k (k-major) or output (mn-major) of the lane's vectors within the tile
  int r0;       // output row (k-major) or k row (mn-major) of the lane's vector 0
  int rv;       // rows (k-major) or outputs (mn-major) of the matrix from the tile's first on
  int krem[2];  // reduction values from the loaded tile's first on

  __device__ __forceinline__ void init(int64_t ld_, int64_t left, int wave, int lane) {
    ld = ld_;
    rv = (int)min<int64_t>(left, 1 << 20);
    r0 = 64 / CH * wave + lane / CH;
    c8 = 8 * dma_chunk<ROWS, KMAJ>(r0, lane % CH);
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int r = r0 + RSTEP * q;
      off[q] = 16 + (KMAJ ? (uint32_t)(min(r, rv - 1) * ld * 2) + 2 * c8
                          : (uint32_t)(r * ld * 2) + (uint32_t)(2 * min(c8, rv - 8)));
    }
  }
  // tile: its first element; kr: reduction values from there on (>= 1)
  template <int P>
  __device__ __forceinline__ void load(const uint16_t* tile, int kr, bool past) {
    krem[P] = kr;
    if constexpr (ANY) {
      const int last = past ? 0 : (KMAJ ? kr : rv) - 1, last_row = past ? 0 : (KMAJ ? rv : kr) - 1;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const uint16_t* row = tile + (int64_t)min(r0 + RSTEP * q, last_row) * ld;
#pragma unroll
        for (int e = 0; e < 8; ++e) v[P][q][e] = row[min(c8 + e, last)];
      }
    } else {
      const uint8_t* base = reinterpret_cast<const uint8_t*>(tile - 8);  // never accessed itself
      const int back = KMAJ ? 2 * max(0, c8 + 8 - kr) : 0;  // k-major: how far past the row's end
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        uint32_t o = off[q];
        if (kr < 64) {  // uniform: the last k tile
          if (KMAJ) o -= back;
          else o -= (uint32_t)(max(0, r0 + RSTEP * q - (kr - 1)) * ld * 2);
        }
        if (past) o = (uint32_t)__builtin_amdgcn_readfirstlane((int)o);
        v[P][q] = *reinterpret_cast<const u32x4_any*>(base + o);
      }
    }
  }
  template <int P>
  __device__ __forceinline__ void store(uint8_t* lds, int wave, int lane) {
    const int n = KMAJ ? krem[P] : rv;
    const bool whole = n >= (KMAJ ? 64 : ROWS);
    const int sh = c8 - min(c8, n - 8);
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      u32x4 x;
      if constexpr (ANY) {
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
          const uint32_t lo = c8 + e < n ? v[P][q][e] : 0, hi = c8 + e + 1 < n ? v[P][q][e + 1] : 0;
          x[e / 2] = lo | (hi << 16);
        }
      } else {
        x = v[P][q];
        if (!whole) x = shr_halves(x, sh);
      }
      if (!KMAJ && r0 + RSTEP * q >= krem[P]) x = u32x4{0u, 0u, 0u, 0u};
      *reinterpret_cast<u32x4*>(lds + 1024 * (wave + NWAVES * q) + 16 * lane) = x;
    }
  }
  // x with its first s elements dropped and zeros after the rest
  __device__ __forceinline__ static u32x4 shr_halves(u32x4 x, int s) {
    const u32x4 o = {__builtin_amdgcn_alignbit(x[1], x[0], 16), __builtin_amdgcn_alignbit(x[2], x[1], 16),
                     __builtin_amdgcn_alignbit(x[3], x[2], 16), x[3] >> 16};
    x = (s & 1) ? o : x;
    x = (s & 2) ? u32x4{x[1], x[2], x[3], 0u} : x;
    x = (s & 4) ? u32x4{x[2], x[3], 0u, 0u} : x;
    return s >= 8 ? u32x4{0u, 0u, 0u, 0u} : x;
  }
};

// Per-lane LDS byte offsets of the MFMA fragments of one operand, for a
// wave whose rows start at w0 within the tile (relative to the tile base).
template <int ROWS, bool KMAJ, int T>
struct FragReader {
  uint32_t base[KMAJ ? 4 : T];
  __device__ __forceinline__ void init(int w0, int lane) {
    if constexpr (KMAJ) {
      const int r = w0 + (lane & 31);
      const int sw = (r >> 1) & 7;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) base[kk] = (uint32_t)(r * 128 + (((2 * kk + (lane >> 5)) ^ sw) << 4));
    } else {
      const int g = lane >> 4, e = (lane >> 2) & 3, t = lane & 3;
      const int kr = 8 * (g >> 1) + e;  // + 16 kk + 4 h
#pragma unroll
      for (int i = 0; i < T; ++i) {
        const int m = w0 + 32 * i + 16 * (g & 1) + 4 * t;
        base[i] = (uint32_t)(kr * ROWS * 2 + (dma_chunk<ROWS, false>(e, m >> 3) << 4) + (m & 7) * 2);
      }
    }
  }
  // fragment i (rows w0 + 32 i ..) at k step kk of the tile at lds
  template <int I, int KK>
  __device__ __forceinline__ uint4 read(uint32_t lds) const {
    if constexpr (KMAJ) {
      return lds_b128(lds + base[KK] + I * 32 * 128);
    } else {
      const uint2 lo = lds_tr_b64(lds + base[I] + KK * 16 * ROWS * 2);
      const uint2 hi = lds_tr_b64(lds + base[I] + KK * 16 * ROWS * 2 + 4 * ROWS * 2);
      return make_uint4(lo.x, lo.y, hi.x, hi.y);
    }
  }
};

// Sum of the 8 half values of an MFMA operand fragment, in a fixed pairwise order.
template <int DT>
__device__ __forceinline__ float frag_sum8(const uint4& f) {
  const uint32_t w[4] = {f.x, f.y, f.z, f.w};
  float p[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) p[k] = h2f<DT>((uint16_t)(w[k] & 0xFFFFu)) + h2f<DT>((uint16_t)(w[k] >> 16));
  return (p[0] + p[1]) + (p[2] + p[3]);
}

// One BM x BN output tile per workgroup, waves of WM x WN, k tiles of 64 in
// two LDS stages.
//
// What bounds it: with random operands and every CU busy the chip runs at its
// power limit (256 x 256 tiles: 1.65 us per k tile, 1.3 PFLOP/s; 1.2 us with
// operands of zeros), so the shape of the tiles matters through the bytes
// moved per MFMA, the rounds a tile count needs, and what each tile costs
// before and after its k loop.  The loop itself has no wait at its top: the
// barrier that publishes k tile kt + 1, and frees the stage of tile kt,
// stands before the last of tile kt's four k steps of 16, whose MFMAs cover the
// fragment reads of tile kt + 1's first step; the copies of tile kt + 2 start
// right behind it and have a whole k tile to land.  (With the barrier at the
// top of each k tile, 128 x 128 tiles took 61.5 / 56.2 / 78.9 us forward at
// 12608 x 2304 x 768, dX there and forward at 12608 x 3072 x 768 in bf16;
// this loop 53.6 / 50.7 / 69.9.)
//
// OCC: waves per SIMD the register budget is sized for.  E: the epilogue
// operations compiled in (EPI_GENERIC: taken from the arguments).
//
// DBS: also sum the rows of A over this workgroup's k range (the bias
// gradient of a weight-gradient product; see GemmArgs::db).  The waves of
// the left half of the tile (wn0 == 0) add up their A fragments as the MFMAs
// consume them: lane l holds 8 consecutive k of row l % 32 (k half l / 32),
// so per lane a running float32 sum per fragment, in k order, and at the end
// lane l plus lane l + 32 give the row's sum.  With split-K the work is
// spread over the C tile columns that share the A rows: the workgroup of
// column c sums the k tiles kt = c, c + C, ... of its split and writes
// partial dbp[row][split * C + c] (the reduction adds a row's C x splits
// partials with one wave, in a fixed order); without split-K column 0 sums
// every k tile and writes db itself.
//
// STG (1; 2 for operands of StagedOperand's ANY form): the operands go
// through registers (StagedOperand) instead of the direct copies: any
// alignment and any reduction length.  Tile kt + 1 is written to the other
// stage and the loads of tile kt + 3 are issued ahead of the MFMAs of tile kt,
// so a load has two k tiles to land.  (One-value loads served these operands
// before: 8415 x 768 x 588 in bf16 forward / dX / dW took 89 / 145 / 157 us.)
template <int DT, int BM, int BN, int WM, int WN, int OCC, bool AK, bool BKM, int E, bool DBS = false,
          int STG = 0>
__global__ __launch_bounds__((BM / WM) * (BN / WN) * 64)
__attribute__((amdgpu_waves_per_eu(OCC, OCC)))
void gemm_tile_kernel(GemmArgs g) {
  constexpr int NWAVES = (BM / WM) * (BN / WN);
  constexpr int TM = WM / 32, TN = WN / 32;
  constexpr int A_BYTES = BM * 64 * 2, B_BYTES = BN * 64 * 2;
  constexpr int STAGE = A_BYTES + B_BYTES;
  constexpr int L = (BM + BN) / 8 / NWAVES;  // copies per lane per k tile
  // LDS read instructions per k step (a k-major fragment is one 16-byte
  // read, an mn-major one two transposing 8-byte reads)
  constexpr int kReads = TM * (AK ? 1 : 2) + TN * (BKM ? 1 : 2);
  // the epilogue works on 64 columns of a wave at a time
  constexpr int EC = WN < 64 ? WN : 64;
  constexpr int EPI = NWAVES * WM * (EC + 4) * 2;
  __shared__ __attribute__((aligned(1024))) uint8_t smem[2 * STAGE > EPI ? 2 * STAGE : EPI];
  const uint32_t lds0 = lds_u32(smem);

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm0 = (wave / (BN / WN)) * WM;
  const int wn0 = (wave % (BN / WN)) * WN;

  int64_t m0, n0;
  tile_origin<BM, BN>(g.M, g.N, m0, n0);
  int64_t z = blockIdx.y;
  int split = 0;
  int64_t offA = 0, offB = 0, offC = 0;
  if (g.splits > 1) {
    split = (int)z;
  } else {
    const int64_t i0 = (uint32_t)z / (uint32_t)g.nb1, i1 = (uint32_t)z % (uint32_t)g.nb1;
    offA = i0 * g.sA0 + i1 * g.sA1;
    offB = i0 * g.sB0 + i1 * g.sB1;
    offC = i0 * g.sC0 + i1 * g.sC1;
  }
  const int64_t kbeg = (int64_t)split * g.k_split;
  const int64_t kend = min(g.K, kbeg + g.k_split);
  const int nk = (int)((kend - kbeg + (STG ? 63 : 0)) / 64);

  const uint16_t* Ab = g.A + offA + (AK ? m0 * g.lda + kbeg : kbeg * g.lda + m0);
  const uint16_t* Bb = g.B + offB + (BKM ? n0 * g.ldb + kbeg : kbeg * g.ldb + n0);
  std::conditional_t<STG != 0, StagedOperand<BM, AK, NWAVES, STG == 2>, DmaOperand<BM, AK, NWAVES>> da;
  std::conditional_t<STG != 0, StagedOperand<BN, BKM, NWAVES, STG == 2>, DmaOperand<BN, BKM, NWAVES>> db;
  if constexpr (STG != 0) {
    da.init(g.lda, g.M - m0, wave, lane);
    db.init(g.ldb, g.N - n0, wave, lane);
  } else {
    da.init(g.lda, (int)min<int64_t>(BM, g.M - m0), wave, lane);
    db.init(g.ldb, (int)min<int64_t>(BN, g.N - n0), wave, lane);
  }

  const bool whole = g.full_epi && m0 + BM <= g.M && n0 + BN <= g.N;  // uniform over the workgroup
  const int64_t mw = m0 + wm0, nw = n0 + wn0;
  // A whole tile's GELU' or residual operand is loaded into registers before
  // the first copies where they fit (the oldest loads, so the first tile's
  // wait covers them): the epilogue then starts without a memory round trip.
  constexpr bool kPF = STG == 0 && E != EPI_GENERIC && (E & (EPI_DACT | EPI_RESID)) != 0 && TN == 2 && TM <= 2;
  u32x4 pf[kPF ? 4 * TM : 1];
  if constexpr (kPF) {
    if (whole) {
      const int64_t ldp = (E & EPI_DACT) ? g.ldc : g.ldr;
      const uint16_t* src = ((E & EPI_DACT) ? g.dact : g.resid) + (mw * ldp + nw);
#pragma unroll
      for (int t = 0; t < 4 * TM; ++t)
        pf[t] = *reinterpret_cast<const u32x4*>(src + (uint32_t)(((lane >> 3) + 8 * t) * ldp + 8 * (lane & 7)));
    }
  }

  auto issue = [&](int kt, auto par) {  // par: STG's register set, kt & 1
    if constexpr (STG != 0) {
      const bool past = kt >= nk;
      kt = min(kt, nk - 1);
      const int krem = (int)min<int64_t>(kend - kbeg - 64 * (int64_t)kt, 1 << 20);
      da.template load<par>(Ab + (int64_t)kt * (AK ? 64 : 64 * g.lda), krem, past);
      db.template load<par>(Bb + (int64_t)kt * (BKM ? 64 : 64 * g.ldb), krem, past);
    } else {
      const uint32_t st = lds0 + (uint32_t)((kt & 1) * STAGE);
      da.issue(reinterpret_cast<const uint16_t*>(reinterpret_cast<const uint8_t*>(Ab) + kt * da.step), st, wave);
      db.issue(reinterpret_cast<const uint16_t*>(reinterpret_cast<const uint8_t*>(Bb) + kt * db.step),
               st + A_BYTES, wave);
    }
  };
  auto put = [&](auto par) {  // STG: a loaded k tile (register set par) into stage par
    if constexpr (STG != 0) {
      da.template store<par>(smem + par * STAGE, wave, lane);
      db.template store<par>(smem + par * STAGE + A_BYTES, wave, lane);
    }
  };
  constexpr std::integral_constant<int, 0> I0{};
  constexpr std::integral_constant<int, 1> I1{};
  constexpr std::integral_constant<int, 2> I2{};
  constexpr std::integral_constant<int, 3> I3{};
  // a single k tile of one-value loads: nothing to prefetch
  const bool one = STG == 2 && nk == 1;
  if constexpr (STG != 0) {
    // no branch around a load in the loop (one would make the waits count the
    // later loads too): past the last k tile something is loaded and not used
    issue(0, I0);
    if (!one) issue(1, I1);
  } else {
    issue(0, I0);
    if (nk > 1) issue(1, I0);
  }

  FragReader<BM, AK, TM> fa;
  FragReader<BN, BKM, TN> fb;
  fa.init(wm0, lane);
  fb.init(wn0, lane);
  f32x16 acc[TM][TN];
  static_for<TM>([&](auto i) {
    static_for<TN>([&](auto j) {
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
    });
  });
  // bias-gradient sums: tile columns sharing the A rows, this one's index,
  // and the next k tile this wave adds up (uniform over the wave)
  const int db_cols = g.splits > 1 ? (int)((g.N + BN - 1) / BN) : 1;
  const int db_col = g.splits > 1 ? (int)(n0 / BN) : 0;
  const bool dbw = DBS && wn0 == 0 && (g.splits > 1 || n0 == 0);
  int db_next = db_col;
  float dbs[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) dbs[i] = 0.0f;

  if constexpr (STG != 0) {
    put(I0);
    if (!one) issue(2, I0);
  } else {
    if (nk > 1) wait_vmcnt<L>();
    else wait_vmcnt<0>();
  }
  __syncthreads();

  // fragments double-buffered over the k steps of 16: the LDS reads of the
  // next step are issued among the MFMAs of the current one
  uint4 af[2][TM], bf[2][TN];
  auto read = [&](auto set, auto kk, uint32_t sa) {
    static_for<TM>([&](auto i) { af[set][i] = fa.template read<i, kk>(sa); });
    static_for<TN>([&](auto j) { bf[set][j] = fb.template read<j, kk>(sa + A_BYTES); });
  };
  auto multiply = [&](auto set, bool db_now) {
    static_for<TM>([&](auto i) {
      static_for<TN>([&](auto j) { acc[i][j] = mfma32<DT>(bf[set][j], af[set][i], acc[i][j]); });
    });
    if constexpr (DBS) {
      if (db_now) static_for<TM>([&](auto i) { dbs[i] += frag_sum8<DT>(af[set][i]); });
    }
    static_for<TM * TN>([&](auto x) {  // each MFMA with its share of the reads
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      constexpr int n = (x + 1) * kReads / (TM * TN) - x * kReads / (TM * TN);
      if constexpr (n > 0) __builtin_amdgcn_sched_group_barrier(0x100, n, 0);
    });
    __builtin_amdgcn_sched_barrier(0);
  };
  read(I0, I0, lds0);
  // one k tile; par = kt & 1 and last, which loads nothing, for STG only
  auto k_tile = [&](int kt, auto par, auto last) {
    const uint32_t sa = lds0 + (uint32_t)((kt & 1) * STAGE);
    const uint32_t sn = lds0 + (uint32_t)(((kt + 1) & 1) * STAGE);
    const bool db_now = dbw && kt == db_next;
    if (db_now) db_next += db_cols;
    if constexpr (STG != 0) {
      // the other stage was read before the last barrier
      constexpr std::integral_constant<int, 1 - par> other{};
      if (kt + 1 < nk) put(other);
      if constexpr (!last) issue(kt + 3, other);
    }
    read(I1, I1, sa);
    multiply(I0, db_now);
    read(I0, I2, sa);
    multiply(I1, db_now);
    read(I1, I3, sa);
    multiply(I0, db_now);
    if (kt + 1 < nk) {
      if constexpr (STG == 0) wait_vmcnt<0>();  // k tile kt + 1 has landed
      __syncthreads();
      if constexpr (STG == 0) {
        if (kt + 2 < nk) issue(kt + 2, I0);
      }
      read(I0, I0, sn);
    }
    multiply(I1, db_now);
  };
  if constexpr (STG != 0) {
    int kt = 0;
    for (; kt + 1 < nk; kt += 2) {
      k_tile(kt, I0, I0);
      k_tile(kt + 1, I1, I0);
    }
    if (kt < nk) k_tile(kt, I0, I1);
  } else {
    for (int kt = 0; kt < nk; ++kt) k_tile(kt, I0, I0);
  }

  if constexpr (DBS) {
    if (dbw) {
      int bad = 0;
      static_for<TM>([&](auto i) {
        const float other = __shfl_xor(dbs[i], 32);  // the row's other 8 k of every step
        const int64_t row = mw + 32 * i + lane;
        if (lane < 32 && row < g.M) {
          const float v = dbs[i] + other;
          if (g.splits > 1) {
            g.dbp[row * ((int64_t)g.splits * db_cols) + (int64_t)split * db_cols + db_col] = v;
          } else {
            const uint16_t h = f2h<DT>(v);
            g.db[row] = h;
            bad += h_nonfinite<DT>(h) ? 1 : 0;
          }
        }
      });
      if (g.nonfinite) add_nonfinite(g.nonfinite, bad);
    }
  }
  // the accumulators hold C^T blocks (the MFMA operands are swapped above)
  if (g.splits > 1) {
    gemm_partials<TM, TN>(g, acc, mw, nw, lane, split);
    return;
  }
  __syncthreads();  // every wave is done reading the stage buffers
  uint16_t* lds = reinterpret_cast<uint16_t*>(smem) + wave * (WM * (EC + 4));
  static_for<(TN + 1) / 2>([&](auto c) {
    constexpr int J0 = 2 * c, TC = TN - J0 < 2 ? TN - J0 : 2;
    if (whole)
      gemm_epilogue_lds<DT, TM, TC, E, false, J0>(g, acc, mw, nw + 32 * J0, lane, offC, lds,
                                                  kPF ? pf : nullptr);
    else
      gemm_epilogue_lds<DT, TM, TC, E, true, J0>(g, acc, mw, nw + 32 * J0, lane, offC, lds, nullptr,
                                                 (int)min<int64_t>(WM, g.M - mw),
                                                 (int)min<int64_t>(32 * TC, g.N - nw - 32 * J0));
  });
}

// Sum of split-K partials in split order, one rounding: C = half(sum_s W[s]),
// one thread per output in the first ceil(MN / 256) workgroups.  The
// workgroups after them reduce the bias-gradient partials dbp[row][p],
// p < dbparts, one wave per row (nrows rows; 0: none): lane l adds p = l,
// l + 64, ... in order, then the fixed wave tree of wave_sum; db = half of
// that.  Non-finite results are added to *nonfinite when it is set.
// VEC (MN a multiple of 4, ws 16-byte and C 8-byte aligned): each thread
// reduces 4 consecutive outputs with 16-byte loads and one 8-byte store, each
// output summed in the same split order as the scalar form (the same bits):
// 3072 x 768 from 2 splits alone 6.3 -> 5.4 us, 768 x 768 from 8 splits 6.2 -> 4.9.
template <int DT, bool VEC>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float* __restrict__ ws, int splits,
                                                            int64_t MN, uint16_t* __restrict__ C,
                                                            int32_t* __restrict__ nonfinite,
                                                            const float* __restrict__ dbp, int dbparts,
                                                            int64_t nrows, uint16_t* __restrict__ db) {
  constexpr int PER = VEC ? 4 : 1;
  const int64_t mn_blocks = (MN + 256 * PER - 1) / (256 * PER);
  if ((int64_t)blockIdx.x < mn_blocks) {
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * PER;
    if (i >= MN) return;
    if constexpr (VEC) {
      f32x4 s = *reinterpret_cast<const f32x4*>(ws + i);
      for (int k = 1; k < splits; ++k) {
        const f32x4 t = *reinterpret_cast<const f32x4*>(ws + (int64_t)k * MN + i);
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] += t[e];
      }
      uint16_t h[4];
      int bad = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        h[e] = f2h<DT>(s[e]);
        bad += h_nonfinite<DT>(h[e]) ? 1 : 0;
      }
      *reinterpret_cast<uint2*>(C + i) =
          make_uint2((uint32_t)h[0] | ((uint32_t)h[1] << 16), (uint32_t)h[2] | ((uint32_t)h[3] << 16));
      if (nonfinite) add_nonfinite(nonfinite, bad);
    } else {
      float s = ws[i];
      for (int k = 1; k < splits; ++k) s += ws[(int64_t)k * MN + i];
      const uint16_t h = f2h<DT>(s);
      C[i] = h;
      if (nonfinite) add_nonfinite(nonfinite, h_nonfinite<DT>(h) ? 1 : 0);
    }
    return;
  }
  const int64_t row = ((int64_t)blockIdx.x - mn_blocks) * 4 + (threadIdx.x >> 6);
  if (row >= nrows) return;  // uniform over the wave
  const int lane = threadIdx.x & 63;
  const float* p = dbp + row * dbparts;
  float s = 0.0f;
  for (int k = lane; k < dbparts; k += 64) s += p[k];
  s = wave_sum(s);
  if (lane == 0) {
    const uint16_t h = f2h<DT>(s);
    db[row] = h;
    if (nonfinite) add_nonfinite(nonfinite, h_nonfinite<DT>(h) ? 1 : 0);
  }
}

// launch shape of splitk_reduce_kernel: MN outputs and nrows bias rows
inline unsigned splitk_reduce_blocks(int64_t MN, int64_t nrows, bool vec) {
  const int64_t per = vec ? 1024 : 256;
  return (unsigned)((MN + per - 1) / per + (nrows + 3) / 4);
}

inline bool splitk_reduce_vec(const float* ws, int64_t MN, const uint16_t* C) {
  return MN % 4 == 0 && (reinterpret_cast<uintptr_t>(ws) & 15u) == 0 &&
         (reinterpret_cast<uintptr_t>(C) & 7u) == 0;
}

// ------------------------------------------------------------ dispatch --

static bool aligned_vec(const void* p, int64_t ld, int64_t s0, int64_t s1) {
  return (reinterpret_cast<uintptr_t>(p) & 15u) == 0 && ld % 8 == 0 && s0 % 8 == 0 && s1 % 8 == 0;
}

static bool operands_aligned(const GemmArgs& g) {
  return aligned_vec(g.A, g.lda, g.sA0, g.sA1) && aligned_vec(g.B, g.ldb, g.sB0, g.sB1);
}

// Epilogue mask of a call: 0 with split-K, whose kernels end before it, and
// EPI_GENERIC for calls that count non-finite outputs (weight gradients).
static int epilogue_mask(const GemmArgs& g) {
  if (g.splits > 1) return 0;
  if (g.nonfinite) return EPI_GENERIC;
  return (g.bias ? EPI_BIAS : 0) | (g.act == MPX_ACT_GELU_TANH ? EPI_GELU : 0) |
         (g.dact ? EPI_DACT : 0) | (g.resid ? EPI_RESID : 0);
}

// Whole-tile epilogue preconditions that do not depend on the tile: output,
// pre-activation, GELU' and residual operands 16-byte aligned with row
// strides a multiple of 8, the bias 8-byte aligned, and the per-lane 32-bit
// offsets in range.
static bool full_epilogue_ok(const GemmArgs& g, int bm) {
  auto al8 = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 7u) == 0; };
  auto al16 = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; };
  const bool strides = g.sC0 % 8 == 0 && g.sC1 % 8 == 0;
  return g.splits == 1 && strides && g.ldc % 8 == 0 && al16(g.C) && (!g.bias || al8(g.bias)) &&
         (!g.pre || al16(g.pre)) && (!g.dact || al16(g.dact)) &&
         (!g.resid || (al16(g.resid) && g.ldr % 8 == 0)) && g.ldc * bm < ((int64_t)1 << 30) &&
         g.ldr * bm < ((int64_t)1 << 30);
}

// The kernel of a call's layouts and epilogue: the epilogues of the library's own
// calls are compiled in, any other takes the generic one, which loads its
// operand row by row between the stores and is several times the code (forward
// with residual 8366 x 856 x 104 bf16 generic / compiled in 23.6 / 16.4 us, 395
// products of 128 x 128 x 128 11.2 / 10.4).  MPX_K(AK, BKM, E, DBS) launches.
#define MPX_BY_EPILOGUE(ALL_LAYOUTS)                                         \
  do {                                                                       \
    const int e = epilogue_mask(g);                                          \
    if (ak && bk) {                                                          \
      switch (e) {                                                           \
        case 0: MPX_K(true, true, 0, false); break;                          \
        case EPI_BIAS: MPX_K(true, true, EPI_BIAS, false); break;            \
        case EPI_BIAS | EPI_GELU: MPX_K(true, true, EPI_BIAS | EPI_GELU, false); break;   \
        case EPI_BIAS | EPI_RESID: MPX_K(true, true, EPI_BIAS | EPI_RESID, false); break; \
        default: MPX_K(true, true, EPI_GENERIC, false);                      \
      }                                                                      \
    } else if (ak) {                                                         \
      switch (e) {                                                           \
        case 0: MPX_K(true, false, 0, false); break;                         \
        case EPI_DACT: MPX_K(true, false, EPI_DACT, false); break;           \
        default: MPX_K(true, false, EPI_GENERIC, false);                     \
      }                                                                      \
    } else if constexpr (ALL_LAYOUTS) {                                      \
      if (bk) {                                                              \
        if (e == 0) MPX_K(false, true, 0, false);                            \
        else MPX_K(false, true, EPI_GENERIC, false);                         \
      } else if (g.db) { /* weight gradient, the bias gradient summed alongside */ \
        if (e == 0) MPX_K(false, false, 0, true);                            \
        else MPX_K(false, false, EPI_GENERIC, true);                         \
      } else {                                                               \
        if (e == 0) MPX_K(false, false, 0, false);                           \
        else MPX_K(false, false, EPI_GENERIC, false);                        \
      }                                                                      \
    } else {                                                                 \
      return hipErrorInvalidValue;                                           \
    }                                                                        \
  } while (0)

// Direct-to-LDS tiles.  The 128 x 128 ones take every layout; the others a
// k-major A (forward, dX) without split-K.
template <int DT, int BM, int BN, int WM, int WN, int OCC>
hipError_t launch_tiles(GemmArgs g, bool ak, bool bk, int64_t nbatch, hipStream_t s) {
  constexpr int NT = (BM / WM) * (BN / WN) * 64;
  const int64_t tiles = ((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN);
  dim3 grid((unsigned)tiles, (unsigned)(g.splits > 1 ? g.splits : nbatch));
  g.full_epi = full_epilogue_ok(g, BM) ? 1 : 0;
#define MPX_K(AKv, BKv, Ev, DBv) \
  gemm_tile_kernel<DT, BM, BN, WM, WN, OCC, AKv, BKv, Ev, DBv><<<grid, NT, 0, s>>>(g)
  MPX_BY_EPILOGUE((BM == 128 && BN == 128));
#undef MPX_K
  return hipGetLastError();
}

// Operands only StagedOperand's ANY form takes: rows of fewer than 8 values (no
// 16-byte load fits) or lane offsets past 31 bits.
inline bool staged_any(const GemmArgs& g, bool ak, bool bk) {
  const int64_t lim = ((int64_t)1 << 31) - 4096;
  return (ak ? g.K : g.M) < 8 || (bk ? g.K : g.N) < 8 || g.lda * 256 >= lim || g.ldb * 256 >= lim;
}

// Operands staged through registers (STG 1: any alignment, any reduction
// length; 2: those of staged_any).
template <int DT, int BM, int BN, int WM, int WN, int STG>
hipError_t launch_staged(GemmArgs g, bool ak, bool bk, int64_t nbatch, hipStream_t s) {
  constexpr int NT = (BM / WM) * (BN / WN) * 64;
  const int64_t tiles = ((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN);
  dim3 grid((unsigned)tiles, (unsigned)(g.splits > 1 ? g.splits : nbatch));
  g.full_epi = full_epilogue_ok(g, BM) ? 1 : 0;
#define MPX_K(AKv, BKv, Ev, DBv) \
  gemm_tile_kernel<DT, BM, BN, WM, WN, 2, AKv, BKv, Ev, DBv, STG><<<grid, NT, 0, s>>>(g)
  MPX_BY_EPILOGUE(true);
#undef MPX_K
  return hipGetLastError();
}

// The launchers are compiled in three sources per half type, which build in
// parallel: the 128 x 128 and 64 x 128 tiles (gemm_f16.hip), the wide ones
// (gemm_wide_f16.hip) and the register-staged ones (gemm_staged_f16.hip);
// likewise for bf16.
#define MPX_GEMM_STAGED(X, DT)                                                              \
  X template hipError_t launch_staged<DT, 64, 64, 32, 32, 1>(GemmArgs, bool, bool, int64_t, hipStream_t); \
  X template hipError_t launch_staged<DT, 64, 64, 32, 32, 2>(GemmArgs, bool, bool, int64_t, hipStream_t); \
  X template hipError_t launch_staged<DT, 128, 128, 64, 64, 1>(GemmArgs, bool, bool, int64_t, hipStream_t);
#define MPX_GEMM_WIDE(X, DT)                                                                \
  X template hipError_t launch_tiles<DT, 256, 256, 128, 64, 2>(GemmArgs, bool, bool, int64_t, hipStream_t); \
  X template hipError_t launch_tiles<DT, 128, 192, 64, 96, 2>(GemmArgs, bool, bool, int64_t, hipStream_t);
#ifndef MPX_GEMM_STAGED_SOURCE
MPX_GEMM_STAGED(extern, MPX_F16)
MPX_GEMM_STAGED(extern, MPX_BF16)
#endif
#ifndef MPX_GEMM_WIDE_SOURCE
MPX_GEMM_WIDE(extern, MPX_F16)
MPX_GEMM_WIDE(extern, MPX_BF16)
#endif

// Tile configurations (the value of mpx_gemm_set_config):
//   1  register-staged 64 x 64, 4 waves of 32 x 32    (any operands)
//   2  register-staged 128 x 128, 4 waves of 64 x 64  (any operands)
// direct-to-LDS:
//   3  256 x 256, 8 waves of 128 x 64, one workgroup per CU    (A k-major)
//   5  128 x 192, 4 waves of 64 x 96, two workgroups per CU    (A k-major; also 4)
//   7  128 x 128, 4 waves of 64 x 64, two workgroups per CU    (also 6, 10)
//   9  64 x 128, 4 waves of 32 x 64, three workgroups per CU   (A k-major; also 11)
//   8  skinny products: one wave (K > 32) or one lane (K <= 32) per output
extern int g_forced_config;  // defined in gemm.hip

// The direct-to-LDS kernel needs 16-byte aligned operands and whole k tiles
// of 64 in every split, and 32-bit per-lane copy offsets.
static bool dma_ok(const GemmArgs& g, bool vec, bool ak, bool bk) {
  if (!vec || g.K % 64 != 0) return false;
  if (g.splits > 1 && g.k_split % 64 != 0) return false;
  const int64_t lim = (int64_t)1 << 31;
  const int64_t spanA = (ak ? 256 : 64) * g.lda * 2, spanB = (bk ? 256 : 64) * g.ldb * 2;
  return spanA < lim && spanB < lim;
}

static bool small_ok(const GemmArgs& g, int64_t nbatch);

// Direct-to-LDS tiles for a k-major A, by estimated time.  A chip of 256 CUs
// runs 256 x per_cu tiles at a time; a round of o tiles per CU takes
// nk x k_us[o - 1] (nk k tiles of 64) plus o x tile_us for what surrounds the
// k loops (tile_us[1]: epilogues that read or write a second matrix), and the
// last round has only as many tiles per CU as are left.  The constants are
// regression coefficients, set for the choice and not for the times, which
// they give too small (median 1.1 to 1.4 by tile; a full chip of 128 x 128 tiles does
// not run at the 1.7 PFLOP/s of 0.65 us): those of least loss on 70% of 2000
// measured products (M 65..57000, N and K 64..4096, a tenth up to 16384; forward
// with bias, GELU or residual, dX, dX through GELU'; operands from HBM), none less
// for more tiles per CU.  On the other 30% the choice is 0.3% slower than the
// fastest tile, 64 x 128 alone 6%, 128 x 128 alone 13%.  256 x 256 is charged 10% more
// than its fit (0.4% then): one workgroup takes a whole CU, and beside a second
// stream it loses that (one-block step, 8320 x 1536 x 384 with GELU and its dX through
// GELU': 348.5 us with 256 x 256, 342 with 128 x 128).  Examples (us;
// 256 x 256, 128 x 192, 128 x 128, 64 x 128): 12608 x 2304 x 768 dX
// 49 / 51 / 51 / 58; 12608 x 768 x 3072 forward 78 / 66 / 80 / 87; 16640 x 384
// x 1536 44 / 34 / 29 / 41; 8320 x 384 x 384 16.6 / 10.0 / 9.0 / 8.9.
struct TileCost {
  int config, bm, bn, per_cu;
  double k_us[3], tile_us[2];
};
static int choose_tiles(const GemmArgs& g, int64_t nbatch) {
  static const TileCost costs[] = {
      {9, 64, 128, 3, {0.48, 0.50, 0.78}, {0.60, 1.25}},
      {7, 128, 128, 2, {0.51, 0.65, 0}, {1.36, 2.75}},
      {5, 128, 192, 2, {0.77, 0.83, 0}, {1.86, 4.49}},
      {3, 256, 256, 1, {1.08, 0, 0}, {7.36, 14.1}},
  };
  const int second = g.pre || g.dact || g.resid ? 1 : 0;
  const double nk = (double)(g.K / 64);
  int best = 7;
  double least = 0.0;
  for (const TileCost& c : costs) {
    const int64_t tiles = ((g.M + c.bm - 1) / c.bm) * ((g.N + c.bn - 1) / c.bn) * nbatch;
    auto round = [&](int64_t o) { return o ? nk * c.k_us[o - 1] + c.tile_us[second] * (double)o : 0.0; };
    const double t = (double)(tiles / (256 * c.per_cu)) * round(c.per_cu) +
                     round((tiles % (256 * c.per_cu) + 255) / 256);
    if (least == 0.0 || t < least) {
      least = t;
      best = c.config;
    }
  }
  return best;
}

static int choose_config(const GemmArgs& g, bool vec, bool ak, bool bk, int64_t nbatch) {
  const bool dma = dma_ok(g, vec, ak, bk);
  const bool small = small_ok(g, nbatch);
  int f = g_forced_config;
  f = f == 4 ? 5 : f == 6 || f == 10 ? 7 : f == 11 ? 9 : f;
  if (f == 8 && small) return 8;
  if (f == 7 && dma) return 7;
  if ((f == 3 || f == 5 || f == 9) && dma && ak && g.splits == 1) return f;
  const bool any = staged_any(g, ak, bk);
  if (f == 1 || f == 2) return any ? 1 : f;
  if (small && (g.M <= 32 || g.N <= 32 || g.K <= 32)) return 8;
  // 64 x 64 register-staged tiles (us, against the tile that would be taken
  // otherwise):
  // - outputs of up to 64 columns or rows: forward 43 x 192 x 64 5.0 / 6.5 with
  //   64 x 128 tiles, 256 x 100 x 384 6.4 / 8.9 and dX there 4.3 / 6.3 with 128 x 128, a
  //   split dW of 64 x 128 over 3310 rows 17 / 24.  Not dX of up to 64 rows on the direct
  //   tiles (equal up to K = 1024; the staged ones gain 8% only beyond).
  // - products the tiles of choose_tiles do not take, with so few 64 x 64 tiles
  //   that smaller ones spread the work: up to two per CU against the staged
  //   128 x 128 tiles (1000 x 768 x 768 dW, unaligned, 0.6 of their time; at 768 tiles
  //   1.1), one per CU against the direct ones (dW and batched products of 256 tiles
  //   0.86 to 1.03, of 512 1.04 to 1.6)
  const int64_t t64 = ((g.M + 63) / 64) * ((g.N + 63) / 64) * nbatch;
  const bool tiles = dma && ak && g.splits == 1;
  if (any || g.N <= 64 || (g.M <= 64 && (bk || !tiles))) return 1;
  if (!tiles && g.splits == 1 && t64 <= (dma ? 256 : 512)) return 1;
  if (tiles) return choose_tiles(g, nbatch);
  return dma ? 7 : 2;
}

// ----------------------------------------------------------- skinny GEMMs --
//
// Products with a dimension of 32 or less (a classifier head: 10 outputs, or
// a reduction over 10 classes) waste most of a 32x32 MFMA tile and run a
// long dependent k loop on very few workgroups.  Here every output element
// gets its own wave when K > 32 (lane l sums k = l, l + 64, ... in float32,
// then a fixed butterfly adds the 64 lane sums) or its own lane when K <= 32
// (a plain k loop).  Both orders are fixed, so results are reproducible.
// Epilogue: bias and residual, h = half(acc + bias[n]), then half(h + R[m,n]).
template <int DT, bool WAVE>
__global__ __launch_bounds__(256) void gemm_small_kernel(GemmArgs g, bool ak, bool bk) {
  const int64_t MN = g.M * g.N;
  const int64_t idx = WAVE ? ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6))
                           : ((int64_t)blockIdx.x * 256 + threadIdx.x);
  if (idx >= MN) return;
  const int64_t m = idx / g.N, n = idx % g.N;
  // opA(m,k) = A[m*lda + k] (k-major) or A[k*lda + m]; opB(n,k) likewise
  const int64_t sam = ak ? g.lda : 1, sak = ak ? 1 : g.lda;
  const int64_t sbn = bk ? g.ldb : 1, sbk = bk ? 1 : g.ldb;
  const uint16_t* a = g.A + m * sam;
  const uint16_t* b = g.B + n * sbn;
  float acc = 0.0f;
  if constexpr (WAVE) {
    const int lane = threadIdx.x & 63;
    for (int64_t k = lane; k < g.K; k += 64) acc += h2f<DT>(a[k * sak]) * h2f<DT>(b[k * sbk]);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) acc += __shfl_xor(acc, o);
    if (lane != 0) return;
  } else {
    for (int64_t k = 0; k < g.K; ++k) acc += h2f<DT>(a[k * sak]) * h2f<DT>(b[k * sbk]);
  }
  const float bias = g.bias ? h2f<DT>(g.bias[n]) : 0.0f;
  uint16_t h = f2h<DT>(acc + bias);
  if (g.resid) h = f2h<DT>(h2f<DT>(h) + h2f<DT>(g.resid[m * g.ldr + n]));
  g.C[m * g.ldc + n] = h;
  if (g.nonfinite) add_nonfinite(g.nonfinite, h_nonfinite<DT>(h) ? 1 : 0);
}

static bool small_ok(const GemmArgs& g, int64_t nbatch) {
  return nbatch == 1 && g.splits == 1 && !g.pre && !g.dact && g.act == MPX_ACT_NONE &&
         g.M * g.N <= ((int64_t)1 << 22);
}

template <int DT>
static hipError_t launch_small(const GemmArgs& g, bool ak, bool bk, hipStream_t s) {
  const int64_t MN = g.M * g.N;
  if (g.K > 32)
    gemm_small_kernel<DT, true><<<(unsigned)((MN + 3) / 4), 256, 0, s>>>(g, ak, bk);
  else
    gemm_small_kernel<DT, false><<<(unsigned)((MN + 255) / 256), 256, 0, s>>>(g, ak, bk);
  return hipGetLastError();
}

// ak: A is k-major; bk: B is k-major.  A call with g.db set (a weight
// gradient whose bias gradient is wanted) gets it from the GEMM when the
// chosen kernel can sum it (the two-stage 128 x 128 kernels, and 64 x 64
// ones without split-K: the split-K partials are laid out for 128-wide tile
// columns); *db_fused tells the caller whether it did,
// and otherwise the caller computes the column sums itself.
template <int DT>
static hipError_t run_gemm(GemmArgs g, bool ak, bool bk, int64_t nbatch, hipStream_t s,
                           bool* db_fused) {
  const int cfg = choose_config(g, operands_aligned(g), ak, bk, nbatch);
  const bool fuse = g.db && (cfg == 7 || cfg == 2 || (cfg == 1 && g.splits == 1)) && !ak && !bk &&
                    nbatch == 1 && (g.splits == 1 || g.dbp);
  if (db_fused) *db_fused = fuse;
  if (!fuse) {
    g.db = nullptr;
    g.dbp = nullptr;
  }
  switch (cfg) {
    case 8: return launch_small<DT>(g, ak, bk, s);
    case 1:
      return staged_any(g, ak, bk) ? launch_staged<DT, 64, 64, 32, 32, 2>(g, ak, bk, nbatch, s)
                                   : launch_staged<DT, 64, 64, 32, 32, 1>(g, ak, bk, nbatch, s);
    case 2: return launch_staged<DT, 128, 128, 64, 64, 1>(g, ak, bk, nbatch, s);
    case 3: return launch_tiles<DT, 256, 256, 128, 64, 2>(g, ak, bk, nbatch, s);
    case 5: return launch_tiles<DT, 128, 192, 64, 96, 2>(g, ak, bk, nbatch, s);
    case 7: return launch_tiles<DT, 128, 128, 64, 64, 2>(g, ak, bk, nbatch, s);
    case 9: return launch_tiles<DT, 64, 128, 32, 64, 3>(g, ak, bk, nbatch, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t run_gemm_f16(const GemmArgs& g, bool ak, bool bk, int64_t nbatch, hipStream_t s,
                        bool* db_fused = nullptr);
hipError_t run_gemm_bf16(const GemmArgs& g, bool ak, bool bk, int64_t nbatch, hipStream_t s,
                         bool* db_fused = nullptr);

}  // namespace mpx
