// Float32 GEMMs on the float32 MFMA (v_mfma_f32_32x32x2_f32) for full-precision
// training, the baseline MPX's mixed precision is measured against (§4: full
// precision vs mixed precision).  128 x 128 output tiles, four waves
// of 64 x 64 (2 x 2 blocks of 32 x 32) and the same epilogue operations as the
// half kernels in float32.  Aligned operands (16-byte rows, a reduction that
// is a multiple of 32) take the direct-to-LDS kernel, any others the one that
// stages k tiles of 16 through registers.
#include "gemm_f32.h"

#include <algorithm>

#include "colsum.h"
#include "common.h"
#include "dma.h"
#include "mfma.h"

namespace mpx {

namespace {

constexpr int kBM = 128, kBN = 128, kBK = 16;
// LDS rows of 128 floats padded to 160: the two half-waves of an operand read
// (k and k + 1) fall 32 banks apart
constexpr int kPitch = 160;

// One operand tile (128 rows of the output dimension x 16 k) into registers
// and then into LDS as [k][row].  KMAJ: element (r, k) at P[r*ld + k]
// (a lane loads 4 consecutive k of one row), otherwise at P[k*ld + r] (4
// consecutive rows of one k).  Out-of-range elements read as zero.
template <bool KMAJ>
struct TileF32 {
  float v[8];
  __device__ __forceinline__ void load(const float* P, int64_t ld, int64_t r0, int64_t rows,
                                       int64_t k0, int64_t kend, bool vec, int tid) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      int64_t r, k;
      if constexpr (KMAJ) {
        r = r0 + (tid >> 2) + 64 * i;
        k = k0 + 4 * (tid & 3);
      } else {
        k = k0 + (tid >> 5) + 8 * i;
        r = r0 + 4 * (tid & 31);
      }
      if (vec && (KMAJ ? (r < rows && k + 4 <= kend) : (k < kend && r + 4 <= rows))) {
        const f32x4 x = *reinterpret_cast<const f32x4*>(P + (KMAJ ? r * ld + k : k * ld + r));
#pragma unroll
        for (int c = 0; c < 4; ++c) v[4 * i + c] = x[c];
      } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const int64_t rr = KMAJ ? r : r + c, kk = KMAJ ? k + c : k;
          v[4 * i + c] = (rr < rows && kk < kend) ? P[KMAJ ? rr * ld + kk : kk * ld + rr] : 0.0f;
        }
      }
    }
  }
  __device__ __forceinline__ void store(float (*S)[kPitch], int tid) const {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      if constexpr (KMAJ) {
        const int r = (tid >> 2) + 64 * i, k = 4 * (tid & 3);
#pragma unroll
        for (int c = 0; c < 4; ++c) S[k + c][r] = v[4 * i + c];
      } else {
        const int k = (tid >> 5) + 8 * i, r = 4 * (tid & 31);
        *reinterpret_cast<f32x4*>(&S[k][r]) = f32x4{v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]};
      }
    }
  }
};

// The wave's 2 x 2 blocks of 32 x 32 from output row mw and column nw on: split-K
// partials, or the epilogue.  Accumulator layout of a block: lane l holds
// column l % 32, value r is row 8 (r / 4) + 4 (l / 32) + r % 4.  32 rows at a time
// go through the wave's own [32][68] floats of LDS, then out 4 rows x 256
// contiguous bytes per access; the operand values of 16 rows are loaded
// together, ahead of the first store (a load behind a store that may alias
// it waits for memory: 247 -> 202 us forward at 16640 x 1536 x 384).  Stores straight
// from the accumulators, 40 KB of code, measured the same.
__device__ __forceinline__ void gemm_f32_epilogue(const GemmF32Args& g, const f32x16 (&acc)[2][2], int64_t mw,
                                                  int64_t nw, int lane, int split, int64_t offC, float* lds) {
  const bool part = g.splits > 1;
  float* out = part ? g.ws + (int64_t)split * g.M * g.N : g.C + offC;
  const int64_t ld = part ? g.N : g.ldc;
  const float* src = part ? nullptr : g.dact ? g.dact : g.resid;  // no call has both
  float* pre = part ? nullptr : g.pre;
  const int c4 = 4 * (lane & 15);
  const int64_t n = nw + c4;
  const int nc = (int)max<int64_t>(0, min<int64_t>(4, g.N - n));
  auto al16 = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; };
  const bool vec = nc == 4 && ld % 4 == 0 && al16(out) && al16(src) && al16(pre);
  auto load4 = [&](const float* p) {
    f32x4 v = {0.0f, 0.0f, 0.0f, 0.0f};
    if (vec) return *reinterpret_cast<const f32x4*>(p);
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if (c < nc) v[c] = p[c];
    return v;
  };
  auto store4 = [&](float* p, f32x4 v) {
    if (vec) {
      *reinterpret_cast<f32x4*>(p) = v;
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (c < nc) p[c] = v[c];
    }
  };
  f32x4 bias = {0.0f, 0.0f, 0.0f, 0.0f};
  if (!part && g.bias) {
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if (c < nc) bias[c] = g.bias[n + c];
  }
  static_for<2>([&](auto i) {
    asm volatile("" ::: "memory");
    static_for<2>([&](auto j) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        lds[(8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * 68 + 32 * j + (lane & 31)] = acc[i][j][r];
    });
    asm volatile("" ::: "memory");  // the wave's own writes come first
#pragma unroll 1
    for (int t = 0; t < 2; ++t) {  // 16 rows
      f32x4 op[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int64_t m = mw + 32 * i + 16 * t + 4 * q + (lane >> 4);
        op[q] = src && m < g.M ? load4(src + offC + m * ld + n) : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int row = 16 * t + 4 * q + (lane >> 4);
        const int64_t m = mw + 32 * i + row;
        if (m >= g.M) continue;
        f32x4 v = *reinterpret_cast<const f32x4*>(lds + row * 68 + c4);
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] += bias[c];
        if (pre) store4(pre + offC + m * ld + n, v);
        if (!part && g.act == MPX_ACT_GELU_TANH) {
#pragma unroll
          for (int c = 0; c < 4; ++c) v[c] = gelu_tanh(v[c]);
        }
        if (src) {
#pragma unroll
          for (int c = 0; c < 4; ++c) v[c] = g.dact ? v[c] * gelu_tanh_grad(op[q][c]) : v[c] + op[q][c];
        }
        store4(out + m * ld + n, v);
      }
    }
  });
}

template <bool AK, bool BKM>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmF32Args g) {
  // the operand tiles; the epilogue's staging (4 x 32 x 68 floats) follows in both
  __shared__ __attribute__((aligned(16))) float smem[4][kBK][kPitch];
  float (*sA)[kBK][kPitch] = smem;
  float (*sB)[kBK][kPitch] = smem + 2;
  static_assert(4 * 32 * 68 <= 4 * kBK * kPitch, "epilogue staging");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm0 = (wave >> 1) * 64, wn0 = (wave & 1) * 64;
  const int64_t tiles_n = (g.N + kBN - 1) / kBN;
  const int64_t m0 = (int64_t)(blockIdx.x / tiles_n) * kBM;
  const int64_t n0 = (int64_t)(blockIdx.x % tiles_n) * kBN;
  int split = 0;
  const float* Ap = g.A;
  const float* Bp = g.B;
  int64_t offC = 0;
  if (g.splits > 1) {
    split = (int)blockIdx.y;
  } else {  // batch entry
    const int64_t i0 = blockIdx.y / g.nb1, i1 = blockIdx.y % g.nb1;
    Ap += i0 * g.sA0 + i1 * g.sA1;
    Bp += i0 * g.sB0 + i1 * g.sB1;
    offC = i0 * g.sC0 + i1 * g.sC1;
  }
  const int64_t kbeg = (int64_t)split * g.k_split;
  const int64_t kend = min(g.K, kbeg + g.k_split);
  const int nk = (int)((kend - kbeg + kBK - 1) / kBK);
  const bool va = (reinterpret_cast<uintptr_t>(Ap) & 15u) == 0 && g.lda % 4 == 0;
  const bool vb = (reinterpret_cast<uintptr_t>(Bp) & 15u) == 0 && g.ldb % 4 == 0;

  f32x16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  TileF32<AK> ta;
  TileF32<BKM> tb;
  if (nk > 0) {
    ta.load(Ap, g.lda, m0, g.M, kbeg, kend, va, tid);
    tb.load(Bp, g.ldb, n0, g.N, kbeg, kend, vb, tid);
    ta.store(sA[0], tid);
    tb.store(sB[0], tid);
  }
  __syncthreads();
  const int hk = lane >> 5, l32 = lane & 31;
  for (int kt = 0; kt < nk; ++kt) {
    const int buf = kt & 1;
    const bool more = kt + 1 < nk;
    if (more) {  // next k tile into registers while this one is multiplied
      ta.load(Ap, g.lda, m0, g.M, kbeg + (int64_t)(kt + 1) * kBK, kend, va, tid);
      tb.load(Bp, g.ldb, n0, g.N, kbeg + (int64_t)(kt + 1) * kBK, kend, vb, tid);
    }
#pragma unroll
    for (int kk = 0; kk < kBK; kk += 2) {
      // lane l supplies row / column l % 32 at k = kk + l / 32
      const float a0 = sA[buf][kk + hk][wm0 + l32], a1 = sA[buf][kk + hk][wm0 + 32 + l32];
      const float b0 = sB[buf][kk + hk][wn0 + l32], b1 = sB[buf][kk + hk][wn0 + 32 + l32];
      acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, b0, acc[0][0], 0, 0, 0);
      acc[0][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, b1, acc[0][1], 0, 0, 0);
      acc[1][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, b0, acc[1][0], 0, 0, 0);
      acc[1][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, b1, acc[1][1], 0, 0, 0);
    }
    if (more) {  // the other buffer was released by the previous barrier
      ta.store(sA[buf ^ 1], tid);
      tb.store(sB[buf ^ 1], tid);
    }
    __syncthreads();
  }

  // the loop's last barrier has passed: the tiles in LDS are read
  gemm_f32_epilogue(g, acc, m0 + wm0, n0 + wn0, lane, split, offC, &smem[0][0][0] + wave * (32 * 68));
}

// ------------------------------------------------- direct-to-LDS kernel --
//
// Bound by the float32 MFMA (157 TFLOP/s dense at 2.4 GHz; 64 cycles per
// 32x32x2, so every wave has to issue them back to back): k tiles of 32 in two
// LDS stages of 32 KiB, two workgroups per CU, the k loop of the half kernel
// (the barrier of the next k tile stands before the last of the four k steps of
// 8).  A k step reads each operand fragment once for 16 MFMAs: a k-major
// fragment is one 16-byte read per lane, whose element e holds k = 8 kk +
// 4 (lane / 32) + e, so MFMA e multiplies k = 8 kk + e and 8 kk + 4 + e (the
// order of the reduction is free as long as A and B agree); an mn-major one is
// four 4-byte reads of the same k values.
// LDS layouts: k-major [row][32 k], 128 B rows, 16-byte chunk c of row r at
// c ^ ((r >> 1) & 7); mn-major [k][128], chunk c of row k at c ^ (8 ((k >> 2) & 1)),
// so the two half-waves of a read, 4 rows apart, fall in different banks.
// Measured at 16640 x 1536 x 384, forward / dX / dW with db: 265 / 272 / 359 + 70 us
// with the register-staged kernel, 200 / 206 / 189 with this (98, 95 and 104
// TFLOP/s; 144 at 4096^3, where it was 106); what is left is 12 us a round of
// 512 tiles outside the k loops and, for dX, 390 tiles on 256 CUs.

// one operand of 128 rows (of M or N) x 32 k per stage, 4 copies per lane
template <bool KMAJ>
struct DmaF32 {
  uint32_t off[4];
  __device__ __forceinline__ void init(int64_t ld, int rv, int wave, int lane) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int at = 64 * (wave + 4 * q) + lane;  // the tile's 16-byte chunk this lane copies
      if constexpr (KMAJ) {
        const int r = at >> 3, c = (at & 7) ^ ((r >> 1) & 7);
        off[q] = (uint32_t)(min(r, rv - 1) * ld * 4 + c * 16);
      } else {
        const int k = at >> 5, c = (at & 31) ^ (8 * ((k >> 2) & 1));
        off[q] = (uint32_t)(k * ld * 4 + (4 * c < rv ? 16 * c : 0));
      }
    }
  }
  __device__ __forceinline__ void issue(const float* base, uint32_t lds, int wave) const {
    const uint64_t p = reinterpret_cast<uint64_t>(base);
    const uint64_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)p);
    const uint64_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(p >> 32));
    const void* sbase = reinterpret_cast<const void*>(lo | (hi << 32));
    const uint32_t slds = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds);
#pragma unroll
    for (int q = 0; q < 4; ++q) dma16(sbase, off[q], slds + 1024u * (uint32_t)(wave + 4 * q));
  }
};

__device__ __forceinline__ float lds_f32(uint32_t addr) {
  return *(const __attribute__((address_space(3))) float*)(uintptr_t)addr;
}

// the fragment of 32 rows from w0 + 32 I on, at k step KK of the tile at lds
template <bool KMAJ>
struct FragF32 {
  uint32_t base[KMAJ ? 4 : 2];
  __device__ __forceinline__ void init(int w0, int lane) {
    if constexpr (KMAJ) {
      const int r = w0 + (lane & 31), sw = (r >> 1) & 7;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) base[kk] = (uint32_t)(r * 128 + (((2 * kk + (lane >> 5)) ^ sw) << 4));
    } else {
      const int hk = lane >> 5;  // k = 8 kk + 4 hk + e
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int m = w0 + 32 * i + (lane & 31);
        base[i] = (uint32_t)(4 * hk * 512 + (((m >> 2) ^ (8 * hk)) << 4) + (m & 3) * 4);
      }
    }
  }
  template <int I, int KK>
  __device__ __forceinline__ f32x4 read(uint32_t lds) const {
    if constexpr (KMAJ) {
      return __builtin_bit_cast(f32x4, lds_b128(lds + base[KK] + I * 32 * 128));
    } else {
      const uint32_t a = lds + base[I] + 8 * KK * 512;
      return f32x4{lds_f32(a), lds_f32(a + 512), lds_f32(a + 1024), lds_f32(a + 1536)};
    }
  }
};

// DBS: the waves of the tile's first 64 columns also sum the rows of A (db),
// when the tile is in the first tile column: per k tile, then over the k tiles.
template <bool AK, bool BKM, bool DBS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_f32_dma_kernel(GemmF32Args g) {
  constexpr int STAGE = 32768, HALF = 16384;
  __shared__ __attribute__((aligned(1024))) uint8_t smem[2 * STAGE];
  const uint32_t lds0 = lds_u32(smem);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm0 = (wave >> 1) * 64, wn0 = (wave & 1) * 64;
  int64_t m0, n0;
  tile_origin<128, 128>(g.M, g.N, m0, n0);
  int split = 0;
  const float* Ap = g.A;
  const float* Bp = g.B;
  int64_t offC = 0;
  if (g.splits > 1) {
    split = (int)blockIdx.y;
  } else {  // batch entry
    const int64_t i0 = (uint32_t)blockIdx.y / (uint32_t)g.nb1, i1 = (uint32_t)blockIdx.y % (uint32_t)g.nb1;
    Ap += i0 * g.sA0 + i1 * g.sA1;
    Bp += i0 * g.sB0 + i1 * g.sB1;
    offC = i0 * g.sC0 + i1 * g.sC1;
  }
  const int64_t kbeg = (int64_t)split * g.k_split;
  const int64_t kend = min(g.K, kbeg + g.k_split);
  const int nk = (int)((kend - kbeg) / 32);
  const float* Ab = Ap + (AK ? m0 * g.lda + kbeg : kbeg * g.lda + m0);
  const float* Bb = Bp + (BKM ? n0 * g.ldb + kbeg : kbeg * g.ldb + n0);
  DmaF32<AK> da;
  DmaF32<BKM> db;
  da.init(g.lda, (int)min<int64_t>(128, g.M - m0), wave, lane);
  db.init(g.ldb, (int)min<int64_t>(128, g.N - n0), wave, lane);
  auto issue = [&](int kt) {
    const uint32_t st = lds0 + (uint32_t)((kt & 1) * STAGE);
    da.issue(Ab + (int64_t)kt * (AK ? 32 : 32 * g.lda), st, wave);
    db.issue(Bb + (int64_t)kt * (BKM ? 32 : 32 * g.ldb), st + HALF, wave);
  };
  issue(0);
  if (nk > 1) issue(1);
  FragF32<AK> fa;
  FragF32<BKM> fb;
  fa.init(wm0, lane);
  fb.init(wn0, lane);
  // the first half of the k tiles is summed apart from the second: half as
  // long chains of float32 additions (dW at 16640 x 1536 x 384: relative
  // error 8.7e-7 -> 6.1e-7 against 64 bits)
  f32x16 acc[2][2], first[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
  const bool dbw = DBS && wn0 == 0 && n0 == 0;  // uniform over the wave
  float dbs[2] = {0.0f, 0.0f}, dbt[2] = {0.0f, 0.0f};
  if (nk > 1) wait_vmcnt<8>();
  else wait_vmcnt<0>();
  __syncthreads();
  f32x4 af[2][2], bf[2][2];
  auto read = [&](auto set, auto kk, uint32_t st) {
    static_for<2>([&](auto i) { af[set][i] = fa.template read<i, kk>(st); });
    static_for<2>([&](auto j) { bf[set][j] = fb.template read<j, kk>(st + HALF); });
  };
  auto multiply = [&](auto set) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(af[set][i][e], bf[set][j][e], acc[i][j], 0, 0, 0);
    if constexpr (DBS) {
      if (dbw) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
          dbt[i] += (af[set][i][0] + af[set][i][1]) + (af[set][i][2] + af[set][i][3]);
      }
    }
  };
  constexpr std::integral_constant<int, 0> I0{};
  constexpr std::integral_constant<int, 1> I1{};
  constexpr std::integral_constant<int, 2> I2{};
  constexpr std::integral_constant<int, 3> I3{};
  read(I0, I0, lds0);
  auto k_tile = [&](int kt) {
    const uint32_t sa = lds0 + (uint32_t)((kt & 1) * STAGE), sn = lds0 + (uint32_t)(((kt + 1) & 1) * STAGE);
    read(I1, I1, sa);
    multiply(I0);
    read(I0, I2, sa);
    multiply(I1);
    read(I1, I3, sa);
    multiply(I0);
    if (kt + 1 < nk) {
      wait_vmcnt<0>();  // k tile kt + 1 has landed
      __syncthreads();
      if (kt + 2 < nk) issue(kt + 2);
      read(I0, I0, sn);
    }
    multiply(I1);
    if constexpr (DBS) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        dbs[i] += dbt[i];
        dbt[i] = 0.0f;
      }
    }
  };
  for (int kt = 0; kt < (nk >> 1); ++kt) k_tile(kt);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        first[i][j][r] = acc[i][j][r];
        acc[i][j][r] = 0.0f;
      }
  for (int kt = nk >> 1; kt < nk; ++kt) k_tile(kt);
  if constexpr (DBS) {
    if (dbw) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const float v = dbs[i] + __shfl_xor(dbs[i], 32);
        const int64_t row = m0 + wm0 + 32 * i + lane;
        if (lane < 32 && row < g.M) {
          if (g.splits > 1) g.dbp[(int64_t)split * g.M + row] = v;
          else g.db[row] = v;
        }
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] += first[i][j][r];
  __syncthreads();  // every wave is done reading the stage buffers
  gemm_f32_epilogue(g, acc, m0 + wm0, n0 + wn0, lane, split, offC,
                    reinterpret_cast<float*>(smem) + wave * (32 * 68));
}

// Sums of the split-K partials in split order, 4 outputs per thread where MN
// allows, and behind them the bias partials, one row per thread.
template <bool VEC>
__global__ __launch_bounds__(256) void splitk_reduce_f32_kernel(const float* __restrict__ ws, int splits,
                                                                int64_t MN, float* __restrict__ C,
                                                                const float* __restrict__ dbp, int64_t rows,
                                                                float* __restrict__ db) {
  constexpr int PER = VEC ? 4 : 1;
  const int64_t blocks = (MN + 256 * PER - 1) / (256 * PER);
  if ((int64_t)blockIdx.x >= blocks) {
    const int64_t r = ((int64_t)blockIdx.x - blocks) * 256 + threadIdx.x;
    if (r >= rows) return;
    float s = dbp[r];
    for (int k = 1; k < splits; ++k) s += dbp[(int64_t)k * rows + r];
    db[r] = s;
    return;
  }
  const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * PER;
  if (i >= MN) return;
  if constexpr (VEC) {
    f32x4 s = *reinterpret_cast<const f32x4*>(ws + i);
    for (int k = 1; k < splits; ++k) {
      const f32x4 t = *reinterpret_cast<const f32x4*>(ws + (int64_t)k * MN + i);
#pragma unroll
      for (int e = 0; e < 4; ++e) s[e] += t[e];
    }
    *reinterpret_cast<f32x4*>(C + i) = s;
  } else {
    float s = ws[i];
    for (int k = 1; k < splits; ++k) s += ws[(int64_t)k * MN + i];
    C[i] = s;
  }
}

// Column sums of a dense float32 matrix: partial sums over row slices (a
// lane per column, rows of the slice in order), then the slices in order.
__global__ __launch_bounds__(256) void colsum_f32_partial_kernel(const float* __restrict__ X, int64_t rows,
                                                                 int64_t cols, int64_t rows_per,
                                                                 float* __restrict__ part) {
  const int64_t col = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (col >= cols) return;
  const int64_t r0 = (int64_t)blockIdx.y * rows_per, r1 = min(rows, r0 + rows_per);
  float s = 0.0f;
  for (int64_t r = r0; r < r1; ++r) s += X[r * cols + col];
  part[(int64_t)blockIdx.y * cols + col] = s;
}

// 32 columns per workgroup, 8 lanes per column: lane group q sums the slices
// q, q + 8, ... in order, then the 8 sums are added pairwise (one lane per
// column, all slices in order, took 41 us for 512 slices of 1536 columns).
__global__ __launch_bounds__(256) void colsum_f32_final_kernel(const float* __restrict__ part, int64_t nparts,
                                                               int64_t cols, float* __restrict__ out) {
  __shared__ float red[8][32];
  const int c = threadIdx.x & 31, q = threadIdx.x >> 5;
  const int64_t col = (int64_t)blockIdx.x * 32 + c;
  float s = 0.0f;
  if (col < cols) {
#pragma unroll 8
    for (int64_t p = q; p < nparts; p += 8) s += part[p * cols + col];
  }
  red[q][c] = s;
  __syncthreads();
  if (q == 0 && col < cols)
    out[col] = ((red[0][c] + red[1][c]) + (red[2][c] + red[3][c])) +
               ((red[4][c] + red[5][c]) + (red[6][c] + red[7][c]));
}

}  // namespace

// What the direct copies need of an operand: 16-byte aligned rows and batch
// entries, whole 16-byte chunks (an mn-major row must not end inside one) and
// 32-bit lane offsets.
static bool dma_f32_operand(const float* p, bool kmaj, int64_t ld, int64_t extent, int64_t s0, int64_t s1) {
  return (reinterpret_cast<uintptr_t>(p) & 15u) == 0 && ld % 4 == 0 && s0 % 4 == 0 && s1 % 4 == 0 &&
         (kmaj || extent % 4 == 0) && ld * 128 * 4 < ((int64_t)1 << 31);
}

bool gemm_f32_direct(const GemmF32Args& g, bool ak, bool bk) {
  return g.K % 32 == 0 && dma_f32_operand(g.A, ak, g.lda, g.M, g.sA0, g.sA1) &&
         dma_f32_operand(g.B, bk, g.ldb, g.N, g.sB0, g.sB1);
}

hipError_t launch_gemm_f32(GemmF32Args g, bool ak, bool bk, int64_t nbatch, hipStream_t s, bool* db_fused) {
  const int64_t tiles = ((g.M + kBM - 1) / kBM) * ((g.N + kBN - 1) / kBN);
  const int64_t gy = g.splits > 1 ? g.splits : nbatch;
  if (tiles > 0x7FFFFFFF || g.splits < 1 || gy < 1 || gy > 65535 || g.nb1 < 1 ||
      (g.splits > 1 && nbatch != 1))
    return hipErrorInvalidValue;
  const dim3 grid((unsigned)tiles, (unsigned)gy);
  const bool dma = gemm_f32_direct(g, ak, bk) && (g.splits == 1 || g.k_split % 32 == 0);
  const bool fuse = dma && !ak && !bk && nbatch == 1 && g.db && (g.splits == 1 || g.dbp);
  if (db_fused) *db_fused = fuse;
  if (dma) {
    if (ak && bk) gemm_f32_dma_kernel<true, true, false><<<grid, 256, 0, s>>>(g);
    else if (ak) gemm_f32_dma_kernel<true, false, false><<<grid, 256, 0, s>>>(g);
    else if (bk) gemm_f32_dma_kernel<false, true, false><<<grid, 256, 0, s>>>(g);
    else if (fuse) gemm_f32_dma_kernel<false, false, true><<<grid, 256, 0, s>>>(g);
    else gemm_f32_dma_kernel<false, false, false><<<grid, 256, 0, s>>>(g);
    return hipGetLastError();
  }
  if (ak && bk) gemm_f32_kernel<true, true><<<grid, 256, 0, s>>>(g);
  else if (ak) gemm_f32_kernel<true, false><<<grid, 256, 0, s>>>(g);
  else if (bk) gemm_f32_kernel<false, true><<<grid, 256, 0, s>>>(g);
  else gemm_f32_kernel<false, false><<<grid, 256, 0, s>>>(g);
  return hipGetLastError();
}

hipError_t launch_splitk_reduce_f32(const float* ws, int splits, int64_t MN, float* C, const float* dbp,
                                    int64_t rows, float* db, hipStream_t s) {
  const bool vec = MN % 4 == 0 && ((reinterpret_cast<uintptr_t>(ws) | reinterpret_cast<uintptr_t>(C)) & 15u) == 0;
  const int64_t per = vec ? 1024 : 256;
  const unsigned blocks = (unsigned)((MN + per - 1) / per + (rows + 255) / 256);
  if (vec) splitk_reduce_f32_kernel<true><<<blocks, 256, 0, s>>>(ws, splits, MN, C, dbp, rows, db);
  else splitk_reduce_f32_kernel<false><<<blocks, 256, 0, s>>>(ws, splits, MN, C, dbp, rows, db);
  return hipGetLastError();
}

hipError_t launch_colsum_f32(const float* X, int64_t rows, int64_t cols, float* ws, float* out,
                             hipStream_t s) {
  // the slice count of the half column sum, so the same workspace size serves
  const int64_t sl = colsum_slices(rows, cols);
  const int64_t per = (rows + sl - 1) / sl;
  const unsigned gx = (unsigned)((cols + 255) / 256);
  colsum_f32_partial_kernel<<<dim3(gx, (unsigned)sl), 256, 0, s>>>(X, rows, cols, per, ws);
  colsum_f32_final_kernel<<<(unsigned)((cols + 31) / 32), 256, 0, s>>>(ws, sl, cols, out);
  return hipGetLastError();
}

}  // namespace mpx
