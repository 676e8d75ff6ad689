// fp32 matrix tiles shared by the fp32 forward and backward kernels (gfx950).
//
// v_mfma_f32_16x16x4_f32: full fp32 products and accumulation, 2048 flops in 32 cycles per SIMD
// (the rate of every fp32 matrix shape, so the smallest tile costs nothing and gives the finest
// split of small problems).  Operand layout for lane l (g = l / 16, n = l % 16):
//   A (16 x 4): row n, k = g     B (4 x 16): column n, k = g     C (16 x 16): column n, rows 4g + r
// The order in which a contraction runs through its index is free as long as A and B agree, so
// both operand kinds are loaded 16 bytes per lane straight from row-major global memory:
//   row fragments (contraction over the head dim): row n, dims 16 s + 4 g .. + 3; product (s, j)
//       contracts dims {16 s + 4 g + j};
//   column fragments (contraction over rows): row 4 g + r, dims 64 c + 4 n .. + 3; product j of a
//       64-dim group has output row i = dim 64 c + 4 i + j, so that a lane's outputs come in quads
//       of consecutive dims too.  Head dims past the last whole group of 64 go in groups of 16,
//       one dim per lane (output row i = dim 16 c + i).
// A C tile of a score block (column = this lane's stationary row, rows 4 g + r) is the B operand
// of the next contraction as it is: product r contracts the rows {4 g + r}.
// Waves read from L1/L2 without LDS: one 256-byte fragment feeds a 32-cycle product, 32 bytes per
// clock and CU with all four SIMDs busy.
#pragma once

#include "ringx_device.h"

namespace ringx {

__device__ __forceinline__ f32x4 mfma16f(float a, float b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Every fragment is a buffer load: a scalar descriptor of the rows at hand (wave-uniform base, size
// of the rows that exist), one 32-bit lane offset fixed for the whole kernel, constants.  So there
// is no per-lane address arithmetic in the loops and no branch: what lies outside, rows past the
// end as well as head dims past d (whose lane offsets are moved outside), reads as zero.

// Which head dims the last 16 of a row may lack.
enum F32Edge {
  kFull = 0,    // d = 16 NS: none
  kQuad = 1,    // d % 4 == 0: whole quads
  kAny = 2,     // any: the last 16 dims are loaded one by one
};

// Rows of a matrix with d columns, for the fragments of one 16-row block (rows past `rows` are
// zero; rows <= 16).
struct RowBlock {
  __amdgpu_buffer_rsrc_t rsrc;
  __device__ __forceinline__ RowBlock(const float* base, int64_t row, int d, int rows)
      : rsrc(__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(uniform_ptr(base + row * d)), 0,
                                               __builtin_amdgcn_readfirstlane(rows * d * 4),
                                               0x00020000)) {}
  __device__ __forceinline__ f32x4 load4(int off) const {
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, off, 0, 0));
  }
  // one value per row (d = 1): rows 4 g .. 4 g + 3
  __device__ __forceinline__ f32x4 load4_rows(int g) const {
    return f32x4{load1(16 * g), load1(16 * g + 4), load1(16 * g + 8), load1(16 * g + 12)};
  }
  __device__ __forceinline__ float load1(int off) const {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc, off, 0, 0));
  }
};
constexpr int kOutside = 1 << 30;   // a byte offset past any block of rows

// Head dims of a [rows, d] fp32 matrix as seen by one lane, padded to 16 NS (16 (NS - 1) < d), and
// the lane's byte offsets into a 16-row block.
template <int NS, int EDGE>
struct F32Dims {
  static constexpr int kG4 = NS / 4;            // 64-dim groups of the column fragments
  static constexpr int kG1 = NS % 4;            // 16-dim groups after them
  int d, n, g;
  int row;          // row n, dim 4 g
  int col[4];       // rows 4 g + r, dim 4 n
  int one[4];       // rows 4 g + r, dim n
  int row_out[4], col_out[4];   // kOutside where the last 16 dims' element j lies past d, else 0

  __device__ __forceinline__ F32Dims(int d_, int lane) : d(d_), n(lane & 15), g(lane >> 4) {
    row = 4 * (n * d + 4 * g);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      col[r] = 4 * ((4 * g + r) * d + 4 * n);
      one[r] = 4 * ((4 * g + r) * d + n);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      row_out[j] = 16 * (NS - 1) + 4 * g + j < d ? 0 : kOutside;
      col_out[j] = (kG1 ? 16 * (NS - 1) + n : 64 * (kG4 - 1) + 4 * n + j) < d ? 0 : kOutside;
    }
  }
  // first dim of output quad t (0 .. NS-1) of this lane (see the accumulators below)
  __device__ __forceinline__ int quad(int t) const {
    return t < 4 * kG4 ? 64 * (t / 4) + 16 * g + 4 * (t % 4) : 64 * kG4 + 16 * (t - 4 * kG4) + 4 * g;
  }
  // four consecutive dims; `edge`: they may reach past d, `out` as above
  __device__ __forceinline__ f32x4 frag4(const RowBlock& b, int off, bool edge,
                                         const int (&out)[4]) const {
    if (EDGE == kFull || !edge) return b.load4(off);
    if (EDGE == kQuad) return b.load4(off + out[0]);
    f32x4 x;
#pragma unroll
    for (int j = 0; j < 4; ++j) x[j] = b.load1(off + 4 * j + out[j]);
    return x;
  }
  // output rows, four dims from `dim` (not in a hot loop)
  __device__ __forceinline__ f32x4 load4(const float* rowp, int dim) const {
    f32x4 x = {};
    if (EDGE != kAny) {
      if (EDGE == kFull || dim < d) x = *reinterpret_cast<const f32x4*>(rowp + dim);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (dim + j < d) x[j] = rowp[dim + j];
    }
    return x;
  }
  __device__ __forceinline__ void store4(float* rowp, int dim, const f32x4& x) const {
    if (EDGE != kAny) {
      if (EDGE == kFull || dim < d) *reinterpret_cast<f32x4*>(rowp + dim) = x;
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (dim + j < d) rowp[dim + j] = x[j];
    }
  }
};

// Row fragments (A or B operand of a contraction over the head dim): row n of the block.
template <int NS>
struct RowFrag {
  f32x4 x[NS];
  template <int EDGE>
  __device__ __forceinline__ void load(const F32Dims<NS, EDGE>& D, const RowBlock& b) {
#pragma unroll
    for (int s = 0; s < NS; ++s) x[s] = D.frag4(b, D.row + 64 * s, s == NS - 1, D.row_out);
  }
};

// A . B over the head dim: rows of `a` against columns of `b`, two chains of products so that
// neither waits for the other's result.
template <int NS>
__device__ __forceinline__ f32x4 dot_rows(const RowFrag<NS>& a, const RowFrag<NS>& b) {
  f32x4 c0 = {}, c1 = {};
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    c0 = mfma16f(a.x[s][0], b.x[s][0], c0);
    c1 = mfma16f(a.x[s][1], b.x[s][1], c1);
    c0 = mfma16f(a.x[s][2], b.x[s][2], c0);
    c1 = mfma16f(a.x[s][3], b.x[s][3], c1);
  }
  return c0 + c1;
}

// Column fragments: rows 4 g + r of the block.
template <int NS>
struct ColFrag {
  static constexpr int kG4 = NS / 4, kG1 = NS % 4;
  f32x4 v[4][kG4 > 0 ? kG4 : 1];
  float s[4][kG1 > 0 ? kG1 : 1];
  template <int EDGE>
  __device__ __forceinline__ void load(const F32Dims<NS, EDGE>& D, const RowBlock& b) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
#pragma unroll
      for (int c = 0; c < kG4; ++c)
        v[r][c] = D.frag4(b, D.col[r] + 256 * c, kG1 == 0 && c == kG4 - 1, D.col_out);
#pragma unroll
      for (int c = 0; c < kG1; ++c)
        s[r][c] = b.load1(D.one[r] + 256 * kG4 + 64 * c +
                          (EDGE != kFull && c == kG1 - 1 ? D.col_out[0] : 0));
    }
  }
};

// Accumulators of a [16 NS dims] x [16 stationary rows] output: this lane holds its stationary
// row n at the dims of D.quad(t), t < NS.
template <int NS>
struct AccF32 {
  static constexpr int kG4 = NS / 4, kG1 = NS % 4;
  f32x4 a4[kG4 > 0 ? kG4 : 1][4];
  f32x4 a1[kG1 > 0 ? kG1 : 1];
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int c = 0; c < kG4; ++c)
#pragma unroll
      for (int j = 0; j < 4; ++j) a4[c][j] = f32x4{};
#pragma unroll
    for (int c = 0; c < kG1; ++c) a1[c] = f32x4{};
  }
  __device__ __forceinline__ void scale(float f) {
#pragma unroll
    for (int c = 0; c < kG4; ++c)
#pragma unroll
      for (int j = 0; j < 4; ++j) a4[c][j] *= f;
#pragma unroll
    for (int c = 0; c < kG1; ++c) a1[c] *= f;
  }
  // += sum over the block's 16 rows of (row's dims) x p (p[r]: row 4 g + r, column n)
  __device__ __forceinline__ void add(const ColFrag<NS>& f, const f32x4& p) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
#pragma unroll
      for (int c = 0; c < kG4; ++c)
#pragma unroll
        for (int j = 0; j < 4; ++j) a4[c][j] = mfma16f(f.v[r][c][j], p[r], a4[c][j]);
#pragma unroll
      for (int c = 0; c < kG1; ++c) a1[c] = mfma16f(f.s[r][c], p[r], a1[c]);
    }
  }
  __device__ __forceinline__ f32x4 quad(int t) const {
    if (t < 4 * kG4) {
      const f32x4(&q)[4] = a4[kG4 > 0 ? t / 4 : 0];
      return f32x4{q[0][t % 4], q[1][t % 4], q[2][t % 4], q[3][t % 4]};
    }
    return a1[kG1 > 0 ? t - 4 * kG4 : 0];
  }
  __device__ __forceinline__ void set_quad(int t, const f32x4& x) {
    if (t < 4 * kG4) {
#pragma unroll
      for (int j = 0; j < 4; ++j) a4[kG4 > 0 ? t / 4 : 0][j][t % 4] = x[j];
    } else {
      a1[kG1 > 0 ? t - 4 * kG4 : 0] = x;
    }
  }
};

// max over / sum of the four lanes that share n (lane ^ 16, lane ^ 32)
__device__ __forceinline__ float max_groups(float x) {
  x = fmaxf(x, __shfl_xor(x, 16));
  return fmaxf(x, __shfl_xor(x, 32));
}
__device__ __forceinline__ float sum_groups(float x) {
  x += __shfl_xor(x, 16);
  return x + __shfl_xor(x, 32);
}

// How many of a workgroup's kF32Waves waves split the streamed rows of one stationary 16-row block
// (a power of two): the fewest that put two waves on every SIMD of the chip (2048), so that one
// wave's loads and exponentials hide behind the other's products, while every wave keeps at least
// two blocks of 16 rows.  The split costs one pass over LDS at the end.
constexpr int kF32Waves = 8;
inline int f32_split(int64_t blocks, int64_t rows) {
  int ks = 1;
  while (ks < kF32Waves && blocks * ks < 2048 && rows >= 64 * (int64_t)ks) ks *= 2;
  return ks;
}

}  // namespace ringx
