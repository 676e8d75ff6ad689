// Multi-fidelity tokenizer of the Turbulence Transformer (arXiv 2507.16697 Sec. III-B; the
// filter / mode-size pairs of Table III): one fidelity mode of a field Y[c, z, y, x] is the
// periodic subdomain selection C(Y) of D/ratio x H/ratio x W/ratio cells around a centre, the k^3
// Gaussian filter F(.) applied with stride k (the D/k x H/k x W/k grid the paper gives for F(Y)),
// and patchify with patch p into tokens [L, C p^3] (token index x fastest, feature
// ((c p + iz) p + iy) p + ix).
//
// HBM-bound: the filter windows do not overlap, so every subdomain cell is read once and every
// token feature written once.  The unfiltered crop with patch 1 (Table III's filter 1) is a copy
// with one thread per cell and contiguous per-token stores.  For k a power of two a wave streams
// 256 consecutive cells, 4 per lane, through the k^2 rows of its windows and accumulates in
// registers; the k cells of a window are then summed within the lane (k <= 4) or across k/4
// lanes by butterfly shuffles.  Other k take a plain kernel with one thread per filtered cell.
// The separable weights w_i w_j w_l come in as kernel arguments (computed on the host,
// normalised to sum 1).

#include "ringx_device.h"
#include "ringx_kernels.h"

namespace ringx {
namespace {

constexpr int kTokThreads = 256;
constexpr int kTokBatch = 8;             // field rows that a wave of the row kernel has in flight
constexpr int64_t kTokGridX = 1 << 22;   // workgroups along x of the row kernel
// four fp32 cells at 4-byte alignment
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

__global__ __launch_bounds__(kTokThreads) void tt_tokenize_kernel(
    const float* __restrict__ field, void* __restrict__ tokens, int C, int D, int H, int W, int k,
    int gz, int gy, int gx, int z0, int y0, int x0, int p, TokWeights w, int out_bf16) {
  const int64_t n_out = (int64_t)C * gz * gy * gx;
  const int64_t idx = (int64_t)blockIdx.x * kTokThreads + threadIdx.x;
  if (idx >= n_out) return;
  const int e = (int)(idx % gx);
  int64_t r = idx / gx;
  const int b = (int)(r % gy);
  r /= gy;
  const int a = (int)(r % gz);
  const int c = (int)(r / gz);

  // first cell of the window in the (periodic) field; z0, y0, x0 are already in [0, D) etc.
  int zb = z0 + k * a;
  zb -= zb >= D ? D : 0;
  int yb = y0 + k * b;
  yb -= yb >= H ? H : 0;
  int xb = x0 + k * e;
  xb -= xb >= W ? W : 0;

  const float* fc = field + (int64_t)c * D * H * W;
  float acc = 0.f;
  for (int i = 0; i < k; ++i) {
    int z = zb + i;
    z -= z >= D ? D : 0;
    float accy = 0.f;
    for (int j = 0; j < k; ++j) {
      int y = yb + j;
      y -= y >= H ? H : 0;
      const float* row = fc + ((int64_t)z * H + y) * W;
      float accx = 0.f;
      for (int l = 0; l < k; ++l) {
        int x = xb + l;
        x -= x >= W ? W : 0;
        accx = __builtin_fmaf(w.w[l], row[x], accx);
      }
      accy = __builtin_fmaf(w.w[j], accx, accy);
    }
    acc = __builtin_fmaf(w.w[i], accy, acc);
  }

  // token (patch) index, x fastest, and feature within the token
  const int Py = gy / p, Px = gx / p;
  const int64_t t = ((int64_t)(a / p) * Py + b / p) * Px + e / p;
  const int f = ((c * p + a % p) * p + b % p) * p + e % p;
  const int64_t o = t * ((int64_t)C * p * p * p) + f;
  if (out_bf16) {
    reinterpret_cast<__bf16*>(tokens)[o] = (__bf16)acc;
  } else {
    reinterpret_cast<float*>(tokens)[o] = acc;
  }
}

// Row-streaming variant, K a power of two.  One wave = 256 subdomain cells (64 lanes x 4 cells): a
// segment of one (c, a, b) filtered row, the segments of a row in neighbouring waves, or with PACK
// (rows of at most 128 cells) 2^(6 - log2_lanes) whole rows of 2^log2_lanes lanes each.  NB field rows
// are in flight; with FAR the segments of a row are a whole sweep of rows apart (tok_rows_form).
// Bound by how many loads are in flight: a wave that loaded and used one field row at a time, with
// a branch around each load for the lane at the field's periodic edge, read 5.3 TB/s of a 512^3 x 4
// field at k = 8 (402 us) and far less of small ones, whose few waves then wait row by row.  Eight
// rows in flight and no branch between them: 342 us (6.3 TB/s; 6.7 with rows on 16-byte boundaries),
// 256^3 x 3 77 -> 35 us, 128^3 59 -> 11 us; k = 16 420 -> 340, 240 -> 48 and 229 -> 37 us.  Four
// rows: 359, 37 and 16 us; sixteen (140 registers, three waves per SIMD): 353, 37 and 12 us.
template <int K, int NB, bool PACK, bool FAR>
__global__ __launch_bounds__(kTokThreads) void tt_tokenize_rows_kernel(
    const float* __restrict__ field, void* __restrict__ tokens, int C, int D, int H, int W, int sx,
    int gz, int gy, int gx, int z0, int y0, int x0, int p, TokWeights w, int out_bf16, uint32_t segs,
    int log2_lanes) {
  const int lane = threadIdx.x & 63;
  // One row at a time the wave's indices and addresses stay per lane: in scalar registers they are a
  // serial chain that such a short wave does not hide (512^3 x 4, k = 2, patch 2: 713 against 665
  // us); with eight rows in flight scalar row addresses are the better ones.
  const int wave = NB == 1 ? threadIdx.x >> 6 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t unit =
      ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * (kTokThreads / 64) + wave;
  const int64_t rows = (int64_t)C * gz * gy;
  int64_t row = unit, seg = 0;
  if constexpr (PACK) {
    row = (unit << (6 - log2_lanes)) + (lane >> log2_lanes);
  } else if constexpr (!FAR) {
    row = unit / segs;
    seg = unit % segs;
  } else {
    seg = unit / rows;
    row = seg < segs ? unit % rows : rows;
  }
  if (row >= rows) return;
  const int b = (int)(row % gy);
  const int a = (int)((row / gy) % gz);
  const int c = (int)(row / ((int64_t)gy * gz));
  // first of this lane's 4 subdomain cells
  const int pos = PACK ? 4 * (lane & ((1 << log2_lanes) - 1)) : (int)seg * 256 + 4 * lane;
  const bool active = pos < sx;                     // sx is a multiple of K and of 4 when K >= 4

  // Every lane reads one quad of cells per field row (4-byte alignment is all a multi-dword load
  // needs).  A lane whose four cells run over the field's end reads the last four cells of the row,
  // and its other cells, from the row's start, by a second load; lanes past the subdomain's end read
  // its last quad along with the lane that owns it.
  int xs = x0 + (active ? pos : sx - 4);
  xs -= xs >= W ? W : 0;
  const int over = xs + 4 - W;      // cells past the end, when positive
  const bool wrap = over > 0;
  xs = wrap ? W - 4 : xs;
  const float* fc = field + (int64_t)c * D * H * W;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  float acc2[4] = {0.f, 0.f, 0.f, 0.f};
  constexpr int kBatch = K * K < NB ? K * K : NB;   // field rows in flight
#pragma unroll 1
  for (int r0 = 0; r0 < K * K; r0 += kBatch) {
    const float* rowp[kBatch];
    float wij[kBatch];
    f32x4 v[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int i = (r0 + u) / K, j = (r0 + u) % K;
      int z = z0 + K * a + i;
      z -= z >= D ? D : 0;
      z -= z >= D ? D : 0;
      int y = y0 + K * b + j;
      y -= y >= H ? H : 0;
      y -= y >= H ? H : 0;
      wij[u] = w.w[i] * w.w[j];
      rowp[u] = fc + ((int64_t)z * H + y) * W;
      // the field is streamed once: non-temporal loads, except for the unfiltered crop (k = 1),
      // whose short row segments are latency-bound
      const f32x4u* vp = reinterpret_cast<const f32x4u*>(rowp[u] + xs);
      v[u] = K > 1 ? __builtin_nontemporal_load(vp) : *vp;
    }
    __builtin_amdgcn_sched_barrier(0);
    if (wrap) {
      cold_path();
      f32x4 v2[kBatch];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) v2[u] = *reinterpret_cast<const f32x4u*>(rowp[u]);
#pragma unroll
      for (int u = 0; u < kBatch; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc2[e] = __builtin_fmaf(wij[u], v2[u][e], acc2[e]);
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] = __builtin_fmaf(wij[u], v[u][e], acc[e]);
  }
  if (wrap) {
    cold_path();
    // cells 0 .. 3 - over are the row's last ones, the others its first
    float cell[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float x = acc2[0];
#pragma unroll
      for (int f = 0; f < 4; ++f) {
        x = e + over == f ? acc[f] : x;
        x = e + over - 4 == f ? acc2[f] : x;
      }
      cell[e] = x;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] = cell[e];
  }
  // x weights, then the window sums: within the lane for K <= 4, across K/4 lanes otherwise
  float part[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) part[e] = acc[e] * w.w[(pos + e) & (K - 1)];
  constexpr int kPerLane = K < 4 ? 4 / K : 1;      // windows completed inside one lane
  float win[kPerLane];
#pragma unroll
  for (int q = 0; q < kPerLane; ++q) {
    float s = 0.f;
#pragma unroll
    for (int e = 0; e < (K < 4 ? K : 4); ++e) s += part[q * (K < 4 ? K : 4) + e];
    win[q] = s;
  }
  if constexpr (K > 4) {
#pragma unroll
    for (int m = 1; m < K / 4; m <<= 1) win[0] += __shfl_xor(win[0], m);
    if ((lane & (K / 4 - 1)) != 0) return;
  }
  if (!active) return;
  const int Py = gy / p, Px = gx / p;
  const int64_t feat = (int64_t)C * p * p * p;
#pragma unroll
  for (int q = 0; q < kPerLane; ++q) {
    const int e = pos / K + q;                       // filtered cell along x
    const int64_t t = ((int64_t)(a / p) * Py + b / p) * Px + e / p;
    const int f = ((c * p + a % p) * p + b % p) * p + e % p;
    if (out_bf16) reinterpret_cast<__bf16*>(tokens)[t * feat + f] = (__bf16)win[q];
    else reinterpret_cast<float*>(tokens)[t * feat + f] = win[q];
  }
}

// The unfiltered crop (k = 1) with patch 1: token t = subdomain cell (z, y, x), x fastest, and its
// C features are the C channels of that cell.  One thread per cell: the channel loads of
// consecutive threads are consecutive cells of a row (coalesced), and each thread writes its C
// features as one contiguous run (16-byte stores of 4 channels when C is a multiple of 4), so
// every output line is written whole by neighbouring threads.
template <bool OUT_BF16>
__global__ __launch_bounds__(kTokThreads) void tt_crop_kernel(
    const float* __restrict__ field, void* __restrict__ tokens, int C, int D, int H, int W,
    int sz, int sy, int sx, int z0, int y0, int x0) {
  const int64_t n = (int64_t)sz * sy * sx;
  const int64_t i = (int64_t)blockIdx.x * kTokThreads + threadIdx.x;
  if (i >= n) return;
  const int x = (int)(i % sx);
  const int64_t r = i / sx;
  const int y = (int)(r % sy);
  const int z = (int)(r / sy);
  int zz = z0 + z, yy = y0 + y, xx = x0 + x;
  zz -= zz >= D ? D : 0;
  yy -= yy >= H ? H : 0;
  xx -= xx >= W ? W : 0;
  const int64_t plane = (int64_t)D * H * W;
  const float* src = field + ((int64_t)zz * H + yy) * W + xx;
  if ((C & 3) == 0) {
    for (int c = 0; c < C; c += 4) {
      const f32x4 v = {src[c * plane], src[(c + 1) * plane], src[(c + 2) * plane],
                       src[(c + 3) * plane]};
      if constexpr (OUT_BF16) {
        u32x2 w2;
        w2[0] = pack_bf16x2(v[0], v[1]);
        w2[1] = pack_bf16x2(v[2], v[3]);
        *reinterpret_cast<u32x2*>(reinterpret_cast<__bf16*>(tokens) + i * C + c) = w2;
      } else {
        *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(tokens) + i * C + c) = v;
      }
    }
  } else {
    for (int c = 0; c < C; ++c) {
      const float v = src[c * plane];
      if constexpr (OUT_BF16) reinterpret_cast<__bf16*>(tokens)[i * C + c] = (__bf16)v;
      else reinterpret_cast<float*>(tokens)[i * C + c] = v;
    }
  }
}

template <int K, int NB, bool PACK, bool FAR>
hipError_t launch_rows(const TokArgs& a, int64_t units, int64_t segs, int log2_lanes) {
  // workgroups along x, then y: a launch dimension holds less than 2^32 threads
  const int64_t blocks = (units + kTokThreads / 64 - 1) / (kTokThreads / 64);
  const int64_t nx = blocks < kTokGridX ? blocks : kTokGridX;
  const dim3 grid((uint32_t)nx, (uint32_t)((blocks + nx - 1) / nx));
  hipLaunchKernelGGL((tt_tokenize_rows_kernel<K, NB, PACK, FAR>), grid, dim3(kTokThreads), 0, a.stream,
                     a.field, a.tokens, (int)a.C, (int)a.D, (int)a.H, (int)a.W, (int)(a.gx * K),
                     (int)a.gz, (int)a.gy, (int)a.gx, (int)a.z0, (int)a.y0, (int)a.x0, (int)a.p,
                     a.w, a.out_bf16 ? 1 : 0, (uint32_t)segs, log2_lanes);
  return hipGetLastError();
}

template <int K>
hipError_t launch_rows(const TokArgs& a) {
  const int64_t rows = a.C * a.gz * a.gy, sx = a.gx * K;
  if (sx > 128) {
    const int64_t segs = (sx + 255) / 256;
    const int64_t u = rows * segs;
    const TokRowsForm f = tok_rows_form(K, rows, sx, a.W, a.x0);
    if constexpr (K == 2)
      if (f.one_row) return launch_rows<K, 1, false, false>(a, u, segs, 6);
    if constexpr (K >= 4 && K <= 16)
      if (f.one_row) return launch_rows<K, 1, false, true>(a, u, segs, 6);
    return launch_rows<K, kTokBatch, false, false>(a, u, segs, 6);
  }
  int l = 0;   // lanes of a row, a power of two that holds whole windows
  while ((4 << l) < sx) ++l;
  return launch_rows<K, kTokBatch, true, false>(a, (rows + (64 >> l) - 1) >> (6 - l), 1, l);
}

}  // namespace

hipError_t launch_tt_tokenize(const TokArgs& a) {
  if (a.k == 1 && a.p == 1) {
    // the unfiltered crop: one thread per subdomain cell (the weight of a 1-cell window is 1)
    const int64_t n = a.gz * a.gy * a.gx;
    const dim3 grid((uint32_t)((n + kTokThreads - 1) / kTokThreads));
    if (a.out_bf16)
      hipLaunchKernelGGL(tt_crop_kernel<true>, grid, dim3(kTokThreads), 0, a.stream, a.field,
                         a.tokens, (int)a.C, (int)a.D, (int)a.H, (int)a.W, (int)a.gz, (int)a.gy,
                         (int)a.gx, (int)a.z0, (int)a.y0, (int)a.x0);
    else
      hipLaunchKernelGGL(tt_crop_kernel<false>, grid, dim3(kTokThreads), 0, a.stream, a.field,
                         a.tokens, (int)a.C, (int)a.D, (int)a.H, (int)a.W, (int)a.gz, (int)a.gy,
                         (int)a.gx, (int)a.z0, (int)a.y0, (int)a.x0);
    return hipGetLastError();
  }
  // the row kernel needs 4-cell lane groups inside the subdomain row: sx % 4 == 0
  const int64_t sx = a.gx * a.k;
  const int64_t units = a.C * a.gz * a.gy * ((sx + 255) / 256);
  if (sx % 4 == 0 && units / (kTokThreads / 64) < 65535 * kTokGridX) {
    switch (a.k) {
      case 1: return launch_rows<1>(a);
      case 2: return launch_rows<2>(a);
      case 4: return launch_rows<4>(a);
      case 8: return launch_rows<8>(a);
      case 16: return launch_rows<16>(a);
      case 32: return launch_rows<32>(a);
      default: break;
    }
  }
  const int64_t n_out = a.C * a.gz * a.gy * a.gx;
  const int64_t blocks = (n_out + kTokThreads - 1) / kTokThreads;
  hipLaunchKernelGGL(tt_tokenize_kernel, dim3((uint32_t)blocks), dim3(kTokThreads), 0, a.stream,
                     a.field, a.tokens, (int)a.C, (int)a.D, (int)a.H, (int)a.W, (int)a.k,
                     (int)a.gz, (int)a.gy, (int)a.gx, (int)a.z0, (int)a.y0, (int)a.x0, (int)a.p,
                     a.w, a.out_bf16 ? 1 : 0);
  return hipGetLastError();
}

}  // namespace ringx
