// Ring-chunked attention forward in fp32 (storage and arithmetic), any head dim 1..128, on the fp32
// matrix cores (tiles and operand layouts in f32_tiles.h).
//
// One wave owns 16 queries, held as B operands, and streams keys 64 at a time:
//   S^T = K Q^T   (lane: its query n, keys 4 g + r of each 16)
//   P^T = exp(scale S^T - m), m the running row maximum, rescaled only when it moves
//   O^T += V^T P^T  with P^T straight from the registers
// A workgroup's 8 waves are 8 / ks query blocks of ks waves each; the ks waves of a block take
// consecutive key ranges and merge (m, l, O) through LDS at the end, so that a problem with few
// query rows still fills the SIMDs (rule in f32_split).
//
// Bound by the fp32 matrix rate (154 TFLOP/s in a large library product on this card) as long as
// every CU has query blocks: H = 3, Nq = 1531, Nk = 3001, d = 100 takes 111 us (34 ms with one
// thread per query row and scalar FMAs), where the 288 query blocks make two rounds over 256 CUs
// (80 us of products on the CUs that get two).  H = 2, Nq = Nk = 1024, d = 64: 6366 -> 15.6 us for
// the call.  The error against 64 bits is smaller than before (4.3e-7 -> 2.9e-7 relative there): the
// scale is fused into the exponent's subtraction and every wave sums fewer terms.
//
// The local results of the R chunks (arXiv 2507.16697 Sec. III-A) merge by Eq. (5) exactly
// whatever reference their exponentials use; in the fused mode all of them share the wave's
// running reference, so that the merge is the running sum itself and only one division and one
// log remain.  Partials mode runs every chunk for itself and writes (loc_out_r, loc_lse_r); step
// mode (R = 1) folds the one chunk into a running fp32 (acc_out, acc_lse) left by earlier ring
// steps, which by the step contract holds the normalised result.

#include "f32_tiles.h"
#include "ringx_kernels.h"

#include <algorithm>
#include <type_traits>

namespace ringx {
namespace {

constexpr int kThreads = 64 * kF32Waves;

template <int NS, int EDGE>
__global__ __launch_bounds__(kThreads, 2) void fwd_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
    float* __restrict__ out, float* __restrict__ lse, int mode, int first, int64_t BH, int H,
    int grp, int64_t Nq, int64_t Nk, int64_t R, int d, float scale, int ks_log2) {
  // the key-split merge: per wave 16 queries x (16 NS dims, m, l)
  constexpr int kRow = 16 * NS + 4;
  __shared__ __attribute__((aligned(16))) float part[kF32Waves * 16 * kRow];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const F32Dims<NS, EDGE> D(d, lane);
  const int ks = 1 << ks_log2;
  const int qg = wave >> ks_log2, kp = wave & (ks - 1), nqg = kF32Waves >> ks_log2;
  const int bh = blockIdx.y;
  const int64_t kvh = (bh / H) * (H / grp) + (bh % H) / grp;
  const float* kb = k + kvh * Nk * d;
  const float* vb = v + kvh * Nk * d;
  const bool partials = mode == (int)FwdMode::kPartials;
  const int64_t chunks = partials ? R : 1;

  for (int64_t qt = blockIdx.x; qt * nqg * 16 < Nq; qt += gridDim.x) {
    const int64_t qi = (qt * nqg + qg) * 16 + D.n;
    const bool active = qi < Nq;
    const int64_t q0 = min<int64_t>((qt * nqg + qg) * 16, Nq - 1);
    RowFrag<NS> qf;
    qf.load(D, RowBlock(q, (int64_t)bh * Nq + q0, d, (int)min<int64_t>(16, Nq - q0)));

    for (int64_t r = blockIdx.z; r < chunks; r += gridDim.z) {
      // keys of this wave: part kp of ks of the chunk's 16-key blocks
      const int64_t lo = partials ? r * (Nk / R) + r * (Nk % R) / R : 0;
      const int64_t hi = partials ? (r + 1) * (Nk / R) + (r + 1) * (Nk % R) / R : Nk;
      const int64_t nb = (hi - lo + 15) / 16;
      int64_t key = lo + 16 * ((nb * kp) >> ks_log2);
      int64_t end = lo + 16 * ((nb * (kp + 1)) >> ks_log2);
      end = end < hi ? end : hi;

      float m = -INFINITY, l = 0.f;
      AccF32<NS> o;
      o.zero();

      RowFrag<NS> kf[2];
      ColFrag<NS> vf[2];
      auto block = [&](const float* base, int64_t row) {   // empty past `end`
        return RowBlock(base, row, d, (int)max<int64_t>(0, min<int64_t>(16, end - row)));
      };
      kf[0].load(D, block(kb, key));
      // NB blocks of 16 keys from `key`, whose first K fragments are in kf[0]; only NB = 1 may be
      // cut short by `end`.  The loads of the fragments that come next go out before each block's
      // products.
      auto tile = [&](auto nbc) {
        constexpr int NB = decltype(nbc)::value;
        f32x4 s[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          if (b + 1 < NB) kf[(b + 1) & 1].load(D, block(kb, key + 16 * (b + 1)));
          else vf[0].load(D, block(vb, key));
          __builtin_amdgcn_sched_barrier(0);
          s[b] = dot_rows(kf[b & 1], qf);
          __builtin_amdgcn_sched_barrier(0);
        }
        const int rows = NB == 1 ? (int)min<int64_t>(16, end - key) : 16;
        if (NB == 1 && rows < 16) {
          // keys past the end add nothing
          cold_path();
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (4 * D.g + i >= rows) s[0][i] = -INFINITY;
        }
        float mx = -INFINITY;
#pragma unroll
        for (int b = 0; b < NB; ++b)
          mx = fmaxf(mx, fmaxf(fmaxf(s[b][0], s[b][1]), fmaxf(s[b][2], s[b][3])));
        const float mnew = fmaxf(m, max_groups(mx) * scale);
        if (__builtin_amdgcn_ballot_w64(mnew > m)) {
          const float alpha = mnew > m ? expf(m - mnew) : 1.f;
          l *= alpha;
          o.scale(alpha);
          m = mnew;
        }
        const float ref = m == -INFINITY ? 0.f : m;   // every score so far -inf: P = 0, not NaN
#pragma unroll
        for (int b = 0; b < NB; ++b) {
#pragma unroll
          for (int i = 0; i < 4; ++i) s[b][i] = expf(__builtin_fmaf(s[b][i], scale, -ref));
          l += (s[b][0] + s[b][1]) + (s[b][2] + s[b][3]);
        }
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          if (b + 1 < NB) vf[(b + 1) & 1].load(D, block(vb, key + 16 * (b + 1)));
          else kf[0].load(D, block(kb, key + 16 * NB));
          __builtin_amdgcn_sched_barrier(0);
          o.add(vf[b & 1], s[b]);
          __builtin_amdgcn_sched_barrier(0);
        }
        key += 16 * NB;
      };
      while (key + 64 <= end) tile(std::integral_constant<int, 4>{});
      while (key < end) tile(std::integral_constant<int, 1>{});
      l = sum_groups(l);

      if (ks > 1) {
        float* mine = part + (wave * 16 + D.n) * kRow;
#pragma unroll
        for (int t = 0; t < NS; ++t) *reinterpret_cast<f32x4*>(mine + D.quad(t)) = o.quad(t);
        if (D.g == 0) {
          mine[16 * NS] = m;
          mine[16 * NS + 1] = l;
        }
        __syncthreads();
        if (kp == 0) {
          // the block's first wave adds the parts in key order
          float M = m;
          for (int p = 1; p < ks; ++p) M = fmaxf(M, mine[p * 16 * kRow + 16 * NS]);
          const float ref = M == -INFINITY ? 0.f : M;
          const float w0 = expf(m - ref);
          l *= w0;
          o.scale(w0);
          for (int p = 1; p < ks; ++p) {
            const float* other = mine + p * 16 * kRow;
            const float w = expf(other[16 * NS] - ref);
            l = __builtin_fmaf(w, other[16 * NS + 1], l);
#pragma unroll
            for (int t = 0; t < NS; ++t) {
              const f32x4 x = *reinterpret_cast<const f32x4*>(other + D.quad(t));
              f32x4 y = o.quad(t);
#pragma unroll
              for (int j = 0; j < 4; ++j) y[j] = __builtin_fmaf(w, x[j], y[j]);
              o.set_quad(t, y);
            }
          }
          m = M;
        }
        __syncthreads();
      }
      if (kp != 0 || !active) continue;

      const float inv = 1.0f / l;
      const float lse_r = m + logf(l);
      const int64_t row = (partials ? r * BH * Nq : 0) + (int64_t)bh * Nq + qi;
      float* orow = out + row * d;
      float wa = 0.f, wb = inv, lnew = lse_r;
      if (mode == (int)FwdMode::kStep && !first) {
        // Eq. (5) with the running result
        const float lold = lse[row];
        const float M = fmaxf(lold, lse_r);
        const float a = expf(lold - M), b = expf(lse_r - M);
        wa = a / (a + b);
        wb = b * inv / (a + b);
        lnew = M + logf(a + b);
#pragma unroll
        for (int t = 0; t < NS; ++t) {
          const f32x4 old = D.load4(orow, D.quad(t)), x = o.quad(t);
          f32x4 y;
#pragma unroll
          for (int j = 0; j < 4; ++j)
            y[j] = (lold == -INFINITY ? 0.f : old[j] * wa) + x[j] * wb;
          D.store4(orow, D.quad(t), y);
        }
      } else {
#pragma unroll
        for (int t = 0; t < NS; ++t) D.store4(orow, D.quad(t), o.quad(t) * wb);
      }
      if (D.g == 0) lse[row] = lnew;
    }
  }
}

template <int NS, int EDGE>
hipError_t launch_edge(const FwdArgs& a, FwdMode mode) {
  const bool partials = mode == FwdMode::kPartials;
  const int64_t blocks = (a.Nq + 15) / 16, chunks = partials ? a.R : 1;
  const int ks = f32_split(blocks * a.BH * chunks, (a.Nk + chunks - 1) / chunks);
  const int64_t tiles = (blocks * ks + kF32Waves - 1) / kF32Waves;
  // a workgroup takes further query tiles and chunks when the grid's limits cut it short
  const dim3 grid((uint32_t)std::min<int64_t>(tiles, 1 << 22), (uint32_t)a.BH,
                  (uint32_t)std::min<int64_t>(chunks, 65535));
  float* out = partials ? a.part_out : mode == FwdMode::kStep ? a.acc_out : (float*)a.out;
  float* lse = partials ? a.part_lse : mode == FwdMode::kStep ? a.acc_lse : a.lse;
  hipLaunchKernelGGL((fwd_f32_kernel<NS, EDGE>), grid, dim3(kThreads), 0, a.stream, (const float*)a.q,
                     (const float*)a.k, (const float*)a.v, out, lse, (int)mode, a.first ? 1 : 0,
                     a.BH, (int)a.H, (int)a.G, a.Nq, a.Nk, a.R, (int)a.d, a.scale,
                     __builtin_ctz(ks));
  return hipGetLastError();
}

template <int NS>
hipError_t launch(const FwdArgs& a, FwdMode mode) {
  if (a.d == 16 * NS) return launch_edge<NS, kFull>(a, mode);
  if (a.d % 4 == 0) return launch_edge<NS, kQuad>(a, mode);
  return launch_edge<NS, kAny>(a, mode);
}

}  // namespace

hipError_t launch_fwd_f32(const FwdArgs& a, FwdMode mode) {
  switch ((a.d + 15) / 16) {
    case 1: return launch<1>(a, mode);
    case 2: return launch<2>(a, mode);
    case 3: return launch<3>(a, mode);
    case 4: return launch<4>(a, mode);
    case 5: return launch<5>(a, mode);
    case 6: return launch<6>(a, mode);
    case 7: return launch<7>(a, mode);
    default: return launch<8>(a, mode);
  }
}

}  // namespace ringx
