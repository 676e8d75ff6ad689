// Recompute backward in fp32 (storage and arithmetic), any head dim 1..128, on the fp32 matrix
// cores (tiles and operand layouts in f32_tiles.h).
//
// Both halves recompute P_ij = exp(scale q_i.k_j - lse_i) from the merged log-sum-exp and
// dS_ij = P_ij (dout_i.v_j - D_i), over all keys whatever their chunk; one wave owns 16 stationary rows as B operands and streams 16
// rows of the other side at a time:
//   dK/dV: 16 keys; S = Q K^T, dP = dO V^T (lane: its key, queries 4 g + r), dV^T += dO^T P,
//          dK^T += Q^T dS, over every query of every query head that shares the K/V head;
//   dQ:    16 queries; S^T = K Q^T, dP^T = V dO^T, dQ^T += K^T dS^T, over every key.
// A workgroup's 8 waves are 8 / ks stationary blocks of ks waves, which take consecutive ranges of
// the stream and add their accumulators through LDS in stream order (rule in f32_split), so the
// result is bitwise reproducible.  The two halves are independent, and each alone leaves SIMDs
// idle on a small problem, so the whole backward is one launch over the tiles of both.
//
// Bound by the fp32 matrix rate (7 products of 2 Nq Nk d executed for the 5 of the definition) and,
// beside it, by what the waves read through L2 (a 256-byte fragment per product): H = 3, Nq = 1531,
// Nk = 3001, d = 100 takes 285 us, 76 TFLOP/s of executed products of the 154 that a large fp32
// library product reaches (63 ms with one thread per row and scalar FMAs).  Eight waves to a block
// instead of four, which share no fragments in L1, took 332 us; loading fragments a block ahead
// changed nothing.

#include "f32_tiles.h"
#include "ringx_kernels.h"

#include <algorithm>
#include <type_traits>

namespace ringx {
namespace {

constexpr int kThreads = 64 * kF32Waves;

struct BwdF32Args {
  const float *q, *k, *v, *dout, *lse, *delta;
  float *dq, *dk, *dv;
  int64_t Nq, Nk;
  int64_t tiles_kv, tiles_q;        // workgroup tiles of one K/V head's keys, one head's queries
  int64_t n_kv, n_q;                // all tiles of the two halves (0: half not wanted)
  int H, grp, d, acc_kv, acc_q;
  int ksl_kv, ksl_q;                // log2 of the waves that share a stationary block
  float scale;
};

// Sum of the ks waves' accumulators of one stationary block, in stream order, into its first wave.
template <int NS, int EDGE>
__device__ __forceinline__ void reduce_parts(AccF32<NS>& a, const F32Dims<NS, EDGE>& D, float* lds,
                                             int wave, int kp, int ks) {
  constexpr int kRow = 16 * NS + 4;
  float* mine = lds + (wave * 16 + D.n) * kRow;
  if (kp > 0) {
#pragma unroll
    for (int t = 0; t < NS; ++t) *reinterpret_cast<f32x4*>(mine + D.quad(t)) = a.quad(t);
  }
  __syncthreads();
  if (kp == 0) {
    for (int p = 1; p < ks; ++p) {
#pragma unroll
      for (int t = 0; t < NS; ++t)
        a.set_quad(t, a.quad(t) + *reinterpret_cast<const f32x4*>(mine + p * 16 * kRow + D.quad(t)));
    }
  }
  __syncthreads();
}

template <int NS, int EDGE>
__device__ __forceinline__ void store_rows(const AccF32<NS>& a, const F32Dims<NS, EDGE>& D, float* row,
                                           float f, int accumulate) {
#pragma unroll
  for (int t = 0; t < NS; ++t) {
    f32x4 x = a.quad(t) * f;
    if (accumulate) x += D.load4(row, D.quad(t));
    D.store4(row, D.quad(t), x);
  }
}

template <int NS, int EDGE>
__device__ __forceinline__ void dkdv_tile(const BwdF32Args& A, const F32Dims<NS, EDGE>& D, int64_t tile,
                                          float* lds, int wave) {
  const int ksl = A.ksl_kv, ks = 1 << ksl, kg = wave >> ksl, kp = wave & (ks - 1);
  const int64_t bh = tile / A.tiles_kv;   // K/V head (of B * H / grp)
  const int64_t key = ((tile % A.tiles_kv) * (kF32Waves >> ksl) + kg) * 16 + D.n;
  const bool active = key < A.Nk;
  const int64_t krow = bh * A.Nk + key;
  const int64_t k0 = min<int64_t>(((tile % A.tiles_kv) * (kF32Waves >> ksl) + kg) * 16, A.Nk - 1);
  const int krows = (int)min<int64_t>(16, A.Nk - k0);
  const int d = D.d;
  RowFrag<NS> kf, vf;
  kf.load(D, RowBlock(A.k, bh * A.Nk + k0, d, krows));
  vf.load(D, RowBlock(A.v, bh * A.Nk + k0, d, krows));
  AccF32<NS> dk, dv;
  dk.zero();
  dv.zero();

  // this wave's 16-query blocks: part kp of ks of the group's grp * nqb blocks
  const int hkv = A.H / A.grp;
  const int64_t qh0 = (bh / hkv) * A.H + (bh % hkv) * A.grp;
  const int64_t nqb = (A.Nq + 15) / 16, total = A.grp * nqb;
  int64_t blk = (total * kp) >> ksl;
  const int64_t end = (total * (kp + 1)) >> ksl;
  int64_t head = qh0 + blk / nqb, i0 = 16 * (blk % nqb);
  // Both forms of a row block are loaded together, so that the second finds its lines in L1 (4% at
  // d = 100), except at d > 96, where the four fragments would spill far more of the 256 registers
  // of a wave than the 4 to 8 (d <= 112) and 16 to 48 that spill as it is.
  constexpr bool kQcEarly = NS < 7;
  // A head's ragged last block is code of its own: its mask in the common loop, as a select or as a
  // branch, costs 4-8% (8 heads x 4096 x 4096, d = 64: 657 us, 665 with the block apart, 691 and 716).
  // At d = 97 .. 112 the second copy costs dK/dV alone 11% (3 x 1531 x 3001, d = 100: 213 -> 237 us)
  // and the branch gains 4% (205), so there the branch it is.
  constexpr bool kApart = NS != 7;
  auto block = [&](int rows, auto ragged) {
    const int64_t row0 = head * A.Nq + i0;
    const RowBlock qb(A.q, row0, d, rows), ob(A.dout, row0, d, rows);
    RowFrag<NS> qa, oa;
    ColFrag<NS> oc, qc;
    const f32x4 ls = RowBlock(A.lse, row0, 1, rows).load4_rows(D.g);
    const f32x4 dl = RowBlock(A.delta, row0, 1, rows).load4_rows(D.g);
    qa.load(D, qb);
    if constexpr (kQcEarly) qc.load(D, qb);
    oa.load(D, ob);
    oc.load(D, ob);
    __builtin_amdgcn_sched_barrier(0);
    const f32x4 s = dot_rows(qa, kf);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (!kQcEarly) qc.load(D, qb);
    const f32x4 dp = dot_rows(oa, vf);
    f32x4 p, ds;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      p[r] = expf(__builtin_fmaf(s[r], A.scale, -ls[r]));
      ds[r] = p[r] * (dp[r] - dl[r]);
    }
    if (decltype(ragged)::value || (!kApart && rows < 16)) {
      if (!kApart) cold_path();
      // queries past the end (zero rows) add nothing: a key with an infinite feature makes their
      // score 0 * inf and their P NaN
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (4 * D.g + r >= rows) p[r] = ds[r] = 0.f;
    }
    dv.add(oc, p);
    dk.add(qc, ds);
  };
  for (; blk < end; ++blk) {
    if (!kApart) {
      block((int)min<int64_t>(16, A.Nq - i0), std::false_type{});
    } else if (i0 + 16 <= A.Nq) {
      block(16, std::false_type{});
    } else {
      cold_path();
      block((int)(A.Nq - i0), std::true_type{});
    }
    i0 += 16;
    if (i0 >= A.Nq) {
      i0 = 0;
      ++head;
    }
  }
  if (ks > 1) {
    reduce_parts(dk, D, lds, wave, kp, ks);
    reduce_parts(dv, D, lds, wave, kp, ks);
  }
  if (kp == 0 && active) {
    store_rows(dk, D, A.dk + krow * d, A.scale, A.acc_kv);
    store_rows(dv, D, A.dv + krow * d, 1.f, A.acc_kv);
  }
}

template <int NS, int EDGE>
__device__ __forceinline__ void dq_tile(const BwdF32Args& A, const F32Dims<NS, EDGE>& D, int64_t tile,
                                        float* lds, int wave) {
  const int ksl = A.ksl_q, ks = 1 << ksl, qg = wave >> ksl, kp = wave & (ks - 1);
  const int64_t bh = tile / A.tiles_q;
  const int64_t qi = ((tile % A.tiles_q) * (kF32Waves >> ksl) + qg) * 16 + D.n;
  const bool active = qi < A.Nq;
  const int64_t qrow = bh * A.Nq + (active ? qi : A.Nq - 1);
  const int64_t q0 = min<int64_t>(((tile % A.tiles_q) * (kF32Waves >> ksl) + qg) * 16, A.Nq - 1);
  const int qrows = (int)min<int64_t>(16, A.Nq - q0);
  const int d = D.d;
  RowFrag<NS> qf, of;
  qf.load(D, RowBlock(A.q, bh * A.Nq + q0, d, qrows));
  of.load(D, RowBlock(A.dout, bh * A.Nq + q0, d, qrows));
  const float nl = -A.lse[qrow], dl = A.delta[qrow];
  AccF32<NS> dq;
  dq.zero();

  const int64_t kvh = kv_head(bh, A.H, A.grp);
  const int64_t nkb = (A.Nk + 15) / 16;
  int64_t j0 = 16 * ((nkb * kp) >> ksl);
  int64_t end = 16 * ((nkb * (kp + 1)) >> ksl);
  end = end < A.Nk ? end : A.Nk;
  auto block = [&](const float* base, int64_t j) {   // empty past `end`
    return RowBlock(base, kvh * A.Nk + j, d, (int)max<int64_t>(0, min<int64_t>(16, end - j)));
  };
  for (; j0 < end; j0 += 16) {
    RowFrag<NS> ka, va;
    ColFrag<NS> kc;
    ka.load(D, block(A.k, j0));
    kc.load(D, block(A.k, j0));
    va.load(D, block(A.v, j0));
    __builtin_amdgcn_sched_barrier(0);
    const f32x4 s = dot_rows(ka, qf);
    const f32x4 dp = dot_rows(va, of);
    f32x4 ds;
#pragma unroll
    for (int r = 0; r < 4; ++r) ds[r] = expf(__builtin_fmaf(s[r], A.scale, nl)) * (dp[r] - dl);
    if (j0 + 16 > end) {
      // keys past the end add nothing (their P = exp(-lse) need not be finite)
      cold_path();
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (j0 + 4 * D.g + r >= end) ds[r] = 0.f;
    }
    dq.add(kc, ds);
  }
  if (ks > 1) reduce_parts(dq, D, lds, wave, kp, ks);
  if (kp == 0 && active) store_rows(dq, D, A.dq + qrow * d, A.scale, A.acc_q);
}

template <int NS, int EDGE>
__global__ __launch_bounds__(kThreads, 2) void bwd_f32_kernel(BwdF32Args A) {
  __shared__ __attribute__((aligned(16))) float lds[kF32Waves * 16 * (16 * NS + 4)];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const F32Dims<NS, EDGE> D(A.d, lane);
  for (int64_t t = xcd_remap(blockIdx.x, gridDim.x); t < A.n_kv + A.n_q; t += gridDim.x) {
    if (t < A.n_kv) dkdv_tile(A, D, t, lds, wave);
    else dq_tile(A, D, t - A.n_kv, lds, wave);
  }
}

template <int NS, int EDGE>
hipError_t launch_edge(const BwdArgs& a, bool want_kv, bool want_q) {
  BwdF32Args A;
  A.q = (const float*)a.q, A.k = (const float*)a.k, A.v = (const float*)a.v;
  A.dout = (const float*)a.dout, A.lse = a.lse, A.delta = a.delta;
  A.dq = a.dq, A.dk = a.dk, A.dv = a.dv, A.Nq = a.Nq, A.Nk = a.Nk;
  A.H = (int)a.H, A.grp = (int)a.G, A.d = (int)a.d, A.scale = a.scale;
  A.acc_kv = a.accumulate_dkv ? 1 : 0, A.acc_q = a.accumulate_dq ? 1 : 0;
  const int64_t bkv = a.BH / a.G, kb = (a.Nk + 15) / 16, qb = (a.Nq + 15) / 16;
  // Both halves count whether or not this launch holds both: sharing a launch, each needs only its
  // share of the waves, and a half launched alone (the stages of the backward) sums in the same
  // order, so that the stages give the whole backward's bits.
  const int64_t all = kb * bkv + qb * a.BH;
  const int ks_kv = f32_split(all, a.G * a.Nq), ks_q = f32_split(all, a.Nk);
  A.ksl_kv = __builtin_ctz(ks_kv), A.ksl_q = __builtin_ctz(ks_q);
  A.tiles_kv = (kb * ks_kv + kF32Waves - 1) / kF32Waves;
  A.tiles_q = (qb * ks_q + kF32Waves - 1) / kF32Waves;
  A.n_kv = want_kv ? A.tiles_kv * bkv : 0;
  A.n_q = want_q ? A.tiles_q * a.BH : 0;
  // a workgroup takes further tiles when the grid's limit cuts it short
  const dim3 grid((uint32_t)std::min<int64_t>(A.n_kv + A.n_q, 1 << 22));
  hipLaunchKernelGGL((bwd_f32_kernel<NS, EDGE>), grid, dim3(kThreads), 0, a.stream, A);
  return hipGetLastError();
}

template <int NS>
hipError_t launch(const BwdArgs& a, bool want_kv, bool want_q) {
  if (a.d == 16 * NS) return launch_edge<NS, kFull>(a, want_kv, want_q);
  if (a.d % 4 == 0) return launch_edge<NS, kQuad>(a, want_kv, want_q);
  return launch_edge<NS, kAny>(a, want_kv, want_q);
}

hipError_t launch_any(const BwdArgs& a, bool want_kv, bool want_q) {
  switch ((a.d + 15) / 16) {
    case 1: return launch<1>(a, want_kv, want_q);
    case 2: return launch<2>(a, want_kv, want_q);
    case 3: return launch<3>(a, want_kv, want_q);
    case 4: return launch<4>(a, want_kv, want_q);
    case 5: return launch<5>(a, want_kv, want_q);
    case 6: return launch<6>(a, want_kv, want_q);
    case 7: return launch<7>(a, want_kv, want_q);
    default: return launch<8>(a, want_kv, want_q);
  }
}

}  // namespace

hipError_t launch_bwd_dkdv_f32(const BwdArgs& a) { return launch_any(a, true, false); }
hipError_t launch_bwd_dq_f32(const BwdArgs& a) { return launch_any(a, false, true); }
hipError_t launch_bwd_f32(const BwdArgs& a) { return launch_any(a, true, true); }

}  // namespace ringx
