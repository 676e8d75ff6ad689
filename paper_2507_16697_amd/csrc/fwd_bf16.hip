// Ring-chunked attention forward, bf16 storage, bf16 MFMA with fp32 accumulation (gfx950).
//
// One workgroup = 8 waves (two per SIMD) = one (b, h) and a tile of 256 queries (32 per wave), so
// that each K/V tile brought into LDS serves 256 queries; problems too small or uneven for that
// take smaller workgroups or split the keys among a workgroup's waves (query_cut in
// ringx_kernels.h).  The key/value sequence is visited as R chunks (ring steps, arXiv 2507.16697
// Sec. III-A), streamed through LDS in tiles of 64 keys that never straddle a chunk boundary; in
// fused mode key streams take the whole sequence in tiles of 64 keys (32 for four streams at
// d = 128) without regard to chunks, whose merge their own then is.  K and V tiles are double
// buffered (the on-chip analogue of the paper's ping-pong buffers) and filled by direct
// global->LDS loads: while tile j is processed, the K tile j+2 and the V tile j+1 are in flight.
//
// Each wave is software pipelined over key tiles: the MFMAs of S_{j+1} = K_{j+1} Q^T are
// interleaved with the exponentials and row sums of tile j, so that the matrix cores and the
// vector ALU work at the same time (the other wave of the SIMD runs its O += V^T P^T products
// meanwhile).  Per wave, with g = lane / 32 and n = lane % 32:
//   S^T = K Q^T   A = K rows from LDS (key n, 8 dims), B = Q^T from registers (query n, 8 dims)
//                 -> lane holds query n and keys 8*(r/4) + 4g + r%4 of each 32-key block;
//   O^T += V^T P^T A = V^T read from the row-major V tile with ds_read_b64_tr_b16 (4 keys per
//                 read), B = P^T straight from the S^T registers (keys 4g..4g+3, 8+4g..8+4g+3).
// LDS tiles are row-major with the 16-byte chunks of each row XOR-swizzled by the row index, so
// that both the 16-byte K reads (16 rows, one chunk) and the transposed V reads (4 rows x 2
// chunks per 16 lanes) hit distinct banks.
//
// Softmax statistics are fp32 in the exp2 domain (t = scale*log2(e)*q.k).  Eqs. (2)-(3) hold for
// any per-row reference m, not only the running maximum, so no row maximum is taken per tile: a
// tile's probabilities exp2(t - m) are formed against the current m, and only when a lane's sum
// of them reaches 2^32 (or is not finite, as on the first tile, whose m is still -inf) is the tile
// redone with m moved to its row maximum and the accumulators rescaled.  A lane's sum bounds each
// of its terms, so every probability stays below 2^32: bf16 and fp32 keep the same relative
// precision at any magnitude, and a row sum or output accumulator of at most 2^32 per key stays
// far inside the fp32 range for any realistic V.  At the end of chunk r (a workgroup without key
// streams) the wave forms the chunk's log-sum-exp loc_lse_r from the chunk's own row sum and folds it into the
// merged lse by Eq. (5).  The output numerator is kept unnormalised: Eq. (5)'s term
// exp(loc_lse_r - M) loc_out_r equals exp(m - M) times the chunk's unnormalised accumulator, so
// one accumulator holds the running sum of all chunk terms and the final division by the Eq. (5)
// denominator is a multiplication by 2^(m - lse).  MODE kPartials instead writes every chunk's
// (loc_out_r, loc_lse_r) and restarts the accumulator; MODE kStep (one chunk, R = 1) merges the
// chunk's result into a running fp32 (acc_out, acc_lse) by Eq. (5), one ring step at a time.

#include "ringx_device.h"
#include "ringx_kernels.h"

#include <type_traits>

namespace ringx {
namespace {

typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;

constexpr float kGuard = 4294967296.0f;   // 2^32: bound on a lane's probability sum

// KS key streams share a workgroup's NW waves (KS = 1: all of them take every key).
template <int D, int KS = 1, int NW = 8>
struct FwdCfg {
  static constexpr int kD = D;
  static constexpr int kThreads = 64 * NW;
  static constexpr int kWaves = NW;
  static constexpr int kSW = kWaves / KS;         // waves per key stream
  static constexpr int kQW = 32;                  // queries per wave
  static constexpr int kBQ = kSW * kQW;           // queries per workgroup
  static constexpr int kBK = KS * D > 256 ? 32 : 64;   // keys per tile (LDS holds 4 KS tiles)
  static constexpr int kRowBytes = D * 2;
  static constexpr int kChunks = D / 8;           // 16-byte chunks per row
  static constexpr int kTileBytes = kBK * kRowBytes;   // 16 KiB (64 keys, d = 128) or 8 KiB
  static constexpr int kKTiles = kBK / 32;        // 32-key blocks per tile
  static constexpr int kDSteps = D / 16;          // MFMA k-steps over the head dim
  static constexpr int kKSteps = kBK / 16;        // MFMA k-steps over the keys
  static constexpr int kCT = D / 32;              // 32-dim blocks of the output
  // Only waves 0..3, one on each SIMD, issue the tile loads: while a wave waits for the CU's load
  // path to take its loads, the other wave of its SIMD keeps the matrix core busy (2% faster at
  // d = 128 and 5% at d = 64 than all eight waves issuing at once; two loader waves: 1% and 3%).
  // With several streams the waves of each load that stream's tiles.
  static constexpr int kLoaders = kSW < 4 ? kSW : 4;
  static constexpr int kLoads = kTileBytes / (kLoaders * 64 * 16);   // 16-byte loads per loader lane
  static_assert(kLoads * kLoaders * 1024 == kTileBytes, "whole tiles per load round");
  // end of the streams: 4 kCT KiB of accumulators and 512 bytes of statistics per wave of the
  // streams after the first, in the tile buffers
  static constexpr int kXchWave = 4 * kCT * 1024 + 512;
  static_assert((kWaves - kSW) * kXchWave <= 4 * KS * kTileBytes, "stream exchange fits");
};

// Swizzled 16-byte chunk of (row, logical chunk c) inside a row-major tile.
template <int D>
__device__ __forceinline__ int swz(int row) {
  if constexpr (D == 128) return ((row & 3) << 2) | ((row >> 2) & 3);
  else return (((row >> 1) & 1) << 2) | ((row >> 2) & 3);
}
template <int D>
__device__ __forceinline__ int tile_off(int row, int c) {   // byte offset
  return row * (D * 2) + ((c ^ swz<D>(row)) << 4);
}


// Per-lane byte offsets (from the tile's first row) of this lane's direct loads: 16-byte slot
// `slot` of the swizzled tile holds logical chunk (slot % chunks) ^ swz(row) of row slot / chunks.
template <typename C>
__device__ __forceinline__ void load_offsets(int (&goff)[C::kLoads], int (&grow)[C::kLoads],
                                             int wave, int lane) {
#pragma unroll
  for (int u = 0; u < C::kLoads; ++u) {
    const int slot = (u * C::kLoaders + (wave % C::kLoaders)) * 64 + lane;
    const int row = slot / C::kChunks;
    const int c = (slot % C::kChunks) ^ swz<C::kD>(row);
    grow[u] = row;
    goff[u] = row * C::kRowBytes + c * 16;
  }
}

// Issue the direct loads of one K or V tile starting at key `start` into the LDS buffer at
// `dst`; rows at or past `hi` (only in the last tile of a chunk) are clamped to hi - 1.
// `wdst` is the loader wave's first 1 KiB slot (wave * 1024, an SGPR).
// `wave` counts within the stream.
template <typename C>
__device__ __forceinline__ void issue_tile(const char* __restrict__ base, uint32_t dst,
                                           uint32_t start, uint32_t hi,
                                           const int (&goff)[C::kLoads],
                                           const int (&grow)[C::kLoads], int wave, uint32_t wdst) {
  if (wave >= C::kLoaders) return;
  const char* src = base + (uint64_t)start * C::kRowBytes;
  if (start + C::kBK <= hi) {
#pragma unroll
    for (int u = 0; u < C::kLoads; ++u)
      load_lds16_s(src, (uint32_t)goff[u], dst + wdst + u * C::kLoaders * 1024);
  } else {
    cold_path();
    const int last = (int)(hi - 1 - start);
#pragma unroll
    for (int u = 0; u < C::kLoads; ++u) {
      const int off = grow[u] <= last ? goff[u] : goff[u] - (grow[u] - last) * C::kRowBytes;
      load_lds16_s(src, (uint32_t)off, dst + wdst + u * C::kLoaders * 1024);
    }
  }
}

// One workgroup = one (b, h), kBQ queries and the chunks [rg R / RG, (rg + 1) R / RG) (RG > 1 in
// partials mode only, where chunks are independent).  With KS > 1 key streams, stream p of the
// workgroup takes every KS-th key tile of the range (the whole range in fused and step mode, one
// chunk after the other in partials mode) and the streams merge through LDS at its end.
template <int D, int MODE, int KS, int NW>
__global__ __launch_bounds__(64 * NW, NW == 8 ? 1 : 3) void fwd_bf16_kernel(
    const __bf16* __restrict__ q, const __bf16* __restrict__ k, const __bf16* __restrict__ v,
    __bf16* __restrict__ out, float* __restrict__ lse, float* __restrict__ part_out,
    float* __restrict__ part_lse, float* __restrict__ acc_out, float* __restrict__ acc_lse,
    int first, int BH, int H, int grp, int64_t Nq, int64_t Nk, int R, int RG, float c2) {
  using C = FwdCfg<D, KS, NW>;
  constexpr bool kPartials = MODE == (int)FwdMode::kPartials;
  constexpr bool kStep = MODE == (int)FwdMode::kStep;
  constexpr bool kFused = MODE == (int)FwdMode::kFused;
  // K buffers of every stream, then V buffers
  __shared__ __attribute__((aligned(1024))) char lds[4 * KS * C::kTileBytes];
  char* const lds_k = lds;
  char* const lds_v = lds + 2 * KS * C::kTileBytes;

  const int t = threadIdx.x;
  const int lane = t & 63;
  const int wave8 = __builtin_amdgcn_readfirstlane(t >> 6);
  const int ks = KS == 1 ? 0 : wave8 / C::kSW;           // key stream
  const int wave = KS == 1 ? wave8 : wave8 % C::kSW;     // wave of the stream
  const int n = lane & 31;
  const int g = lane >> 5;

  const int64_t nqt = (Nq + C::kBQ - 1) / C::kBQ;
  uint32_t wg = xcd_remap(blockIdx.x, gridDim.x);
  const int64_t q0 = (wg % nqt) * C::kBQ + wave * C::kQW;
  wg /= nqt;
  const int64_t bh = kPartials ? wg / RG : wg;
  if (bh >= BH) return;

  const uint32_t nk = (uint32_t)Nk;
  // this workgroup's chunks and their keys [key_lo, key_hi)
  int r0 = 0;
  uint32_t key_lo = 0, key_hi = nk;
  ChunkWalk walk{nk, nk / (uint32_t)R, nk % (uint32_t)R, 0, (uint32_t)R};
  int r_end = R;
  if (kPartials && RG > 1) {
    const uint32_t rg = wg % RG;
    r0 = (int)((uint64_t)rg * R / RG);
    r_end = (int)((uint64_t)(rg + 1) * R / RG);
    key_lo = (uint32_t)((uint64_t)r0 * nk / R);
    key_hi = (uint32_t)((uint64_t)r_end * nk / R);
    walk.Nk = key_hi;
    walk.racc = (uint32_t)((uint64_t)r0 * walk.rem % (uint32_t)R);
  }

  const __bf16* qb = q + bh * Nq * D;
  const int64_t kvh = kv_head(bh, H, grp);
  // wave-uniform bases in SGPRs, so that the per-tile load addresses are scalar arithmetic
  const char* kb =
      static_cast<const char*>(uniform_ptr(reinterpret_cast<const char*>(k + kvh * Nk * D)));
  const char* vb =
      static_cast<const char*>(uniform_ptr(reinterpret_cast<const char*>(v + kvh * Nk * D)));
  int goff[C::kLoads], grow[C::kLoads];
  load_offsets<C>(goff, grow, wave, lane);

  uint32_t wdst = (uint32_t)__builtin_amdgcn_readfirstlane(wave * 1024);
  // Tiles of this wave's stream: t0 the current one, t1 and t2 the next two.  `key_end`: a tile
  // that starts there or later does not exist.
  KeyTile t0, t1, t2;
  uint32_t key_end = key_hi;
  int it = 0, nit = 0;        // KS > 1: the range's tile round and number of rounds
  auto next_tile = [&](const KeyTile& x) -> KeyTile {
    if constexpr (KS == 1) return walk.next<C::kBK>(x);
    else return KeyTile{x.start + KS * C::kBK, x.hi};
  };

  // LDS byte addresses of the two K and two V buffers of the stream
  const int st_off = 2 * ks * C::kTileBytes;
  const char* const my_k = lds_k + st_off;
  const char* const my_v = lds_v + st_off;
  const uint32_t lk = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds_k + st_off;
  const uint32_t lv = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds_v + st_off;

  // K_0, V_0 and K_1 of the range that starts at `lo` (KS > 1: and ends at `hi`)
  auto start_range = [&](uint32_t lo, uint32_t hi) {
    if constexpr (KS == 1) {
      t0 = walk.first(lo);
    } else {
      key_end = hi;
      it = 0;
      nit = (int)(((hi - lo + C::kBK - 1) / C::kBK + KS - 1) / KS);
      t0 = KeyTile{lo + ks * C::kBK, hi};
    }
    t1 = next_tile(t0);
    t2 = next_tile(t1);
    if (KS == 1 || t0.start < key_end) {
      issue_tile<C>(kb, lk, t0.start, t0.hi, goff, grow, wave, wdst);
      issue_tile<C>(vb, lv, t0.start, t0.hi, goff, grow, wave, wdst);
    }
    if (t1.start < key_end)
      issue_tile<C>(kb, lk + C::kTileBytes, t1.start, t1.hi, goff, grow, wave, wdst);
  };
  // in flight while Q is loaded
  if constexpr (KS > 1 && kPartials) {
    uint32_t hi0 = key_lo + walk.q_sz;
    if (walk.racc + walk.rem >= walk.R) ++hi0;
    start_range(key_lo, hi0);
  } else {
    start_range(key_lo, key_hi);
  }

  // Q fragments (B operand of S^T = K Q^T): query n of this wave, dims 16*ks + 8g .. +8.
  bf16x8 qf[C::kDSteps];
  {
    int64_t qi = q0 + n;
    qi = qi < Nq ? qi : Nq - 1;
#pragma unroll
    for (int s = 0; s < C::kDSteps; ++s)
      qf[s] = *reinterpret_cast<const bf16x8*>(qb + qi * D + s * 16 + g * 8);
  }

  // per-lane LDS byte offsets (tile-relative)
  int koff[C::kDSteps];   // K fragment of 32-key block 0 at k-step s (block kt adds kt*32 rows)
#pragma unroll
  for (int s = 0; s < C::kDSteps; ++s) koff[s] = tile_off<D>(n, 2 * s + g);
  // V^T fragments via transposed reads: for 16-lane group G, rows j0 + (lane%16)/4 with
  // j0 = 16*ks + 4g (+8 for the second half), columns 32*ct + 16*(G%2) + 4*(lane%4).
  int voff[2][C::kCT];
  {
    const int G = lane >> 4;
    const int rr = (lane & 15) >> 2;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int ct = 0; ct < C::kCT; ++ct) {
        const int row = 4 * g + 8 * h + rr;
        const int col = 32 * ct + 16 * (G & 1) + 4 * (lane & 3);
        voff[h][ct] = tile_off<D>(row, col >> 3) + (col & 7) * 2;
      }
  }

  f32x16 oacc[C::kCT];
#pragma unroll
  for (int c = 0; c < C::kCT; ++c) oacc[c] = f32x16{};
  float m2 = -INFINITY;     // reference max of the row (exp2 domain)
  float lc = 0.f;           // this lane's share of the chunk's row sum, relative to m2
  float lse2m = -INFINITY;  // merged log2-sum-exp over finished chunks (Eq. (5))

  f32x16 sa[C::kKTiles], sb[C::kKTiles];
  // S_0, once K_0 has landed
  auto first_scores = [&] {
    wait_vmem_all();
    __syncthreads();
#pragma unroll
    for (int kt = 0; kt < C::kKTiles; ++kt) sa[kt] = f32x16{};
#pragma unroll
    for (int s = 0; s < C::kDSteps; ++s)
#pragma unroll
      for (int kt = 0; kt < C::kKTiles; ++kt)
        sa[kt] = mfma32(*reinterpret_cast<const bf16x8*>(my_k + koff[s] + kt * 32 * C::kRowBytes),
                        qf[s], sa[kt]);
  };

  // The result of chunk r (its row sum `lrow` and log2-sum-exp `lse2r`, the accumulators as they
  // are) where it goes: folded into the running (acc_out, acc_lse), or to the partials.
  auto put_step = [&](float lrow, float lse2r) {
    // Eq. (5) with the running result: out_acc <- (out_acc a + loc_out b) / (a + b)
    const int64_t qi = q0 + n;
    if (qi < Nq) {
      const int64_t row = bh * Nq + qi;
      float* ao = acc_out + row * D;
      const float inv = 1.0f / lrow;
      float wa = 0.f, wb = inv;
      float lnew = lse2r;
      if (!first) {
        const float lold = acc_lse[row] * kLog2e;
        const float M = fmaxf(lold, lse2r);
        const float a = fast_exp2(lold - M);
        const float b = fast_exp2(lse2r - M);
        const float den = a + b;
        wa = a / den;
        wb = b * inv / den;
        lnew = M + fast_log2(den);
      }
#pragma unroll
      for (int c = 0; c < C::kCT; ++c)
#pragma unroll
        for (int rq = 0; rq < 4; ++rq) {
          f32x4* dst = reinterpret_cast<f32x4*>(ao + c * 32 + 8 * rq + 4 * g);
          const f32x4 prev = first ? f32x4{} : *dst;
          f32x4 val;
#pragma unroll
          for (int e = 0; e < 4; ++e) val[e] = prev[e] * wa + oacc[c][4 * rq + e] * wb;
          *dst = val;
        }
      if (g == 0) acc_lse[row] = lnew * kLn2;
    }
  };
  auto put_partial = [&](int r, float lrow, float lse2r) {
    const int64_t qi = q0 + n;
    if (qi < Nq) {
      const float inv = 1.0f / lrow;
      const int64_t row = ((int64_t)r * BH + bh) * Nq + qi;
      float* po = part_out + row * D;
#pragma unroll
      for (int c = 0; c < C::kCT; ++c)
#pragma unroll
        for (int rq = 0; rq < 4; ++rq) {
          f32x4 val = {oacc[c][4 * rq] * inv, oacc[c][4 * rq + 1] * inv,
                       oacc[c][4 * rq + 2] * inv, oacc[c][4 * rq + 3] * inv};
          *reinterpret_cast<f32x4*>(po + c * 32 + 8 * rq + 4 * g) = val;
        }
      if (g == 0) part_lse[row] = lse2r * kLn2;
    }
  };

  // One pipelined iteration for tile t0 (scores in `cur`); parity P selects the buffers: K_{j+1}
  // is read from K buffer 1-P, V_j from V buffer P; K_{j+2} lands in K buffer P, V_{j+1} in V
  // buffer 1-P.  Returns true after the last tile.
  auto step = [&](f32x16 (&cur)[C::kKTiles], f32x16 (&nxt)[C::kKTiles], auto parity) -> bool {
    constexpr int P = decltype(parity)::value;
    // K_{j+1} and V_j landed (issued one iteration ago); every wave is done with K_j, V_{j-1}
    wait_vmem_all();
    __syncthreads();
    // wdst counts as redefined here, so that the load slots' addresses are formed at each use
    // (scalar adds) instead of being held in registers across the loop
    asm volatile("" : "+s"(wdst));
    if (t2.start < key_end)
      issue_tile<C>(kb, lk + P * C::kTileBytes, t2.start, t2.hi, goff, grow, wave, wdst);
    if (t1.start < key_end)
      issue_tile<C>(vb, lv + (1 - P) * C::kTileBytes, t1.start, t1.hi, goff, grow, wave, wdst);
    // a stream's last round may hold no tile of its own
    if (KS > 1 && t0.start >= key_end) return ++it >= nit;
    // The vector work of this half (exponentials, row sums) is the longer chain; it issues ahead
    // of the other wave's matrix products on the SIMD, which fill the gaps (priority drops again
    // for the P V half).
    __builtin_amdgcn_s_setprio(1);

    // last tile of a chunk: keys past the chunk end (clamped copies of its last key) add nothing
    const int nvalid = (int)min<uint32_t>(C::kBK, t0.hi - t0.start);
    if (nvalid < C::kBK) {
      cold_path();
      const int thr = nvalid - 4 * g;   // key 4g + off is past the end iff off >= thr
#pragma unroll
      for (int kt = 0; kt < C::kKTiles; ++kt)
#pragma unroll
        for (int rr = 0; rr < 16; ++rr)
          if (kt * 32 + 8 * (rr >> 2) + (rr & 3) >= thr) cur[kt][rr] = -INFINITY;
    }
    // S_{j+1} = K_{j+1} Q^T on the matrix cores, P_j = exp2(t - m) on the vector ALU
    const char* kbuf = my_k + (1 - P) * C::kTileBytes;
#pragma unroll
    for (int kt = 0; kt < C::kKTiles; ++kt) nxt[kt] = f32x16{};
#pragma unroll
    for (int s = 0; s < C::kDSteps; ++s)
#pragma unroll
      for (int kt = 0; kt < C::kKTiles; ++kt)
        nxt[kt] = mfma32(*reinterpret_cast<const bf16x8*>(kbuf + koff[s] + kt * 32 * C::kRowBytes),
                         qf[s], nxt[kt]);
    bf16x8 pf[C::kKSteps];
    float la = 0.f, lb = 0.f;
#pragma unroll
    for (int kt = 0; kt < C::kKTiles; ++kt)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        u32x4 w;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float p0 = fast_exp2(__builtin_fmaf(cur[kt][8 * h + 2 * e], c2, -m2));
          const float p1 = fast_exp2(__builtin_fmaf(cur[kt][8 * h + 2 * e + 1], c2, -m2));
          la += p0;
          lb += p1;
          w[e] = pack_bf16x2(p0, p1);
        }
        pf[2 * kt + h] = __builtin_bit_cast(bf16x8, w);
      }
    // at d = 128, four vector-ALU instructions (and, with them, two exponentials) beside each of
    // the 16 S products spread the tile's exponentials evenly over them (seven per product
    // front-loaded them onto the first nine and ran 1.5% slower; three and five were 0.3% and
    // 1.1% slower); d = 64 has half as many products for the same vector work and takes eight
    // per product (2-4% faster than seven, nine or ten)
    constexpr int kValuPerProduct = D == 128 ? 4 : 8;
    __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
    for (int i = 0; i < C::kDSteps * C::kKTiles; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, kValuPerProduct, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    // the reference m moves only when a probability of the tile could reach 2^32: the rare tile
    // that fails the check is redone against its row maximum
    if (__builtin_amdgcn_ballot_w64(!(la + lb < kGuard))) {
      cold_path();
      float ma = -INFINITY;
#pragma unroll
      for (int kt = 0; kt < C::kKTiles; ++kt)
#pragma unroll
        for (int rr = 0; rr < 16; ++rr) ma = fmaxf(ma, cur[kt][rr]);
      float mnew = fmaxf(m2, max_halves(ma) * c2);
      // a stream may meet scores of -inf alone (keys masked by an infinite feature) that one stream
      // over all keys would weigh at 0: a finite reference keeps its sums 0 instead of NaN
      if constexpr (KS > 1) mnew = fmaxf(mnew, -3e38f);
      const float alpha = fast_exp2(m2 - mnew);
      m2 = mnew;
      lc *= alpha;
#pragma unroll
      for (int c = 0; c < C::kCT; ++c) oacc[c] *= alpha;
      la = 0.f;
      lb = 0.f;
#pragma unroll
      for (int kt = 0; kt < C::kKTiles; ++kt)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          u32x4 w;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float p0 = fast_exp2(__builtin_fmaf(cur[kt][8 * h + 2 * e], c2, -m2));
            const float p1 = fast_exp2(__builtin_fmaf(cur[kt][8 * h + 2 * e + 1], c2, -m2));
            la += p0;
            lb += p1;
            w[e] = pack_bf16x2(p0, p1);
          }
          pf[2 * kt + h] = __builtin_bit_cast(bf16x8, w);
        }
    }
    lc += la + lb;

    __builtin_amdgcn_s_setprio(0);
    // O += V_j^T P_j on the matrix cores
    const char* vbuf = my_v + P * C::kTileBytes;
#pragma unroll
    for (int s = 0; s < C::kKSteps; ++s)
#pragma unroll
      for (int c = 0; c < C::kCT; ++c) {
        const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
            (lds_bf16x4*)(vbuf + voff[0][c] + s * 16 * C::kRowBytes));
        const bf16x4 hi4 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
            (lds_bf16x4*)(vbuf + voff[1][c] + s * 16 * C::kRowBytes));
        oacc[c] = mfma32(__builtin_shufflevector(lo, hi4, 0, 1, 2, 3, 4, 5, 6, 7), pf[s], oacc[c]);
      }
    __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
    for (int i = 0; i < C::kKSteps * C::kCT; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
    }
    __builtin_amdgcn_sched_barrier(0);

    // the last tile of its chunk?  (step mode has one chunk, whose end is the loop's)
    const bool chunk_end = KS == 1 && !kStep && t0.start + C::kBK >= t0.hi;
    if (kFused && chunk_end) {
      // end of chunk r0: loc_lse_r from the chunk's own row sum, merged by Eq. (5) on the
      // log-sum-exps; the numerator terms already share the reference m2
      const float lse2r = m2 + fast_log2(sum_halves(lc));
      const float M = fmaxf(lse2m, lse2r);
      lse2m = M + fast_log2(fast_exp2(lse2m - M) + fast_exp2(lse2r - M));
      lc = 0.f;
    }
    t0 = t1;
    t1 = t2;
    t2 = next_tile(t2);
    if constexpr (KS == 1) return kPartials ? chunk_end : t0.start >= key_end;
    else return ++it >= nit;
  };
  auto run_range = [&] {
    first_scores();
    while (true) {
      if (step(sa, sb, std::integral_constant<int, 0>{})) break;
      if (step(sb, sa, std::integral_constant<int, 1>{})) break;
    }
  };

  if constexpr (KS == 1 && kPartials) {
    // Chunk ends leave the tile loop and come back to it where they left, pipeline intact: with
    // the stores inside the loop the compiler orders the exponentials so that each waits for its
    // own result (26 wait states per tile at d = 64).
    first_scores();
    bool odd = false;
    while (true) {
      while (true) {
        if (!odd) {
          odd = true;
          if (step(sa, sb, std::integral_constant<int, 0>{})) break;
        }
        odd = false;
        if (step(sb, sa, std::integral_constant<int, 1>{})) break;
      }
      const float lrow = sum_halves(lc);
      put_partial(r0, lrow, m2 + fast_log2(lrow));
      if (t0.start >= key_end) break;
#pragma unroll
      for (int c = 0; c < C::kCT; ++c) oacc[c] = f32x16{};
      m2 = -INFINITY;
      lc = 0.f;
      ++r0;
    }
  } else if constexpr (KS == 1) {
    run_range();
    if constexpr (kStep) {
      const float lrow = sum_halves(lc);
      put_step(lrow, m2 + fast_log2(lrow));
    }
  } else {
    while (true) {
      const uint32_t hi = key_end;
      run_range();
      // The streams' (m, l, O) of this range through LDS into stream 0, in stream order.  Every
      // wave is past its last tile read once all have met here.
      __syncthreads();
      char* const xch = lds;
      float lrow = sum_halves(lc);
      if (ks > 0) {
        char* mine = xch + ((ks - 1) * C::kSW + wave) * C::kXchWave;
#pragma unroll
        for (int c = 0; c < C::kCT; ++c)
#pragma unroll
          for (int rq = 0; rq < 4; ++rq)
            *reinterpret_cast<f32x4*>(mine + (c * 4 + rq) * 1024 + lane * 16) =
                f32x4{oacc[c][4 * rq], oacc[c][4 * rq + 1], oacc[c][4 * rq + 2],
                      oacc[c][4 * rq + 3]};
        *reinterpret_cast<f32x2*>(mine + C::kCT * 4096 + lane * 8) = f32x2{m2, lrow};
      }
      __syncthreads();
      if (ks == 0) {
        const char* const others = xch + wave * C::kXchWave;
        float M = m2;
        f32x2 st[KS - 1];
#pragma unroll
        for (int p = 0; p < KS - 1; ++p) {
          st[p] = *reinterpret_cast<const f32x2*>(others + p * C::kSW * C::kXchWave +
                                                  C::kCT * 4096 + lane * 8);
          M = fmaxf(M, st[p][0]);
        }
        const float w0 = fast_exp2(m2 - M);
        lrow *= w0;
#pragma unroll
        for (int c = 0; c < C::kCT; ++c) oacc[c] *= w0;
#pragma unroll
        for (int p = 0; p < KS - 1; ++p) {
          const float w = fast_exp2(st[p][0] - M);
          lrow = __builtin_fmaf(w, st[p][1], lrow);
#pragma unroll
          for (int c = 0; c < C::kCT; ++c)
#pragma unroll
            for (int rq = 0; rq < 4; ++rq) {
              const f32x4 x = *reinterpret_cast<const f32x4*>(
                  others + p * C::kSW * C::kXchWave + (c * 4 + rq) * 1024 + lane * 16);
#pragma unroll
              for (int e = 0; e < 4; ++e)
                oacc[c][4 * rq + e] = __builtin_fmaf(w, x[e], oacc[c][4 * rq + e]);
            }
        }
        const float lse2r = M + fast_log2(lrow);
        if constexpr (kFused) {
          m2 = M;
          lse2m = lse2r;
        } else if constexpr (kStep) {
          put_step(lrow, lse2r);
        } else {
          put_partial(r0, lrow, lse2r);
        }
      }
      if constexpr (!kPartials) break;
      // the next chunk of this workgroup
      if (++r0 >= r_end) break;
      __syncthreads();
#pragma unroll
      for (int c = 0; c < C::kCT; ++c) oacc[c] = f32x16{};
      m2 = -INFINITY;
      lc = 0.f;
      start_range(hi, (uint32_t)((uint64_t)(r0 + 1) * nk / R));
    }
  }

  if (kFused && ks == 0) {
    const int64_t qi = q0 + n;
    if (qi < Nq) {
      // out = numerator / Eq. (5) denominator = oacc * 2^(m - lse)
      const float f = fast_exp2(m2 - lse2m);
      __bf16* ob = out + (bh * Nq + qi) * D;
#pragma unroll
      for (int c = 0; c < C::kCT; ++c)
#pragma unroll
        for (int rq = 0; rq < 4; ++rq) {
          u32x2 w;
          w[0] = pack_bf16x2(oacc[c][4 * rq] * f, oacc[c][4 * rq + 1] * f);
          w[1] = pack_bf16x2(oacc[c][4 * rq + 2] * f, oacc[c][4 * rq + 3] * f);
          *reinterpret_cast<u32x2*>(ob + c * 32 + 8 * rq + 4 * g) = w;
        }
      if (g == 0) lse[bh * Nq + qi] = lse2m * kLn2;
    }
  }
}

template <int D, int MODE, int KS, int NW>
hipError_t launch(const FwdArgs& a, int64_t RG) {
  using C = FwdCfg<D, KS, NW>;
  const int64_t nwg = (a.Nq + C::kBQ - 1) / C::kBQ * a.BH * RG;
  hipLaunchKernelGGL((fwd_bf16_kernel<D, MODE, KS, NW>), dim3((uint32_t)nwg), dim3(C::kThreads), 0,
                     a.stream, (const __bf16*)a.q, (const __bf16*)a.k, (const __bf16*)a.v,
                     (__bf16*)a.out, a.lse, a.part_out, a.part_lse, a.acc_out, a.acc_lse,
                     a.first ? 1 : 0, (int)a.BH, (int)a.H, (int)a.G, a.Nq, a.Nk, (int)a.R, (int)RG,
                     a.scale * kLog2e);
  return hipGetLastError();
}

template <int D, int MODE>
hipError_t launch_plan(const FwdArgs& a) {
  const FwdPlan p = fwd_plan((a.Nq + 255) / 256 * a.BH, a.Nk, a.R, D, MODE == (int)FwdMode::kPartials);
  if constexpr (D == 64)
    if (p.cut.half) return launch<D, MODE, 1, 4>(a, p.rg);
  if constexpr (MODE != (int)FwdMode::kPartials)
    if (p.cut.ks == 4) return launch<D, MODE, 4, 8>(a, p.rg);
  if (p.cut.ks == 2) return launch<D, MODE, 2, 8>(a, p.rg);
  return launch<D, MODE, 1, 8>(a, p.rg);
}

template <int D>
hipError_t launch_mode(const FwdArgs& a, FwdMode mode) {
  switch (mode) {
    case FwdMode::kPartials: return launch_plan<D, (int)FwdMode::kPartials>(a);
    case FwdMode::kStep: return launch_plan<D, (int)FwdMode::kStep>(a);
    default: return launch_plan<D, (int)FwdMode::kFused>(a);
  }
}

}  // namespace

int64_t fwd_bf16_workgroups(int64_t BH, int64_t Nq, int64_t d) {
  (void)d;
  const int64_t bq = FwdCfg<128>::kBQ;
  static_assert(FwdCfg<128>::kBQ == FwdCfg<64>::kBQ, "one query tile size");
  return BH * ((Nq + bq - 1) / bq);
}

hipError_t launch_fwd_bf16(const FwdArgs& a, FwdMode mode) {
  return a.d == 128 ? launch_mode<128>(a, mode) : launch_mode<64>(a, mode);
}

}  // namespace ringx
