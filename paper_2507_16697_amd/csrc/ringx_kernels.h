// Host-side launch interface between the C ABI layer (ringx_api.cpp) and the kernel files.
// Arguments arrive here already validated.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ringx {

// What the forward does with each chunk's local result (loc_out_r, loc_lse_r).
enum class FwdMode {
  kFused = 0,     // Eq. (5) merge of all R chunks in registers -> out, lse
  kPartials = 1,  // write every chunk's result -> part_out, part_lse
  kStep = 2,      // R = 1: merge the one chunk into the running fp32 acc_out, acc_lse
};

// How the query-stationary bf16 kernels (forward, dQ) cut a launch.  Whole: workgroups of 256
// queries, one per CU, so n of them take ceil(n / 256) rounds, and with few of them, or few in the
// last round, most of the chip is idle.
struct QueryCut {
  int ks = 1;          // key streams: an 8-wave workgroup takes 256 / ks queries, its waves split the
                       // keys ks ways
  bool half = false;   // 4-wave workgroups of 128 queries, three per CU (d = 64)
};
// What a kernel gains beyond rounds that are half empty or emptier.  A kernel with half-size workgroups
// takes them in ragged launches, and in full rounds from n = half_from on, up to half_keys keys;
// one without (half_from = 0) takes two streams in ragged launches, from split_keys[0] keys on up
// to two rounds and from split_keys[1] on up to three.
struct CutRule {
  int64_t half_from, half_keys;
  int64_t split_keys[2];
};
// n = B H ceil(Nq / 256); `keys` that one workgroup visits.  Measured at 8192 keys, two heads (us; one,
// two and four streams, *half-size):
//   n =            96           128          192          288              384              768
//   forward d=64   130 84 96    123 82 92    127 148 136  260 222 195*     259 240 217*     422 458 419*
//   forward d=128  178 127 152  168 130 152  200 222 230  388 338          387 370          679 731
//   dQ d=64        156 94 106   157 103 112  162 180 165  327 275 249*     329 299 282*     566 586
//   dQ d=128       263 157 199  263 181 212  270 311 316  575 485          576 528          963 1043
// and at n = 64, 4096 keys: 66 40 28, 88 54 45, 81 46 34 and 138 81 64.  So: four streams as long
// as one round holds the quarter-size workgroups, two while it holds the half-size ones; where the
// last round is at most half full, half-size workgroups, which end closer together.  In full rounds
// splitting loses, because a tile serves fewer queries, unless three half-size workgroups on a CU
// gain more by covering each other's barriers, first and last tiles:
// the d = 64 forward does up to 16384 keys (n = 1024: 1024 keys 97 -> 85, 4096 301 -> 284, 16384
// 1130 -> 1072; 2% slower at 262144), dQ up to 4096 keys and from three rounds on (1024 keys 118 ->
// 110, n = 768 at 2048 keys 160 -> 153, n = 3072 at 4096 1138 -> 1108; n = 512 197 against 204).
// At d = 128, without half-size workgroups, two streams in a ragged launch have a fixed cost (a
// merge, and a wave's own Q for half as many keys) and pay only where the round they save is long.
// Speed-up over one stream by n and keys (lowest and highest of five n in each range):
//   forward     300         512         1500        4096        8192        16384       32768
//   257 .. 384  0.86 0.89   0.91 0.94   0.96 1.05   1.03 1.09   1.02 1.11   1.06 1.12   1.17 1.24
//   513 .. 640  0.79 0.83   0.85 0.89   0.91 0.94   0.95 0.99   0.98 1.00   0.97 1.09   1.04 1.14
//   769 .. 896  0.74 0.80   0.79 0.82   0.87 0.91   0.91 0.96   0.93 0.97   0.98 1.05   1.01 1.04
//   dQ
//   257 .. 384  1.02 1.06   1.07 1.13   1.07 1.17   1.10 1.11   1.10 1.12   1.12 1.15   1.15 1.26
//   513 .. 640  0.97 0.99   0.99 1.09   1.01 1.03   0.99 1.04   1.01 1.05   1.04 1.13   1.04 1.12
//   769 .. 896  0.96 0.98   0.96 0.98   0.98 1.03   0.96 1.00   0.95 0.99   1.00 1.12   1.00 1.02
inline QueryCut query_cut(int64_t n, int64_t keys, const CutRule& r) {
  QueryCut c;
  const bool ragged = n > 256 && n < 1024 && (n - 1) % 256 < 128;
  if (r.half_from > 0 && (ragged || (n >= r.half_from && keys <= r.half_keys))) c.half = true;
  else if (n <= 64) c.ks = 4;
  else if (n <= 128) c.ks = 2;
  else if (ragged && n <= 768 && keys >= r.split_keys[n <= 512 ? 0 : 1]) c.ks = 2;
  while (c.ks > 1 && keys < 64 * c.ks) c.ks /= 2;
  return c;
}
// half-size forms exist at d = 64 only
inline CutRule fwd_cut_rule(int64_t d) {
  return d == 64 ? CutRule{512, 16384, {0, 0}} : CutRule{0, 0, {2048, 16384}};
}
inline CutRule dq_cut_rule(int64_t d) {
  return d == 64 ? CutRule{768, 4096, {0, 0}} : CutRule{0, 0, {0, 1024}};
}

struct FwdPlan {
  QueryCut cut;
  int64_t rg = 1;   // chunk groups (partials)
};

// n = B H ceil(Nq / 256) as above, R chunks of Nk keys.
// Partials: chunks are independent, so they are spread over workgroups, over as few groups as give
// the shortest launch (480 workgroups, whose two rounds are nearly full, lose 2% to four groups),
// and up to four rounds where one is at most half full (Nq = 2048, 8 chunks of 4096, 16 heads,
// d = 128: 664 us whole, 479 in one round, 453 in four).  A launch's length is its rounds times the
// chunks of the largest group; at d = 128 a chunk costs as much as 320 keys more (its stores) and a
// workgroup 370 (its queries, the first tiles), fitted to the times of whole and grouped launches
// of 130 .. 2000 workgroups, 2 .. 8 chunks of 300 .. 4000 keys.  Without these two, 200 workgroups
// of 8 chunks of 300 keys took eight groups and 1.30 times as long as whole (1000 keys: 1.08).
// d = 64, whose workgroups are half as large in such launches, gained in every grouped launch.
inline FwdPlan fwd_plan(int64_t n, int64_t Nk, int64_t R, int64_t d, bool partials) {
  FwdPlan p;
  if (partials) {
    const double chunk = (double)Nk / (double)R + (d == 128 ? 320 : 0), start = d == 128 ? 370 : 0;
    auto length = [&](int64_t rg) {
      return (double)((n * rg + 255) / 256) * ((double)((R + rg - 1) / rg) * chunk + start);
    };
    for (int64_t rg = 1; rg < R && n * rg < 2048;) {
      rg = 2 * rg < R ? 2 * rg : R;
      if (length(rg) < 0.97 * length(p.rg) || (n <= 128 && n * rg <= 1024)) p.rg = rg;
    }
  }
  p.cut = query_cut(n * p.rg, Nk / p.rg, fwd_cut_rule(d));
  if (partials) {
    // two streams at most, as the launch is split over chunks already (four 128-key chunks of 4
    // heads x 512 queries: 8.9 us four ways, 10.2 two ways, 12.3 whole), and only where a chunk, not
    // just its group, has a tile for each: the streams split one chunk after the other
    if (p.cut.ks > 2) p.cut.ks = 2;
    if (Nk / R < 64 * p.cut.ks) p.cut.ks = 1;
  }
  return p;
}

// dQ from stored dS: the key-stream kernel (32 queries per workgroup, one of them to a CU) for slabs
// that leave half of the CUs or more without a group of 128 queries and the others with one group
// to hide its own loads.  Its speed-up over the 128-query kernel, R = 1, by keys:
//   groups x queries     32    128   256   512   1000  2000  4000  8000  16000
//   32 x 128             1.16  1.20  1.31  1.48  1.63  1.80  1.91  1.98  2.04
//   64 x 128             1.13  1.16  1.27  1.40  1.56  1.66  1.79  1.86  2.11
//   128 x 32             0.86  0.93  1.08  1.30  1.44  1.48  2.24  2.30  2.18
//   128 x 64             0.96  1.00  1.12  1.33  1.33  1.47  2.06  2.18  2.05
//   96 x 128             0.71  0.73  0.76  0.83  0.88  0.94  0.97  0.99  1.29
//   128 x 128            0.70  0.72  0.77  0.82  0.89  0.98  1.33  1.33  1.32
// (100 chunks of 20 keys, 128 x 128: 1.27; 192 groups even, 256 groups 0.89.)  So: as long as its
// workgroups fit one round, for more than 64 groups from 256 keys on; in two rounds only where
// the 128-query kernel walks many tiles.
inline bool dq_ds_streams(int64_t nh, int64_t Nq, int64_t Nk, int64_t R) {
  const int64_t groups = nh * ((Nq + 127) / 128), wgs = nh * ((Nq + 31) / 32);
  const int64_t tiles = R * (((Nk + R - 1) / R + 63) / 64);
  if (groups > 128) return false;
  if (wgs <= 256) return groups <= 64 || Nk >= 256;
  return tiles >= 96;
}

// The row-streaming tokenizer kernel on rows of more than 128 cells: one field row in flight instead of
// eight (then with a row's 256-cell segments in neighbouring waves at k = 2, a whole sweep of rows
// apart otherwise).
struct TokRowsForm {
  bool one_row = false;
};
// Measured (us; a kernel that loads with a branch per row / one row, segments near / one row, far /
// eight rows, near; 4 channels; crops that start on a 16-byte boundary, off one, and on one with
// the field's edge inside; 64^2 x 512 and 640 with 2 channels):
//   k = 2   512^3, patch 2     670 769 720    665 739 690    686 763 727    704 751 735
//           1024^3, ratio 2    761 808 815    751 774 715    767 812 819    789 812 748
//   k = 4   512^3              390 468 437    384 391 395    391 433 438    374 382 391
//           1024^3, ratio 2    380 423 424    486 506 433    384 426 429    495 515 422
//           1024^2 x 1536, r 2 615 686 707    592 628 655    615 684 709    590 629 653
//   k = 8   512^3              343 389 383    360 382 363    343 381 384    332 353 350
//           1024^3             2698 3110 3037 2874 2987 2909 2675 3006 3017 2881 2952 3014
//           1024^3, ratio 2    329 368 366    333 357 359    330 368 368    354 381 357
//           64^2 x 640         33 52 33       33 34 34       33 33 33       9 10 9
//   k = 16  512^3              327 432 364    336 367 352    326 359 363    326 348 351
//           1024^3, ratio 2    313 348 348    314 338 340    316 352 351    360 386 341
//   k = 4   1024^3              3002 3703 3453  3103 3234 3127  3048 3573 3469  3152 3394 3185
//   k = 2   64^2 x 512          5.3 6.5 5.1     5.8 5.7 5.4     -               4.9 5.0 4.9
// Small fields take eight rows: they come from caches, and few waves need the loads in flight.
// Large ones take one row at k = 2, whose waves are short; where a crop narrower than its field
// reads whole segments (k = 4: of rows a multiple of 4 KiB apart); at k = 8 for rows of three
// segments or more that start on a boundary; and at k = 4 for whole rows of the largest fields.
inline TokRowsForm tok_rows_form(int64_t k, int64_t rows, int64_t sx, int64_t W, int64_t x0) {
  TokRowsForm f;
  const int64_t cells = rows * k * k * sx;
  if (cells < (int64_t(1) << 27)) return f;
  const bool crop = sx > 256 && sx % 256 == 0 && sx < W;
  if (k == 2) f.one_row = true;
  if (k == 4) f.one_row = (crop && W % 1024 == 0) || (sx == W && x0 == 0 && cells >= int64_t(1) << 31);
  if (k == 8) f.one_row = crop || (sx > 512 && x0 % 4 == 0 && W % 4 == 0);
  if (k == 16) f.one_row = crop;
  return f;
}

struct FwdArgs {
  const void* q = nullptr;
  const void* k = nullptr;
  const void* v = nullptr;
  void* out = nullptr;          // merged output (fused mode)
  float* lse = nullptr;         // merged lse (fused mode)
  float* part_out = nullptr;    // [R,B,H,Nq,d] (partials mode)
  float* part_lse = nullptr;    // [R,B,H,Nq]   (partials mode)
  float* acc_out = nullptr;     // [B,H,Nq,d] running merged output (step mode)
  float* acc_lse = nullptr;     // [B,H,Nq]   running merged lse (step mode)
  bool first = false;           // step mode: the accumulator holds nothing yet
  int64_t BH = 0, Nq = 0, Nk = 0, d = 0, R = 1;
  int64_t H = 1, G = 1;         // query heads per batch; query heads per K/V head (GQA)
  float scale = 1.f;
  hipStream_t stream = nullptr;
};

struct MergeArgs {
  const float* part_out = nullptr;
  const float* part_lse = nullptr;
  void* out = nullptr;
  float* lse = nullptr;
  int64_t R = 1, BH = 0, Nq = 0, d = 0;
  bool out_bf16 = false;
  hipStream_t stream = nullptr;
};

struct BwdArgs {
  const void* q = nullptr;
  const void* k = nullptr;
  const void* v = nullptr;
  const void* out = nullptr;
  const void* dout = nullptr;
  const float* lse = nullptr;
  float* dq = nullptr;
  float* dk = nullptr;
  float* dv = nullptr;
  float* delta = nullptr;       // D_i = dout_i . out_i, [B,H,Nq]
  float* nl = nullptr;          // -lse_i * log2(e), [B,H,Nq] (the exponent's offset, base 2)
  int64_t BH = 0, Nq = 0, Nk = 0, d = 0, R = 1;   // BH = B * H query heads
  int64_t H = 1, G = 1;         // query heads per batch; query heads per K/V head (GQA)
  float scale = 1.f;
  bool accumulate_dkv = false;  // dk, dv += instead of =
  bool accumulate_dq = false;   // dq += instead of =
  char* ds = nullptr;           // store mode of the dK/dV kernel: -dS of every score, bf16
  hipStream_t stream = nullptr;
};

// Stored dS (written by the dK/dV kernel in store mode, read by bwd_dq_ds.hip): per query head j,
// 32-key block kb of the padded key axis (chunk r, 128-key tile t, block w: kb = 4 (r tpc + t) + w,
// nkb = 4 R tpc blocks), 128-query group qg and 32-query block qs of the group, one unit of
// kDsUnitBytes.  The query axis runs fastest, so that each wave of the writer, which owns one key
// block and sweeps the queries, writes one contiguous stream.
constexpr int64_t kDsUnitBytes = 2048;
__host__ __device__ inline int64_t ds_unit_offset(int64_t j, int64_t qg, int64_t kb, int64_t qs,
                                                  int64_t nqg, int64_t nkb) {
  return (((j * nkb + kb) * nqg + qg) * 4 + qs) * kDsUnitBytes;
}
// 128-key tiles per chunk (the longest chunk, ceil(Nk / R) keys, rounded up)
__host__ __device__ inline int64_t ds_tiles_per_chunk(int64_t Nk, int64_t R) {
  return ((Nk + R - 1) / R + 127) / 128;
}
// bytes of stored dS for nh query heads
inline int64_t ds_bytes(int64_t nh, int64_t Nq, int64_t Nk, int64_t R) {
  return nh * ((Nq + 127) / 128) * 4 * R * ds_tiles_per_chunk(Nk, R) * 4 * kDsUnitBytes;
}

struct DsArgs {
  const void* ds = nullptr;     // stored -dS of nh query heads
  const void* k = nullptr;      // K of the nh / G K/V heads, [nh / G, Nk, 128] bf16
  float* dq = nullptr;          // [nh, Nq, 128] fp32, overwritten
  int64_t nh = 0, G = 1, Nq = 0, Nk = 0, R = 1, tpc = 1;
  float scale = 1.f;
  hipStream_t stream = nullptr;
};

// One fidelity mode of the multi-fidelity tokenizer (tt_tokenize.hip).
constexpr int kMaxTokFilter = 32;
struct TokWeights {
  float w[kMaxTokFilter];       // normalised 1D Gaussian weights, w[0 .. k-1]
};
struct TokArgs {
  const float* field = nullptr;  // [C, D, H, W] fp32
  void* tokens = nullptr;        // [L, C p^3], fp32 or bf16
  int64_t C = 0, D = 0, H = 0, W = 0, k = 1, p = 1;
  int64_t gz = 0, gy = 0, gx = 0;   // filtered grid: subdomain size / k
  int64_t z0 = 0, y0 = 0, x0 = 0;   // first subdomain cell, in [0, D) x [0, H) x [0, W)
  TokWeights w{};
  bool out_bf16 = false;
  hipStream_t stream = nullptr;
};

hipError_t launch_fwd_bf16(const FwdArgs& a, FwdMode mode);
hipError_t launch_fwd_f32(const FwdArgs& a, FwdMode mode);
hipError_t launch_lse_merge(const MergeArgs& a);
hipError_t launch_bwd_pre(const BwdArgs& a, bool bf16);
hipError_t launch_bwd_dkdv_bf16(const BwdArgs& a);
hipError_t launch_bwd_dkdv_bf16_d64(const BwdArgs& a);   // d = 64 (bwd_bf16_d64.hip)
hipError_t launch_bwd_dq_bf16(const BwdArgs& a);
// d = 64, and d = 128 where the launch is split into key streams (bwd_dq_bf16_d64.hip)
hipError_t launch_bwd_dq_bf16_two_waves(const BwdArgs& a, const QueryCut& c);
hipError_t launch_bwd_dkdv_f32(const BwdArgs& a);
hipError_t launch_bwd_dq_f32(const BwdArgs& a);
hipError_t launch_bwd_f32(const BwdArgs& a);      // both halves of the fp32 backward
hipError_t launch_bwd_dq_ds(const DsArgs& a);   // d = 128, bf16 dS (bwd_dq_ds.hip)

hipError_t launch_tt_tokenize(const TokArgs& a);

int64_t fwd_bf16_workgroups(int64_t BH, int64_t Nq, int64_t d);

}  // namespace ringx
