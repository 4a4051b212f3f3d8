// api.cpp -- the C entry points: argument checks on the host, workspace
// carving, and the launch sequence of the forward and backward passes.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>

#include "kernels.h"
#include "plan.h"

namespace {

using namespace dsv;

constexpr int64_t kMaxDim = 1 << 20;

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }
bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }
int64_t ld_rank(int32_t r_max) { return (r_max + 7) & ~7; }  // 16-byte rows of rank entries

// Compute units of the current device (0 if the query fails).
int device_cus() {
  static int cached[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0) return 0;
  if (dev < 64 && cached[dev] > 0) return cached[dev];
  int n = 0;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  if (dev < 64) cached[dev] = n;
  return n;
}

// GEMM launch plan: tile shape and work split.  Candidates, costed in
// CU-time (one 128 x 128 x C tile on one CU = 1):
//   128 x 128, two workgroups per CU, whole tiles in whole waves of 2 * CUs;
//   256 x 256 (4 units, at a relative matrix-core efficiency kEff256), one
//     workgroup per CU, whole tiles in whole waves of CUs;
//   the same with the r tiles of a last, partial wave split into
//     s = CUs / r equal K ranges (one workgroup per piece, at least
//     kMinSkIters K-steps each), so that wave takes 1/s of a tile's time,
//     plus kSplitCost64 for the pieces' fp32 partials and the kernel that sums
//     them (relative to a tile of 64 K-steps, so smaller for longer tiles).
//   the same with the r <= CUs / 2 tiles of a last, partial wave run as two
//     halves of 128 rows each, on twice the CUs (no pieces to sum, and the same
//     bits as whole tiles; 6144 x 4096 x 4096, 1.5 waves: 160 us, against 182 with
//     the tiles split in two).  Among the 256 x 256 forms only: the masked
//     low-rank term of the 128 x 128 form keeps a NaN in its own column, that of
//     the 256 x 256 form does not.  Not a forward whose only wave is split in two:
//     about 120 to 146 K-steps by the costs above, over which the split form gains more
//     per K-step than its sum costs (1007 x 9016 x 5880: 131 us, 161 in halves; 69 such
//     calls: halves 9% longer in the mean).  dX keeps halves there: split in two, 58 such dX
//     took 4% longer with W as it is and 4% less transposed, and both must give the same bits.
// The constants were fitted to timings of the Llama-3-8B projections
// (forward and dX) on MI355X.
struct GemmPlan {
  int tm = 128, tn = 128;
  int32_t n_mtiles = 0, n_ntiles = 0;
  int32_t dp_tiles = 0, sk_tiles = 0, sk_split = 0, half_tiles = 0;
};
constexpr int kMinSkIters = 8;
constexpr double kEff256 = 1.12;
constexpr double kSplitCost64 = 0.4;
constexpr double kHalfTile = 0.55;

GemmPlan plan_gemm(int32_t m256, int32_t m128, int32_t n_out, int32_t C, bool fwd, bool allow_split = true) {
  GemmPlan best;
  best.n_mtiles = m128;
  best.n_ntiles = (n_out + 127) / 128;
  best.dp_tiles = best.n_mtiles * best.n_ntiles;
  const int cus = device_cus();
  if (cus <= 0) return best;
  const int64_t t128 = (int64_t)m128 * best.n_ntiles;
  const double cost128 = (double)((t128 + 2 * cus - 1) / (2 * cus)) * 2.0;

  const int64_t n256 = (n_out + 255) / 256, t256 = (int64_t)m256 * n256;
  const int64_t nk = (C + 63) / 64;
  if (t256 <= 0) return best;
  GemmPlan p;
  p.tm = p.tn = 256;
  p.n_mtiles = m256;
  p.n_ntiles = (int32_t)n256;
  p.dp_tiles = (int32_t)t256;
  const int64_t full = t256 / cus, r = t256 % cus;
  double cost256 = (double)(full + (r > 0)) * 4.0 / kEff256;
  const int64_t split = r > 0 ? std::min<int64_t>(cus / r, nk / kMinSkIters) : 0;
  if (allow_split && split >= 2 && ((full * cus) & 7) == 0) {
    const double cost_split =
        ((double)full + 1.0 / (double)split) * 4.0 / kEff256 + kSplitCost64 * 64.0 / (double)nk;
    if (cost_split < cost256) {
      cost256 = cost_split;
      p.dp_tiles = (int32_t)(full * cus);
      p.sk_tiles = (int32_t)r;
      p.sk_split = (int32_t)split;
    }
  }
  if (cost256 >= cost128) return best;
  const bool only_split = fwd && full == 0 && p.sk_split == 2;
  if (r > 0 && 2 * r <= cus && !only_split && ((double)full + kHalfTile) * 4.0 / kEff256 < cost256) {
    p.dp_tiles = (int32_t)(full * cus);
    p.half_tiles = (int32_t)r;
    p.sk_tiles = p.sk_split = 0;
  }
  return p;
}

// GEMM in pieces (launch_part_gemm) for a batch's projections, or the tile kernels
// above.  Of the pieces' forms the one with the smallest cost is taken: rounds of
// workgroups over the CUs times K-steps per piece times the configuration's time per
// step (at least the weights at 5.5 TB/s), plus the fp32 pieces written and read once
// each at 5 TB/s.  Then the pieces are estimated beside the tiles, in microseconds, and
// the smaller one wins.  The constants below were fitted, by the time that wrong choices
// cost either way, to 5902 calls timed both ways on MI355X: single, groups of two and three,
// forward and dX, masked and not, 1 .. 8192 rows, 8 .. 28672 columns, Llama shapes, random
// ones, and tables of decode, prefill and training segments:
//   tiles    kTileStep per K-step and kTileEnd per round of the form (kHalfStep, kHalfEnd
//            for half tiles, forward and dX; a split round and its sum: kSplitSum and the fp32 pieces at
//            5 TB/s more), at least the stream of the weights
//   pieces   kPieceStep per K-step of a piece and kPieceEnd per round, at least the stream
//            of the weights; kPieceElemUs per fp32 element of the pieces; kPieceBase
// Of the calls, those of Llama shapes and serving tables lose 0.3% (single) and 0.3 .. 2.7%
// (grouped) to the best choice of each, the random ones 1% and 2.5 .. 8% (groups of unequal
// projections, whose pieces need that every single call takes pieces or splits its tiles).
//   K = N = 4096, 8 rows: 12 us in pieces, 38 in tiles; two K = 4096, N = 14336, 90 rows: 62
//   and 100; K = 1024, N = 32768, 128 rows: 34 and 23, so tiles
//   kTieUs: a small single call may lose that much by its pieces, so that its group has them
//   kRowsMargin: above 512 rows a forward's pieces must be that much ahead
//   kSideUs: above 2048 rows tiles hide the grouped backward's dA reduction (two K = 1024, N =
//   3072, 3399 rows: 84 us, in pieces 100)
// Narrow outputs take pieces at thousands of rows too (K = 2048, N = 64, 16384 training rows:
// dX 54 us, tiles 73).  There the forward's shrink fills CUs that the pieces want: above 2048
// rows a growing part of its read of X is added to them, from 8192 all of it (K = 8192, N =
// 512, 8192 rows: 114 us, tiles 102), and no forward beyond takes them (K = 4096, N = 256, 32768
// rows: 160 and 135; three K = 4096, N = 64, 16384 rows: 218 and 178); nor dX above the 32768
// rows timed, which keeps the sum's grid of rows within 65535 however many adapters they have.
// A forward's choice depends on the number of rows and the shapes, never on how the
// rows are grouped into segments or whether training rows are masked (the launch that
// gathered rows cost the tiles, about 6 us, and the masked shrink's that pieces need, as
// much, are left out for that): the base product of a row is the same bits in every
// table of as many rows.
struct PartPlan {
  bool use = false;
  int cfg = 0;
  int32_t n_m[kMaxGroup] = {}, n_n[kMaxGroup] = {}, split[kMaxGroup] = {};
  size_t off[kMaxGroup] = {}, bytes = 0;  // the pieces' buffers, past the rest of the workspace
  size_t h_off[kMaxGroup] = {};           // forward: the shrink's pieces
  size_t bytes_any = 0;                   // forward: the most `bytes` of any grouping of the rows
};
constexpr int kMinPartSteps = 4, kFwdPartRows = 8192, kBwdPartRows = 32768;
constexpr double kPartBytesPerUs = 5e6, kWeightBytesPerUs = 5.5e6;
// 128 x 128 tiles with one workgroup per CU, with two, 256 x 256 tiles
constexpr double kTileStep[3] = {0.68, 0.76, 1.37}, kTileEnd[3] = {0.27, 4.53, 5.72}, kTileWeightBytesPerUs[3] = {3.47e6, 5.2e6, 5.05e6};
constexpr double kOneTileBytesPerUs = 0.129e6, kHalfStep[2] = {1.08, 0.9}, kHalfStepRows128 = 1.18, kHalfEnd = 5.23, kSplitSum = 11.2, kSplitBytesPerUs = 5.02e6;
constexpr double kPieceStep[kPartCfgs] = {0.21, 0.47, 0.56, 0.89}, kPieceEnd[kPartCfgs] = {0.01, 0.63, 1.54, 0.42};
constexpr double kPieceWeightBytesPerUs[kPartCfgs] = {6.63e6, 6.5e6, 6.59e6, 4.69e6}, kPieceElemUs = 1.87e-6;
// what the pieces' other launches cost more than the tiles': up to 256 rows, above; forward, dX; single, grouped
constexpr double kPieceBase[2][2][2] = {{{-1.9, -9.5}, {1.3, -10.8}}, {{-2.3, 0.7}, {-0.5, -8.7}}};
constexpr double kShrinkBytesPerUs = 7.16e6, kSideUs = 15.0, kTieUs[2] = {1.5, 5.0}, kRowsMargin = 1.1;

// Time of 256 x 256 tiles at least: the stream of their weights.
double stream256_us(double weight_bytes, double tiles) {
  return weight_bytes / std::min(kTileWeightBytesPerUs[2], kOneTileBytesPerUs * tiles);
}
double half_us(bool fwd, int32_t M, double nk) { return (M <= 128 ? kHalfStepRows128 : kHalfStep[!fwd]) * nk + kHalfEnd; }
double tiles_us(bool fwd, const GemmPlan& g, int32_t M, int32_t Nout, int32_t C) {
  const int64_t cus = device_cus(), nk = (C + 63) / 64;
  if (cus <= 0) return 0.0;  // no device: no launch plan either
  const int form = g.tm == 256 ? 2 : g.dp_tiles <= cus ? 0 : 1;
  const int64_t per = form == 1 ? 2 * cus : cus;
  double t = (double)((g.dp_tiles + per - 1) / per) * (kTileStep[form] * nk + kTileEnd[form]);
  if (g.half_tiles > 0) t += half_us(fwd, M, nk);
  if (g.sk_tiles > 0)
    t += kTileStep[2] * nk / g.sk_split + kSplitSum + (double)g.sk_tiles * g.sk_split * g.tm * g.tn * 8 / kSplitBytesPerUs;
  const double w_bytes = 2.0 * Nout * C;
  return std::max(t, form == 2 ? stream256_us(w_bytes, (double)g.n_mtiles * g.n_ntiles) : w_bytes / kTileWeightBytesPerUs[form]);
}

// p (forward): the plan whose shrink runs beside the pieces.
PartPlan part_plan(const dsv_plan* p, int32_t M, int32_t n, const int32_t* Nout, const int32_t* C, double t_tiles) {
  PartPlan best;
  const int cus = device_cus();
  if (cus <= 0 || M <= 0 || M > (p ? kFwdPartRows : kBwdPartRows)) return best;
  static const int kSplits[] = {1, 2, 3, 4, 5, 6, 8, 10, 12, 16};
  double w_bytes = 0, x_bytes = 0, w_us, piece_us = 0, t_best = HUGE_VAL;
  int32_t nk[kMaxGroup], nk_max = 1;
  for (int i = 0; i < n; ++i) {
    nk[i] = (C[i] + 63) / 64;
    w_bytes += 2.0 * Nout[i] * C[i];
    x_bytes += 2.0 * M * C[i];
    nk_max = std::max(nk_max, nk[i]);
  }
  w_us = w_bytes / kWeightBytesPerUs;
  for (int cfg = 0; cfg < kPartCfgs; ++cfg) {
    const PartCfg& pc = kPartCfg[cfg];
    if (pc.tm < 64 && M > pc.tm) continue;  // the 32-row tile is for batches of one row tile
    const int64_t slots = (int64_t)cus * pc.per_cu;
    int32_t last = 0;
    for (const int s : kSplits) {
      const int32_t t = std::max((nk_max + s - 1) / s, std::min(kMinPartSteps, nk_max));
      if (t == last) break;
      last = t;
      int64_t wgs = 0, elems = 0;
      for (int i = 0; i < n; ++i) {
        const int64_t sp = (nk[i] + t - 1) / t;
        wgs += sp * ((M + pc.tm - 1) / pc.tm) * ((Nout[i] + pc.tn - 1) / pc.tn);
        elems += sp * M * Nout[i];
      }
      if (wgs > INT32_MAX) break;
      const int64_t rounds = (wgs + slots - 1) / slots;
      const double us = std::max((double)(rounds * t) * pc.step_us, w_us) + (double)elems * 8 / kPartBytesPerUs;
      if (us < t_best) {
        t_best = us;
        best.cfg = cfg;
        int32_t steps = 0;
        for (int i = 0; i < n; ++i) {
          best.split[i] = (nk[i] + t - 1) / t;
          steps = std::max(steps, (nk[i] + best.split[i] - 1) / best.split[i]);
        }
        piece_us = std::max(rounds * (kPieceStep[cfg] * steps + kPieceEnd[cfg]), w_bytes / kPieceWeightBytesPerUs[cfg]) +
                   kPieceElemUs * elems;
      }
    }
  }
  if (t_best == HUGE_VAL) return best;
  piece_us += kPieceBase[M > 256][p == nullptr][n > 1];
  if (p) piece_us += std::min(1.0, std::max(0.0, (M - 2048) / 6144.0)) * x_bytes / kShrinkBytesPerUs;
  if (p && M > 512) piece_us *= kRowsMargin;
  if (!p && n > 1 && M > 2048) piece_us += kSideUs;
  best.use = piece_us < t_tiles + (n == 1 && M <= 256 ? kTieUs[p == nullptr] : 0.0);
  if (best.use)
    for (int i = 0; i < n; ++i) {
      best.n_m[i] = (M + kPartCfg[best.cfg].tm - 1) / kPartCfg[best.cfg].tm;
      best.n_n[i] = (Nout[i] + kPartCfg[best.cfg].tn - 1) / kPartCfg[best.cfg].tn;
      best.off[i] = best.bytes;
      const size_t part = align256((size_t)best.split[i] * M * Nout[i] * 4);
      best.bytes += part;
      if (!p) continue;
      int32_t pieces, cpp;
      skinny_split(C[i], p->n_shrink, &pieces, &cpp);
      best.h_off[i] = best.bytes;
      best.bytes += align256((size_t)pieces * M * p->r_max * 4);
      skinny_split(C[i], (M + kRankItemRows - 1) / kRankItemRows, &pieces, &cpp);  // the fewest items: the most pieces
      best.bytes_any += part + align256((size_t)pieces * M * p->r_max * 4);
    }
  return best;
}

struct FwdWs {
  size_t h_all, delta, keep, sk_part, rk_part, total;
};
struct BwdWs {
  size_t g, hrec, part_b, part_a, keep, sk_part, g_part, h_part, total;
};

// Dropout bitmask of the training rows: ceil(K / 32) words per row.
size_t keep_bytes(const dsv_plan& p, int32_t K) { return (size_t)p.T_t * ((K + 31) / 32) * 4; }

// Split-tile scratch of a GEMM plan: one fp32 partial tile per piece.
size_t carve_sk(const GemmPlan& gp, size_t off, size_t* part) {
  *part = off;
  if (gp.sk_tiles <= 0) return off;
  return align256(off + (size_t)gp.sk_tiles * gp.sk_split * gp.tm * gp.tn * 4);
}

FwdWs fwd_ws(const dsv_plan& p, dsv_dtype dt, int32_t K, int32_t N, const GemmPlan& gp) {
  FwdWs w{};
  size_t off = 0;
  if (dt == DSV_BF16) {
    w.h_all = off;
    off = align256(off + (size_t)p.T * ld_rank(p.r_max) * 2);
    w.delta = off;
    off = align256(off + (size_t)p.n_gather * N * 4);
    off = carve_sk(gp, off, &w.sk_part);
    w.rk_part = off;  // pieces of a split shrink
    off = align256(off + skinny_part_bytes(K, p.n_shrink, p.T, p.r_max));
  } else {
    w.h_all = off;
    off = align256(off + (size_t)p.T * p.r_max * 4);
    w.delta = off;
  }
  w.keep = off;  // dropout mask of the training rows
  off = align256(off + keep_bytes(p, K));
  w.total = off;
  return w;
}

BwdWs bwd_ws(const dsv_plan& p, dsv_dtype dt, int32_t K, int32_t N, const GemmPlan& gp) {
  BwdWs w{};
  size_t off = 0;
  if (dt == DSV_BF16) {
    w.g = off;
    off = align256(off + (size_t)p.T_t * ld_rank(p.r_max) * 2);
    w.hrec = off;  // h of the training rows, recomputed when H_save is not kept
    off = align256(off + (size_t)p.T_t * ld_rank(p.r_max) * 2);
    w.part_b = off;
    off = align256(off + (size_t)p.n_chunks * N * p.r_max * 4);
    w.part_a = off;
    off = align256(off + (size_t)p.n_chunks * K * p.r_max * 4);
    off = carve_sk(gp, off, &w.sk_part);
    w.g_part = off;  // g's partials, one per 256-column block of N
    off = align256(off + (size_t)token_col_blocks(N) * p.T_t * p.r_max * 4);
    w.h_part = off;  // pieces of a split recomputed h
    off = align256(off + skinny_part_bytes(K, p.n_shrink, p.T_t, p.r_max));
  } else {
    w.g = off;
    off = align256(off + (size_t)p.T_t * p.r_max * 4);
    w.hrec = off;
    off = align256(off + (size_t)p.T_t * p.r_max * 4);
  }
  w.keep = off;  // dropout mask of the training rows
  off = align256(off + keep_bytes(p, K));
  w.total = off;
  return w;
}

GemmPlan fwd_gemm_plan(const dsv_plan& p, dsv_dtype dt, int32_t K, int32_t N, bool allow_split = true) {
  if (dt != DSV_BF16 || p.T == 0) return GemmPlan{};
  return plan_gemm(p.n_ftiles, p.n_ftiles128, N, K, true, allow_split);
}
GemmPlan bwd_gemm_plan(const dsv_plan& p, dsv_dtype dt, int32_t K, int32_t N) {
  if (dt != DSV_BF16 || p.T_t == 0) return GemmPlan{};
  return plan_gemm(p.n_btiles, p.n_btiles128, K, N, false);
}

// Pieces or tiles of one projection's forward / dX GEMM.
PartPlan fwd_part_plan(const dsv_plan& p, dsv_dtype dt, int32_t K, int32_t N, bool allow_split = true) {
  if (dt != DSV_BF16 || p.T == 0) return PartPlan{};
  return part_plan(&p, p.T, 1, &N, &K, tiles_us(true, fwd_gemm_plan(p, dt, K, N, allow_split), p.T, N, K));
}
PartPlan bwd_part_plan(const dsv_plan& p, dsv_dtype dt, int32_t K, int32_t N) {
  if (dt != DSV_BF16 || p.T_t == 0) return PartPlan{};
  return part_plan(nullptr, p.T_t, 1, &K, &N, tiles_us(false, bwd_gemm_plan(p, dt, K, N), p.T_t, K, N));
}
// ... of a grouped call, whose tiles share one launch of whole 256 x 256 tiles.
// A projection whose single call splits no contraction keeps its whole tiles
// (its grouped result is the single call's, bit for bit).
template <typename Proj, typename ShapeOf>
PartPlan group_part_plan(const dsv_plan& p, int pass, int32_t n, const Proj* pr, ShapeOf shape) {
  const int32_t M = pass == 0 ? p.T : p.T_t, mtiles = pass == 0 ? p.n_ftiles : p.n_btiles;
  const int cus = device_cus();
  if (cus <= 0 || M == 0) return PartPlan{};
  int32_t Nout[DSV_MAX_GROUP], C[DSV_MAX_GROUP];
  double tiles = 0, steps = 0, longest = 0, shortest = HUGE_VAL, long_tiles = 0, w_bytes = 0;
  for (int i = 0; i < n; ++i) {
    shape(pr[i], &Nout[i], &C[i]);
    const double nk = (C[i] + 63) / 64, t = (double)mtiles * ((Nout[i] + 255) / 256);
    if (nk > longest) longest = nk, long_tiles = 0;
    if (nk == longest) long_tiles += t;
    shortest = std::min(shortest, nk);
    tiles += t / cus;
    steps += nk * t / cus;
    w_bytes += 2.0 * Nout[i] * C[i];
  }
  auto round = [](double nk) { return kTileStep[2] * nk + kTileEnd[2]; };
  double whole;
  if (shortest == longest) {  // rounds over the CUs, the last one of halves where they fit
    const double part = tiles - std::floor(tiles);
    whole = (std::floor(tiles) + (part > 0.5 ? 1.0 : 0.0)) * round(longest);
    if (part > 0.0 && part <= 0.5) whole += half_us(pass == 0, M, longest);
  } else {  // the shorter ones fill up behind the longest
    whole = std::max(std::ceil(long_tiles / cus) * round(longest),
                     kTileStep[2] * (steps + 0.5 * shortest) + kTileEnd[2] * (tiles + 0.5));
  }
  whole = std::max(whole, stream256_us(w_bytes, tiles * cus));
  const PartPlan pp = part_plan(pass == 0 ? &p : nullptr, M, n, Nout, C, whole);
  for (int i = 0; pp.use && i < n; ++i)
    if (!(pass == 0 ? fwd_gemm_plan(p, DSV_BF16, pr[i].K, pr[i].N) : bwd_gemm_plan(p, DSV_BF16, pr[i].K, pr[i].N)).sk_tiles &&
        !(pass == 0 ? fwd_part_plan(p, DSV_BF16, pr[i].K, pr[i].N) : bwd_part_plan(p, DSV_BF16, pr[i].K, pr[i].N)).use)
      return PartPlan{};
  return pp;
}
PartPlan fwd_group_part(const dsv_plan& p, dsv_dtype dt, int32_t n, const dsv_fwd_proj* pr) {
  if (dt != DSV_BF16) return PartPlan{};
  return group_part_plan(p, 0, n, pr, [](const dsv_fwd_proj& q, int32_t* o, int32_t* c) { *o = q.N, *c = q.K; });
}
PartPlan bwd_group_part(const dsv_plan& p, dsv_dtype dt, int32_t n, const dsv_bwd_proj* pr) {
  if (dt != DSV_BF16) return PartPlan{};
  return group_part_plan(p, 1, n, pr, [](const dsv_bwd_proj& q, int32_t* o, int32_t* c) { *o = q.K, *c = q.N; });
}

int check_common(const dsv_plan* p, dsv_dtype dt, int32_t K, int32_t N) {
  if (!p) return DSV_ERR_ARG;
  if (dt != DSV_BF16 && dt != DSV_F32) return DSV_ERR_RANGE;
  if (K <= 0 || N <= 0 || (K & 7) || (N & 7) || K > kMaxDim || N > kMaxDim) return DSV_ERR_SIZE;
  return DSV_OK;
}

int ptr_ok(const void* p) { return p && aligned16(p); }

// Row strides (elements) of one projection's caller buffers: X [T][x],
// W [N][w], Y [T][y], dY [T_t][dy], dX [T_t][dx], Wt [K][wt].
struct Strides {
  int64_t x, w, y, dy, dx, wt;
};
Strides dense_strides(int32_t K, int32_t N) { return Strides{K, K, N, N, K, N}; }
// A caller's stride: 0 is the dense row length; any other value must hold a
// row (>= len), keep rows 16-byte aligned (a multiple of 8 elements) and
// stay within the kernels' 32-bit panel offsets (<= kMaxDim).
int row_stride(int32_t given, int32_t len, int64_t* out) {
  if (given == 0) {
    *out = len;
    return DSV_OK;
  }
  if (given < len || (given & 7) || given > kMaxDim) return DSV_ERR_SIZE;
  *out = given;
  return DSV_OK;
}
int fwd_strides(const dsv_fwd_proj& q, Strides* st) {
  *st = dense_strides(q.K, q.N);
  int rc = row_stride(q.ldx, q.K, &st->x);
  if (rc == DSV_OK) rc = row_stride(q.ldw, q.K, &st->w);
  if (rc == DSV_OK) rc = row_stride(q.ldy, q.N, &st->y);
  return rc;
}
int bwd_strides(const dsv_bwd_proj& q, Strides* st) {
  *st = dense_strides(q.K, q.N);
  int rc = row_stride(q.ldx, q.K, &st->x);
  if (rc == DSV_OK) rc = row_stride(q.ldw, q.K, &st->w);
  if (rc == DSV_OK) rc = row_stride(q.lddy, q.N, &st->dy);
  if (rc == DSV_OK) rc = row_stride(q.lddx, q.K, &st->dx);
  if (rc == DSV_OK) rc = row_stride(q.ldwt, q.N, &st->wt);
  return rc;
}

template <typename T>
T* at(void* base, size_t off) {
  return reinterpret_cast<T*>(static_cast<char*>(base) + off);
}

void set_split(GemmArgs& g, const GemmPlan& gp, void* ws, size_t part_off) {
  g.n_mtiles = gp.n_mtiles;
  g.n_ntiles = gp.n_ntiles;
  g.dp_tiles = gp.dp_tiles;
  g.sk_tiles = gp.sk_tiles;
  g.sk_split = gp.sk_split;
  g.half_tiles = gp.half_tiles;
  g.sk_part = gp.sk_tiles > 0 ? at<float>(ws, part_off) : nullptr;
}

// Benchmark timing of the GEMM launches (dsv_timing_enable / dsv_timing_read).
struct Timing {
  static constexpr int kMaxPairs = 4096;
  bool on = false;
  int n = 0;
  hipEvent_t ev[kMaxPairs][2] = {};
  int kind[kMaxPairs] = {};  // 0 forward GEMM, 1 dX GEMM
};
Timing g_timing;

// Hands the events of a timed launch to the next GEMM launch (they are
// recorded within its kernels' dispatches); returns the pair index or -1.
int timing_begin(int kind, hipStream_t s) {
  (void)s;
  Timing& t = g_timing;
  if (!t.on || t.n >= Timing::kMaxPairs) return -1;
  const int i = t.n;
  for (int k = 0; k < 2; ++k)
    if (!t.ev[i][k] && hipEventCreate(&t.ev[i][k]) != hipSuccess) return -1;
  set_launch_events(t.ev[i][0], t.ev[i][1]);
  t.kind[i] = kind;
  t.n = i + 1;
  return i;
}

// A pair whose launch launched nothing (or failed before its last kernel) is
// dropped: its events were never recorded.
void timing_end(int i, hipStream_t s) {
  (void)s;
  if (i < 0 || !launch_events_pending()) return;
  set_launch_events(nullptr, nullptr);
  if (i == g_timing.n - 1) g_timing.n = i;
}

}  // namespace

extern "C" int dsv_timing_enable(int32_t on) {
  g_timing.on = on != 0;
  return DSV_OK;
}

extern "C" int dsv_timing_read(double* fwd_ms, int32_t* fwd_n, double* bwd_ms, int32_t* bwd_n) {
  double ms[2] = {0.0, 0.0};
  int32_t cnt[2] = {0, 0};
  int rc = DSV_OK;
  for (int i = 0; i < g_timing.n; ++i) {
    float e = 0.f;
    if (hipEventSynchronize(g_timing.ev[i][1]) != hipSuccess ||
        hipEventElapsedTime(&e, g_timing.ev[i][0], g_timing.ev[i][1]) != hipSuccess) {
      rc = DSV_ERR_DEVICE;
      continue;
    }
    ms[g_timing.kind[i]] += e;
    cnt[g_timing.kind[i]] += 1;
  }
  g_timing.n = 0;
  if (fwd_ms) *fwd_ms = ms[0];
  if (fwd_n) *fwd_n = cnt[0];
  if (bwd_ms) *bwd_ms = ms[1];
  if (bwd_n) *bwd_n = cnt[1];
  return rc;
}

namespace {

// AdamW of up to DSV_MAX_GROUP projections in one launch (dsv_adamw_step is a
// group of one): validation first, nothing launched on any error.
int adamw_impl(const dsv_plan* p, dsv_dtype dt, int32_t n, const dsv_adamw_proj* projs, int32_t step,
               const dsv_adamw_hparams* hp, hipStream_t stream) {
  if (!p) return DSV_ERR_ARG;
  if (n < 1 || n > DSV_MAX_GROUP) return DSV_ERR_RANGE;
  if (!projs) return DSV_ERR_ARG;
  for (int32_t i = 0; i < n; ++i) {
    const int rc = check_common(p, dt, projs[i].K, projs[i].N);
    if (rc != DSV_OK) return rc;
  }
  if (!p->d_meta || !hp) return DSV_ERR_ARG;
  if (step < 1 || !std::isfinite(hp->lr) || hp->lr < 0.0 || !std::isfinite(hp->weight_decay) ||
      hp->weight_decay < 0.0 || !(hp->beta1 >= 0.0 && hp->beta1 < 1.0) ||
      !(hp->beta2 >= 0.0 && hp->beta2 < 1.0) || !(hp->eps > 0.0) || !std::isfinite(hp->eps))
    return DSV_ERR_RANGE;
  for (int32_t i = 0; i < n; ++i) {
    const dsv_adamw_proj& q = projs[i];
    if (!ptr_ok(q.dA) || !ptr_ok(q.dB) || !ptr_ok(q.A_master) || !ptr_ok(q.B_master) || !ptr_ok(q.A_m) ||
        !ptr_ok(q.A_v) || !ptr_ok(q.B_m) || !ptr_ok(q.B_v) || (q.A && !aligned16(q.A)) ||
        (q.B && !aligned16(q.B)))
      return DSV_ERR_ARG;
  }
  if (p->n_tads == 0) return DSV_OK;
  AdamWArgs a{};
  a.r_max = p->r_max;
  a.n_proj = n;
  a.bf16 = dt == DSV_BF16;
  a.train_ads = p->dptr(p->lay.train_ads);
  a.ranks = p->dptr(p->lay.ranks);
  // B in float4 units when every training rank and the rank stride are multiples of 4
  bool bvec = (p->r_max & 3) == 0;
  for (int32_t s = 0; s < p->n_tads; ++s) bvec = bvec && (p->ranks[p->meta[p->lay.train_ads + s]] & 3) == 0;
  a.bvec = bvec ? 1 : 0;
  // factors formed in double on the host, rounded once to fp32
  const double bc1 = 1.0 - std::pow(hp->beta1, (double)step);
  const double bc2 = 1.0 - std::pow(hp->beta2, (double)step);
  a.decay = (float)(1.0 - hp->lr * hp->weight_decay);
  a.b1 = (float)hp->beta1;
  a.b2 = (float)hp->beta2;
  a.c1 = (float)(1.0 - hp->beta1);
  a.c2 = (float)(1.0 - hp->beta2);
  a.eps = (float)hp->eps;
  a.step_size = (float)(hp->lr / bc1);
  a.sqrt_bc2 = (float)std::sqrt(bc2);
  int64_t blocks = 0;
  for (int32_t i = 0; i < n; ++i) {
    const dsv_adamw_proj& q = projs[i];
    // units of the largest training rank; smaller ranks leave threads idle
    const int64_t r = p->r_train;
    const int64_t units = r * q.K / 4 + (bvec ? (int64_t)q.N * r / 4 : (int64_t)q.N * r);
    const int64_t bpa = (units + 255) / 256;
    if (bpa * 256 > INT32_MAX) return DSV_ERR_SIZE;  // the kernel indexes units in 32 bits
    AdamWProj& d = a.proj[i];
    d.K = q.K;
    d.N = q.N;
    d.blk_begin = (int32_t)blocks;
    d.bpa = (int32_t)bpa;
    d.dA = q.dA;
    d.dB = q.dB;
    d.pA = q.A_master;
    d.pB = q.B_master;
    d.mA = q.A_m;
    d.vA = q.A_v;
    d.mB = q.B_m;
    d.vB = q.B_v;
    d.A = q.A;
    d.B = q.B;
    blocks += bpa * p->n_tads;
    if (blocks > INT32_MAX) return DSV_ERR_SIZE;
  }
  return launch_adamw(a, blocks, stream) == hipSuccess ? DSV_OK : DSV_ERR_DEVICE;
}

}  // namespace

extern "C" int dsv_adamw_step(const dsv_plan* p, dsv_dtype dt, int32_t K, int32_t N, int32_t step,
                              const dsv_adamw_hparams* hp, const float* dA, const float* dB, float* A_master,
                              float* B_master, float* A_m, float* A_v, float* B_m, float* B_v, void* A,
                              void* B, void* hip_stream) {
  const dsv_adamw_proj one{K, N, dA, dB, A_master, B_master, A_m, A_v, B_m, B_v, A, B};
  return adamw_impl(p, dt, 1, &one, step, hp, static_cast<hipStream_t>(hip_stream));
}

extern "C" int dsv_adamw_step_grouped(const dsv_plan* p, dsv_dtype dt, int32_t n_proj,
                                      const dsv_adamw_proj* projs, int32_t step, const dsv_adamw_hparams* hp,
                                      void* hip_stream) {
  return adamw_impl(p, dt, n_proj, projs, step, hp, static_cast<hipStream_t>(hip_stream));
}

extern "C" int dsv_gemm_config(const dsv_plan* p, dsv_dtype dt, int32_t K, int32_t N, int32_t pass,
                               int32_t out[6]) {
  int rc = check_common(p, dt, K, N);
  if (rc != DSV_OK) return rc;
  if (!out || (pass != 0 && pass != 1)) return DSV_ERR_ARG;
  for (int i = 0; i < 6; ++i) out[i] = 0;
  if (dt != DSV_BF16 || (pass == 0 ? p->T : p->T_t) == 0) return DSV_OK;
  const PartPlan pp = pass == 0 ? fwd_part_plan(*p, dt, K, N) : bwd_part_plan(*p, dt, K, N);
  if (pp.use) {
    out[0] = kPartCfg[pp.cfg].tm;
    out[1] = kPartCfg[pp.cfg].tn;
    out[2] = pp.n_m[0];
    out[3] = pp.n_n[0];
    out[4] = pp.n_m[0] * pp.n_n[0];
    out[5] = pp.split[0];
    return DSV_OK;
  }
  const GemmPlan gp = pass == 0 ? fwd_gemm_plan(*p, dt, K, N) : bwd_gemm_plan(*p, dt, K, N);
  out[0] = gp.tm;
  out[1] = gp.tn;
  out[2] = gp.n_mtiles;
  out[3] = gp.n_ntiles;
  out[4] = gp.sk_tiles;
  out[5] = gp.sk_split;
  return DSV_OK;
}

extern "C" int dsv_cobatch_fwd_workspace(const dsv_plan* p, dsv_dtype dt, int32_t K, int32_t N,
                                         size_t* bytes) {
  int rc = check_common(p, dt, K, N);
  if (rc != DSV_OK) return rc;
  if (!bytes) return DSV_ERR_ARG;
  *bytes = fwd_ws(*p, dt, K, N, fwd_gemm_plan(*p, dt, K, N)).total + fwd_part_plan(*p, dt, K, N).bytes;
  return DSV_OK;
}

extern "C" int dsv_lora_bwd_workspace(const dsv_plan* p, dsv_dtype dt, int32_t K, int32_t N,
                                      size_t* bytes) {
  int rc = check_common(p, dt, K, N);
  if (rc != DSV_OK) return rc;
  if (!bytes) return DSV_ERR_ARG;
  *bytes = bwd_ws(*p, dt, K, N, bwd_gemm_plan(*p, dt, K, N)).total + bwd_part_plan(*p, dt, K, N).bytes;
  return DSV_OK;
}

extern "C" int dsv_lora_bwd_dropout_workspace(const dsv_plan* p, dsv_dtype dt, int32_t K, int32_t N,
                                              size_t* bytes) {
  int rc = check_common(p, dt, K, N);
  if (rc != DSV_OK) return rc;
  if (!bytes) return DSV_ERR_ARG;
  *bytes = bwd_ws(*p, dt, K, N, bwd_gemm_plan(*p, dt, K, N)).total + bwd_part_plan(*p, dt, K, N).bytes;
  return DSV_OK;
}

namespace {

// Dropout parameters -> mask spec; false when they are out of range.
bool dropout_spec(const dsv_dropout* d, DropoutSpec* out) {
  if (!d || !std::isfinite(d->p) || d->p < 0.0 || d->p >= 1.0) return false;
  const double t = std::floor(d->p * 4294967296.0);
  out->thr = t >= 4294967295.0 ? 0xFFFFFFFFu : (uint32_t)t;
  out->scale = (float)(1.0 / (1.0 - d->p));
  out->seed = d->seed;
  out->offset = d->offset;
  return true;
}

// The caller's mask buffer must hold 32-bit words.
bool mask_aligned(const dsv_dropout* d) { return !d || !d->mask || (reinterpret_cast<uintptr_t>(d->mask) & 3) == 0; }

// Where a projection's mask lives: the caller's buffer, else the workspace.
uint32_t* mask_buffer(const dsv_dropout* d, void* ws_keep) {
  return d && d->mask ? d->mask : static_cast<uint32_t*>(ws_keep);
}

// The sum of the pieces over the forward's items / the backward's.
FinishGroup fwd_finish(const dsv_plan& p) {
  FinishGroup f{};
  f.row_train = p.dptr(p.lay.row_train);
  f.r_max = p.r_max;
  f.items = p.dptr(p.lay.shrink_items);
  f.rows = p.dptr(p.lay.shrink_rows);
  f.ranks = p.dptr(p.lay.ranks);
  f.scales = reinterpret_cast<const float*>(p.dptr(p.lay.scales));
  return f;
}
FinishGroup bwd_finish(const dsv_plan& p) {
  FinishGroup f{};
  f.r_max = p.r_max;
  f.items = p.dptr(p.lay.train_items);
  f.ranks = p.dptr(p.lay.ranks);
  return f;
}
// Appends projection i of the plan to the launch of the pieces and to their sum.
void add_part(PartGroup& pg, FinishGroup& fg, const PartPlan& pp, int i, PartArgs a, char* parts, const uint16_t* L,
              int64_t ldl, const void* Q, void* out, int64_t ldo, const uint32_t* keep, int32_t keep_words,
              float keep_scale) {
  a.n_m = pp.n_m[i];
  a.n_n = pp.n_n[i];
  a.split = pp.split[i];
  a.part = reinterpret_cast<float*>(parts + pp.off[i]);
  pg.a[pg.n] = a;
  pg.off[pg.n + 1] = pg.off[pg.n] + a.n_m * a.n_n * a.split;
  ++pg.n;
  fg.a[fg.n++] = FinishArgs{a.part, a.split, a.M, a.Nout, L, ldl, nullptr, 0, nullptr, static_cast<const uint16_t*>(Q),
                            static_cast<uint16_t*>(out), ldo, keep, keep_words, keep_scale, 1};
}
// Puts the shrink of the last appended projection (i of the plan) beside its
// pieces; its h then reaches the sum as pieces.
void add_part_shrink(const dsv_plan& p, PartGroup& pg, FinishGroup& fg, const PartPlan& pp, int i, const void* A,
                     char* parts, void* H_save) {
  const PartArgs& a = pg.a[pg.n - 1];
  PartShrink& h = pg.sh[pg.n - 1];
  h.X = a.P;
  h.ldx = a.ldp;
  h.A = static_cast<const uint16_t*>(A);
  h.C = a.C;
  h.part = reinterpret_cast<float*>(parts + pp.h_off[i]);
  skinny_split(a.C, p.n_shrink, &h.pieces, &h.cpp);
  pg.sh_off[pg.n] = pg.sh_off[pg.n - 1] + p.n_shrink * h.pieces;
  pg.items = p.dptr(p.lay.shrink_items);
  pg.rows = p.dptr(p.lay.shrink_rows);
  pg.ranks = p.dptr(p.lay.ranks);
  pg.n_items = p.n_shrink;
  pg.T = p.T;
  pg.r_max = p.r_max;
  FinishArgs& f = fg.a[fg.n - 1];
  f.h_part = h.part;
  f.h_pieces = h.pieces;
  f.h_save = p.T_t > 0 ? static_cast<uint16_t*>(H_save) : nullptr;
}

// noalloc: the allocation-free form (dsv_cobatch_fwd_noalloc): the workspace is
// the library's device scratch, the GEMM plan splits no 256 x 256 tile along the
// contraction (a split needs a partial tile per piece, tens of MB; batches of few
// rows run in pieces where those fit), and no benchmark timing events are created.
int fwd_impl(const dsv_plan* p, dsv_dtype dt, int32_t K, int32_t N, const void* X, const void* W, const void* A,
             const void* B, void* Y, void* H_save, const dsv_dropout* drop, void* workspace,
             size_t workspace_bytes, void* hip_stream, const Strides* lds = nullptr, bool noalloc = false) {
  int rc = check_common(p, dt, K, N);
  if (rc != DSV_OK) return rc;
  const Strides ld = lds ? *lds : dense_strides(K, N);
  DropoutSpec ds{};
  if (drop && !dropout_spec(drop, &ds)) return DSV_ERR_RANGE;
  if (!mask_aligned(drop)) return DSV_ERR_ARG;
  const bool dropping = drop && drop->p > 0.0 && p->T_t > 0;
  if (!p->d_meta) return DSV_ERR_ARG;
  if (p->T == 0) return DSV_OK;  // empty batch: nothing to read or write
  if (!ptr_ok(X) || !ptr_ok(W) || !ptr_ok(A) || !ptr_ok(B) || !ptr_ok(Y)) return DSV_ERR_ARG;
  if (H_save && !aligned16(H_save)) return DSV_ERR_ARG;
  const GemmPlan gp = fwd_gemm_plan(*p, dt, K, N, !noalloc);
  const FwdWs ws = fwd_ws(*p, dt, K, N, gp);
  if (ws.total > 0) {
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255)) return DSV_ERR_ARG;
    if (workspace_bytes < ws.total) return DSV_ERR_SIZE;
  }
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  const MetaLayout& L = p->lay;
  const int32_t* ranks = p->dptr(L.ranks);
  const float* scales = reinterpret_cast<const float*>(p->dptr(L.scales));
  hipError_t e = hipSuccess;

  // 0. dropout mask of the training rows' adapter input (into the caller's
  //    buffer when one is given, for the backward to read).
  uint32_t* keep_w = dropping ? mask_buffer(drop, at<uint32_t>(workspace, ws.keep)) : nullptr;
  const uint32_t* keep = keep_w;
  const int32_t keep_words = (K + 31) / 32;
  if (dropping && (e = launch_dropout_mask(keep_w, p->T_t, K, ds, s)) != hipSuccess) return DSV_ERR_DEVICE;

  if (dt == DSV_F32) {
    F32Args a{};
    a.T = p->T;
    a.Tt = p->T_t;
    a.K = K;
    a.N = N;
    a.r_max = p->r_max;
    a.keep = keep;
    a.keep_words = keep_words;
    a.drop_scale = ds.scale;
    a.row_adapter = p->dptr(L.row_adapter);
    a.row_train = p->dptr(L.row_train);
    a.shrink_items = p->dptr(L.shrink_items);
    a.shrink_rows = p->dptr(L.shrink_rows);
    a.n_shrink = p->n_shrink;
    a.r_used = p->r_used;
    a.ranks = ranks;
    a.scales = scales;
    a.X = static_cast<const float*>(X);
    a.W = static_cast<const float*>(W);
    a.A = static_cast<const float*>(A);
    a.B = static_cast<const float*>(B);
    a.Y = static_cast<float*>(Y);
    a.ldx = ld.x;
    a.ldw = ld.w;
    a.ldy = ld.y;
    a.Hsave = p->T_t > 0 ? static_cast<float*>(H_save) : nullptr;
    a.Hall = at<float>(workspace, ws.h_all);
    e = launch_f32_fwd(a, s);
    return e == hipSuccess ? DSV_OK : DSV_ERR_DEVICE;
  }

  const int64_t ldh = ld_rank(p->r_max);
  uint16_t* h_all = at<uint16_t>(workspace, ws.h_all);
  float* delta = p->n_gather > 0 ? at<float>(workspace, ws.delta) : nullptr;

  // 1. shrink: h of every row, grouped by adapter.
  SkinnyArgs sk{};
  sk.P = static_cast<const uint16_t*>(X);
  sk.ldp = ld.x;
  sk.rows = p->dptr(L.shrink_rows);
  sk.items = p->dptr(L.shrink_items);
  sk.Q = static_cast<const uint16_t*>(A);
  sk.q_ad = (int64_t)p->r_max * K;
  sk.ldq = K;
  sk.qsel = nullptr;
  sk.ranks = ranks;
  sk.scales = nullptr;
  sk.C = K;
  sk.out1 = h_all;
  sk.ld1 = ldh;
  sk.out2 = p->T_t > 0 ? static_cast<uint16_t*>(H_save) : nullptr;
  sk.ld2 = p->r_max;
  sk.row_train = p->dptr(L.row_train);
  sk.keep = keep;
  sk.keep_words = keep_words;
  sk.drop_scale = ds.scale;
  sk.part = at<float>(workspace, ws.rk_part);
  sk.part_n = p->T;
  sk.r_max = p->r_max;
  sk.split_items = p->n_shrink;
  // 1a. few rows: the base product in pieces, the shrink beside them (a launch of
  //     its own where dropout masks it), then their sum with the low-rank term of
  //     every row.  A workspace without room for the pieces takes the tiles.  The
  //     fixed scratch of the allocation-free form has room or not for any grouping of
  //     the rows alike: its pieces need none of the other regions (no dropout there).
  const PartPlan pp = fwd_part_plan(*p, dt, K, N, !noalloc);
  char* parts = at<char>(workspace, noalloc ? 0 : ws.total);
  if (pp.use && (noalloc ? workspace_bytes >= pp.bytes_any : workspace_bytes - ws.total >= pp.bytes)) {
    if (keep && launch_shrink(sk, p->n_shrink, p->r_used, s) != hipSuccess) return DSV_ERR_DEVICE;
    PartGroup pg{};
    FinishGroup fg = fwd_finish(*p);
    add_part(pg, fg, pp, 0, PartArgs{static_cast<const uint16_t*>(X), ld.x, static_cast<const uint16_t*>(W), ld.w, p->T, N, K},
             parts, h_all, ldh, B, Y, ld.y, nullptr, 0, 1.f);
    if (!keep) add_part_shrink(*p, pg, fg, pp, 0, A, parts, H_save);
    const int tk = noalloc ? -1 : timing_begin(0, s);
    e = launch_part_gemm(pg, pp.cfg, p->r_used, false, s);
    if (e == hipSuccess) e = launch_part_finish(fg, p->n_shrink, p->r_used, false, s);
    timing_end(tk, s);
    return e == hipSuccess ? DSV_OK : DSV_ERR_DEVICE;
  }
  if ((e = launch_shrink(sk, p->n_shrink, p->r_used, s)) != hipSuccess) return DSV_ERR_DEVICE;

  // 2. gathered rows: fp32 low-rank term, each touched adapter read once.
  if (p->n_gather > 0) {
    e = launch_gather_expand(h_all, ldh, static_cast<const uint16_t*>(B), N, p->r_max,
                             p->dptr(L.gather_items), p->n_gitems, p->dptr(L.gather_rows), ranks,
                             scales, delta, s);
    if (e != hipSuccess) return DSV_ERR_DEVICE;
  }

  // 3. base GEMM with the low-rank prologue, one rounding.
  GemmArgs g{};
  g.P = static_cast<const uint16_t*>(X);
  g.ldp = ld.x;
  g.Q = static_cast<const uint16_t*>(W);
  g.ldq = ld.w;
  g.out = static_cast<uint16_t*>(Y);
  g.ldo = ld.y;
  g.M = p->T;
  g.Nout = N;
  g.C = K;
  g.tiles = p->dptr(gp.tm == 256 ? L.fwd_tiles : L.fwd_tiles128);
  g.uniform_rows = gp.tm == 256;
  set_split(g, gp, workspace, ws.sk_part);
  g.Lp = h_all;
  g.ldl = ldh;
  g.Lq = static_cast<const uint16_t*>(B);
  g.lq_ad = (int64_t)N * p->r_max;
  g.lq_j = 1;
  g.lq_col = p->r_max;
  g.ranks = ranks;
  g.scales = scales;
  g.delta = delta;
  g.gslot = p->dptr(L.gslot);
  const int tk = noalloc ? -1 : timing_begin(0, s);
  e = launch_gemm_nt(g, gp.tm, gp.tn, s);
  timing_end(tk, s);
  if (e != hipSuccess) return DSV_ERR_DEVICE;
  return DSV_OK;
}

// Wt (optional, bf16): the frozen weight transposed, [K][N]; the dX GEMM then
// reads it K-contiguous like the forward's W instead of transposing W on the fly.
// A second stream of the current device (default priority, non-blocking)
// and two events, created on first use: the grouped bf16 backward runs its
// dA reductions and final sums there, beside the dX GEMMs on the caller's
// stream, which need neither.  The fork and join are enqueued under a lock, so calls
// from several host threads do not interleave on the shared events; the side
// work of successive calls queues up on the one side stream.
struct SideStream {
  hipStream_t s = nullptr;
  hipEvent_t fork = nullptr, join = nullptr;
};
std::mutex g_side_mu;
SideStream g_side[64];

// The current device's side stream (created if needed), or nullptr.
SideStream* side_stream() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
  SideStream& sd = g_side[dev];
  if (!sd.s) {
    hipStream_t st = nullptr;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (hipStreamCreateWithFlags(&st, hipStreamNonBlocking) != hipSuccess) return nullptr;
    if (hipEventCreateWithFlags(&e0, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&e1, hipEventDisableTiming) != hipSuccess) {
      if (e0) (void)hipEventDestroy(e0);
      (void)hipStreamDestroy(st);
      return nullptr;
    }
    sd.fork = e0;
    sd.join = e1;
    sd.s = st;
  }
  return &sd;
}

int bwd_impl(const dsv_plan* p, dsv_dtype dt, int32_t K, int32_t N, const void* X, const void* W, const void* A,
             const void* B, const void* H_save, const void* dY, float* dA, float* dB, void* dX,
             int32_t accumulate, const dsv_dropout* drop, const void* Wt, void* workspace,
             size_t workspace_bytes, void* hip_stream, const Strides* lds = nullptr) {
  int rc = check_common(p, dt, K, N);
  if (rc != DSV_OK) return rc;
  const Strides ld = lds ? *lds : dense_strides(K, N);
  DropoutSpec ds{};
  if (drop && !dropout_spec(drop, &ds)) return DSV_ERR_RANGE;
  if (!mask_aligned(drop)) return DSV_ERR_ARG;
  const bool dropping = drop && drop->p > 0.0;
  if (accumulate != 0 && accumulate != 1) return DSV_ERR_RANGE;
  if (!p->d_meta) return DSV_ERR_ARG;
  if (p->T_t == 0) return DSV_OK;  // no training rows: nothing to read or write
  if (!ptr_ok(X) || !ptr_ok(W) || !ptr_ok(A) || !ptr_ok(B) || !ptr_ok(dA) || !ptr_ok(dB))
    return DSV_ERR_ARG;
  if (dX && !aligned16(dX)) return DSV_ERR_ARG;
  if (!ptr_ok(dY) || (H_save && !aligned16(H_save)) || (Wt && !aligned16(Wt))) return DSV_ERR_ARG;
  const GemmPlan gp = bwd_gemm_plan(*p, dt, K, N);
  const BwdWs ws = bwd_ws(*p, dt, K, N, gp);
  if (ws.total > 0) {
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255)) return DSV_ERR_ARG;
    if (workspace_bytes < ws.total) return DSV_ERR_SIZE;
  }
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  const MetaLayout& L = p->lay;
  const int32_t* ranks = p->dptr(L.ranks);
  const float* scales = reinterpret_cast<const float*>(p->dptr(L.scales));
  hipError_t e = hipSuccess;

  // 0. the forward's dropout mask: the caller's buffer, or regenerated from
  //    the same seed and offset.
  uint32_t* keep = dropping ? mask_buffer(drop, at<uint32_t>(workspace, ws.keep)) : nullptr;
  const int32_t keep_words = (K + 31) / 32;
  if (dropping && !drop->mask && (e = launch_dropout_mask(keep, p->T_t, K, ds, s)) != hipSuccess)
    return DSV_ERR_DEVICE;

  if (dt == DSV_F32) {
    F32Args a{};
    a.T = p->T;
    a.Tt = p->T_t;
    a.K = K;
    a.N = N;
    a.r_max = p->r_max;
    a.keep = keep;
    a.keep_words = keep_words;
    a.drop_scale = ds.scale;
    a.train_rows = p->dptr(L.train_rows);
    a.train_adapter = p->dptr(L.train_adapter);
    a.train_ads = p->dptr(L.train_ads);
    a.n_tads = p->n_tads;
    a.tad_ptr = p->dptr(L.tad_chunk_ptr);
    a.tad_chunks = p->dptr(L.tad_chunks);
    a.chunks = p->dptr(L.chunks);
    a.train_items = p->dptr(L.train_items);
    a.n_titems = p->n_titems;
    a.r_train = p->r_train;
    a.ranks = ranks;
    a.scales = scales;
    a.X = static_cast<const float*>(X);
    a.W = static_cast<const float*>(W);
    a.A = static_cast<const float*>(A);
    a.B = static_cast<const float*>(B);
    a.Hs = static_cast<const float*>(H_save);
    a.Hrec = at<float>(workspace, ws.hrec);
    a.dY = static_cast<const float*>(dY);
    a.G = at<float>(workspace, ws.g);
    a.dA = dA;
    a.dB = dB;
    a.dX = static_cast<float*>(dX);
    a.ldx = ld.x;
    a.ldw = ld.w;
    a.lddy = ld.dy;
    a.lddx = ld.dx;
    a.accumulate = accumulate;
    e = launch_f32_bwd(a, s);
    return e == hipSuccess ? DSV_OK : DSV_ERR_DEVICE;
  }

  const int64_t ldh = ld_rank(p->r_max);
  uint16_t* gm = at<uint16_t>(workspace, ws.g);
  float* part_b = at<float>(workspace, ws.part_b);
  float* part_a = at<float>(workspace, ws.part_a);
  const int32_t* train_ads = p->dptr(L.train_ads);

  // 1. H_save not kept (residual-only retention): recompute h of the training
  //    rows from X with the forward's shrink (same values, bit for bit).
  const uint16_t* hs = static_cast<const uint16_t*>(H_save);
  int64_t ldhs = p->r_max;
  if (!hs) {
    uint16_t* hrec = at<uint16_t>(workspace, ws.hrec);
    SkinnyArgs sh{};
    sh.P = static_cast<const uint16_t*>(X);
    sh.ldp = ld.x;
    sh.rows = p->dptr(L.train_rows);
    sh.items = p->dptr(L.train_items);
    sh.Q = static_cast<const uint16_t*>(A);
    sh.q_ad = (int64_t)p->r_max * K;
    sh.ldq = K;
    sh.qsel = nullptr;
    sh.ranks = ranks;
    sh.scales = nullptr;
    sh.C = K;
    sh.out1 = nullptr;
    sh.out2 = hrec;
    sh.ld2 = ldh;
    sh.row_train = p->dptr(L.row_train);
    sh.keep = keep;
    sh.keep_words = keep_words;
    sh.drop_scale = ds.scale;
    sh.part = at<float>(workspace, ws.h_part);
    sh.part_n = p->T_t;
    sh.r_max = p->r_max;
    sh.split_items = p->n_shrink;  // the forward shrink's split: the same sums
    if ((e = launch_shrink_train(sh, p->n_titems, p->r_train, s)) != hipSuccess) return DSV_ERR_DEVICE;
    hs = hrec;
    ldhs = ldh;
  }

  // 2. per-chunk fp32 partials of dy^T h (-> dB); the same pass writes the
  //    per-column-block partials of dy B_a (-> g), reading dy once.
  TokenReduceGroup tb{};
  tb.n = 1;
  TokenReduceArgs& rb = tb.a[0];
  rb.P = static_cast<const uint16_t*>(dY);
  rb.ldp = ld.dy;
  rb.prow = nullptr;
  rb.Q = hs;
  rb.ldq = ldhs;
  rb.chunks = p->dptr(L.chunks);
  rb.ranks = ranks;
  rb.C = N;
  rb.r_max = p->r_max;
  rb.part = part_b;
  rb.B = static_cast<const uint16_t*>(B);
  rb.gpart = at<float>(workspace, ws.g_part);
  rb.gpart_n = p->T_t;
  tb.yoff[1] = token_col_blocks(N);
  if ((e = launch_token_reduce_group(tb, p->n_chunks, p->r_train, s)) != hipSuccess) return DSV_ERR_DEVICE;

  // 3. g = s_a dy B_a: the block partials summed in order, rounded once -> G [T_t][ldh]
  SkinnyGroup gf{};
  gf.n = 1;
  SkinnyArgs& sk = gf.a[0];
  sk.items = p->dptr(L.train_items);
  sk.ranks = ranks;
  sk.scales = scales;
  sk.out1 = gm;
  sk.ld1 = ldh;
  sk.part = rb.gpart;
  sk.part_n = p->T_t;
  sk.r_max = p->r_max;
  sk.pieces = token_col_blocks(N);
  if ((e = launch_g_finish_group(gf, p->n_titems, s)) != hipSuccess) return DSV_ERR_DEVICE;

  // 4. per-chunk fp32 partials of x^T g (-> dA)
  TokenReduceGroup ta{};
  ta.n = 1;
  TokenReduceArgs& ra = ta.a[0];
  ra.P = static_cast<const uint16_t*>(X);
  ra.ldp = ld.x;
  ra.prow = p->dptr(L.train_rows);
  ra.Q = gm;
  ra.ldq = ldh;
  ra.chunks = p->dptr(L.chunks);
  ra.ranks = ranks;
  ra.C = K;
  ra.r_max = p->r_max;
  ra.part = part_a;
  ra.keep = keep;  // dA contracts the masked input
  ra.keep_words = keep_words;
  ta.yoff[1] = token_col_blocks(K);

  // 5. fixed-order sums into dB (scaled by s_a) and dA.
  const int32_t* tad_ptr = p->dptr(L.tad_chunk_ptr);
  const int32_t* tad_chunks = p->dptr(L.tad_chunks);
  const ReduceOutArgs ob{part_b, N, scales, 0, dB, 1.f};
  const ReduceOutArgs oa{part_a, K, nullptr, 1, dA, dropping ? ds.scale : 1.f};
  auto dA_and_sums = [&](hipStream_t sx) -> int {
    if (launch_token_reduce_group(ta, p->n_chunks, p->r_train, sx) != hipSuccess) return DSV_ERR_DEVICE;
    if (launch_reduce_out(ob, oa, p->r_max, p->r_train, train_ads, p->n_tads, tad_ptr, tad_chunks, ranks, accumulate,
                          sx) != hipSuccess)
      return DSV_ERR_DEVICE;
    return DSV_OK;
  };
  if (!dX) return dA_and_sums(s);

  // 6. dx = dy W + g A_a on the matrix cores (W read with a transposing load).
  //    Under dropout g A_a passes through the input's mask (in the accumulators,
  //    between the low-rank prologue and the main loop).
  const PartPlan pp = bwd_part_plan(*p, dt, K, N);
  auto dx_gemm = [&](hipStream_t s) -> int {
    if (pp.use && workspace_bytes - ws.total >= pp.bytes) {  // few rows: in pieces, as in the forward
      PartGroup pg{};
      FinishGroup fg = bwd_finish(*p);
      add_part(pg, fg, pp, 0, PartArgs{static_cast<const uint16_t*>(dY), ld.dy, static_cast<const uint16_t*>(Wt ? Wt : W),
                                       Wt ? ld.wt : ld.w, p->T_t, K, N},
               at<char>(workspace, ws.total), gm, ldh, A, dX, ld.dx, keep, keep_words, ds.scale);
      const int tk = timing_begin(1, s);
      hipError_t e = launch_part_gemm(pg, pp.cfg, p->r_train, Wt == nullptr, s);
      if (e == hipSuccess) e = launch_part_finish(fg, p->n_titems, p->r_train, true, s);
      timing_end(tk, s);
      return e == hipSuccess ? DSV_OK : DSV_ERR_DEVICE;
    }
    GemmArgs g{};
    g.P = static_cast<const uint16_t*>(dY);
    g.ldp = ld.dy;
    g.Q = static_cast<const uint16_t*>(Wt ? Wt : W);
    g.ldq = Wt ? ld.wt : ld.w;
    g.out = static_cast<uint16_t*>(dX);
    g.ldo = ld.dx;
    g.M = p->T_t;
    g.Nout = K;
    g.C = N;
    g.tiles = p->dptr(gp.tm == 256 ? L.bwd_tiles : L.bwd_tiles128);
    g.uniform_rows = gp.tm == 256 && p->btiles_uniform;
    set_split(g, gp, workspace, ws.sk_part);
    if (g.half_tiles > 0 && !Wt && !nn16_fits(g)) {  // the 8-wave form has whole tiles only
      g.dp_tiles += g.half_tiles;
      g.half_tiles = 0;
    }
    g.Lp = gm;
    g.ldl = ldh;
    g.Lq = static_cast<const uint16_t*>(A);
    g.lq_ad = (int64_t)p->r_max * K;
    g.lq_j = K;
    g.lq_col = 1;
    g.ranks = ranks;
    g.scales = nullptr;
    g.delta = nullptr;
    g.gslot = nullptr;
    g.keep = keep;
    g.keep_words = keep_words;
    g.keep_scale = ds.scale;
    const int tk = timing_begin(1, s);
    const hipError_t e = Wt ? launch_gemm_nt(g, gp.tm, gp.tn, s) : launch_gemm_nn(g, gp.tm, gp.tn, s);
    timing_end(tk, s);
    return e == hipSuccess ? DSV_OK : DSV_ERR_DEVICE;
  };
  // One projection's dA work is too small to pay for a fork to the side
  // stream (the grouped call forks): everything on the caller's stream.
  if ((rc = dA_and_sums(s)) != DSV_OK) return rc;
  return dx_gemm(s);
}

}  // namespace

extern "C" int dsv_cobatch_fwd(const dsv_plan* p, dsv_dtype dt, int32_t K, int32_t N, const void* X,
                               const void* W, const void* A, const void* B, void* Y, void* H_save,
                               void* workspace, size_t workspace_bytes, void* hip_stream) {
  return fwd_impl(p, dt, K, N, X, W, A, B, Y, H_save, nullptr, workspace, workspace_bytes, hip_stream);
}

extern "C" int dsv_cobatch_fwd_noalloc(const dsv_plan* p, dsv_dtype dt, int32_t K, int32_t N, const void* X,
                                       const void* W, const void* A, const void* B, void* Y, void* H_save,
                                       void* hip_stream) {
  // the device scratch replaces the workspace: its address on the current
  // device (looked up on the device's first call), never the array's name
  void* scratch = nullptr;
  if (noalloc_scratch(&scratch) != hipSuccess) return DSV_ERR_DEVICE;
  return fwd_impl(p, dt, K, N, X, W, A, B, Y, H_save, nullptr, scratch, kNoAllocScratchBytes, hip_stream,
                  /*lds=*/nullptr, /*noalloc=*/true);
}

extern "C" int dsv_cobatch_fwd_dropout(const dsv_plan* p, dsv_dtype dt, int32_t K, int32_t N, const void* X,
                                       const void* W, const void* A, const void* B, void* Y, void* H_save,
                                       const dsv_dropout* dropout, void* workspace, size_t workspace_bytes,
                                       void* hip_stream) {
  if (!dropout) return DSV_ERR_ARG;
  return fwd_impl(p, dt, K, N, X, W, A, B, Y, H_save, dropout, workspace, workspace_bytes, hip_stream);
}

extern "C" int dsv_lora_bwd(const dsv_plan* p, dsv_dtype dt, int32_t K, int32_t N, const void* X,
                            const void* W, const void* A, const void* B, const void* H_save,
                            const void* dY, float* dA, float* dB, void* dX, int32_t accumulate,
                            void* workspace, size_t workspace_bytes, void* hip_stream) {
  return bwd_impl(p, dt, K, N, X, W, A, B, H_save, dY, dA, dB, dX, accumulate, nullptr, nullptr, workspace,
                  workspace_bytes, hip_stream);
}

extern "C" int dsv_lora_bwd_dropout(const dsv_plan* p, dsv_dtype dt, int32_t K, int32_t N, const void* X,
                                    const void* W, const void* A, const void* B, const void* H_save,
                                    const void* dY, float* dA, float* dB, void* dX, int32_t accumulate,
                                    const dsv_dropout* dropout, void* workspace, size_t workspace_bytes,
                                    void* hip_stream) {
  if (!dropout) return DSV_ERR_ARG;
  return bwd_impl(p, dt, K, N, X, W, A, B, H_save, dY, dA, dB, dX, accumulate, dropout, nullptr, workspace,
                  workspace_bytes, hip_stream);
}

// ---------------------------------------------------------------------------
// Grouped launches: several projections of one batch (one plan) with one
// launch per step kind.  GEMMs take whole 256x256 tiles of every projection in
// one launch, longest contraction first, so the tail of one projection is
// filled by the tiles of the next instead of being split.
// ---------------------------------------------------------------------------
namespace {

static_assert(kMaxGroup == DSV_MAX_GROUP, "group size of the kernels and the interface");

GemmPlan whole256(int32_t m256, int32_t n_out) {
  GemmPlan g;
  g.tm = g.tn = 256;
  g.n_mtiles = m256;
  g.n_ntiles = (n_out + 255) / 256;
  g.dp_tiles = g.n_mtiles * g.n_ntiles;
  return g;
}

// Halves the tiles of a grouped launch's last, partial wave where they fill at
// most half the CUs (plan_gemm's rule).  Only for projections of one contraction
// length, whose waves end together; ok: the launch's kernels have half tiles.
// beside_wide: dX beside the dA reduction of ranks above 32 on the side stream.  Halves
// on nearly every CU leave that work none to run on, which costs more than they gain
// while the contraction is short (501 rows through two 512 x 8192, rank 64: 128 tiles 69
// us, 256 halves 82; at 64 K-steps the halves win): seven CUs of eight at most there.
void halve_last_wave(GemmGroup& G, bool ok, bool beside_wide = false) {
  const int cus = device_cus();
  const int most = beside_wide && (G.a[0].C + 63) / 64 <= 32 ? cus - cus / 8 : cus;
  for (int p = 1; p < G.n; ++p) ok = ok && (G.a[p].C + 63) / 64 == (G.a[0].C + 63) / 64;
  int32_t r = ok && cus > 0 ? G.off[G.n] % cus : 0;
  if (2 * r > most) r = 0;
  for (int p = G.n - 1; p >= 0 && r > 0; --p) {
    GemmArgs& g = G.a[p];
    g.half_tiles = std::min(r, g.dp_tiles);
    g.dp_tiles -= g.half_tiles;
    r -= g.half_tiles;
  }
  for (int p = 0; p < G.n; ++p) {
    G.off[p + 1] = G.off[p] + G.a[p].dp_tiles;
    G.hoff[p + 1] = G.hoff[p] + 2 * G.a[p].half_tiles;
  }
}

int check_group(const dsv_plan* p, dsv_dtype dt, int32_t n, const void* projs) {
  if (!p || !projs) return DSV_ERR_ARG;
  if (n < 1 || n > DSV_MAX_GROUP) return DSV_ERR_RANGE;
  if (dt != DSV_BF16 && dt != DSV_F32) return DSV_ERR_RANGE;
  return DSV_OK;
}

// Workspace of a grouped call: each projection's single-call regions (without
// split-tile partials for bf16), one after the other.
size_t fwd_group_ws(const dsv_plan& p, dsv_dtype dt, int32_t n, const dsv_fwd_proj* pr, size_t* base,
                    FwdWs* w) {
  size_t off = 0;
  for (int i = 0; i < n; ++i) {
    const GemmPlan gp = dt == DSV_BF16 ? whole256(p.n_ftiles, pr[i].N) : GemmPlan{};
    w[i] = fwd_ws(p, dt, pr[i].K, pr[i].N, gp);
    base[i] = off;
    off = align256(off + w[i].total);
  }
  return off;
}

size_t bwd_group_ws(const dsv_plan& p, dsv_dtype dt, int32_t n, const dsv_bwd_proj* pr, size_t* base,
                    BwdWs* w) {
  size_t off = 0;
  for (int i = 0; i < n; ++i) {
    const GemmPlan gp = dt == DSV_BF16 ? whole256(p.n_btiles, pr[i].K) : GemmPlan{};
    w[i] = bwd_ws(p, dt, pr[i].K, pr[i].N, gp);
    base[i] = off;
    off = align256(off + w[i].total);
  }
  return off;
}

// projections in launch order: longest contraction first (stable)
void by_contraction(int32_t n, const int32_t* C, int32_t* order) {
  for (int i = 0; i < n; ++i) order[i] = i;
  std::stable_sort(order, order + n, [&](int32_t a, int32_t b) { return C[a] > C[b]; });
}

}  // namespace

extern "C" int32_t dsv_row_stride(int32_t n, dsv_dtype dt) {
  if (n <= 0 || (dt != DSV_BF16 && dt != DSV_F32)) return 0;
  if (dt == DSV_BF16 && n > 8192 && ((int64_t)n * 2) % 4096 == 0) return n + 64;
  return n;
}

extern "C" int dsv_cobatch_fwd_grouped_workspace(const dsv_plan* p, dsv_dtype dt, int32_t n_proj,
                                                 const dsv_fwd_proj* projs, size_t* bytes) {
  int rc = check_group(p, dt, n_proj, projs);
  if (rc != DSV_OK) return rc;
  if (!bytes) return DSV_ERR_ARG;
  if (n_proj == 1) return dsv_cobatch_fwd_workspace(p, dt, projs[0].K, projs[0].N, bytes);
  for (int i = 0; i < n_proj; ++i)
    if ((rc = check_common(p, dt, projs[i].K, projs[i].N)) != DSV_OK) return rc;
  size_t base[DSV_MAX_GROUP];
  FwdWs w[DSV_MAX_GROUP];
  *bytes = fwd_group_ws(*p, dt, n_proj, projs, base, w) + fwd_group_part(*p, dt, n_proj, projs).bytes;
  return DSV_OK;
}

extern "C" int dsv_lora_bwd_grouped_workspace(const dsv_plan* p, dsv_dtype dt, int32_t n_proj,
                                              const dsv_bwd_proj* projs, size_t* bytes) {
  int rc = check_group(p, dt, n_proj, projs);
  if (rc != DSV_OK) return rc;
  if (!bytes) return DSV_ERR_ARG;
  if (n_proj == 1) return dsv_lora_bwd_workspace(p, dt, projs[0].K, projs[0].N, bytes);
  for (int i = 0; i < n_proj; ++i)
    if ((rc = check_common(p, dt, projs[i].K, projs[i].N)) != DSV_OK) return rc;
  size_t base[DSV_MAX_GROUP];
  BwdWs w[DSV_MAX_GROUP];
  *bytes = bwd_group_ws(*p, dt, n_proj, projs, base, w) + bwd_group_part(*p, dt, n_proj, projs).bytes;
  return DSV_OK;
}

namespace {

// Dropout of a grouped call: every projection's mask spec (projections with
// p = 0 get an all-keeping mask of scale 1 when another one drops, which
// leaves their results bit for bit as without dropout).
int group_dropout(const dsv_dropout* drops, int32_t n, int32_t T_t, DropoutSpec* ds, bool* any) {
  *any = false;
  for (int i = 0; i < n; ++i) ds[i] = DropoutSpec{0u, 1.f, 0, 0};
  if (!drops) return DSV_OK;
  for (int i = 0; i < n; ++i) {
    if (!dropout_spec(&drops[i], &ds[i])) return DSV_ERR_RANGE;
    if (!mask_aligned(&drops[i])) return DSV_ERR_ARG;
    if (drops[i].p > 0.0 && T_t > 0) *any = true;
  }
  return DSV_OK;
}

int fwd_grouped_impl(const dsv_plan* p, dsv_dtype dt, int32_t n_proj, const dsv_fwd_proj* projs,
                     const dsv_dropout* drops, void* workspace, size_t workspace_bytes, void* hip_stream) {
  int rc = check_group(p, dt, n_proj, projs);
  if (rc != DSV_OK) return rc;
  Strides st[DSV_MAX_GROUP];
  if (n_proj == 1) {
    const dsv_fwd_proj& q = projs[0];
    if ((rc = check_common(p, dt, q.K, q.N)) != DSV_OK || (rc = fwd_strides(q, &st[0])) != DSV_OK) return rc;
    return fwd_impl(p, dt, q.K, q.N, q.X, q.W, q.A, q.B, q.Y, q.H_save, drops, workspace, workspace_bytes,
                    hip_stream, &st[0]);
  }
  // every check before any launch
  for (int i = 0; i < n_proj; ++i) {
    const dsv_fwd_proj& q = projs[i];
    if ((rc = check_common(p, dt, q.K, q.N)) != DSV_OK) return rc;
    if ((rc = fwd_strides(q, &st[i])) != DSV_OK) return rc;
  }
  DropoutSpec ds[DSV_MAX_GROUP];
  bool dropping = false;
  if ((rc = group_dropout(drops, n_proj, p->T_t, ds, &dropping)) != DSV_OK) return rc;
  if (!p->d_meta) return DSV_ERR_ARG;
  if (p->T == 0) return DSV_OK;
  for (int i = 0; i < n_proj; ++i) {
    const dsv_fwd_proj& q = projs[i];
    if (!ptr_ok(q.X) || !ptr_ok(q.W) || !ptr_ok(q.A) || !ptr_ok(q.B) || !ptr_ok(q.Y)) return DSV_ERR_ARG;
    if (q.H_save && !aligned16(q.H_save)) return DSV_ERR_ARG;
  }
  size_t base[DSV_MAX_GROUP];
  FwdWs w[DSV_MAX_GROUP];
  const size_t total = fwd_group_ws(*p, dt, n_proj, projs, base, w);
  if (total > 0) {
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255)) return DSV_ERR_ARG;
    if (workspace_bytes < total) return DSV_ERR_SIZE;
  }
  char* wsb = static_cast<char*>(workspace);
  if (dt == DSV_F32) {  // the fp32 check path: the single-projection kernels, one projection at a time
    for (int i = 0; i < n_proj; ++i) {
      const dsv_fwd_proj& q = projs[i];
      rc = fwd_impl(p, dt, q.K, q.N, q.X, q.W, q.A, q.B, q.Y, q.H_save, drops ? &drops[i] : nullptr, wsb + base[i],
                    w[i].total, hip_stream, &st[i]);
      if (rc != DSV_OK) return rc;
    }
    return DSV_OK;
  }
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  const MetaLayout& L = p->lay;
  const int32_t* ranks = p->dptr(L.ranks);
  const float* scales = reinterpret_cast<const float*>(p->dptr(L.scales));
  const int64_t ldh = ld_rank(p->r_max);

  // 0. dropout masks of the training rows' adapter input, every projection in
  //    one launch (into the caller's buffers where given)
  uint32_t* keepg[DSV_MAX_GROUP] = {};
  if (dropping) {
    DropoutMaskGroup mg{};
    mg.n = n_proj;
    for (int i = 0; i < n_proj; ++i) {
      keepg[i] = mask_buffer(&drops[i], at<uint32_t>(wsb + base[i], w[i].keep));
      mg.bits[i] = keepg[i];
      mg.K[i] = projs[i].K;
      mg.d[i] = ds[i];
    }
    if (launch_dropout_mask_group(mg, p->T_t, s) != hipSuccess) return DSV_ERR_DEVICE;
  }

  // 1. shrink of every projection in one launch
  SkinnyGroup sg{};
  sg.n = n_proj;
  for (int i = 0; i < n_proj; ++i) {
    const dsv_fwd_proj& q = projs[i];
    SkinnyArgs& sk = sg.a[i];
    sk.P = static_cast<const uint16_t*>(q.X);
    sk.ldp = st[i].x;
    sk.rows = p->dptr(L.shrink_rows);
    sk.items = p->dptr(L.shrink_items);
    sk.Q = static_cast<const uint16_t*>(q.A);
    sk.q_ad = (int64_t)p->r_max * q.K;
    sk.ldq = q.K;
    sk.ranks = ranks;
    sk.C = q.K;
    sk.out1 = at<uint16_t>(wsb + base[i], w[i].h_all);
    sk.ld1 = ldh;
    sk.out2 = p->T_t > 0 ? static_cast<uint16_t*>(q.H_save) : nullptr;
    sk.ld2 = p->r_max;
    sk.row_train = p->dptr(L.row_train);
    sk.part = at<float>(wsb + base[i], w[i].rk_part);
    sk.part_n = p->T;
    sk.r_max = p->r_max;
    sk.split_items = p->n_shrink;
    if (dropping) {
      sk.keep = keepg[i];
      sk.keep_words = (q.K + 31) / 32;
      sk.drop_scale = ds[i].scale;
    }
  }
  // 1a. few rows: every base product in pieces, the shrinks beside them (a launch
  //     of their own where dropout masks them), then their sums with the low-rank terms
  const PartPlan pp = fwd_group_part(*p, dt, n_proj, projs);
  if (pp.use && workspace_bytes - total >= pp.bytes) {
    if (dropping && launch_shrink_group(sg, p->n_shrink, p->r_used, s) != hipSuccess) return DSV_ERR_DEVICE;
    PartGroup pg{};
    FinishGroup fg = fwd_finish(*p);
    for (int i = 0; i < n_proj; ++i) {
      const dsv_fwd_proj& q = projs[i];
      add_part(pg, fg, pp, i, PartArgs{static_cast<const uint16_t*>(q.X), st[i].x, static_cast<const uint16_t*>(q.W),
                                       st[i].w, p->T, q.N, q.K},
               wsb + total, sg.a[i].out1, ldh, q.B, q.Y, st[i].y, nullptr, 0, 1.f);
      if (!dropping) add_part_shrink(*p, pg, fg, pp, i, q.A, wsb + total, q.H_save);
    }
    const int tk = timing_begin(0, s);
    hipError_t e = launch_part_gemm(pg, pp.cfg, p->r_used, false, s);
    if (e == hipSuccess) e = launch_part_finish(fg, p->n_shrink, p->r_used, false, s);
    timing_end(tk, s);
    return e == hipSuccess ? DSV_OK : DSV_ERR_DEVICE;
  }
  if (launch_shrink_group(sg, p->n_shrink, p->r_used, s) != hipSuccess) return DSV_ERR_DEVICE;

  // 2. gathered rows of every projection in one launch
  if (p->n_gather > 0) {
    GatherGroup gg{};
    gg.n = n_proj;
    for (int i = 0; i < n_proj; ++i) {
      gg.a[i] = GatherArgs{sg.a[i].out1, static_cast<const uint16_t*>(projs[i].B), projs[i].N,
                           at<float>(wsb + base[i], w[i].delta)};
      gg.yoff[i + 1] = gg.yoff[i] + (projs[i].N + 255) / 256;
    }
    if (launch_gather_group(gg, ldh, p->r_max, p->dptr(L.gather_items), p->n_gitems, p->dptr(L.gather_rows),
                            ranks, scales, s) != hipSuccess)
      return DSV_ERR_DEVICE;
  }

  // 3. every base GEMM in one launch, longest contraction first
  int32_t Cs[DSV_MAX_GROUP], order[DSV_MAX_GROUP];
  for (int i = 0; i < n_proj; ++i) Cs[i] = projs[i].K;
  by_contraction(n_proj, Cs, order);
  GemmGroup G{};
  G.n = n_proj;
  for (int k = 0; k < n_proj; ++k) {
    const int i = order[k];
    const dsv_fwd_proj& q = projs[i];
    GemmArgs& g = G.a[k];
    g.P = static_cast<const uint16_t*>(q.X);
    g.ldp = st[i].x;
    g.Q = static_cast<const uint16_t*>(q.W);
    g.ldq = st[i].w;
    g.out = static_cast<uint16_t*>(q.Y);
    g.ldo = st[i].y;
    g.M = p->T;
    g.Nout = q.N;
    g.C = q.K;
    g.tiles = p->dptr(L.fwd_tiles);
    g.uniform_rows = 1;
    set_split(g, whole256(p->n_ftiles, q.N), nullptr, 0);
    g.Lp = sg.a[i].out1;
    g.ldl = ldh;
    g.Lq = static_cast<const uint16_t*>(q.B);
    g.lq_ad = (int64_t)q.N * p->r_max;
    g.lq_j = 1;
    g.lq_col = p->r_max;
    g.ranks = ranks;
    g.scales = scales;
    g.delta = p->n_gather > 0 ? at<float>(wsb + base[i], w[i].delta) : nullptr;
    g.gslot = p->dptr(L.gslot);
    G.off[k + 1] = G.off[k] + g.n_mtiles * g.n_ntiles;
  }
  halve_last_wave(G, true);
  const int tk = timing_begin(0, s);
  const hipError_t e = launch_gemm_group_nt(G, s);
  timing_end(tk, s);
  return e == hipSuccess ? DSV_OK : DSV_ERR_DEVICE;
}

int bwd_grouped_impl(const dsv_plan* p, dsv_dtype dt, int32_t n_proj, const dsv_bwd_proj* projs, int32_t accumulate,
                     const dsv_dropout* drops, void* workspace, size_t workspace_bytes, void* hip_stream) {
  int rc = check_group(p, dt, n_proj, projs);
  if (rc != DSV_OK) return rc;
  Strides st[DSV_MAX_GROUP];
  if (n_proj == 1) {
    const dsv_bwd_proj& q = projs[0];
    if ((rc = check_common(p, dt, q.K, q.N)) != DSV_OK || (rc = bwd_strides(q, &st[0])) != DSV_OK) return rc;
    return bwd_impl(p, dt, q.K, q.N, q.X, q.W, q.A, q.B, q.H_save, q.dY, q.dA, q.dB, q.dX, accumulate, drops, q.Wt,
                    workspace, workspace_bytes, hip_stream, &st[0]);
  }
  for (int i = 0; i < n_proj; ++i) {
    if ((rc = check_common(p, dt, projs[i].K, projs[i].N)) != DSV_OK) return rc;
    if ((rc = bwd_strides(projs[i], &st[i])) != DSV_OK) return rc;
  }
  DropoutSpec ds[DSV_MAX_GROUP];
  bool dropping = false;
  if ((rc = group_dropout(drops, n_proj, p->T_t, ds, &dropping)) != DSV_OK) return rc;
  if (accumulate != 0 && accumulate != 1) return DSV_ERR_RANGE;
  if (!p->d_meta) return DSV_ERR_ARG;
  if (p->T_t == 0) return DSV_OK;
  for (int i = 0; i < n_proj; ++i) {
    const dsv_bwd_proj& q = projs[i];
    if (!ptr_ok(q.X) || !ptr_ok(q.W) || !ptr_ok(q.A) || !ptr_ok(q.B) || !ptr_ok(q.dA) || !ptr_ok(q.dB) ||
        !ptr_ok(q.dY))
      return DSV_ERR_ARG;
    if ((q.dX && !aligned16(q.dX)) || (q.H_save && !aligned16(q.H_save)) || (q.Wt && !aligned16(q.Wt)))
      return DSV_ERR_ARG;
  }
  size_t base[DSV_MAX_GROUP];
  BwdWs w[DSV_MAX_GROUP];
  const size_t total = bwd_group_ws(*p, dt, n_proj, projs, base, w);
  if (total > 0) {
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255)) return DSV_ERR_ARG;
    if (workspace_bytes < total) return DSV_ERR_SIZE;
  }
  char* wsb = static_cast<char*>(workspace);
  if (dt == DSV_F32) {
    for (int i = 0; i < n_proj; ++i) {
      const dsv_bwd_proj& q = projs[i];
      rc = bwd_impl(p, dt, q.K, q.N, q.X, q.W, q.A, q.B, q.H_save, q.dY, q.dA, q.dB, q.dX, accumulate,
                    drops ? &drops[i] : nullptr, q.Wt, wsb + base[i], w[i].total, hip_stream, &st[i]);
      if (rc != DSV_OK) return rc;
    }
    return DSV_OK;
  }
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  const MetaLayout& L = p->lay;
  const int32_t* ranks = p->dptr(L.ranks);
  const float* scales = reinterpret_cast<const float*>(p->dptr(L.scales));
  const int64_t ldh = ld_rank(p->r_max);
  const int32_t* train_ads = p->dptr(L.train_ads);
  uint16_t* gm[DSV_MAX_GROUP];
  uint32_t* keep[DSV_MAX_GROUP];
  for (int i = 0; i < n_proj; ++i) {
    gm[i] = at<uint16_t>(wsb + base[i], w[i].g);
    keep[i] = dropping ? mask_buffer(&drops[i], at<uint32_t>(wsb + base[i], w[i].keep)) : nullptr;
  }

  // 0. the forward's dropout masks: the caller's buffers, or regenerated from
  //    the same seeds and offsets (one launch for those)
  if (dropping) {
    DropoutMaskGroup mg{};
    mg.n = n_proj;
    for (int i = 0; i < n_proj; ++i) {
      mg.bits[i] = drops[i].mask ? nullptr : keep[i];
      mg.K[i] = projs[i].K;
      mg.d[i] = ds[i];
    }
    if (launch_dropout_mask_group(mg, p->T_t, s) != hipSuccess) return DSV_ERR_DEVICE;
  }

  // 1. h of the training rows for projections whose forward kept no H_save
  const uint16_t* hs[DSV_MAX_GROUP];
  int64_t ldhs[DSV_MAX_GROUP];
  SkinnyGroup rg{};
  for (int i = 0; i < n_proj; ++i) {
    const dsv_bwd_proj& q = projs[i];
    hs[i] = static_cast<const uint16_t*>(q.H_save);
    ldhs[i] = p->r_max;
    if (hs[i]) continue;
    uint16_t* hrec = at<uint16_t>(wsb + base[i], w[i].hrec);
    SkinnyArgs& sh = rg.a[rg.n++];
    sh.P = static_cast<const uint16_t*>(q.X);
    sh.ldp = st[i].x;
    sh.rows = p->dptr(L.train_rows);
    sh.items = p->dptr(L.train_items);
    sh.Q = static_cast<const uint16_t*>(q.A);
    sh.q_ad = (int64_t)p->r_max * q.K;
    sh.ldq = q.K;
    sh.ranks = ranks;
    sh.C = q.K;
    sh.out2 = hrec;
    sh.ld2 = ldh;
    sh.row_train = p->dptr(L.row_train);
    sh.keep = keep[i];
    sh.keep_words = (q.K + 31) / 32;
    sh.drop_scale = ds[i].scale;
    sh.part = at<float>(wsb + base[i], w[i].h_part);
    sh.part_n = p->T_t;
    sh.r_max = p->r_max;
    sh.split_items = p->n_shrink;  // the forward shrink's split: the same sums
    hs[i] = hrec;
    ldhs[i] = ldh;
  }
  if (rg.n > 0 && launch_shrink_train_group(rg, p->n_titems, p->r_train, s) != hipSuccess) return DSV_ERR_DEVICE;

  // 2. chunk partials of dy^T h (dB), every projection; the same pass writes
  //    the column-block partials of dy B_a (g), reading dy once
  TokenReduceGroup tbg{};
  tbg.n = n_proj;
  for (int i = 0; i < n_proj; ++i) {
    const dsv_bwd_proj& q = projs[i];
    TokenReduceArgs& tb = tbg.a[i];
    tb.P = static_cast<const uint16_t*>(q.dY);
    tb.ldp = st[i].dy;
    tb.Q = hs[i];
    tb.ldq = ldhs[i];
    tb.chunks = p->dptr(L.chunks);
    tb.ranks = ranks;
    tb.C = q.N;
    tb.r_max = p->r_max;
    tb.part = at<float>(wsb + base[i], w[i].part_b);
    tb.B = static_cast<const uint16_t*>(q.B);
    tb.gpart = at<float>(wsb + base[i], w[i].g_part);
    tb.gpart_n = p->T_t;
    tbg.yoff[i + 1] = tbg.yoff[i] + token_col_blocks(q.N);
  }
  if (launch_token_reduce_group(tbg, p->n_chunks, p->r_train, s) != hipSuccess) return DSV_ERR_DEVICE;

  // 3. g = s_a dy B_a of every projection: block partials summed in order, rounded once
  SkinnyGroup gf{};
  gf.n = n_proj;
  for (int i = 0; i < n_proj; ++i) {
    SkinnyArgs& sk = gf.a[i];
    sk.items = p->dptr(L.train_items);
    sk.ranks = ranks;
    sk.scales = scales;
    sk.out1 = gm[i];
    sk.ld1 = ldh;
    sk.part = tbg.a[i].gpart;
    sk.part_n = p->T_t;
    sk.r_max = p->r_max;
    sk.pieces = token_col_blocks(projs[i].N);
  }
  if (launch_g_finish_group(gf, p->n_titems, s) != hipSuccess) return DSV_ERR_DEVICE;

  // 4. chunk partials of x^T g (dA), every projection
  TokenReduceGroup tag{};
  tag.n = n_proj;
  for (int i = 0; i < n_proj; ++i) {
    const dsv_bwd_proj& q = projs[i];
    TokenReduceArgs& ta = tag.a[i];
    ta.P = static_cast<const uint16_t*>(q.X);
    ta.ldp = st[i].x;
    ta.prow = p->dptr(L.train_rows);
    ta.Q = gm[i];
    ta.ldq = ldh;
    ta.chunks = p->dptr(L.chunks);
    ta.ranks = ranks;
    ta.C = q.K;
    ta.r_max = p->r_max;
    ta.part = at<float>(wsb + base[i], w[i].part_a);
    ta.keep = keep[i];  // dA contracts the masked input
    ta.keep_words = (q.K + 31) / 32;
    tag.yoff[i + 1] = tag.yoff[i] + token_col_blocks(q.K);
  }

  // 5. fixed-order sums into dB (scaled by s_a) and dA, every projection
  ReduceOutGroup og{};
  og.n = 2 * n_proj;
  for (int i = 0; i < n_proj; ++i) {
    og.a[2 * i] = ReduceOutArgs{tbg.a[i].part, projs[i].N, scales, 0, projs[i].dB, 1.f};
    og.a[2 * i + 1] = ReduceOutArgs{tag.a[i].part, projs[i].K, nullptr, 1, projs[i].dA,
                                    dropping ? ds[i].scale : 1.f};
  }
  auto dA_and_sums = [&](hipStream_t sx) -> int {
    if (launch_token_reduce_group(tag, p->n_chunks, p->r_train, sx) != hipSuccess) return DSV_ERR_DEVICE;
    if (launch_reduce_out_group(og, p->r_max, p->r_train, train_ads, p->n_tads, p->dptr(L.tad_chunk_ptr),
                                p->dptr(L.tad_chunks), ranks, accumulate, sx) != hipSuccess)
      return DSV_ERR_DEVICE;
    return DSV_OK;
  };

  // 6. every dX GEMM in one launch, longest contraction first (projections with a
  //    transposed weight in one NT launch, the others in one NN launch)
  const PartPlan pp = bwd_group_part(*p, dt, n_proj, projs);
  auto dx_all = [&](hipStream_t s) -> int {
    if (pp.use && workspace_bytes - total >= pp.bytes) {  // few rows: in pieces, one sum for all
      FinishGroup fg = bwd_finish(*p);
      const int tk = timing_begin(1, s);
      hipError_t e = hipSuccess;
      for (int nt = 1; nt >= 0 && e == hipSuccess; --nt) {
        PartGroup pg{};
        for (int i = 0; i < n_proj; ++i) {
          const dsv_bwd_proj& q = projs[i];
          if (!q.dX || (q.Wt != nullptr) != (nt == 1)) continue;
          add_part(pg, fg, pp, i, PartArgs{static_cast<const uint16_t*>(q.dY), st[i].dy,
                                           static_cast<const uint16_t*>(nt ? q.Wt : q.W), nt ? st[i].wt : st[i].w,
                                           p->T_t, q.K, q.N},
                   wsb + total, gm[i], ldh, q.A, q.dX, st[i].dx, keep[i], (q.K + 31) / 32, ds[i].scale);
        }
        if (pg.n > 0) e = launch_part_gemm(pg, pp.cfg, p->r_train, nt == 0, s);
      }
      if (fg.n > 0 && e == hipSuccess) e = launch_part_finish(fg, p->n_titems, p->r_train, true, s);
      timing_end(tk, s);
      return e == hipSuccess ? DSV_OK : DSV_ERR_DEVICE;
    }
    int32_t Cs[DSV_MAX_GROUP], order[DSV_MAX_GROUP];
    for (int i = 0; i < n_proj; ++i) Cs[i] = projs[i].N;
    by_contraction(n_proj, Cs, order);
    for (int nt = 1; nt >= 0; --nt) {
      GemmGroup G{};
      for (int k = 0; k < n_proj; ++k) {
        const int i = order[k];
        const dsv_bwd_proj& q = projs[i];
        if (!q.dX || (q.Wt != nullptr) != (nt == 1)) continue;
        GemmArgs& g = G.a[G.n];
        g.P = static_cast<const uint16_t*>(q.dY);
        g.ldp = st[i].dy;
        g.Q = static_cast<const uint16_t*>(nt ? q.Wt : q.W);
        g.ldq = nt ? st[i].wt : st[i].w;
        g.out = static_cast<uint16_t*>(q.dX);
        g.ldo = st[i].dx;
        g.M = p->T_t;
        g.Nout = q.K;
        g.C = q.N;
        g.tiles = p->dptr(L.bwd_tiles);
        g.uniform_rows = p->btiles_uniform;
        set_split(g, whole256(p->n_btiles, q.K), nullptr, 0);
        g.Lp = gm[i];
        g.ldl = ldh;
        g.Lq = static_cast<const uint16_t*>(q.A);
        g.lq_ad = (int64_t)p->r_max * q.K;
        g.lq_j = q.K;
        g.lq_col = 1;
        g.ranks = ranks;
        g.keep = keep[i];  // dropout: g A_a through the input's mask
        g.keep_words = (q.K + 31) / 32;
        g.keep_scale = ds[i].scale;
        G.off[G.n + 1] = G.off[G.n] + g.n_mtiles * g.n_ntiles;
        ++G.n;
      }
      if (G.n > 0) {
        bool ok = true;
        for (int k = 0; k < G.n; ++k) ok = ok && (nt || nn16_fits(G.a[k]));
        halve_last_wave(G, ok, p->r_train > 32);
        const int tk = timing_begin(1, s);
        const hipError_t e = nt ? launch_gemm_group_nt(G, s) : launch_gemm_group_nn(G, s);
        timing_end(tk, s);
        if (e != hipSuccess) return DSV_ERR_DEVICE;
      }
    }
    return DSV_OK;
  };

  // dX needs g only: the dA reduction and the final sums run beside it on the
  // side stream (joined back into the caller's stream before the call returns).
  // Not beside pieces: those are short and fill every CU's LDS, so the side work
  // waits for them anyway (256 rows through gate and up: 118.6 us forked here, 127
  // with dB and g on the side stream as well, 113.7 on one stream).
  if (!(pp.use && workspace_bytes - total >= pp.bytes)) {
    std::lock_guard<std::mutex> lk(g_side_mu);
    if (SideStream* sd = side_stream()) {
      if (hipEventRecord(sd->fork, s) != hipSuccess) return DSV_ERR_DEVICE;
      if ((rc = dx_all(s)) != DSV_OK) return rc;
      if (hipStreamWaitEvent(sd->s, sd->fork, 0) != hipSuccess) return DSV_ERR_DEVICE;
      if ((rc = dA_and_sums(sd->s)) != DSV_OK) return rc;
      if (hipEventRecord(sd->join, sd->s) != hipSuccess || hipStreamWaitEvent(s, sd->join, 0) != hipSuccess)
        return DSV_ERR_DEVICE;
      return DSV_OK;
    }
  }
  if ((rc = dA_and_sums(s)) != DSV_OK) return rc;
  return dx_all(s);
}

}  // namespace

extern "C" int dsv_cobatch_fwd_grouped(const dsv_plan* p, dsv_dtype dt, int32_t n_proj, const dsv_fwd_proj* projs,
                                       void* workspace, size_t workspace_bytes, void* hip_stream) {
  return fwd_grouped_impl(p, dt, n_proj, projs, nullptr, workspace, workspace_bytes, hip_stream);
}

extern "C" int dsv_cobatch_fwd_grouped_dropout(const dsv_plan* p, dsv_dtype dt, int32_t n_proj,
                                               const dsv_fwd_proj* projs, const dsv_dropout* dropouts,
                                               void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (!dropouts) return DSV_ERR_ARG;
  return fwd_grouped_impl(p, dt, n_proj, projs, dropouts, workspace, workspace_bytes, hip_stream);
}

extern "C" int dsv_lora_bwd_grouped(const dsv_plan* p, dsv_dtype dt, int32_t n_proj, const dsv_bwd_proj* projs,
                                    int32_t accumulate, void* workspace, size_t workspace_bytes, void* hip_stream) {
  return bwd_grouped_impl(p, dt, n_proj, projs, accumulate, nullptr, workspace, workspace_bytes, hip_stream);
}

extern "C" int dsv_lora_bwd_grouped_dropout(const dsv_plan* p, dsv_dtype dt, int32_t n_proj,
                                            const dsv_bwd_proj* projs, int32_t accumulate,
                                            const dsv_dropout* dropouts, void* workspace, size_t workspace_bytes,
                                            void* hip_stream) {
  if (!dropouts) return DSV_ERR_ARG;
  return bwd_grouped_impl(p, dt, n_proj, projs, accumulate, dropouts, workspace, workspace_bytes, hip_stream);
}
