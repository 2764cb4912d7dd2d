// Host planner (see plan.h).  Builds, for a list of matrices and shard grids
// (Sec. 3, "How blocks align with model-parallel shards"), the tables used by
// the kernels.  No HIP call is made here.
#include "plan.h"

#include <algorithm>
#include <limits>
#include <utility>

namespace muonbp {

namespace {

int64_t round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }
int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

constexpr int64_t kMaxDim = int64_t(1) << 30;    // int32 leading dims stay valid
constexpr int64_t kMaxTiles = int64_t(1) << 16;  // tile index packs in 16 bits

// Byte offsets inside one NS operand are 32-bit in the GEMM kernels (buffer
// descriptors and per-lane offsets), so no operand may reach 2^31 bytes.
constexpr int64_t kMaxOperandBytes = int64_t(1) << 31;

// Appends the workspace buffers of one problem; returns false on overflow.
// nn (the apply reads Z row-major, so no Z^T is kept between iterations):
// Z[0], Z[1], A, B, with each Z buffer large enough for either layout (S x
// Lp or L x Sp); U of a transposed unit is written as Z^T into the buffer
// the last apply would otherwise fill (off_zt aliases off_z).  Otherwise
// (the transposed-copy apply, or the register-loop kernels): Z[2], Z^T[2],
// A, B.  A Gram-space unit adds Q[2] and T (S x Sp each).
bool place_problem(Problem* p, int64_t* cursor, int64_t align_elems, bool nn) {
  auto take = [&](int64_t n) {
    int64_t at = *cursor;
    *cursor = round_up(at + n, align_elems);
    return at;
  };
  const int64_t zs = p->S * p->Lp, zts = p->L * p->Sp, as = p->S * p->Sp;
  if (nn) {
    const int64_t both = std::max(zs, zts);
    p->off_z[0] = p->off_zt[0] = take(both);
    p->off_z[1] = p->off_zt[1] = take(both);
  } else {
    p->off_z[0] = take(zs);
    p->off_z[1] = take(zs);
    p->off_zt[0] = take(zts);
    p->off_zt[1] = take(zts);
  }
  p->off_a = take(as);
  p->off_b = take(as);
  if (p->gram) {
    p->off_q[0] = take(as);
    p->off_q[1] = take(as);
    p->off_t = take(as);
  }
  return *cursor > 0 && *cursor < (int64_t(1) << 46);
}

// A plan of both kinds of iteration has a Gram and an apply launch for every
// iteration (its units as printed) on top of the Gram-space products: 23
// launches for K = 5, against 17 where every unit runs the Gram-space
// iteration.  Down to L = S that is no more flops (20 S^3 either way), only
// more of them in the slower products, so where the launches saved are worth
// more than that, the remaining units follow: none below kGramMinS (one such
// unit leaves the whole plan as it is), and none above 512 rows.  A launch
// of a small plan costs 4-5 us; rates as for kGramMinS, halved (launches of
// few tiles).  The block step of one layer of width 512: 210 -> 188 us.
//
// 512 rows is where the measurements behind the model ended, not the break-even.
// One S x S unit beside one S x 4 S / four beside three / sixteen beside twelve,
// us, both kinds of iteration against Gram space only: S = 520 188 / 252 / 534
// against 145 / 204 / 457, 768 230 / 387 / 854 against 172 / 297 / 771, 1024 314
// / 506 / 1331 against 258 / 415 / 1379.
//
// Distance of U from 64 bits in Gram space over that as printed, of the units
// that follow (L <= 1.17 S, S = 128 to 512, paper's quintic): 0.67 to 0.89 for
// gradients of rank 4 to 128 with noise, whose distance is the largest (0.6 to
// 1.8% as printed).  Full-rank Gaussian inputs, closer to 64 bits either way
// (0.4 to 0.5%): 1.13 at S = 128, 1.09 at 192, 1.01 at 256, 0.99 at 320, 0.87 at
// 512.  Orthonormal rows (0.3 to 0.4% as printed): 0.62 to 2.2, at most 0.66%.
void unify_iteration(std::vector<Problem>* probs, int ns_steps) {
  double extra_us = 0;
  bool some = false, all = true;
  for (const Problem& p : *probs) {
    if (p.gram) {
      some = true;
      continue;
    }
    all = false;
    if (p.S < kGramMinS || p.S > 512) return;
    const double s = double(p.S), l = double(p.L), gram = s * s * l / 550e6, sym = s * s * s / 445e6,
                 apply = 2 * s * s * l / 495e6;
    double in_gram = 0;
    for (int k0 = 0; k0 < ns_steps; k0 += kGramSegment)
      in_gram += gram + (4.0 * std::min(kGramSegment, ns_steps - k0) - 3.0) * sym + apply;
    extra_us += in_gram - ns_steps * (gram + sym + apply);
  }
  const int segments = (ns_steps + kGramSegment - 1) / kGramSegment;
  if (!some || all || extra_us > 2 * (ns_steps - segments) * 4.0) return;
  for (Problem& p : *probs) p.gram = true;
}

// Largest operand of a problem in bytes (Z in either layout, A, B).
int64_t max_operand_bytes(const Problem& p, int es) {
  return std::max(std::max(p.S * p.Lp, p.L * p.Sp), p.S * p.Sp) * int64_t(es);
}

void add_pack_tiles(Plan* plan, int32_t prob) {
  const Problem& p = plan->probs[prob];
  const int64_t pr = ceil_div(p.rows, kPackTile), pc = ceil_div(p.cols, kPackTile);
  for (int64_t i = 0; i < pr; ++i)
    for (int64_t j = 0; j < pc; ++j)
      plan->pack_tiles.push_back(TileRef{prob, int32_t((i << 16) | j)});
}

// Rows x columns of C for one product of problem p.
void gemm_dims(const Problem& p, GemmKind kind, int64_t* m, int64_t* n, int64_t* k) {
  *m = p.S;
  *n = kind == kApply ? p.L : p.S;
  *k = kind == kGram ? p.L : p.S;
}

int64_t count_tiles(const std::vector<Problem>& probs, GemmKind kind, int v) {
  int64_t n = 0;
  for (const Problem& p : probs) {
    int64_t m, c, k;
    gemm_dims(p, kind, &m, &c, &k);
    const int64_t tm = ceil_div(m, kGemmTileRows[v]), tn = ceil_div(c, kGemmTileCols[v]);
    n += kind == kApply ? tm * tn : tm * (tm + 1) / 2;
  }
  return n;
}

// Logical tile order of one product of one problem: bands of `group` tile
// rows, each band walked column by column (rows inside a column first).  An
// XCD's concurrent tiles then form a group x (tiles / group) block of C that
// shares `group` X panels and as many Y panels as it has columns, instead of
// one X panel and a Y panel per tile.  Tiles taller than 128 rows take
// bands of 4, or of 8 for the polynomial and apply products of a unit with
// at least 16 rows of tiles (measured on the 8B-shaped model: bands of 8
// make the full-step apply, 16 x 56 tiles, 1.7% faster; on the block
// steps' 7-row units they leave the time unchanged and raise the apply's
// traffic by 60%, and the Gram is 2% slower with them; bands of 2 make the
// apply 5% slower).
void append_tiles(const Problem& p, GemmKind kind, int v, int32_t desc,
                  std::vector<TileRef>* out) {
  int64_t m, c, k;
  gemm_dims(p, kind, &m, &c, &k);
  const int64_t tm = ceil_div(m, kGemmTileRows[v]), tn = ceil_div(c, kGemmTileCols[v]);
  const bool small_tiles = kGemmTileRows[v] <= 128 && v != kGemm128x128Split2;
  const int64_t group = small_tiles || (kind != kGram && tm >= 16) ? 8 : 4;
  for (int64_t g0 = 0; g0 < tm; g0 += group)
    for (int64_t j = (kind == kApply ? 0 : g0); j < tn; ++j)
      for (int64_t i = g0; i < std::min(tm, g0 + group); ++i)
        if (kind == kApply || i <= j) out->push_back(TileRef{desc, int32_t((i << 16) | j)});
}

}  // namespace

int32_t gram_apply_slot(int ns_steps, int sg) {
  const int n = std::min(kGramSegment, ns_steps - sg * kGramSegment);
  const int nseg = (ns_steps + kGramSegment - 1) / kGramSegment;
  return kSlotGApply0 + (sg & 1) + 2 * ((n - 1) & 1) + 4 * (sg == nseg - 1);
}

int32_t first_apply_slot(const Problem& p, int ns_steps) {
  if (p.gram) return gram_apply_slot(ns_steps, 0);
  return ns_steps == 1 ? kSlotApplyLast : kSlotApply0;
}

namespace {

// One unit's tiles in a launch's logical order, and their K slices.
struct UnitTiles {
  int64_t begin, end, slices;
};

// Workgroup order of a launch with more tiles than CUs.  Each XCD's share is
// the same work instead of the same number of tiles (a tile of a 4096-wide
// matrix's shard takes four times as long as one of a 1024-wide one's): of
// the units of one shape each XCD takes as many as every other, the rest is
// handed out tile by tile where least is.  A share is walked longest tiles
// first, so that no long one is left for the end, and its units in reverse
// where `reverse` is set: a launch then starts on what the one before it left
// in the last-level cache.  Workgroup w runs on XCD w % 8: shorter shares are
// filled up with empty entries (prob = -1), which the kernels skip.  Measured
// against equal runs of tiles in problem order (us): Gram of the 1024 x 7168
// and 3584 x 2048 shards of two MLP matrices 367 -> 281 and their apply 490 ->
// 428; apply of one layer of the 8B-shaped model's block step 732 -> 626, Gram
// of its full step 2705 -> 2046; 8192 x 256 next to 2048 x 1024 shards, Gram
// 1000 -> 794; the reversal alone 0.3-2.3% of a step.
std::vector<TileRef> balanced_order(const std::vector<TileRef>& logical, std::vector<UnitTiles> units, bool reverse) {
  constexpr int64_t kFixed = 14;  // a tile's prologue and epilogue, in K slices
  auto longer = [](const UnitTiles& a, const UnitTiles& b) { return a.slices > b.slices; };
  std::stable_sort(units.begin(), units.end(), longer);
  std::vector<UnitTiles> share[kNumXCDs], rest;
  int64_t load[kNumXCDs] = {}, total = 0;
  auto weight = [](const UnitTiles& u) { return (u.end - u.begin) * (u.slices + kFixed); };
  for (size_t i = 0; i < units.size();) {
    size_t j = i;
    while (j < units.size() && units[j].slices == units[i].slices &&
           units[j].end - units[j].begin == units[i].end - units[i].begin)
      ++j;
    const size_t each = (j - i) / kNumXCDs;
    for (size_t k = i; k < j; ++k) {
      total += weight(units[k]);
      const size_t x = each > 0 ? (k - i) / each : size_t(kNumXCDs);
      if (x < size_t(kNumXCDs)) {
        share[x].push_back(units[k]);
        load[x] += weight(units[k]);
      } else {
        rest.push_back(units[k]);
      }
    }
    i = j;
  }
  // The rest: the least loaded XCD takes tiles up to the mean.
  const int64_t mean = (total + kNumXCDs - 1) / kNumXCDs;
  for (UnitTiles u : rest)
    while (u.begin < u.end) {
      const int x = int(std::min_element(load, load + kNumXCDs) - load);
      const int64_t per = u.slices + kFixed;
      const int64_t n = std::min(u.end - u.begin, std::max<int64_t>(1, (mean - load[x] + per - 1) / per));
      share[x].push_back(UnitTiles{u.begin, u.begin + n, u.slices});
      load[x] += n * per;
      u.begin += n;
    }
  int64_t size = 0;
  for (int x = 0; x < kNumXCDs; ++x) {
    if (reverse) std::reverse(share[x].begin(), share[x].end());
    std::stable_sort(share[x].begin(), share[x].end(), longer);
    int64_t n = 0;
    for (const UnitTiles& u : share[x]) n += u.end - u.begin;
    if (n > 0) size = std::max(size, (n - 1) * kNumXCDs + x + 1);
  }
  std::vector<TileRef> out(size_t(size), TileRef{-1, 0, 0, 0});
  for (int x = 0; x < kNumXCDs; ++x) {
    size_t w = size_t(x);
    for (const UnitTiles& u : share[x])
      for (int64_t j = 0; j < u.end - u.begin; ++j, w += kNumXCDs)
        out[w] = logical[size_t(reverse ? u.end - 1 - j : u.begin + j)];
  }
  return out;
}

int32_t slot_of(GemmKind kind, int iter, int ns_steps, int poly_slots) {
  const int q = iter & 1;
  return kind == kGram   ? kSlotGram0 + q
         : kind == kPoly ? kSlotPoly0 + std::min(iter, poly_slots - 1)
         : iter == ns_steps - 1 ? kSlotApplyLast
                                : kSlotApply0 + q;
}

// Launch schedule of the K NS iterations.  Per iteration: the Gram (every
// unit that iterates as printed; a Gram-space unit at the start of each
// segment), the polynomial (every unit; a segment's first into Q[0]), then
// for the Gram-space units the products Q_j = P_j Q_{j-1} and T = A_j P_j
// together, and A_{j+1} = T P_j (none in a segment's last iteration), then
// the apply (every unit that iterates as printed; a Gram-space unit's Z <-
// Q Z at the end of each segment).  The Gram-space products take the
// polynomial's tile shape (all are S x S x S).
void build_phases(Plan* plan, int ns_steps, int poly_slots, int desc_per_problem, int ns_elem_bytes, bool lean) {
  plan->phases.clear();
  plan->split_floats = plan->split_slots = 0;
  const int32_t np = int32_t(plan->probs.size());
  using Item = std::pair<int32_t, int32_t>;  // (problem, descriptor slot)
  // The workgroup orders of this plan, with an item's number in place of its
  // descriptor: launches of one kind over the same problems differ in the
  // descriptors only.
  struct Order {
    GemmKind kind;
    bool reverse;
    std::vector<int32_t> probs;
    bool long_k;
    std::vector<TileRef> tiles;
  };
  std::vector<Order> orders;
  auto order_for = [&](GemmKind kind, bool reverse, const std::vector<Item>& items) -> const Order& {
    for (const Order& o : orders)
      if (o.kind == kind && o.reverse == reverse &&
          std::equal(items.begin(), items.end(), o.probs.begin(), o.probs.end(),
                     [](const Item& it, int32_t pi) { return it.first == pi; }))
        return o;
    const int32_t variant = plan->variant[kind], nsplit = plan->nsplit[kind];
    Order o{kind, reverse, {}, false, {}};
    std::vector<UnitTiles> units;
    std::vector<TileRef> logical;
    // Items of a launch are the plan's problems, or each of them twice.
    logical.reserve(size_t(plan->tiles_per_iter[kind]));
    for (const Item& it : items) {
      const Problem& p = plan->probs[size_t(it.first)];
      int64_t m, n, k;
      gemm_dims(p, kind, &m, &n, &k);
      if (ns_elem_bytes == 4 && !gemm_is_dmap(variant)) o.long_k = o.long_k || k > kLongK;
      const int64_t t0 = int64_t(logical.size());
      append_tiles(p, kind, variant, int32_t(o.probs.size()), &logical);
      units.push_back(UnitTiles{t0, int64_t(logical.size()), ceil_div(k, 32)});
      o.probs.push_back(it.first);
    }
    if (nsplit > 1) {
      // The shares of one tile are adjacent, so that the XCD order below
      // keeps them on one XCD (one L2) as a rule.
      std::vector<TileRef> parts;
      parts.reserve(logical.size() * size_t(nsplit));
      for (size_t ti = 0; ti < logical.size(); ++ti)
        for (int32_t q = 0; q < nsplit; ++q)
          parts.push_back(TileRef{logical[ti].prob, logical[ti].ij, int32_t(ti), q});
      plan->split_slots = std::max<int64_t>(plan->split_slots, int64_t(logical.size()));
      plan->split_floats = std::max<int64_t>(
          plan->split_floats, int64_t(logical.size()) * nsplit * kGemmTileRows[variant] * kGemmTileCols[variant]);
      logical.swap(parts);
    }
    // A launch of several rounds: the XCDs' shares balanced, and the units
    // walked the other way round in every second launch.
    if (!lean && nsplit == 1 && int64_t(logical.size()) > kNumCUs)
      o.tiles = balanced_order(logical, std::move(units), reverse);
    else
      o.tiles = xcd_order(logical);
    orders.push_back(std::move(o));
    return orders.back();
  };
  auto add_phase = [&](GemmKind kind, const std::vector<Item>& items) {
    if (items.empty()) return;
    const Order& o = order_for(kind, plan->phases.size() % 2 == 1, items);
    GemmPhase phase;
    phase.variant = plan->variant[kind];
    phase.kind = kind;
    phase.nsplit = plan->nsplit[kind];
    phase.nn = kind == kApply && plan->nn_apply;
    phase.long_k = o.long_k;
    phase.tiles = o.tiles;
    for (TileRef& t : phase.tiles)
      if (t.prob >= 0) {
        const Item& it = items[size_t(t.prob)];
        t.prob = it.first * desc_per_problem + it.second;
      }
    plan->phases.push_back(std::move(phase));
  };
  for (int iter = 0; iter < ns_steps; ++iter) {
    std::vector<Item> gram, poly, qt, upd, apply;
    for (int32_t pi = 0; pi < np; ++pi) {
      const Problem& p = plan->probs[size_t(pi)];
      // An in-place unit's first Gram and first apply read the momentum.
      const bool first_m = p.in_place && iter == 0;
      if (!p.gram) {
        gram.push_back({pi, first_m ? kSlotGramM : slot_of(kGram, iter, ns_steps, poly_slots)});
        poly.push_back({pi, slot_of(kPoly, iter, ns_steps, poly_slots)});
        apply.push_back({pi, first_m ? kSlotApplyM : slot_of(kApply, iter, ns_steps, poly_slots)});
        continue;
      }
      // Segment sg of n iterations, j-th of them.
      const int sg = iter / kGramSegment, j = iter % kGramSegment;
      const int n = std::min(kGramSegment, ns_steps - sg * kGramSegment);
      const int32_t poly_b = slot_of(kPoly, iter, ns_steps, poly_slots);
      if (j == 0) gram.push_back({pi, first_m ? kSlotGramM : kSlotGram0 + (sg & 1)});
      poly.push_back({pi, j == 0 ? poly_b + poly_slots : poly_b});
      if (j > 0) qt.push_back({pi, (j & 1) ? kSlotQ1 : kSlotQ0});
      if (j < n - 1) {
        qt.push_back({pi, j == 0 ? kSlotT0 : kSlotT});
        upd.push_back({pi, j == 0 ? kSlotA0 : kSlotA});
      } else {
        apply.push_back({pi, p.in_place && sg == 0 ? kSlotApplyM : gram_apply_slot(ns_steps, sg)});
      }
    }
    add_phase(kGram, gram);
    add_phase(kPoly, poly);
    add_phase(kPoly, qt);
    add_phase(kPoly, upd);
    add_phase(kApply, apply);
  }
}

}  // namespace

std::vector<TileRef> xcd_order(const std::vector<TileRef>& logical) {
  const int64_t n = int64_t(logical.size());
  const int64_t q = n / kNumXCDs, r = n % kNumXCDs;
  std::vector<TileRef> out(logical.size());
  for (int64_t w = 0; w < n; ++w) {
    const int64_t x = w % kNumXCDs, j = w / kNumXCDs;
    out[w] = logical[x * q + std::min(x, r) + j];
  }
  return out;
}

// padded: every kernel that writes an operand of this plan fills the rows'
// last chunk of 8 elements with zeros (the pack and the DMA kernels' epilogues
// do), so the DMA kernels may read it whole whatever K is.
bool dma_allowed(const std::vector<Problem>& probs, GemmKind kind, int ns_elem_bytes, bool padded) {
  if (ns_elem_bytes != 2) return false;
  if (padded) return true;
  for (const Problem& p : probs) {
    int64_t m, n, k;
    gemm_dims(p, kind, &m, &n, &k);
    if (k % 8 != 0) return false;
  }
  return true;
}

// Time model of one launch of the interleaved DMA kernel, in microseconds,
// fitted to per-launch measurements on MI355X (engine clock about 1.7 GHz
// under sustained MFMA load): rounds of resident workgroups x (fixed cost +
// K slices x time per 32-deep slice).  The fixed cost (launch, ring fill,
// epilogue) is 6.5 us.  A slice costs the tile's MFMA cycles over an
// efficiency that grows with the MFMAs per wave and K step: 4 (128 x 128):
// 0.49, 8: 0.55, 16 (256 x 256): 0.61.  128 x 128 tiles fit two per CU,
// and then take 0.65 us per slice each; larger tiles fit one.
double dmap_launch_us(const std::vector<Problem>& probs, GemmKind kind, int v) {
  int64_t tiles = 0;
  double slices = 0;
  for (const Problem& p : probs) {
    int64_t m, c, k;
    gemm_dims(p, kind, &m, &c, &k);
    const int64_t tm = ceil_div(m, kGemmTileRows[v]), tn = ceil_div(c, kGemmTileCols[v]);
    const int64_t nt = kind == kApply ? tm * tn : tm * (tm + 1) / 2;
    tiles += nt;
    slices += double(nt) * double(ceil_div(k, 32));
  }
  if (tiles == 0) return 0;
  slices /= double(tiles);
  const int nm = (kGemmTileRows[v] / 64) * (kGemmTileCols[v] / 64);
  const double eff = nm <= 4 ? 0.49 : nm <= 8 ? 0.49 + 0.015 * (nm - 4)
                                              : std::min(0.61, 0.55 + 0.0075 * (nm - 8));
  const double slice_us = nm * 2 * 32 / eff / 1700.0;
  constexpr double kFixedUs = 6.5;
  const double one = kFixedUs + slices * slice_us;  // a round with one tile per CU
  if (v != kGemmDmaP128x128) return double(ceil_div(tiles, kNumCUs)) * one;
  const double two = kFixedUs + slices * 0.65;      // a round with two tiles per CU
  const int64_t full = tiles / (2 * kNumCUs), rest = tiles % (2 * kNumCUs);
  return double(full) * two + (rest == 0 ? 0.0 : rest <= kNumCUs ? one : two);
}

// The same for kGemmWaveK64 (two workgroups per CU).  A wave runs a quarter
// of the slices, so a launch that fits one workgroup per CU is little more
// than its fixed cost; with more tiles than that, each of which fetches its
// own operand rows, the time follows the copies.  Measured (us, against the
// 128 x 128 tiles): 48 tiles of 4 / 16 slices 4.8 / 5.7 (6.1 / 8.2), 30 of 32
// 6.9 (12.9), 432 of 16 8.7 (10.2), 624 of 24 14.8 (13.1), 640 of 8 10.9
// (8.5), 528 of 192 79 (59).
double wave_k_launch_us(const std::vector<Problem>& probs, GemmKind kind) {
  int64_t tiles = 0;
  double slices = 0;
  for (const Problem& p : probs) {
    int64_t m, c, k;
    gemm_dims(p, kind, &m, &c, &k);
    const int64_t tm = ceil_div(m, kGemmTileRows[kGemmWaveK64]), tn = ceil_div(c, kGemmTileCols[kGemmWaveK64]);
    const int64_t nt = kind == kApply ? tm * tn : tm * (tm + 1) / 2;
    tiles += nt;
    slices += double(nt) * double(ceil_div(k, 32));
  }
  if (tiles == 0) return 0;
  slices /= double(tiles);
  const double one = 2.0 + 0.08 * slices, two = 3.5 + 0.23 * slices;
  const int64_t full = tiles / (2 * kNumCUs), rest = tiles % (2 * kNumCUs);
  return 2.4 + double(full) * two + (rest == 0 ? 0.0 : rest <= kNumCUs ? one : two);
}

// Whether kGemmWaveK64 may take a launch whose best DMA kernel is `dma`: where
// neither that kernel nor its K split over three workgroups is the faster one
// (measured per launch, us; slices are the longest product's).
//  * Up to three tiles per CU: 720 tiles of 10 / 80 slices 15.4 / 36.6 against
//    17.9 / 42.9; beyond, 1440 of 10 24.5 against 20.5, 960 of 106 60.8 against
//    50.8.
//  * With more than one tile per CU up to 128 slices: 440 of 112 and 440 of 80
//    0.92 of the DMA kernel's time, 275 of 160 49.8 against 43.7, 360 of 240
//    70.2 against 60.6 (0.81 to 1.16 from 144 slices on, 1.02 in the mean).
//  * Where the split kernel would run at one workgroup per CU (three per tile):
//    with more than one tile per CU not at all (312 of 128 / 512 slices 31.3 /
//    129.6 against 25.2 / 63.4 split), else below 320 slices (144 of 192 / 256
//    25.8 / 29.7 against 26.6 / 32.6; 84 of 384 52.6 against 44.7), or below
//    192 with fewer than 20 tiles (12 of 128 18.9 against 19.6; 12 of 192 / 384
//    / 3125 28.3 / 53.1 / 427.6 against 23.6 / 35.5 / 265.5).
bool wave_k_allowed(const std::vector<Problem>& probs, GemmKind kind, int32_t dma) {
  const int64_t tiles = count_tiles(probs, kind, kGemmWaveK64);
  int64_t slices = 0;
  for (const Problem& p : probs) {
    int64_t m, c, k;
    gemm_dims(p, kind, &m, &c, &k);
    slices = std::max(slices, ceil_div(k, 32));
  }
  const int32_t split = choose_split(probs, kind, dma, 0);
  const bool split_fits = split > 1 && split * count_tiles(probs, kind, dma) <= kNumCUs;
  if (tiles > 3 * kNumCUs) return false;
  if (tiles > kNumCUs) return slices <= 128 && !split_fits;
  return !split_fits || slices < (tiles < 20 ? 192 : 320);
}

// The kernel of one fp32 launch, by time models of the three tile shapes whose
// operands are split into bf16 parts, in us: 128 x 128 tiles, one per CU at a
// time, 8 + 1.2 a 32-column slice each; 64 x 64 tiles, 6.7 a launch and 0.46 a
// slice (0.5 alone on a CU); 32 x 32 tiles with the slices shared by the
// waves, 5.7 a launch and 0.29 a slice.  Measured at 128 / 64 / 32: one 256 x
// 256 unit 20 / 11 / 8, one 1024 x 1024 45 / 24 / 32, 144 tiles of 128 at K =
// 4096 155 / 155 / 274, 1088 at K = 2048 443 / 464 / 988.  A shape whose tile
// rows or columns do not fit 16 bits is out (build_layout's limit on the sides
// leaves 64 x 64 tiles in).  -1: a product over more than kLongK terms, which
// takes the kernel that restarts its sums.
int32_t f32_split_variant(const std::vector<Problem>& probs, GemmKind kind) {
  int64_t tiles[3] = {0, 0, 0};
  bool fits[3] = {true, true, true};
  static const int32_t variant[3] = {kGemmF32x128, kGemmF32x64, kGemmF32WaveK32};
  double slices = 0;
  for (const Problem& p : probs) {
    int64_t m, c, k;
    gemm_dims(p, kind, &m, &c, &k);
    if (k > kLongK) return -1;
    for (int v = 0; v < 3; ++v) {
      const int64_t tm = ceil_div(m, kGemmTileRows[variant[v]]), tn = ceil_div(c, kGemmTileCols[variant[v]]);
      const int64_t nt = kind == kApply ? tm * tn : tm * (tm + 1) / 2;
      tiles[v] += nt;
      fits[v] = fits[v] && tm < kMaxTiles && tn < kMaxTiles;
      if (v == 0) slices += double(nt) * double(ceil_div(k, 32));
    }
  }
  slices /= double(tiles[0]);
  auto per_cu = [&](int v) { return std::max(1.0, double(tiles[v]) / kNumCUs); };
  double us[3] = {double(ceil_div(tiles[0], kNumCUs)) * (8 + 1.2 * slices),
                  6.7 + std::max(0.5, 0.46 * per_cu(1)) * slices, 5.7 + 0.29 * per_cu(2) * slices};
  for (int v = 0; v < 3; ++v)
    if (!fits[v]) us[v] = std::numeric_limits<double>::infinity();
  return variant[std::min_element(us, us + 3) - us];
}

int32_t choose_variant(const std::vector<Problem>& probs, GemmKind kind, int tile_policy,
                       int ns_elem_bytes, bool wave_k, bool lean) {
  const bool sym = kind != kApply;
  // With the planner's own choice all three products run on DMA kernels; a
  // forced shape keeps the register K loop where K is not a multiple of 8.
  const bool dma = dma_allowed(probs, kind, ns_elem_bytes, tile_policy == 0 && !lean);
  if (tile_policy > 0) {
    int v = tile_policy - 1;
    // The block-ordered LDS-DMA loop these variants named was removed (the
    // interleaved loop of the same tile shape was 20-25% faster on every
    // launch): they select the interleaved kernel.
    if (v >= kGemmDma128x128 && v <= kGemmDma256x256) v += kGemmDmaP128x128 - kGemmDma128x128;
    // Symmetric products take square tiles; without the DMA path, the
    // register K loop on the same (or, for 192-wide tiles, the nearest) shape.
    if (sym && kGemmTileRows[v] != kGemmTileCols[v]) {
      static const int32_t square[kNumGemmVariants] = {0, 0, 2, 3, 3, 5, 6, 7, 7, 9, 12, 12, 12, 13,
                                                        12, 12};
      v = square[v];
    }
    if (kGemmIsDma[v] && !dma) {
      static const int32_t twin[kNumGemmVariants] = {0, 1, 2, 0, 1, 2, 6, 0, 1, 2, 2, 2, 0, 2,
                                                      2, 2};
      v = twin[v];
    }
    return v;
  }
  // With the interleaved DMA loop (bf16): the tile shape
  // the time model above puts first (square shapes for the symmetric
  // products).  Register K loop otherwise (rules from per-launch
  // measurements on MI355X):
  // symmetric products on 128 x 128 tiles (split over two K groups below two
  // tiles per CU), the apply product on 256 x 256 tiles from two per CU.
  if (dma) {
    // 256 x 256 tiles run on the 8-wave kernel (two waves per SIMD): 4-19%
    // faster than the 4-wave one on every measured launch, never slower.
    // 192 x 256 and 256 x 192 tiles too, since the two waves of a SIMD swap
    // issue priority every slice: the 2048 x 768 shards' apply 700 against
    // 649 TFLOP/s, the 2048 x 6144 step 2.5% faster (before the swap the
    // launches after them ran slower and the step did not gain).
    static const int32_t sym_cands[] = {kGemmDmaP128x128, kGemmDmaP192x192, kGemmDmaP256x256W8};
    static const int32_t gen_cands[] = {kGemmDmaP128x128, kGemmDmaP256x128, kGemmDmaP192x256,
                                        kGemmDmaP256x192, kGemmDmaP256x256W8};
    int32_t best = kGemmDmaP128x128;
    double best_us = dmap_launch_us(probs, kind, best);
    const int32_t* c = sym ? sym_cands : gen_cands;
    const int nc = sym ? 3 : 5;
    for (int i = 1; i < nc; ++i) {
      const double us = dmap_launch_us(probs, kind, c[i]);
      if (us < best_us) {
        best = c[i];
        best_us = us;
      }
    }
    // The 128 x 128 model above is for full launches: where few CUs are busy
    // a launch takes 1.5-3 us less, hence the margin.
    if (wave_k && wave_k_launch_us(probs, kind) < 0.9 * best_us && wave_k_allowed(probs, kind, best))
      return kGemmWaveK64;
    if (best == kGemmDmaP192x256) best = kGemmDmaP192x256W8;
    if (best == kGemmDmaP256x192) best = kGemmDmaP256x192W8;
    return best;
  }
  const int64_t n128 = count_tiles(probs, kind, kGemm128x128);
  if (ns_elem_bytes == 4 && !lean) {
    const int32_t v = f32_split_variant(probs, kind);
    if (v >= 0) return v;
  }
  const int32_t small = n128 < 2 * kNumCUs ? kGemm128x128Split2 : kGemm128x128;
  if (sym) return small;
  if (count_tiles(probs, kind, kGemm256x256) >= 2 * kNumCUs) return kGemm256x256;
  return small;
}

// K split of the interleaved DMA kernels: each tile shared by q workgroups,
// each on about 1/q of the K slices, the last to finish adding the partial
// sums.  Only on request (k_split > 0): the partial sums have to cross the
// per-XCD caches, and on MI355X that traffic (a full fp32 tile per share)
// cost more than the extra CUs gained on every launch measured (the 2048 x
// 6144 shards' Gram: 35 us split 3 ways against 27 us unsplit).
// With k_split = 0 the planner splits 3 ways only a launch that leaves
// most CUs idle and has a long K loop everywhere (fewer tiles than 0.6 x
// the CUs, at least 128 K slices per product): there the extra CUs win
// over the partial-sum traffic (the whole 2048 x 6144 matrix's Gram, 136
// tiles at K = 6144: 56 against 60 us a launch).
int32_t choose_split(const std::vector<Problem>& probs, GemmKind kind, int32_t v, int k_split) {
  if (!gemm_is_dmap(v)) return 1;
  if (k_split > 0) return k_split;
  const int64_t tiles = count_tiles(probs, kind, v);
  if (tiles == 0 || 10 * tiles > 6 * kNumCUs) return 1;
  for (const Problem& p : probs) {
    int64_t m, c, k;
    gemm_dims(p, kind, &m, &c, &k);
    if (ceil_div(k, 32) < 128) return 1;
  }
  return 3;
}

double ns_unit_flops(int64_t S, int64_t L, int K, bool gram) {
  const double s = double(S), l = double(L);
  // Gram Z Z^T: S(S+1)/2 distinct entries x 2L; a symmetric S x S x S
  // product (A A, and the Gram-space Q, T and A products): S(S+1)/2 x 2S;
  // B Z (the apply): S x L entries x 2S.
  const double gram_zz = s * (s + 1) * l, sym = s * s * (s + 1), apply = 2 * s * s * l;
  if (!gram || K == 0) return double(K) * (gram_zz + sym + apply);
  // Per segment of n iterations: one Gram, n polynomials, n - 1 Q products,
  // 2 (n - 1) A updates, one apply.
  double f = 0;
  for (int k0 = 0; k0 < K; k0 += kGramSegment) {
    const int n = std::min(kGramSegment, K - k0);
    f += gram_zz + (4.0 * n - 3.0) * sym + apply;
  }
  return f;
}

double ns_unit_dense_flops(int64_t S, int64_t L, int K) {
  const double s = double(S), l = double(L);
  return 2.0 * K * (2.0 * l * s * s + s * s * s);
}

std::string build_layout(const MatrixShape* mats, int32_t n_mats,
                         int ns_elem_bytes, int ns_steps, int poly_slots, int tile_policy,
                         int k_split, int apply_mode, Layout* out, bool* shape_error, int gram_mode,
                         bool in_place_input, bool lean, bool quintic, int lists) {
  *shape_error = false;
  if (!mats || n_mats <= 0) return "mats must be a non-empty array";
  if (ns_steps < 0) return "ns_steps must be >= 0";
  if (poly_slots < 1 || poly_slots > 64) return "poly_slots out of range";
  if (tile_policy < 0 || tile_policy > kNumGemmVariants) return "tile_policy out of range";
  if (k_split < 0 || k_split > kMaxKSplit) return "k_split out of range";
  if (gram_mode < 0 || gram_mode > 2) return "gram_mode out of range";
  Layout L;
  L.mats.assign(mats, mats + n_mats);
  int64_t elems = 0;
  for (int32_t k = 0; k < n_mats; ++k) {
    const MatrixShape& m = mats[k];
    if (m.rows <= 0 || m.cols <= 0 || m.grid_rows <= 0 || m.grid_cols <= 0 ||
        m.rows > kMaxDim || m.cols > kMaxDim || m.rows % m.grid_rows ||
        m.cols % m.grid_cols) {
      *shape_error = true;
      return "matrix " + std::to_string(k) + ": sizes must be positive, at most 2^30, "
             "and the grid must divide rows and cols";
    }
    if (ceil_div(std::max(m.rows, m.cols), 64) >= kMaxTiles) {
      *shape_error = true;
      return "matrix " + std::to_string(k) + " is too large";
    }
    L.mat_off.push_back(elems);
    elems += m.rows * m.cols;
  }
  L.total_elems = elems;
  L.poly_slots = poly_slots;
  L.desc_per_problem = kSlotPoly0 + 2 * poly_slots;

  // Elements per segment: kSegTarget, or fewer (at least 2048, one 16-byte
  // chunk of bf16 per thread) where that many would leave CUs without a
  // workgroup; with windows off the 16-byte grid, whose chunks go four at a
  // time with more index work each, where they leave fewer than four per CU
  // (3.2 M elements in odd windows: momentum 17.8 -> 10.4 us, update 17.3 ->
  // 8.8).  Aligned windows gain nothing beyond one workgroup per CU, and every
  // segment is one more term of its unit's scale (12.6 M elements in twice the
  // segments: k_scale 8.0 -> 10.7 us).
  bool aligned = true;
  for (const MatrixShape& m : L.mats) aligned = aligned && m.cols / m.grid_cols % 8 == 0;
  const int64_t least = (aligned ? 1 : 4) * kNumCUs;
  int64_t seg_target = kSegTarget;
  while (!lean && seg_target > 2048 && elems / seg_target < least) seg_target /= 2;

  // Blocks in matrix order, row-major inside each grid; segments per block.
  for (int32_t k = 0; k < n_mats; ++k) {
    const MatrixShape& m = mats[k];
    const int64_t br = m.rows / m.grid_rows, bc = m.cols / m.grid_cols;
    const int64_t rows_per_seg = std::max<int64_t>(1, std::min(br, seg_target / bc));
    for (int32_t i = 0; i < m.grid_rows; ++i)
      for (int32_t j = 0; j < m.grid_cols; ++j) {
        BlockPlan b{k, i * br, j * bc, br, bc, int32_t(L.segs.size()), 0};
        for (int64_t r = 0; r < br; r += rows_per_seg) {
          if (L.segs.size() >= size_t(std::numeric_limits<int32_t>::max()))
            return "too many segments";
          L.segs.push_back(SegDesc{int32_t(L.blocks.size()), int32_t(r),
                                   int32_t(std::min(rows_per_seg, br - r)),
                                   int32_t(L.segs.size())});
        }
        b.seg_end = int32_t(L.segs.size());
        L.blocks.push_back(b);
      }
  }
  // Launch order: the r-th segment of every block of one block row of a
  // matrix, then the (r+1)-th, ...  For a column-sharded matrix the
  // workgroups that run together then cover whole rows of the matrix instead
  // of one block's narrow row pieces (a 4096 x 1024 matrix in 8 shards has
  // 256-byte pieces of 2 KB rows); for a single column of blocks it is the
  // block order.
  {
    std::vector<SegDesc> order;
    order.reserve(L.segs.size());
    int32_t bi = 0;
    for (int32_t k = 0; k < n_mats; ++k) {
      const MatrixShape& m = mats[k];
      for (int32_t i = 0; i < m.grid_rows; ++i) {
        const int32_t b0 = bi + i * m.grid_cols;
        const int32_t nseg = L.blocks[b0].seg_end - L.blocks[b0].seg_begin;
        for (int32_t r = 0; r < nseg; ++r)
          for (int32_t j = 0; j < m.grid_cols; ++j) order.push_back(L.segs[L.blocks[b0 + j].seg_begin + r]);
      }
      bi += m.grid_rows * m.grid_cols;
    }
    L.segs.swap(order);
  }

  const int64_t align_elems = kWsAlignBytes / ns_elem_bytes;
  const bool padded = tile_policy == 0 && !lean;  // operands read in whole chunks (dma_allowed)
  for (int full = 0; full < 2; ++full) {
    Plan& plan = L.plan[full];
    plan.full = full != 0;
    int32_t bi = 0;
    // The units: every block (block plan) or every matrix (full plan).
    for (int32_t k = 0; k < n_mats; ++k) {
      const MatrixShape& m = mats[k];
      const int32_t nb = m.grid_rows * m.grid_cols;
      auto add = [&](int64_t r0, int64_t c0, int64_t rows, int64_t cols, int32_t first_block,
                     int32_t n_blocks) {
        Problem p{};
        p.mat = k;
        p.row0 = r0;
        p.col0 = c0;
        p.rows = rows;
        p.cols = cols;
        p.trans = rows > cols;
        p.S = std::min(rows, cols);
        p.L = std::max(rows, cols);
        p.Sp = round_up(p.S, 8);
        p.Lp = round_up(p.L, 8);
        p.first_block = first_block;
        p.n_blocks = n_blocks;
        p.seg_begin = L.blocks[first_block].seg_begin;
        p.seg_end = L.blocks[first_block + n_blocks - 1].seg_end;
        plan.probs.push_back(p);
      };
      if (full) {
        add(0, 0, m.rows, m.cols, bi, nb);
      } else {
        for (int32_t b = 0; b < nb; ++b) {
          const BlockPlan& bp = L.blocks[bi + b];
          add(bp.row0, bp.col0, bp.rows, bp.cols, bi + b, 1);
        }
      }
      bi += nb;
    }
    for (const Problem& p : plan.probs)
      if (max_operand_bytes(p, ns_elem_bytes) >= kMaxOperandBytes) {
        *shape_error = true;
        return "matrix " + std::to_string(p.mat) + (full ? "" : " (one block)") + ": a " +
               std::to_string(p.S) + " x " + std::to_string(p.L) +
               " orthogonalization operand reaches 2^31 bytes, beyond the 32-bit byte offsets "
               "of the NS kernels";
      }
    for (int kind = 0; kind < 3; ++kind) {
      plan.variant[kind] = choose_variant(plan.probs, GemmKind(kind), tile_policy, ns_elem_bytes,
                                          k_split == 0 && !lean, lean);
      plan.nsplit[kind] = choose_split(plan.probs, GemmKind(kind), plan.variant[kind], k_split);
      plan.tiles_per_iter[kind] = count_tiles(plan.probs, GemmKind(kind), plan.variant[kind]);
      if (plan.tiles_per_iter[kind] * plan.nsplit[kind] > int64_t(std::numeric_limits<int32_t>::max() / 2))
        return "too many tiles";
    }
    plan.nn_apply = apply_mode == 0 && gemm_reads_rows(plan.variant[kApply]);
    // Steeper polynomials than the paper's quintic lose precision in Gram
    // space (U of 129 x 1000 with a = 3.44 in two iterations: 0.87% from 64
    // bits as printed, 2.7% in Gram space; with the quintic 0.95% and 0.73%, at
    // odd sizes from 129 x 300 to 999 x 1333 0.59 to 0.88 of the distance as
    // printed for gradients of rank 4 to 128 with noise, 0.81 to 0.98 for
    // Gaussian inputs, 0.72 to 1.7 for orthonormal rows):
    // with other coefficients only the plans that have always run it do,
    // those whose units' smaller sides are all multiples of 8.
    bool chunks = true;
    for (const Problem& p : plan.probs) chunks = chunks && p.S % 8 == 0;
    for (Problem& p : plan.probs)
      p.gram = gram_mode != 1 && ns_elem_bytes == 2 && plan.nn_apply && ns_steps >= 2 &&
               (quintic || chunks) && (gram_mode == 2 || (p.S >= kGramMinS && 4 * p.L >= 5 * p.S));
    if (gram_mode == 0 && padded && quintic) unify_iteration(&plan.probs, ns_steps);
    int64_t cursor = 0, packed = 0;
    const bool with_lists = lists < 0 || lists == full;
    for (int32_t pi = 0; pi < int32_t(plan.probs.size()); ++pi) {
      Problem& p = plan.probs[pi];
      // The momentum window as a GEMM operand: rows of whole 16-byte chunks
      // (the arena is 16-byte aligned), within the kernels' 32-bit byte offsets.
      const MatrixShape& mm = mats[p.mat];
      const int64_t mom_off = L.mat_off[p.mat] + p.row0 * mm.cols + p.col0;
      p.in_place = in_place_input && ns_elem_bytes == 2 && ns_steps >= 1 && plan.nn_apply && !p.trans &&
                   mm.cols % 8 == 0 && (!padded || p.cols % 8 == 0) && mom_off % 8 == 0 &&
                   p.rows * mm.cols * ns_elem_bytes < kMaxOperandBytes;
      if (!place_problem(&p, &cursor, align_elems, plan.nn_apply)) return "workspace too large";
      if (!p.in_place) {
        packed += ceil_div(p.rows, kPackTile) * ceil_div(p.cols, kPackTile);
        if (with_lists) add_pack_tiles(&plan, pi);
      }
      plan.ns_flops += ns_unit_flops(p.S, p.L, ns_steps, p.gram);
      plan.ns_dense_flops += ns_unit_dense_flops(p.S, p.L, ns_steps);
    }
    plan.ws_elems = cursor;
    if (with_lists) build_phases(&plan, ns_steps, poly_slots, L.desc_per_problem, ns_elem_bytes, lean);
    if (packed > int64_t(std::numeric_limits<int32_t>::max() / 2)) return "too many tiles";
  }
  *out = std::move(L);
  return "";
}

}  // namespace muonbp
