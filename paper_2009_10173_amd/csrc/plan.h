// Launch plan of a staged apply: which workgroup rows the launch has, in which order they are
// dispatched, and which tiles are cut into pieces (host code only, no device types, so that
// it can be built and tested on its own).
//
// A staged launch has one workgroup per (piece, position patch).  A piece is a range of one
// output tile's stage units.  An uncut tile is one piece, which writes the output; a cut
// tile is several pieces (each loads the whole LDS ring for its first unit), and each of them
// writes its partial sums to its own slot, which a second kernel adds in slot order.  The slots of a
// tile are consecutive and follow the tile's unit order, so the sum is deterministic.
#pragma once

#include <algorithm>
#include <cmath>
#include <functional>
#include <queue>
#include <vector>

namespace aroam {

struct PlanPiece {
  int tile, u0, u1;  // units [u0, u1) of the tile
  int slot;          // partial slot, or -1 for the single piece of an uncut tile
  double work;
};

// Costs besides the units', in units of work.
struct PlanCosts {
  double workgroup = 1.0;  // start and end of a workgroup
  double add = 0.0;        // the launch that adds the slots of cut tiles
  double add_slot = 0.0;   // and each slot of its most cut tile
};

// Costs of a launch: of a unit, added to its work, and those besides.
struct LaunchCosts {
  double unit;
  PlanCosts plan;
};

// FP64 and FP32, in bundles (of the 128 positions of a patch, about 0.1 us): a unit's staging and
// barrier, a workgroup's first and last accesses, the slot sums.  Where few workgroups run, these are
// what a finer cut has to pay for; measured on the 40 x 40 FISTA (1.13 -> 0.80 ms a pair of applies
// with them, 1.02 with none), the 64 x 64 FP32 forward (177 -> 162 us, 177 with none) and the 23 x 19
// FP64 one (75 -> 51 us, 56 with none).  Slots at 40 and 2 instead of 20 and 1 cut the smallest scans
// too little: the 23 x 19 forward takes 51.6 us instead of 47.6, an LSQR solve on 16 x 16 368 instead
// of 356; at 80 and 4 that takes 440.
constexpr LaunchCosts kRingCosts{8, {24, 20, 1}};

// BF16 in half bundles (of the 256 positions of a patch), FP8 in its own.  With them and cuts at any
// unit, BF16 and FP8 applies of 40 x 40 to 96 x 96 scans take 0.32 to 0.75 of their time with cuts at
// chunk starts (forward 96 x 96 x 64, K 20: BF16 172 -> 126 us, FP8 216 -> 151 us).  Larger or smaller
// costs, and three or four workgroups per CU in the simulation, measured slower.  A BF16 unit costs
// 30: with 16 the batch of three served scans takes 350 us instead of 332, with 44 the 200 x 200 x 128
// forward 911 instead of 862.  FP8 units: 8 and 30 within 1 % of 16.
constexpr LaunchCosts kBf16Costs{30, {60, 200, 6}}, kFp8Costs{16, {30, 60, 3}};

constexpr int kMaxCut = 64;  // largest D of a launch

struct LaunchPlan {
  std::vector<PlanPiece> pieces;     // in dispatch order
  std::vector<int> tile_pieces;      // [tile] pieces of the tile
  std::vector<int> tile_first_slot;  // [tile] slot of its first piece, -1 when uncut
  int n_slots = 0;
  int cut = 1;                       // D of the chosen cut (1: no tile cut)
  bool heaviest_first = false;
  double time = 0;                   // simulated finishing time (work units)
  double uncut_time = 0;             // the same without cuts
};

// Finishing time of a launch whose workgroups (every patch of each piece, pieces in the given
// order) take the first of `slots` free places and last as long as their work.
inline double simulate_launch(const std::vector<double>& piece_work, int n_patches, int slots) {
  if ((double)piece_work.size() * n_patches <= slots)  // every workgroup has a place at once
    return piece_work.empty() ? 0.0 : *std::max_element(piece_work.begin(), piece_work.end());
  std::priority_queue<double, std::vector<double>, std::greater<double>> free_at;
  for (int i = 0; i < slots; ++i) free_at.push(0.0);
  double end = 0;
  for (double w : piece_work)
    for (int p = 0; p < n_patches; ++p) {
      const double t = free_at.top() + w;
      free_at.pop();
      free_at.push(t);
      end = std::max(end, t);
    }
  return end;
}

// Plan a launch.  tile_units[t] .. tile_units[t + 1] are tile t's units; chunk_starts[t]
// lists the units of tile t where a piece may start (the first is tile_units[t] when the tile
// has units); unit_work[u] is unit u's work.  For D = 1 .. max_cut (in steps of a quarter from 8
// on) every tile is cut into about
// (its work) / (largest tile work / D) pieces of similar work, each cut at the start
// whose prefix work is nearest to its share, and the pieces are dispatched in tile order or
// heaviest first, whichever the simulation (`slots` places, one workgroup per piece and
// patch, costs.workgroup added to each for its fixed costs and, for a cut, those of adding
// slots) finishes sooner.  A cut
// is taken only when `allow_cut`, when it shortens the simulated launch by more than 10 %,
// and when its slots (slot_bytes per piece and patch) fit in max_slot_bytes.
inline LaunchPlan plan_launch(const std::vector<int>& tile_units,
                              const std::vector<std::vector<int>>& chunk_starts,
                              const std::vector<double>& unit_work, int n_patches, int slots,
                              bool allow_cut, double slot_bytes, double max_slot_bytes,
                              int max_cut = 8, const PlanCosts& costs = PlanCosts()) {
  const int nT = (int)tile_units.size() - 1;
  std::vector<double> prefix(unit_work.size() + 1, 0.0);
  for (size_t u = 0; u < unit_work.size(); ++u) prefix[u + 1] = prefix[u] + unit_work[u];
  double wmax = 0;
  for (int t = 0; t < nT; ++t)
    wmax = std::max(wmax, prefix[tile_units[t + 1]] - prefix[tile_units[t]]);
  auto cut = [&](int D, std::vector<PlanPiece>& out, std::vector<int>& npieces) {
    out.clear();
    npieces.assign(nT, 1);
    for (int t = 0; t < nT; ++t) {
      const int a = tile_units[t], b = tile_units[t + 1];
      const double wt = prefix[b] - prefix[a];
      const std::vector<int>& cs = chunk_starts[t];
      int S = 1;
      if (D > 1 && wt > 0 && wmax > 0)
        S = std::max(1, std::min((int)cs.size(), (int)std::lround(wt * D / wmax)));
      std::vector<int> cuts;
      size_t j = 1;
      for (int k = 1; k < S && j < cs.size(); ++k, ++j) {
        const double goal = prefix[a] + wt * k / S;
        while (j + 1 < cs.size() &&
               std::fabs(prefix[cs[j + 1]] - goal) <= std::fabs(prefix[cs[j]] - goal))
          ++j;
        cuts.push_back(cs[j]);
      }
      cuts.push_back(b);
      int u = a;
      for (int v : cuts) {
        out.push_back(PlanPiece{t, u, v, -1, prefix[v] - prefix[u]});
        u = v;
      }
      npieces[t] = (int)cuts.size();  // a tile without units keeps one piece that writes zeros
    }
  };
  auto launch_time = [&](const std::vector<PlanPiece>& order) {
    std::vector<double> w;
    for (const PlanPiece& p : order) w.push_back(p.work + costs.workgroup);
    return simulate_launch(w, n_patches, slots);
  };
  LaunchPlan best;
  std::vector<PlanPiece> cur;
  std::vector<int> cur_np;
  for (int D = 1; D <= (allow_cut ? max_cut : 1); D += std::max(1, D / 4)) {
    cut(D, cur, cur_np);
    long long nslots = 0;
    for (int t = 0; t < nT; ++t) nslots += cur_np[t] > 1 ? cur_np[t] : 0;
    if (D > 1 && ((double)nslots * n_patches * slot_bytes > max_slot_bytes ||
                  cur.size() > 65535))  // rows of a grid
      break;
    std::vector<PlanPiece> heavy = cur;
    std::stable_sort(heavy.begin(), heavy.end(),
                     [](const PlanPiece& x, const PlanPiece& y) { return x.work > y.work; });
    double time = launch_time(cur);
    double time_heavy = launch_time(heavy);
    if (nslots > 0) {
      const double add =
          costs.add + costs.add_slot * *std::max_element(cur_np.begin(), cur_np.end());
      time += add;
      time_heavy += add;
    }
    const bool hf = time_heavy <= time;
    if (hf) {
      time = time_heavy;
      cur.swap(heavy);
    }
    if (D == 1) best.uncut_time = time;
    if (D == 1 || (time < 0.9 * best.uncut_time && time < best.time)) {
      best.pieces = cur;
      best.tile_pieces = cur_np;
      best.cut = D;
      best.heaviest_first = hf;
      best.time = time;
    } else if (D > 8 && time > 1.05 * best.time) {
      break;  // finer cuts only add workgroups and slots from here on
    }
  }
  // slots: consecutive per cut tile, in unit order
  best.tile_first_slot.assign(nT, -1);
  best.n_slots = 0;
  for (int t = 0; t < nT; ++t)
    if (best.tile_pieces[t] > 1) {
      best.tile_first_slot[t] = best.n_slots;
      best.n_slots += best.tile_pieces[t];
    }
  std::vector<int> order(best.pieces.size());
  for (size_t i = 0; i < order.size(); ++i) order[i] = (int)i;
  std::stable_sort(order.begin(), order.end(), [&](int x, int y) {
    return best.pieces[x].u0 < best.pieces[y].u0;
  });
  std::vector<int> seen(nT, 0);
  for (int i : order) {
    PlanPiece& p = best.pieces[i];
    if (best.tile_pieces[p.tile] > 1) p.slot = best.tile_first_slot[p.tile] + seen[p.tile]++;
  }
  return best;
}

}  // namespace aroam
