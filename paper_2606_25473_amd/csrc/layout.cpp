// layout.cpp -- host side of the mask: chunk-layout validation, the query-group
// table, pair counts and the work-group tile order.  Plain C++17, no HIP.
#include "layout.hpp"

#include "args.hpp"
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <string>
#include <utility>
#include <vector>

namespace attn {

namespace {
// cut_tiles: tiles that end at group bounds may be this many more
constexpr double kMaxCutGrowth = 1.15;

bool fail(std::string* err, const std::string& msg) {
  if (err) *err = msg;
  return false;
}

// Open group n of the table: it owns rows up to q_end and has no key range yet.
void begin_group(GroupTable* gt, int q_end) {
  const int g = gt->n++;
  gt->q_end[g] = q_end;
  gt->r_begin[g + 1] = gt->r_begin[g];
}

// Append key range [k0, k1) (non-empty, after the group's last range and not touching
// it) to the last group.
bool add_range(GroupTable* gt, int k0, int k1, std::string* err) {
  const int r = gt->r_begin[gt->n];
  if (r == kMaxRanges)
    return fail(err, "more than " + std::to_string(kMaxRanges) + " key ranges in all (ATTN_MAX_RANGES)");
  gt->k[2 * r] = k0;
  gt->k[2 * r + 1] = k1;
  gt->r_begin[gt->n] = (uint16_t)(r + 1);
  return true;
}

std::string at_group(int g) { return " (group " + std::to_string(g) + ")"; }

// ATTN_MASK_RANGES: query-group bounds, per-group range offsets and key ranges.
bool build_range_list(const attn_chunk_layout* layout, int L, GroupTable* gt, std::string* err) {
  const int G = layout->num_chunks;
  if (G < 1 || G > ATTN_MAX_GROUPS)
    return fail(err, "number of query groups must be in [1, " + std::to_string(ATTN_MAX_GROUPS) + "], got " +
                         std::to_string(G));
  const int32_t* qb = layout->chunk_offsets;
  const int32_t* ro = layout->range_offsets;
  if (!qb) return fail(err, "chunk_offsets (the query-group bounds) is NULL");
  if (!ro) return fail(err, "range_offsets is NULL");
  if (qb[0] != 0) return fail(err, "the first query group must start at row 0");
  if (ro[0] != 0) return fail(err, "range_offsets[0] must be 0");
  for (int g = 0; g < G; ++g) {
    if (qb[g + 1] <= qb[g]) return fail(err, "query-group bounds must be strictly increasing" + at_group(g));
    if (ro[g + 1] < ro[g]) return fail(err, "range_offsets must not decrease" + at_group(g));
  }
  if (qb[G] != L)
    return fail(err, "query groups cover " + std::to_string(qb[G]) + " rows but L = " + std::to_string(L));
  const int32_t* rk = layout->ranges;
  if (ro[G] > 0 && !rk) return fail(err, "ranges is NULL");
  std::vector<std::pair<int, int>> K;
  for (int g = 0; g < G; ++g) {
    K.clear();
    for (int64_t r = ro[g]; r < ro[g + 1]; ++r) {
      const int k0 = rk[2 * r], k1 = rk[2 * r + 1];
      if (k0 < 0 || k0 > k1 || k1 > L)
        return fail(err, "key ranges must satisfy 0 <= begin <= end <= L" + at_group(g));
      if (k1 > k0) K.emplace_back(k0, k1);
    }
    std::sort(K.begin(), K.end());
    begin_group(gt, qb[g + 1]);
    for (size_t i = 0; i < K.size(); ++i) {
      if (i > 0 && K[i].first < K[i - 1].second) return fail(err, "key ranges overlap" + at_group(g));
      const int r = gt->r_begin[gt->n];
      if (i > 0 && K[i].first == K[i - 1].second) {
        gt->k[2 * r - 1] = K[i].second;  // touches the previous range: extend it
        continue;
      }
      if (!add_range(gt, K[i].first, K[i].second, err)) return false;
    }
  }
  return true;
}
}  // namespace

bool build_groups(const attn_chunk_layout* layout, int L, GroupTable* gt, std::string* err) {
  if (!layout) return fail(err, "layout is NULL");
  if (L <= 0) return fail(err, "sequence length L must be positive, got " + std::to_string(L));
  gt->n = 0;
  gt->r_begin[0] = 0;
  const int kind = layout->kind;
  if (kind == ATTN_MASK_FULL) {
    begin_group(gt, L);
    return add_range(gt, 0, L, err);
  }
  if (kind == ATTN_MASK_RANGES) return build_range_list(layout, L, gt, err);
  if (kind != ATTN_MASK_BLOCK_CAUSAL && kind != ATTN_MASK_TEACHER_FORCING)
    return fail(err, "unknown mask kind " + std::to_string(kind));
  const int N = layout->num_chunks;
  if (N < 1 || N > ATTN_MAX_CHUNKS)
    return fail(err, "num_chunks must be in [1, " + std::to_string(ATTN_MAX_CHUNKS) + "], got " +
                         std::to_string(N));
  const int32_t* o = layout->chunk_offsets;
  if (!o) return fail(err, "chunk_offsets is NULL");
  if (o[0] != 0) return fail(err, "chunk_offsets[0] must be 0");
  for (int i = 0; i < N; ++i)
    if (o[i + 1] <= o[i]) return fail(err, "chunk_offsets must be strictly increasing (index " +
                                               std::to_string(i + 1) + ")");
  const int half = o[N];
  if (kind == ATTN_MASK_BLOCK_CAUSAL) {
    if (L != half)
      return fail(err, "block-causal layout covers " + std::to_string(half) + " tokens but L = " +
                           std::to_string(L));
    for (int j = 0; j < N; ++j) {
      begin_group(gt, o[j + 1]);
      add_range(gt, 0, o[j + 1], err);
    }
    return true;
  }
  if ((int64_t)L != 2 * (int64_t)half)
    return fail(err, "teacher-forcing layout needs L = 2 * chunk_offsets[N] = " +
                         std::to_string(2 * (int64_t)half) + ", got L = " + std::to_string(L));
  // clean chunk j: clean chunks <= j (N ranges)
  for (int j = 0; j < N; ++j) {
    begin_group(gt, o[j + 1]);
    add_range(gt, 0, o[j + 1], err);
  }
  // noisy chunk i: clean chunks < i, then its own noisy chunk (2N - 1 ranges; 3N - 1 <=
  // kMaxRanges for N <= ATTN_MAX_CHUNKS)
  for (int i = 0; i < N; ++i) {
    begin_group(gt, half + o[i + 1]);
    if (i > 0) add_range(gt, 0, o[i], err);
    add_range(gt, half + o[i], half + o[i + 1], err);
  }
  return true;
}

int64_t count_pairs(const GroupTable& gt) {
  int64_t total = 0;
  for (int g = 0; g < gt.n; ++g) {
    const int64_t rows = gt.q_end[g] - group_q_begin(gt, g);
    int64_t keys = 0;
    for (int r = gt.r_begin[g]; r < gt.r_begin[g + 1]; ++r) keys += gt.k[2 * r + 1] - gt.k[2 * r];
    total += rows * keys;
  }
  return total;
}

int64_t count_computed_pairs(const GroupTable& gt, int L, int br, int bc) {
  int64_t total = 0;
  for (int q0 = 0; q0 < L; q0 += br) {
    const int q1 = q0 + br < L ? q0 + br : L;
    const TilePlan p = plan_tile(gt, q0, q1, bc);
    const int nb = plan_num_blocks(p);
    for (int i = 0; i < nb; ++i) {
      const int k0 = plan_block(p, i) * bc;
      const int k1 = k0 + bc < L ? k0 + bc : L;
      total += (int64_t)(q1 - q0) * (k1 - k0);
    }
  }
  return total;
}

namespace {
// keys of the group that admits most
int64_t most_keys(const GroupTable& gt) {
  int64_t longest = 0;
  for (int g = 0; g < gt.n; ++g) {
    int64_t keys = 0;
    for (int r = gt.r_begin[g]; r < gt.r_begin[g + 1]; ++r) keys += gt.k[2 * r + 1] - gt.k[2 * r];
    longest = std::max(longest, keys);
  }
  return longest;
}

// queries of the key that most admit: rows enter and leave at the ends of the key ranges
int64_t most_rows(const GroupTable& gt) {
  std::vector<std::pair<int, int>> ends;
  ends.reserve(2 * gt.r_begin[gt.n]);
  for (int g = 0; g < gt.n; ++g) {
    const int rows = gt.q_end[g] - group_q_begin(gt, g);
    for (int r = gt.r_begin[g]; r < gt.r_begin[g + 1]; ++r) {
      ends.emplace_back(gt.k[2 * r], rows);
      ends.emplace_back(gt.k[2 * r + 1], -rows);
    }
  }
  std::sort(ends.begin(), ends.end());  // (at one key, leaving rows come first)
  int64_t now = 0, longest = 0;
  for (const auto& e : ends) longest = std::max(longest, now += e.second);
  return longest;
}
}  // namespace

namespace {

// What a launch would take with tiles of one size (bf16), for the three rules below.
//
// A run is `n` tiles of one (batch, head) that walk `len` blocks of 32 each.
struct Run {
  double len, n;
};

// Rows (keys) [begin, end) that admit (are admitted by) `count` keys (rows).
struct Seg {
  int begin, end;
  double count;
};

// (segments of up to 32 rows together count as one)
void add_seg(std::vector<Seg>* s, const Seg& x) {
  if (!s->empty() && s->back().end == x.begin && x.end - s->back().begin <= 32) {
    s->back().end = x.end;
    s->back().count = std::max(s->back().count, x.count);
  } else {
    s->push_back(x);
  }
}

std::vector<Seg> query_segs(const GroupTable& gt) {
  std::vector<Seg> s;
  for (int g = 0; g < gt.n; ++g) {
    double keys = 0;
    for (int r = gt.r_begin[g]; r < gt.r_begin[g + 1]; ++r) keys += gt.k[2 * r + 1] - gt.k[2 * r];
    add_seg(&s, {group_q_begin(gt, g), gt.q_end[g], keys});
  }
  return s;
}

std::vector<Seg> key_segs(const GroupTable& gt) {
  std::vector<std::pair<int, int>> ends;  // rows enter and leave at the ends of the key ranges
  for (int g = 0; g < gt.n; ++g) {
    const int rows = gt.q_end[g] - group_q_begin(gt, g);
    for (int r = gt.r_begin[g]; r < gt.r_begin[g + 1]; ++r) {
      ends.emplace_back(gt.k[2 * r], rows);
      ends.emplace_back(gt.k[2 * r + 1], -rows);
    }
  }
  std::sort(ends.begin(), ends.end());
  std::vector<Seg> s;
  double now = 0;
  for (size_t i = 0; i < ends.size(); ++i) {
    now += ends[i].second;
    if (i + 1 == ends.size() || ends[i + 1].first == ends[i].first) continue;
    add_seg(&s, {ends[i].first, ends[i + 1].first, now});
  }
  return s;
}

// The runs of tiles of br rows.  Cut tiles end with their segment; of the others one per segment
// spans into the next ones and walks the blocks of both: span_blocks(begin, end) of them, or
// about the longest's where there are many segments.
template <class F>
void tile_runs(const std::vector<Seg>& segs, int br, bool cut, F span_blocks, std::vector<Run>* out) {
  out->clear();
  const int ns = (int)segs.size();
  for (int i = 0; i < ns; ++i) {
    double n = (double)(segs[i].end - segs[i].begin) / br, span = 0;
    if (cut) {
      n = std::ceil(n);
    } else if (i + 1 < ns) {
      double blocks = segs[i].count / kMfmaBc;
      if (ns <= kMaxSegs) {
        const int begin = std::max(0, segs[i].end - br / 2);
        blocks = span_blocks(begin, std::min(begin + br, segs[ns - 1].end));
      } else {
        for (int j = i + 1; j < ns && 2 * (segs[j].begin - segs[i].end) < br; ++j) blocks = std::max(blocks, segs[j].count / kMfmaBc);
      }
      span = std::min(n, 1.0);
      out->push_back({blocks, span});
    }
    if (!cut && i + 1 == ns) n += std::ceil((double)segs[i].end / br) - (double)segs[i].end / br;  // (the last tile)
    if (n > span) out->push_back({segs[i].count / kMfmaBc, n - span});
  }
}

// Blocks of 32 that a tile of rows (keys) [begin, end) walks.
auto query_blocks(const GroupTable& gt) {
  return [&gt](int begin, int end) { return (double)plan_num_blocks(plan_tile(gt, begin, end, kMfmaBc)); };
}
auto key_blocks(const GroupTable& gt) {
  return [&gt](int begin, int end) { return (double)plan_num_blocks(plan_key_tile(gt, begin, end, kMfmaBc)); };
}

// Measured times of a tile in us: of a round (one block of every split) and of the rest (plan,
// first loads, merge, stores).  A CU holds one tile of 8 waves, or up to three of 4 waves, whose
// rounds then take 1 + share (its other tiles) times as long.
struct TileCost {
  int br, splits;
  double step, fixed, share;
};

// Lengths within a sixteenth of each other count as one, so that few runs are left.
void merge_runs(std::vector<Run>* runs) {
  std::sort(runs->begin(), runs->end(), [](const Run& x, const Run& y) { return x.len > y.len; });
  size_t k = 0;
  double first = 0;
  for (const Run& r : *runs) {
    Run& m = (*runs)[k > 0 ? k - 1 : 0];
    if (k > 0 && r.len > 0.94 * first) {
      m.len = (m.len * m.n + r.len * r.n) / (m.n + r.n);
      m.n += r.n;
    } else {
      first = r.len;
      (*runs)[k++] = r;
    }
  }
  runs->resize(k);
}

// The launch: work-groups take the tiles as slot_of does, head group after head group, longest
// first in each, on the slot that is free first; at most kMaxFollowed runs are followed (or two
// head groups), the head groups before them fill the slots evenly.  A launch that leaves CUs idle
// runs at a higher clock (the card is at its power limit otherwise): with none busy but the
// longest tile's, a quarter faster.  (The rules take about 6 us of host time, at most 50, for launches
// of one to a few tiles per CU, and under 1 us for smaller and larger ones.)
constexpr int kMaxFollowed = 48;

double launch_cost(std::vector<Run>* runs, int nbh, int head_group, const TileCost& c) {
  double tiles = 0, work = 0, last = 0;  // (work: of one pair)
  for (const Run& r : *runs) tiles += r.n * nbh;
  const double others = c.share > 0 ? std::min(2.0, std::max(0.0, tiles / 256.0 - 1)) : 0;
  const double step = c.step * (1 + c.share * others), slots = 256.0 * (1 + std::ceil(others - 1e-9));
  auto time = [&](const Run& r) { return std::ceil(r.len / c.splits) * step + c.fixed; };
  if (tiles > slots) merge_runs(runs);
  for (const Run& r : *runs) {
    work += r.n * time(r);
    last = std::max(last, time(r));
  }
  if (tiles > slots) {
    const int groups = (nbh + head_group - 1) / head_group, follow = std::max(2, kMaxFollowed / (int)runs->size());
    const int h0 = std::max(0, groups - follow) * head_group;
    // how many slots are free from when on, earliest first
    using Free = std::pair<double, double>;
    std::vector<Free> heap{{work * h0 / slots, slots}};
    const auto later = [](const Free& x, const Free& y) { return x.first > y.first; };
    for (int h = h0; h < nbh; h += head_group) {
      for (const Run& r : *runs) {
        const double t = time(r);
        for (double n = r.n * std::min(head_group, nbh - h); n > 1e-3;) {
          Free f = heap.front();
          if (f.second - n < 1e-3) {  // the run takes every slot of this time
            std::pop_heap(heap.begin(), heap.end(), later);
            heap.pop_back();
          } else {
            heap.front().second -= n;
            f.second = n;
          }
          n -= f.second;
          f.first += t;
          last = std::max(last, f.first);
          heap.push_back(f);
          std::push_heap(heap.begin(), heap.end(), later);
        }
      }
    }
  }
  return last > 0 ? last * (0.75 + 0.25 * std::min(1.0, work * nbh / slots / last)) : 0;
}

// As cut_tiles would cut tiles of br rows.
bool tiles_are_cut(const GroupTable& gt, int L, int br) {
  if (gt.n < 2 || gt.n > kMaxSegs) return false;
  int nt = 0;
  for (int g = 0; g < gt.n; ++g) nt += (gt.q_end[g] - group_q_begin(gt, g) + br - 1) / br;
  return nt <= kMaxCutGrowth * ((L + br - 1) / br);
}

// Whether tiles of br rows, cut or not, all run at once: the smallest ones are then the best.
bool fit_at_once(int L, int nbh, int br) {
  return (int64_t)((L + br - 1) / br * kMaxCutGrowth + 1) * nbh <= 256;
}

// Full tiles per CU beyond which no split was faster in any measured launch.
constexpr int kMaxFullTilesPerCu = 4;
// A split of br rows has to promise this much of the full tiles' time at most, in its pass: the
// estimates are off by 5 % (half of the launches) to 20 % (one in ten), more where the tiles
// span many groups.  Where the forward and the JVP share the choice, the forward, which gains
// least, has to lose nothing.
double split_gain(const GroupTable& gt, int L, int nbh, int br) {
  if (L < 256 * gt.n) return 0.85;
  return (int64_t)((L + br - 1) / br) * nbh <= 256 ? 0.975 : 0.94;
}
struct SharedGain {
  double fwd, jvp;
};
SharedGain shared_gain(const GroupTable& gt, int L, int nbh, int br) {
  if (L < 256 * gt.n) return {1.0, 0.8};
  if ((int64_t)((L + br - 1) / br) * nbh <= 256) return {0.99, 0.97};
  return {0.97, 0.94};
}

}  // namespace

int choose_ksplit(const GroupTable& gt, int L, int nbh, int D) {
  // Forward, JVP and zero-clean JVP take the same tiles (their outputs agree bit for bit), so a
  // split must be worth it to the forward and to the JVP alike: the forward's full tiles have
  // 128 rows and 4 waves, three of which share a CU, the JVP's 256 rows.  Costs fitted to 1500
  // launches (full, block-causal, teacher-forcing and window masks, 1-40 heads, L = 64-30000): the
  // choice is 1.3 % (forward) and 2.4 % (JVP) off the best one on average, since one must serve
  // both; 6 forwards and 11 JVPs of them are more than 3 % slower than full tiles.  (With the
  // longest tile, the mean load and half a tile of tail alone: 93, and 2.5 and 3.4 % on average.)
  // Forward / JVP, us with full tiles and 2 and 4 splits:
  //   12 heads, D = 64, full, L = 1955                    44 /  73,   32 /  48,   36 /  59
  //    6 heads, D = 128, full, L = 5590                  154 / 295,  183 / 438,  179 / 400
  //    6 heads, D = 64, full, L = 11762                  301 / 874,  393 / 764,  359 / 740
  //    4 heads, D = 128, teacher forcing, L = 7866       143 / 317,   69 / 162,   77 / 171
  //    4 heads, D = 128, block-causal, L = 6460          138 / 335,  101 / 240,   75 / 167
  constexpr TileCost kFwdCost[2][3] = {
      {{128, 1, 0.51, 9.0, 0.32}, {128, 2, 0.70, 8.0, 0}, {64, 4, 0.75, 5.0, 0}},     // D = 64
      {{128, 1, 0.75, 10.0, 0.40}, {128, 2, 0.98, 10.5, 0}, {64, 4, 1.22, 6.8, 0}}};    // D = 128
  constexpr TileCost kJvpCost[2][3] = {
      {{256, 1, 1.28, 22.0, 0}, {128, 2, 1.36, 11.0, 0}, {64, 4, 1.55, 5.5, 0}},
      {{256, 1, 2.06, 40.0, 0}, {128, 2, 2.52, 16.0, 0}, {64, 4, 2.95, 10.0, 0}}};
  if ((int64_t)((L + kMfmaBr - 1) / kMfmaBr) * nbh > 256 * kMaxFullTilesPerCu) return 1;
  if (fit_at_once(L, nbh, kMfmaBr / 4)) return 4;
  const std::vector<Seg> segs = query_segs(gt);
  std::vector<Run> runs;
  int best = 1;
  double best_cost[2] = {0, 0};
  for (int i = 0; i < 3; ++i) {
    double c[2];
    for (int p = 0; p < 2; ++p) {
      const TileCost& tc = (p ? kJvpCost : kFwdCost)[D == 128][i];
      tile_runs(segs, tc.br, i > 0 && tiles_are_cut(gt, L, tc.br), query_blocks(gt), &runs);
      c[p] = launch_cost(&runs, nbh, kHeadGroup, tc);
    }
    // (4 splits against 2: the better for both)
    const SharedGain gain = best > 1 ? SharedGain{0.97, 0.97} : shared_gain(gt, L, nbh, kMfmaBr >> i);
    if (i == 0 || (c[0] <= gain.fwd * best_cost[0] && c[1] <= gain.jvp * best_cost[1])) {
      best = 1 << i;
      best_cost[0] = c[0];
      best_cost[1] = c[1];
    }
  }
  return best;
}

int choose_bwd_ksplit(const GroupTable& gt, int L, int nbh, int D) {
  // The same for the query-tile pass of the backward alone.  Backward call, us with full query
  // tiles and 2 and 4 splits (128-key tiles):
  //   12 heads, D = 128, full, L = 2753                   245 / 286 / 277
  //   40 heads, D = 64, block-causal, L = 840            59.7 / 67.6 / 63.2
  //    6 heads, D = 64, full, L = 11762                  1088 / 1045 / 992
  //    4 heads, D = 128, teacher forcing, L = 7866        368 / 262 / 266
  // (5 heads, D = 128, full, L = 73: 21.8 / 23.2 / 25.0, so the one tile of a short
  // sequence is not split.)
  if (D == 128 && L <= 4 * kMfmaBc && gt.n <= 4) return 1;
  constexpr TileCost kCost[2][3] = {{{256, 1, 0.50, 16.0, 0}, {128, 2, 0.50, 10.0, 0}, {64, 4, 0.50, 7.0, 0}},
                                    {{256, 1, 0.85, 29.0, 0}, {128, 2, 0.94, 16.5, 0}, {64, 4, 1.03, 11.7, 0}}};
  if ((int64_t)((L + kMfmaBr - 1) / kMfmaBr) * nbh > 256 * kMaxFullTilesPerCu) return 1;
  if (fit_at_once(L, nbh, kMfmaBr / 4)) return 4;
  const std::vector<Seg> segs = query_segs(gt);
  std::vector<Run> runs;
  int best = 1;
  double best_cost = 0;
  for (int i = 0; i < 3; ++i) {
    const TileCost& tc = kCost[D == 128][i];
    tile_runs(segs, tc.br, i > 0 && tiles_are_cut(gt, L, tc.br), query_blocks(gt), &runs);
    const double c = launch_cost(&runs, nbh, kHeadGroup, tc) / (i == 0 ? 1.0 : split_gain(gt, L, nbh, tc.br));
    if (i == 0 || c < best_cost) {
      best = 1 << i;
      best_cost = c;
    }
  }
  return best;
}

int choose_qsplit(const GroupTable& gt, int L, int nbh, int D) {
  // The key-tile pass.  Backward call, us with 128-key tiles / 64-key tiles (full query tiles):
  //   12 heads, D = 128, full, L = 2753                  245 / 234
  //    6 heads, D = 128, block-causal, L = 14718        1170 / 1251
  //   40 heads, D = 64, block-causal, L = 840           59.7 / 61.3
  //    4 heads, D = 128, teacher forcing, L = 7866       368 / 309
  constexpr TileCost kCost[2][2] = {{{kBwdKeysPerTile, 1, 0.67, 9.0, 0}, {kBwdKeysPerSplitTile, 2, 0.71, 6.7, 0}},
                                    {{kBwdKeysPerTile, 1, 1.06, 12.5, 0}, {kBwdKeysPerSplitTile, 2, 1.20, 8.5, 0}}};
  if ((int64_t)((L + kBwdKeysPerTile - 1) / kBwdKeysPerTile) * nbh > 2 * 256 * kMaxFullTilesPerCu) return 1;
  if (fit_at_once(L, nbh, kBwdKeysPerSplitTile)) return kBwdQuerySplits;
  const std::vector<Seg> segs = key_segs(gt);
  std::vector<Run> runs;
  double c[2];
  for (int i = 0; i < 2; ++i) {
    const TileCost& tc = kCost[D == 128][i];
    tile_runs(segs, tc.br, i > 0 && tiles_are_cut(gt, L, tc.br), key_blocks(gt), &runs);
    c[i] = launch_cost(&runs, nbh, kHeadGroupWide, tc);
  }
  return c[1] < (L < 256 * gt.n ? 0.85 : 0.975) * c[0] ? kBwdQuerySplits : 1;
}

int choose_f32_tiles(const GroupTable& gt, int L, int nbh, int D, F32Kernel kernel) {
  // 64-row tiles as long as twice as many tiles still fit the 256 CUs at once: a work-group then
  // has half the matrix work per block, but splits the block's rows into bf16 parts with half
  // as many threads.  Measured, us with 128 / 64 rows: JVP, D = 128, 2 heads, L = 1024 (16
  // tiles) 231 / 178; D = 64, 2 heads, teacher forcing L = 128 (2 tiles) 27 / 20.
  const int64_t tiles = (int64_t)((L + kF32Br - 1) / kF32Br) * nbh;
  if (tiles <= 128) return 2;
  // Beyond that at D = 128 where the tangent's or the backward's longest tile outlasts the mean
  // load by enough (a 64-row step takes 0.77 of a 128-row one).  The forward and D = 64 share a
  // CU between two 64-row work-groups, whose steps then take as long as the larger ones'.
  // Measured, us with 128 / 64 rows, D = 128:
  //                                          JVP          backward     forward
  //   5 heads, block-causal, L = 4000    713 /  642    943 /  781    322 / 414
  //   8 heads, block-causal, L = 3251    586 /  514    751 /  695    267 / 303
  //   8 heads, full, L = 3000            547 /  848    714 / 1097    248 / 298
  //   3 heads, teacher f., L = 12480    1160 / 1529   2109 / 1979    505 / 577
  //     (64-key tiles and 128-row query tiles, as chosen here:  1714)
  //   12 heads, teacher f., L = 6552    1248 / 1449   1752 / 2128    538 / 620
  // and at D = 64 (5 heads, block-causal, L = 4000) 404 / 486, 542 / 575, 206 / 221.
  if (D == 64 || kernel == F32Kernel::kForward) return 1;
  constexpr double kStep[2] = {1.0, 0.77}, kFixed = 4.0, kCus = 256.0, kTail = 0.35;
  const double longest = (double)(kernel == F32Kernel::kKeyTiles ? most_rows(gt) : most_keys(gt)) / 32.0;
  const double steps = (double)count_pairs(gt) * nbh / (32.0 * kF32Br);  // of 128 rows, over all tiles
  double cost[2];
  for (int i = 0; i < 2; ++i) {
    const int br = kF32Br >> i;
    const double n = (double)((L + br - 1) / br) * nbh;
    const double total = kStep[i] * (1 + i) * steps + n * kFixed;
    cost[i] = std::max(kStep[i] * longest + kFixed, n > kCus ? total / kCus + kTail * total / n : 0.0);
  }
  return cost[1] < cost[0] ? 2 : 1;
}

TileOrder make_tile_order(const attn_chunk_layout* layout, int L, int br) {
  TileOrder o{};
  o.nt = (L + br - 1) / br;
  o.split = o.nt;
  o.first = -1;
  o.mode = 0;
  if (layout->kind == ATTN_MASK_BLOCK_CAUSAL) o.mode = 1;
  if (layout->kind == ATTN_MASK_TEACHER_FORCING) {
    o.mode = 2;
    const int half = L / 2;
    o.split = (half + br - 1) / br;  // the tile holding the clean/noisy boundary counts as clean
  }
  return o;
}

void cut_tiles(TileOrder* o, const GroupTable& gt, int L, int br) {
  // A tile that spans a bound visits the union of both groups' blocks and masks them all; it is
  // one of the longest of its launch.  Cutting leaves a part-filled tile per group instead, which
  // pays while the tiles grow by at most 15 % (measured, JVP, 3 heads, teacher forcing with two
  // chunks of 1560: 116 us spanning, 90 us cut, 98 and 100 tiles per head).
  if (gt.n < 2 || gt.n > kMaxSegs) return;
  int nt = 0;
  for (int g = 0; g < gt.n; ++g) {
    const int rows = gt.q_end[g] - group_q_begin(gt, g);
    o->row[g] = group_q_begin(gt, g);
    o->tile[g] = nt;
    nt += (rows + br - 1) / br;
  }
  if (nt > kMaxCutGrowth * ((L + br - 1) / br)) return;
  o->row[gt.n] = L;
  o->tile[gt.n] = nt;
  o->nseg = gt.n;
  // the first tile of the upper half of the order (teacher forcing: the half is a bound)
  if (o->mode == 2)
    for (int g = 0; g < gt.n; ++g)
      if (o->row[g] <= L / 2) o->split = o->tile[g];
  o->nt = nt;
  if (o->mode != 2) o->split = nt;
}

TileOrder make_tile_order_zero_clean(const GroupTable& gt, int L, int br, int bc, int t0, const TileOrder* cuts) {
  TileOrder o{};
  o.nt = (L + br - 1) / br;
  o.split = t0 / br;  // tiles wholly below t0 need the primal only; the boundary tile is upper
  o.first = -1;
  o.mode = 2;
  bool straddle = t0 % br != 0;
  if (cuts && cuts->nseg > 0) {  // (t0 is a bound)
    o = *cuts;
    straddle = false;
  }
  if (o.nt - (straddle ? 1 : 0) > kMaxMergeTiles) return o;  // merge bits for at most this many
  // Cost of a tile in key-block contractions: 2 per block (scores, output) for a tile
  // without tangent rows, 4 per block of keys without tangents (+ the dQ term of the
  // score tangent and the H~ term of the output tangent), 6 per block with tangent keys.
  auto cost = [&](int t) {
    int q0, q1;
    tile_rows(o, t, br, L, &q0, &q1);
    const TilePlan p = plan_tile(gt, q0, q1, bc);
    const int64_t nb = plan_num_blocks(p), clean = plan_blocks_below(p, t0 / bc);
    return q1 <= t0 ? 2 * nb : 4 * clean + 6 * (nb - clean);
  };
  o.mode = 3;
  // A tile straddling t0 holds the last clean chunk, which sees every clean key with
  // the dQ term: one of the heaviest tiles, and out of place at the low end of the
  // upper half.  It goes first.
  int lo = o.split - 1, hi = o.nt - 1, stop = o.split;
  if (straddle) {
    o.first = o.split;
    stop = o.split + 1;
  }
  int64_t clo = lo >= 0 ? cost(lo) : 0, chi = hi >= stop ? cost(hi) : 0;
  for (int t = 0; t < o.nt - (o.first >= 0 ? 1 : 0); ++t) {
    const bool take_hi = lo < 0 || (hi >= stop && chi >= clo);
    if (take_hi) {
      o.merge[t >> 5] |= 1u << (t & 31);
      --hi;
      chi = hi >= stop ? cost(hi) : 0;
    } else {
      --lo;
      clo = lo >= 0 ? cost(lo) : 0;
    }
  }
  return o;
}

}  // namespace attn
