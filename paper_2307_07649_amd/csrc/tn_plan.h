// How the workgroups of a weight-gradient launch (k_gemm.hip, gemm_tn_kernel) are laid out: chunk lengths and placement on the
// eight XCDs.  Host code, plain C++.
#pragma once
#include <algorithm>
#include <cstring>
#include <functional>

namespace tgnn {

constexpr int TT = 64;          // bulk tile edge
constexpr int TN_ROWS = 32;     // row chunks are multiples of this
constexpr int TN_MAX_ROWS = 4096, TN_MIN_UNITS = 4;   // longest chunk that the plan looks at, and the shortest (a step per wavefront)
constexpr int TN_MAX_GROUP = 10;

// A length is cut into 64-wide pieces plus one narrower one (16, 32 or again 64 wide) for the remainder.  (A remainder of
// 33 .. 48 as a 32- and a 16-wide piece instead of a padded 64-wide one: fewer MFMAs, one more tile; measured on MI355X the
// extra tile costs more than the padding, 83 against 77 us on 4,000 events.)
constexpr int tn_pieces(int len) { return len / TT + (len % TT == 0 ? 0 : 1); }

// A problem as the plan sees it: rows (`counted`: an estimate of what the device has counted), columns of D and of A that its
// tiles cover (per head, with the column of ones), heads, tiles.
struct TnShape {
  int rows;
  bool counted;
  int n, k, heads, tiles;
};

// Workgroup b of the launch runs on XCD b % 8; the workgroups of XCD x form a queue of their own (position b / 8).  The queue has
// the problems one after the other: order qprob, starts qbegin[x], closed by the end of the queue and padded with INT_MAX (the
// kernel reads them with two scalar loads).  Of problem i, XCD x works on the chunks in mine[x][i], all tiles of a chunk in a
// row, so that the rows of a chunk are fetched into one L2 only; a bit stands for 2^shift chunks, so that a mask of 64 holds them.
struct TnPlan {
  unsigned long long mine[8][TN_MAX_GROUP];
  int qbegin[8][16];
  unsigned char qprob[16];
  int chunks[TN_MAX_GROUP];   // chunks | shift << 24
};
constexpr int tn_chunks(int word) { return word & 0xffffff; }
constexpr int tn_shift(int word) { return word >> 24; }
// rows per chunk
constexpr int tn_chunk_rows(int rows, int chunks) { return ((rows + chunks - 1) / chunks + TN_ROWS - 1) / TN_ROWS * TN_ROWS; }

// Chunking and placement.  A workgroup's life is a first wait for data, its share of the rows at the pace at which its
// compute unit's loads come in, and a reduction with one float atomic per tile element.  An XCD holds 64 workgroups at
// once (two per compute unit) and takes the rest of its queue as these end, so what a chunk length costs is decided by
// rounds.  The rule is the shortest chunks with which no queue exceeds TN_QUEUE workgroups, a round (chunks of TN_BASE_ROWS if
// that cannot be), unless a walk of the most loaded XCD's queue
// (tn_makespan) finds another length more than 15 % faster: the walk's constants are fitted to 18 launches of five shapes
// and its error is up to 20 %, so smaller differences mean nothing (taken for them, 80 -> 86 us on 4,000 events, 18.6 ->
// 21.9 on 600).  All problems of a launch use the same chunk length.  Queues of at most 60 / 64 / 80, launches in us: 4,000 events
// 69.8 / 69.8 / 70.0, edge classes 50.1 / 50.5 / 54.7, no edge features 19.8 / 20.8 / 19.8, four negative sets 26.9 / 27.2 /
// 27.2, stand-alone backward call 34.0 / 35.2 / 35.4, 600 events 20.2 all, eight replicas 110 all.
// What in-kernel timestamps say about such a launch: a workgroup sees its first rows 3 to 5 us after it starts
// (argument block, device-side row count, then the rows: three dependent round trips); the reduction and the atomics
// take 2 to 3 us.  Four wavefronts per workgroup, two workgroups per compute unit: one's reduction runs beside the
// other's products (eight: 108 against 90 us on a 4,000-event step, 21.7 against 18.3 us on a 600-event one, both with
// chunks of 1,024 rows at most).
constexpr int TN_SLOTS = 64;            // workgroups an XCD holds at once
constexpr int TN_QUEUE = 60, TN_BASE_ROWS = 2048, TN_MAX_CHUNKS = 64;
constexpr float TN_PLAN_GAIN = 0.85f;
constexpr float TN_COST_WG = 8.0f;      // us: start, reduction, atomics
constexpr float TN_COST_ROW = 0.020f;   // us per row of a 64 x 64 tile
constexpr float TN_COST_LOADS = 0.3f;   // share of that which follows the columns loaded, the rest follows the products

// Chunks of `rows_per_chunk` rows for every problem, of a long one no more than TN_MAX_CHUNKS as long as TN_BASE_ROWS rows each are
// enough for that: the workgroups of a tile all add to the same few lines of memory, one after the other, at 0.4 us per chunk
// (stand-alone backward call of d_m = 34, 19,404 rows: 64 chunks 31 us, 87 chunks 40).  Then the placement on the eight XCDs: chunks in order of decreasing
// size (tiles), each to the least loaded XCD so far.  (Dealt out in turn, chunk c to XCD (c + rotation) % 8, the longest queue
// was up to a fifth longer than the mean: 79 instead of 70 us on 4,000 events, 116 instead of 110 on eight replicas.)  Returns
// the length of the longest XCD queue.
inline int tn_place(TnPlan& plan, const TnShape* p, int n, int rows_per_chunk) {
  int order[TN_MAX_GROUP], load[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (int i = 0; i < n; ++i) order[i] = i;
  std::sort(order, order + n, [&](int a, int b) { return p[a].tiles != p[b].tiles ? p[a].tiles > p[b].tiles : a < b; });
  for (int oi = 0; oi < n; ++oi) {
    const int i = order[oi], rows = p[i].rows;
    int chunks = (rows + rows_per_chunk - 1) / rows_per_chunk, shift = 0;
    chunks = std::min(chunks, std::max(TN_MAX_CHUNKS, (rows + TN_BASE_ROWS - 1) / TN_BASE_ROWS));
    if (!p[i].counted) chunks = (rows + tn_chunk_rows(rows, chunks) - 1) / tn_chunk_rows(rows, chunks);
    while ((chunks - 1) >> shift >= 64) ++shift;
    plan.chunks[i] = chunks | shift << 24;
    plan.qprob[oi] = (unsigned char)i;
    for (int x = 0; x < 8; ++x) { plan.mine[x][i] = 0; plan.qbegin[x][oi] = load[x]; }
    for (int c = 0; c << shift < chunks; ++c) {
      const int x = (int)(std::min_element(load, load + 8) - load);
      plan.mine[x][i] |= 1ull << c;
      load[x] += p[i].tiles * (std::min((c + 1) << shift, chunks) - (c << shift));
    }
  }
  for (int x = 0; x < 8; ++x) {
    plan.qbegin[x][n] = load[x];
    for (int t = n + 1; t < 16; ++t) plan.qbegin[x][t] = 0x7fffffff;
  }
  return *std::max_element(load, load + 8);
}

// What the launch would take, after tn_place: the most loaded XCD's queue on TN_SLOTS slots, each taking the next workgroup
// as it gets free.
inline float tn_makespan(const TnPlan& plan, const TnShape* p, int n) {
  float cost[TN_MAX_GROUP][4][4], load[8];   // of a workgroup, by the widths of its tile in units of 16
  int chunks_of[8][TN_MAX_GROUP];
  for (int i = 0; i < n; ++i) {
    const int chunks = tn_chunks(plan.chunks[i]), r = (p[i].rows + chunks - 1) / chunks;
    for (int a = 0; a < 4; ++a)
      for (int b = 0; b < 4; ++b)
        cost[i][a][b] = TN_COST_WG + TN_COST_ROW * r * (TN_COST_LOADS * (a + b + 2) / 8.0f + (1.0f - TN_COST_LOADS) * (a + 1) * (b + 1) / 16.0f);
  }
  auto widths = [](int len, int idx) { const int r = len - idx * TT; return r > 32 ? 3 : r > 16 ? 1 : 0; };   // of piece idx, in 16s less one
  auto each_tile = [&](int i, auto&& f) {
    for (int h = 0; h < p[i].heads; ++h)
      for (int a = 0; a < tn_pieces(p[i].n); ++a)
        for (int b = 0; b < tn_pieces(p[i].k); ++b) f(cost[i][widths(p[i].n, a)][widths(p[i].k, b)]);
  };
  int worst = 0;
  for (int x = 0; x < 8; ++x) {
    load[x] = 0.f;
    for (int o = 0; o < n; ++o) {
      const int i = plan.qprob[o];
      chunks_of[x][o] = (plan.qbegin[x][o + 1] - plan.qbegin[x][o]) / p[i].tiles;
      float sum = 0.f;
      each_tile(i, [&](float c) { sum += c; });
      load[x] += sum * chunks_of[x][o];
    }
    if (load[x] > load[worst]) worst = x;
  }
  float heap[TN_SLOTS] = {}, end = 0.f;   // when each slot gets free, smallest at the front
  for (int o = 0; o < n; ++o)
    for (int c = 0; c < chunks_of[worst][o]; ++c)
      each_tile(plan.qprob[o], [&](float t) {
        std::pop_heap(heap, heap + TN_SLOTS, std::greater<float>());
        heap[TN_SLOTS - 1] += t;
        end = std::max(end, heap[TN_SLOTS - 1]);
        std::push_heap(heap, heap + TN_SLOTS, std::greater<float>());
      });
  return end;
}

// The chunk length (in units of TN_ROWS) for a launch.  Depends on the problems' shapes only; the last few are remembered, per
// thread, so that a program that calls an operator again does not walk the queues again.
inline int tn_chunk_units(const TnShape* p, int n) {
  struct Kept {
    int key[1 + 5 * TN_MAX_GROUP], units;
  };
  constexpr int KEEP = 8;
  static thread_local Kept kept[KEEP] = {};
  static thread_local int next = 0;
  Kept q = {};
  q.key[0] = n;
  int most = 0;
  for (int i = 0; i < n; ++i) {
    const int key[5] = {p[i].counted ? -p[i].rows : p[i].rows, p[i].n, p[i].k, p[i].heads, p[i].tiles};
    memcpy(q.key + 1 + 5 * i, key, sizeof(key));
    most = std::max(most, p[i].rows);
  }
  for (const Kept& k : kept)
    if (memcmp(k.key, q.key, sizeof(q.key)) == 0) return k.units;
  TnPlan plan;
  // the shortest chunks with which no queue exceeds TN_QUEUE (a round)
  int lo = TN_MIN_UNITS, hi = TN_BASE_ROWS / TN_ROWS;   // hi: taken if nothing smaller fits
  if (tn_place(plan, p, n, hi * TN_ROWS) <= TN_QUEUE)
    while (lo < hi) {
      const int mid = (lo + hi) / 2;
      if (tn_place(plan, p, n, mid * TN_ROWS) <= TN_QUEUE) hi = mid; else lo = mid + 1;
    }
  q.units = hi;
  tn_place(plan, p, n, hi * TN_ROWS);
  float best = TN_PLAN_GAIN * tn_makespan(plan, p, n);
  // lengths whose chunk counts differ for the longest problem
  int last = 0;
  for (int chunks = std::max(1, (most + TN_MAX_ROWS - 1) / TN_MAX_ROWS); chunks <= 64; chunks += 1 + chunks / 6) {
    const int units = std::max(TN_MIN_UNITS, ((most + chunks - 1) / chunks + TN_ROWS - 1) / TN_ROWS);
    if (units == last) { if (units == TN_MIN_UNITS) break; continue; }
    last = units;
    tn_place(plan, p, n, units * TN_ROWS);
    const float t = tn_makespan(plan, p, n);
    if (t < best) { best = t; q.units = units; }
  }
  kept[next] = q;
  next = (next + 1) % KEEP;
  return q.units;
}

}  // namespace tgnn
