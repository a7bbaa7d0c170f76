// Planner of the cell launches: splits the variables into at most two stages whose connected
// components are small, packs components into cells (one workgroup's LDS each) and writes each
// cell's program.
//
// Why stages. Take any prefix A of the processing order and the rest B. Along every row the levels
// of A come before those of B, so the forward pass is A's part, then B's part, and the backward pass
// is B's part, then A's part. Two variables of B that are not connected through rows by variables
// of B exchange nothing inside B's part, and the same holds for A. So an iteration is: A forward,
// B forward and backward (each component of B by itself), A backward, and over a run of iterations
// A's backward part and the next iteration's forward part join too. A component's inner messages
// never leave the workgroup that runs it: they are functions of the multipliers (the backward
// sweep of the multipliers, or the forward sweep), recomputed in LDS instead of being kept in HBM.
// On a grid MRF the order lists all unaries before all pairwise variables: A's components are the
// nodes, B's the edges.
//
// Visiting a component's variables by local steps (longest chain of row predecessors inside the
// component) follows every row's order, so the iterates are those of the sequential algorithm.
#include <algorithm>
#include <atomic>
#include <exception>
#include <mutex>
#include <numeric>
#include <thread>
#include <unordered_map>

#include "internal.h"

namespace bddmp {

namespace {

// bytes of LDS one layer takes: multiplier, link, its share of a row part; descriptors too unless the
// plan has levels of more than two nodes (those stages keep them in global memory, and 18 bytes for the
// 15 a layer takes keep the largest cell under kCellMaxLayers)
int32_t layer_weight(int32_t wc, bool wide_plan) { return wide_plan ? 18 + (wc > 2 ? 8 : 0) : 22; }

struct UnionFind {
  std::vector<int32_t> up, size;
  int32_t largest = 0;
  explicit UnionFind(int32_t n) : up(size_t(n)), size(size_t(n)) {}
  void clear() { largest = 0; }
  void add(int32_t i, int32_t w) {
    up[size_t(i)] = i;
    size[size_t(i)] = w;
    largest = std::max(largest, w);
  }
  int32_t find(int32_t i) {
    while (up[size_t(i)] != i) {
      up[size_t(i)] = up[size_t(up[size_t(i)])];
      i = up[size_t(i)];
    }
    return i;
  }
  void join(int32_t a, int32_t b) {
    a = find(a);
    b = find(b);
    if (a == b) return;
    if (size[size_t(a)] < size[size_t(b)]) std::swap(a, b);
    up[size_t(b)] = a;
    size[size_t(a)] += size[size_t(b)];
    largest = std::max(largest, size[size_t(a)]);
  }
};

// chunks [b, e) of [0, n) on host threads, first exception rethrown
template <class F>
void on_threads(int64_t n, int64_t min_chunk, F &&f) {
  const unsigned hw = std::thread::hardware_concurrency();
  const int64_t nt = std::min<int64_t>({int64_t(hw ? hw : 1), 16, (n + min_chunk - 1) / min_chunk});
  if (nt <= 1) {
    if (n > 0) f(int64_t(0), n);
    return;
  }
  const int64_t chunk = (n + nt - 1) / nt;
  std::exception_ptr err;
  std::mutex mu;
  auto run = [&](int64_t k) {
    try {
      if (k * chunk < n) f(k * chunk, std::min(n, (k + 1) * chunk));
    } catch (...) {
      std::lock_guard<std::mutex> lk(mu);
      if (!err) err = std::current_exception();
    }
  };
  std::vector<std::thread> th;
  int64_t k = 1;
  try {
    for (; k < nt; ++k) th.emplace_back(run, k);
  } catch (...) {
    for (; k < nt; ++k) run(k);
  }
  run(0);
  for (auto &t : th) t.join();
  if (err) std::rethrow_exception(err);
}

// cells to a host thread, at least: some 16384 layers, however large the cells
int64_t cell_share(int64_t cells, int64_t layers) {
  return std::max<int64_t>(1, cells * 16384 / std::max<int64_t>(layers, 1));
}

}  // namespace

// Chooses the stages: per instance the cut of its processing order that makes A's and B's largest
// components together smallest (no cut, everything in B, when the whole instance fits one workgroup).
// The stages run one after the other and a large component's steps in sequence, so the sum follows the
// time: tracking chains are cut above their links and not in their middle, 32 of them with 200 to 1967
// detections 141 us per iteration instead of 177. Leaves P.cell_kind 0 when no cut brings the components
// within a workgroup's LDS.
void choose_cells(const Problem &p, Plan &P, const std::vector<int64_t> &iptr, const std::vector<int32_t> &ilist,
                  const std::vector<int32_t> &inc_row) {
  P.cell_kind = 0;
  if (P.n_cuts || P.I == 0 || P.max_j > kCellMaxRows || P.max_width > kCellMaxWidth) return;
  const int32_t n = P.n;
  std::vector<int32_t> wt(size_t(n), 0);
  for (int32_t i = 0; i < n; ++i)
    for (int64_t q = iptr[size_t(i)]; q < iptr[size_t(i) + 1]; ++q) {
      const int32_t c = ilist[size_t(q)], j = inc_row[size_t(c)];
      const Shape &sh = P.shapes[size_t(P.row_shape[size_t(j)])];
      const int32_t l = int32_t(c - P.canon_off[size_t(j)]);
      wt[size_t(i)] += layer_weight(l + 1 < sh.k ? sh.first[size_t(l) + 2] - sh.first[size_t(l) + 1] : 0, P.max_width > 2);
    }
  // each instance's variables in processing order
  std::vector<int64_t> iv = p.inst_var.empty() ? std::vector<int64_t>{0, n} : p.inst_var;
  const size_t n_inst = iv.size() - 1;
  std::vector<int32_t> ord(static_cast<size_t>(n));
  if (n_inst == 1) {
    ord = P.order;
  } else {
    std::vector<int32_t> inst_of(size_t(n), 0);
    for (size_t k = 0; k < n_inst; ++k)
      for (int64_t i = iv[k]; i < iv[k + 1]; ++i) inst_of[size_t(i)] = int32_t(k);
    std::vector<int64_t> fill(iv.begin(), iv.end() - 1);
    for (int32_t i : P.order) ord[size_t(fill[size_t(inst_of[size_t(i)])]++)] = i;
  }
  UnionFind uf(n);
  std::vector<uint8_t> in(size_t(n), 0);
  auto add = [&](int32_t i, int dir) {
    uf.add(i, wt[size_t(i)]);
    in[size_t(i)] = 1;
    for (int64_t q = iptr[size_t(i)]; q < iptr[size_t(i) + 1]; ++q) {
      const int64_t c = ilist[size_t(q)], j = inc_row[size_t(c)];
      const int64_t o = c + dir;
      if (o < P.canon_off[size_t(j)] || o >= P.canon_off[size_t(j) + 1]) continue;
      const int32_t v = P.inc_var[size_t(o)];
      if (in[size_t(v)]) uf.join(i, v);
    }
  };
  std::vector<int64_t> cut(n_inst, 0);
  std::vector<int32_t> largest;  // of the prefix of each length
  bool two = false;
  for (size_t k = 0; k < n_inst; ++k) {
    const int64_t v0 = iv[k], v1 = iv[k + 1];
    uf.clear();
    largest.assign(1, 0);
    for (int64_t r = v0; r < v1; ++r) {
      add(ord[size_t(r)], -1);
      if (uf.largest > kCellLdsMax) break;
      largest.push_back(uf.largest);
    }
    for (int64_t r = v0; r < v1; ++r) in[size_t(ord[size_t(r)])] = 0;
    const int64_t rmax = int64_t(largest.size()) - 1;  // longest prefix that fits
    if (rmax == v1 - v0) continue;                     // the whole instance fits: no cut
    uf.clear();
    int64_t best = -1;
    std::pair<int32_t, int32_t> cost{INT32_MAX, INT32_MAX};
    for (int64_t r = v1 - v0; r >= 0; --r) {
      if (r < v1 - v0) add(ord[size_t(v0 + r)], 1);
      if (uf.largest > kCellLdsMax || uf.largest > cost.first) break;
      if (r > rmax) continue;
      const int32_t a = largest[size_t(r)], b = uf.largest;
      const std::pair<int32_t, int32_t> c{a + b, std::max(a, b)};
      if (c < cost) {
        cost = c;
        best = r;
      }
    }
    for (int64_t r = v0; r < v1; ++r) in[size_t(ord[size_t(r)])] = 0;
    if (best < 0) return;
    cut[k] = best;
    two = true;
  }
  // components of each stage, numbered by first appearance
  P.var_stage.assign(size_t(n), 1);
  P.var_comp.assign(size_t(n), -1);
  for (size_t k = 0; k < n_inst; ++k)
    for (int64_t r = 0; r < cut[k]; ++r) P.var_stage[size_t(ord[size_t(iv[k] + r)])] = 0;
  uf.clear();
  for (int32_t i : ord) {
    uf.add(i, wt[size_t(i)]);
    for (int64_t q = iptr[size_t(i)]; q < iptr[size_t(i) + 1]; ++q) {
      const int64_t c = ilist[size_t(q)];
      if (c == P.canon_off[size_t(inc_row[size_t(c)])]) continue;
      const int32_t v = P.inc_var[size_t(c) - 1];
      if (P.var_stage[size_t(v)] == P.var_stage[size_t(i)]) uf.join(i, v);
    }
  }
  std::vector<int32_t> id(size_t(n), -1);
  int32_t next = 0;
  for (int32_t i : ord) {
    if (!P.var_nj[size_t(i)]) continue;
    int32_t &c = id[size_t(uf.find(i))];
    if (c < 0) c = next++;
    P.var_comp[size_t(i)] = c;
  }
  P.n_comp = next;
  P.cell_kind = two ? 2 : 1;
  // B's components follow the first component of A they hang on, so that neighbours in storage share
  // what A hands on (on a grid the edges then follow their nodes, however the order lists them)
  std::vector<int32_t> key(static_cast<size_t>(next)), by(static_cast<size_t>(next)), to(static_cast<size_t>(next));
  for (int32_t c = 0; c < next; ++c) key[size_t(c)] = by[size_t(c)] = c;
  for (int32_t i : ord) {
    if (!P.var_nj[size_t(i)] || P.var_stage[size_t(i)] == 0) continue;
    for (int64_t q = iptr[size_t(i)]; q < iptr[size_t(i) + 1]; ++q) {
      const int64_t c = ilist[size_t(q)];
      if (c == P.canon_off[size_t(inc_row[size_t(c)])]) continue;
      const int32_t v = P.inc_var[size_t(c) - 1];
      if (P.var_stage[size_t(v)] == 0) key[size_t(P.var_comp[size_t(i)])] = std::min(key[size_t(P.var_comp[size_t(i)])], P.var_comp[size_t(v)]);
    }
  }
  std::stable_sort(by.begin(), by.end(), [&](int32_t a, int32_t b) { return key[size_t(a)] < key[size_t(b)]; });
  for (int32_t c = 0; c < next; ++c) to[size_t(by[size_t(c)])] = c;
  for (int32_t i : ord)
    if (P.var_comp[size_t(i)] >= 0) P.var_comp[size_t(i)] = to[size_t(P.var_comp[size_t(i)])];
}

namespace {

// Lanes of a stage's workgroups and the layers a cell is filled up to. total: layers of the stage;
// largest: the layers of each step of its largest component (big in all).
//
// Small components go to one-wavefront cells, whose steps need no barrier. Cells of two-row variables
// (one lane each) hold up to 1024 layers, others (one lane per layer) up to 256: a step then fills about
// one wavefront on the grid workloads, and ten or more cells fit a compute unit's LDS. Measured, us per
// iteration with pairs of 512 / 1024 / 2048: Potts 256x256x8 165 / 168 / 233, 128x128x4 25 / 28 / 36, 300x300x4
// 65 / 75 / 99, 40x40x16 57 / 52 / 54 (512 would be the better line for up to eight labels); others of 128 / 256
// / 512: Potts 256x256x8 181 / 168 / 174, 128x128x4 28 / 28 / 39, a million layers of random pairs 9 / 11 / 15,
// of disjoint rows of ten 22 / 13 / 11. Plans of few cells share the layers out so that every compute unit
// gets two, down to 64 layers: total / 256, / 512, / 1024 on 64x64x4 24.3, 20.0, 19.1, on 32x32x8 29.2, 28.3,
// 28.6; at least 32, 64, 128, 256 layers on 16x16x4 16.1, 15.8, 16.6, 18.1.
//
// A larger component is a cell by itself, on the fewest lanes that take at most a quarter more chunks
// than 512 lanes would: 64, 128, 256, 512 lanes on Potts 8x8x3 45, 26, 16, 10.5, on a component of eight steps
// of 600 layers 94, 52, 33, 22; 256 are taken for a tracking instance of 1400 detections, 148, 93, 80, 73, and
// for 5x5x2 9.9, 6.9, 5.2, 5.1 (512 would gain up to 9% there).
void cell_shape(int32_t big, int64_t total, const std::vector<int32_t> &largest, bool pairs, int32_t &block, int32_t &room) {
  const int32_t most = pairs ? 1024 : 256;
  if (big <= most) {
    block = 64;
    room = int32_t(std::min<int64_t>(most, std::max<int64_t>(total / 512, 64)));
    return;
  }
  auto chunks = [&](int32_t b) {
    int64_t n = 0;
    for (int32_t c : largest) n += (c + b - 1) / b;
    return n;
  };
  block = 64;
  while (block < 512 && 4 * chunks(block) > 5 * chunks(512)) block *= 2;
  room = big;
}

// regular levels (lo0, hi0, lo1, hi1 as 2-bit codes): 0-arcs keep the node, and either node 0's 1-arc
// moves to node 1 (a counting level) or node 1's to node 0 (a taking level)
constexpr uint32_t kArcsCount = 0u | (1u << 2) | (1u << 4) | (kC2Bot << 6);
constexpr uint32_t kArcsTake = 0u | (kC2Bot << 2) | (1u << 4) | (0u << 6);

// The arcs of a narrow layer for the cell kernels: a last level's terminals become the values x0, y0
// (0 if set, else +inf) behind nodes 0 and 1 of a virtual child level, chosen so that the level is
// regular where it can be; a root's second node never carries a message, so its arcs are free.
uint32_t cell_arcs(uint32_t arcs, bool last, bool root, bool &x0, bool &y0) {
  x0 = y0 = false;
  auto code = [](uint32_t a, int q) { return (a >> (2 * q)) & 3u; };
  const int used = root ? 2 : 4;
  for (uint32_t pat : {kArcsCount, kArcsTake})
    for (int xy = 0; xy < (last ? 4 : 1); ++xy) {
      // bit 0 of xy: the virtual node 0 is TOP, bit 1: node 1
      bool ok = true;
      for (int q = 0; q < used && ok; ++q) {
        const uint32_t c = code(pat, q), o = code(arcs, q);
        ok = last ? (c < 2u && ((xy >> c) & 1)) == (o == kC2Top) : c == o;
      }
      if (ok) {
        x0 = xy & 1;
        y0 = xy & 2;
        return pat;
      }
    }
  if (!last) return arcs;
  // TOP as virtual node 0
  uint32_t out = 0;
  for (int q = 0; q < 4; ++q) out |= (code(arcs, q) == kC2Top ? 0u : kC2Bot) << (2 * q);
  x0 = true;
  return out;
}

// one cell's program, before the arrays of equal cells are shared
struct CellProg {
  // per layer: area of the parent's link | kCellCount, w1, child and parent layer (0xFFFF: not in the
  // cell); step: first layer of each step, then the end; plans with wide levels: own area and arcs
  std::vector<uint32_t> h, w1, kid, dad, row, step, own, arc;
  int32_t nl = 0, ns = 0, xa = 0;  // layers, steps, areas
  bool pairs = true;               // every variable in two rows, every level regular
  bool wide = false;               // some level or child level has more than two nodes
  void clear() {
    for (auto *v : {&h, &w1, &kid, &dad, &row, &step, &own, &arc}) v->clear();
    nl = ns = xa = 0;
    pairs = true;
    wide = false;
  }
  uint64_t hash() const {
    uint64_t x = 1469598103934665603ull;
    auto mix = [&](uint64_t v) { x = (x ^ v) * 1099511628211ull; x ^= x >> 29; };
    for (const auto *a : {&h, &w1, &kid, &dad, &row, &step, &own, &arc}) {
      for (uint32_t v : *a) mix(v);
      mix(a->size());
    }
    mix(uint64_t(uint32_t(xa)));
    return x;
  }
  bool same(const CellProg &o) const {
    return nl == o.nl && ns == o.ns && xa == o.xa && h == o.h && w1 == o.w1 && kid == o.kid && dad == o.dad && row == o.row &&
           step == o.step && own == o.own && arc == o.arc;
  }
};

struct CellBuilder {
  const Plan &P;
  const std::vector<int32_t> &ownw, &childw, &vstep;
  int32_t bwp;                 // pairs of floats per link above a row part
  std::vector<uint16_t> &loc;  // local index of each layer in its cell

  bool same_stage(int32_t L, uint8_t st) const { return L >= 0 && P.var_stage[size_t(P.layer_var[size_t(L)])] == st; }

  // layers (with pads) and row parts of the cell of these variables; false when they are too many
  bool measure(const int32_t *vars, size_t nv, int32_t &nl, int32_t &nrow) const {
    const uint8_t st = nv ? P.var_stage[size_t(vars[0])] : 0;
    int32_t j = 0, s0 = 0, cur = -1;
    nl = nrow = 0;
    for (size_t k = 0; k < nv; ++k) {
      const int32_t i = vars[k], nj = P.var_nj[size_t(i)];
      if (vstep[size_t(i)] != cur) {
        cur = vstep[size_t(i)];
        s0 = j;
      }
      if (((j - s0) & 63) + nj > 64) j = s0 + ((j - s0 + 63) & ~63);
      j += nj;
      if (j >= kCellMaxLayers) return false;
      for (int32_t q = 0; q < nj; ++q) nrow += !same_stage(P.parent[size_t(P.var_first[size_t(i)] + q)], st);
    }
    nl = (j + 3) & ~3;
    return true;
  }

  // vars: the cell's variables by (step, storage), as measured; layer: the storage layer of each local
  // one. False when the program's fields overflow.
  bool build(const int32_t *vars, size_t nv, CellProg &C, int32_t *layer) const {
    C.clear();
    // local indices: steps one after another, a variable's layers never across a 64-lane boundary of
    // its step (pads hold no layer)
    int32_t j = 0, s0 = 0, cur = -1;
    std::vector<int32_t> at(nv);
    for (size_t k = 0; k < nv; ++k) {
      const int32_t i = vars[k], nj = P.var_nj[size_t(i)];
      if (vstep[size_t(i)] != cur) {
        cur = vstep[size_t(i)];
        s0 = j;
        C.step.push_back(uint32_t(j));
      }
      if (((j - s0) & 63) + nj > 64) j = s0 + ((j - s0 + 63) & ~63);
      at[k] = j;
      for (int32_t q = 0; q < nj; ++q) loc[size_t(P.var_first[size_t(i)] + q)] = uint16_t(j + q);
      j += nj;
    }
    const bool wide_plan = P.max_width > 2;
    C.nl = (j + 3) & ~3;
    C.ns = int32_t(C.step.size());
    C.step.push_back(uint32_t(j));
    C.h.assign(size_t(C.nl), 0u);
    C.w1.assign(size_t(C.nl), 0u);
    C.kid.assign(size_t(C.nl), 0xFFFFu);
    if (wide_plan) {
      C.dad.assign(size_t(C.nl), 0xFFFFu);
      C.own.assign(size_t(C.nl), 0u);
      C.arc.assign(4 * size_t(C.nl), 0u);
    }
    auto each = [&](auto &&f) {
      for (size_t k = 0; k < nv; ++k)
        for (int32_t q = 0; q < P.var_nj[size_t(vars[k])]; ++q) f(vars[k], q, P.var_first[size_t(vars[k])] + q, at[k] + q);
    };
    const uint8_t st = nv ? P.var_stage[size_t(vars[0])] : 0;
    // row parts, numbered by their first layer; each layer's row part by its walk
    std::vector<int32_t> part(size_t(C.nl), -1), link(size_t(C.nl), 0);
    each([&](int32_t, int32_t, int32_t L, int32_t jj) {
      if (same_stage(P.parent[size_t(L)], st)) return;
      const int32_t k = int32_t(C.row.size());
      int32_t e = L;
      for (;; e = P.child[size_t(e)]) {
        part[loc[size_t(e)]] = k;
        if (!same_stage(P.child[size_t(e)], st)) break;
      }
      C.row.push_back(uint32_t(jj) | uint32_t(loc[size_t(e)]) << 13);
    });
    C.xa = C.nl + int32_t(C.row.size()) * bwp;
    each([&](int32_t, int32_t, int32_t L, int32_t jj) {
      link[size_t(jj)] = jj;
      if (childw[size_t(L)] > 2) {
        link[size_t(jj)] = C.xa;
        C.xa += (childw[size_t(L)] + 1) / 2;
      }
      C.wide = C.wide || ownw[size_t(L)] > 2 || childw[size_t(L)] > 2;
    });
    C.xa = (C.xa + 1) & ~1;
    if (wide_plan) C.xa += 2;  // the constants
    if (C.xa > 0x7FFF) return false;
    each([&](int32_t i, int32_t q, int32_t L, int32_t jj) {
      const uint32_t meta = P.meta[size_t(L)];
      const int32_t ch = P.child[size_t(L)], pa = P.parent[size_t(L)], k = part[size_t(jj)], nj = P.var_nj[size_t(i)];
      const bool inner_c = same_stage(ch, st), inner_p = same_stage(pa, st), last = ch < 0, root = pa <= -2;
      const int32_t w = ownw[size_t(L)], wc = childw[size_t(L)];
      uint32_t h = uint32_t(inner_p ? link[loc[size_t(pa)]] : C.nl + k * bwp);
      uint32_t w1 = uint32_t(nj) | uint32_t(q) << kCellPosShift | (last ? kCellLast : 0u);
      if (inner_c) C.kid[size_t(jj)] = uint32_t(loc[size_t(ch)]);
      bool x0 = false, y0 = false;
      if (w > 2 || wc > 2) {
        C.pairs = false;
      } else {
        const uint32_t arcs = cell_arcs(meta & 0xFFu, last, root, x0, y0);
        w1 |= arcs << 16;
        if (arcs == kArcsCount) h |= kCellCount;
        C.pairs = C.pairs && nj == 2 && (arcs == kArcsCount || arcs == kArcsTake);
      }
      if (wide_plan) {
        if (inner_p) C.dad[size_t(jj)] = uint32_t(loc[size_t(pa)]);
        C.own[size_t(jj)] = uint32_t(link[size_t(jj)]) | uint32_t(w) << 16 | uint32_t(wc) << 20;
        const uint32_t consts = 2u * uint32_t(C.xa - 2), f0 = 2u * uint32_t(link[size_t(jj)]);
        auto at_float = [&](uint32_t c) { return c < kTop ? f0 + c : consts + (c == kTop ? 0u : 1u); };
        for (int32_t u = 0; u < 4; ++u) {
          const uint32_t a = u < w ? P.garcs[size_t(P.own_slot[size_t(L)] + u)] : kBot | kBot << 16;
          C.arc[4 * size_t(jj) + size_t(u)] = at_float(a & 0xFFFFu) | at_float(a >> 16) << 16;
        }
      }
      uint32_t &r = C.row[size_t(k)];
      if (root) r |= kCellRowRoot;
      if (last) r |= kCellRowLast | (x0 ? kCellRowTermX : 0u) | (y0 ? kCellRowTermY : 0u);
      C.h[size_t(jj)] = h;
      C.w1[size_t(jj)] = w1;
      layer[jj] = L;
    });
    return true;
  }
};

// The class bits of layers [j0, j1).
uint32_t chunk_class(const CellProg &C, int32_t kind, int32_t j0, int32_t j1) {
  uint32_t cls = kCellRegular | kCellTakes | kCellCounts, longest = 1, nodes = 1;
  for (int32_t j = j0; j < j1; ++j) {
    const uint32_t y = C.w1[size_t(j)];
    if (!(y & 0x7Fu)) continue;
    longest = std::max(longest, y & 0x7Fu);
    if (kind == kCellGen) nodes = std::max(nodes, (C.own[size_t(j)] >> 16) & 0xFu);
    const uint32_t a = y >> 16;
    if (a != kArcsCount) cls &= ~kCellCounts;
    if (a != kArcsTake) cls &= ~kCellTakes;
    if (a != kArcsCount && a != kArcsTake) cls &= ~kCellRegular;
  }
  if (kind == kCellGen) cls = (nodes - 1u) << 24;
  return cls | std::min(longest - 1, 15u) << 28;
}

// LDS of a cell: the kernel's arrays, and slack for the reads of lanes past a chunk's end
int32_t cell_lds(int32_t nl, int32_t nrow, int32_t xa, int32_t kind, int32_t block) {
  return 8 * xa + 4 * nl + (kind == kCellPair ? 2 : (kind == kCellLayers ? 8 : 0)) * nl + 4 * nrow + 16 * block;
}

}  // namespace

// Builds the cells of both stages; false (no cells) when a program's fields overflow.
bool build_cells(Plan &P, const std::vector<int64_t> &iptr, const std::vector<int32_t> &ilist,
                 const std::vector<int32_t> &inc_row, const std::vector<int32_t> &ownw,
                 const std::vector<int32_t> &childw) {
  const int32_t n = P.n;
  // local steps: longest chain of row predecessors in the same stage
  std::vector<int32_t> vstep(size_t(n), 0);
  for (int32_t i : P.order) {
    int32_t t = -1;
    for (int64_t q = iptr[size_t(i)]; q < iptr[size_t(i) + 1]; ++q) {
      const int64_t c = ilist[size_t(q)];
      if (c == P.canon_off[size_t(inc_row[size_t(c)])]) continue;
      const int32_t v = P.inc_var[size_t(c) - 1];
      if (P.var_stage[size_t(v)] == P.var_stage[size_t(i)]) t = std::max(t, vstep[size_t(v)]);
    }
    vstep[size_t(i)] = t + 1;
  }
  // floats of a boundary message: the widest level whose parent lies in the other stage
  int32_t bw = 2;
  for (int64_t L = 0; L < P.I; ++L) {
    const int32_t pa = P.parent[size_t(L)];
    if (pa >= 0 && P.var_stage[size_t(P.layer_var[size_t(pa)])] != P.var_stage[size_t(P.layer_var[size_t(L)])])
      bw = std::max(bw, (ownw[size_t(L)] + 1) & ~1);
  }
  // components: stage, group and layers; packed into cells in (stage, group, component) order
  std::vector<int32_t> clayers(size_t(P.n_comp), 0), cgroup(size_t(P.n_comp), 0), cell_of(size_t(P.n_comp), -1);
  std::vector<uint8_t> cstage(size_t(P.n_comp), 0);
  bool pairs[2] = {true, true};
  int32_t steps[2] = {0, 0};
  for (int32_t i = 0; i < n; ++i) {
    const int32_t c = P.var_comp[size_t(i)];
    if (c < 0) continue;
    clayers[size_t(c)] += P.var_nj[size_t(i)];
    cgroup[size_t(c)] = P.var_group[size_t(i)];
    cstage[size_t(c)] = P.var_stage[size_t(i)];
    steps[P.var_stage[size_t(i)]] = std::max(steps[P.var_stage[size_t(i)]], vstep[size_t(i)] + 1);
    pairs[P.var_stage[size_t(i)]] = pairs[P.var_stage[size_t(i)]] && P.var_nj[size_t(i)] == 2;
  }
  std::vector<int32_t> corder(static_cast<size_t>(P.n_comp));
  for (int32_t c = 0; c < P.n_comp; ++c) corder[size_t(c)] = c;
  std::stable_sort(corder.begin(), corder.end(), [&](int32_t a, int32_t b) {
    return std::make_pair(cstage[size_t(a)], cgroup[size_t(a)]) < std::make_pair(cstage[size_t(b)], cgroup[size_t(b)]);
  });
  std::vector<uint16_t> loc(size_t(P.I), 0);
  std::vector<int32_t> part_of(size_t(P.I), -1);  // global row part starting (B) or ending (A) at a layer
  for (int st = 1; st >= 0; --st) {
    CellStage &S = P.cell[st];
    S = CellStage{};
    S.bw = bw;
    const CellBuilder B{P, ownw, childw, vstep, bw / 2, loc};
    int32_t big = 0;
    for (int32_t c : corder)
      if (cstage[size_t(c)] == st) big = std::max(big, clayers[size_t(c)]);
    if (!big) continue;
    int64_t total = 0;
    for (int32_t c : corder)
      if (cstage[size_t(c)] == st) total += clayers[size_t(c)];
    int32_t room = 0;
    std::vector<int32_t> hist(size_t(steps[st]), 0);
    int32_t bigc = -1;
    for (int32_t c : corder)
      if (cstage[size_t(c)] == st && clayers[size_t(c)] == big) bigc = c;
    if (big > 256)
      for (int32_t i = 0; i < n; ++i)
        if (P.var_comp[size_t(i)] == bigc) hist[size_t(vstep[size_t(i)])] += P.var_nj[size_t(i)];
    cell_shape(big, total, hist, pairs[st] && st == 1, S.block, room);
    room = std::max(room, big);
    int32_t nc = 0, fill = 0, g = -1;
    for (int32_t c : corder) {
      if (cstage[size_t(c)] != st) continue;
      if (nc == 0 || fill + clayers[size_t(c)] > room || cgroup[size_t(c)] != g) {
        ++nc;
        fill = 0;
        g = cgroup[size_t(c)];
      }
      cell_of[size_t(c)] = nc - 1;
      fill += clayers[size_t(c)];
    }
    S.n_cells = nc;
    // each cell's variables, by step (below), then storage
    std::vector<int64_t> vp(size_t(nc) + 1, 0);
    for (int32_t i = 0; i < n; ++i)
      if (P.var_comp[size_t(i)] >= 0 && P.var_stage[size_t(i)] == st) vp[size_t(cell_of[size_t(P.var_comp[size_t(i)])]) + 1]++;
    for (int32_t k = 0; k < nc; ++k) vp[size_t(k) + 1] += vp[size_t(k)];
    std::vector<int32_t> vars(static_cast<size_t>(vp[size_t(nc)]));
    {
      std::vector<int64_t> at(vp.begin(), vp.end() - 1);
      for (int64_t L = 0; L < P.I; L += P.var_nj[size_t(P.layer_var[size_t(L)])]) {
        const int32_t i = P.layer_var[size_t(L)];
        if (P.var_stage[size_t(i)] == st) vars[size_t(at[size_t(cell_of[size_t(P.var_comp[size_t(i)])])]++)] = i;
      }
    }
    auto nvars = [&](int64_t k) { return size_t(vp[size_t(k) + 1] - vp[size_t(k)]); };
    // sizes of the cells, and where each one's layers and row parts start
    std::vector<int64_t> lbase(size_t(nc) + 1, 0), rbase(size_t(nc) + 1, 0);
    std::atomic<bool> ok{true}, all_pairs{true};
    const int64_t share = cell_share(nc, total);
    on_threads(nc, share, [&](int64_t k0, int64_t k1) {
      std::vector<int32_t> at, by;
      for (int64_t k = k0; k < k1; ++k) {
        int32_t *v = vars.data() + vp[size_t(k)];
        // stable counting sort by step
        at.assign(1, 0);
        for (size_t q = 0; q < nvars(k); ++q) {
          const size_t t = size_t(vstep[size_t(v[q])]) + 1;
          if (t >= at.size()) at.resize(t + 1, 0);
          ++at[t];
        }
        for (size_t t = 1; t < at.size(); ++t) at[t] += at[t - 1];
        by.resize(nvars(k));
        for (size_t q = 0; q < by.size(); ++q) by[size_t(at[size_t(vstep[size_t(v[q])])]++)] = v[q];
        std::copy(by.begin(), by.end(), v);
        int32_t nl = 0, nrow = 0;
        if (!B.measure(v, nvars(k), nl, nrow)) ok = false;
        lbase[size_t(k) + 1] = nl;
        rbase[size_t(k) + 1] = nrow;
      }
    });
    if (!ok) return false;
    for (int32_t k = 0; k < nc; ++k) {
      lbase[size_t(k) + 1] += lbase[size_t(k)];
      rbase[size_t(k) + 1] += rbase[size_t(k)];
    }
    if (lbase[size_t(nc)] >= INT32_MAX / 2 || rbase[size_t(nc)] * bw >= INT32_MAX / 2) return false;
    S.layer.assign(size_t(lbase[size_t(nc)]), -1);
    S.link.assign(size_t(rbase[size_t(nc)]), -1);
    S.term.assign(size_t(rbase[size_t(nc)]), -1);
    // the cells: storage layers in cell order, the row parts' bound terms, where they start (B) or end (A)
    // for the links, and the programs, equal ones once (by hash, then compared). Each thread keeps the
    // first program of each hash in its run of cells; a cell's template is numbered among them at first.
    struct Run {
      int64_t k0;
      std::vector<CellProg> prog;
    };
    std::vector<Run> runs;
    std::mutex mu;
    std::vector<int32_t> tmpl(size_t(nc), -1);
    on_threads(nc, share, [&](int64_t k0, int64_t k1) {
      CellProg C;
      Run run{k0, {}};
      std::unordered_multimap<uint64_t, int32_t> by_hash;
      for (int64_t k = k0; k < k1; ++k) {
        int32_t *lay = S.layer.data() + lbase[size_t(k)];
        if (!B.build(vars.data() + vp[size_t(k)], nvars(k), C, lay)) {
          ok = false;
          return;
        }
        if (!C.pairs) all_pairs = false;
        const uint64_t h = C.hash();
        int32_t t = -1;
        const auto eq = by_hash.equal_range(h);
        for (auto it = eq.first; it != eq.second && t < 0; ++it)
          if (C.same(run.prog[size_t(it->second)])) t = it->second;
        if (t < 0) {
          t = int32_t(run.prog.size());
          run.prog.push_back(C);
          by_hash.emplace(h, t);
        }
        tmpl[size_t(k)] = t;
        for (size_t q = 0; q < C.row.size(); ++q) {
          const int32_t Lb = lay[C.row[q] & 0x1FFFu], Le = lay[(C.row[q] >> 13) & 0x1FFFu];
          const int64_t r = rbase[size_t(k)] + int64_t(q);
          if (P.parent[size_t(Lb)] <= -2) S.term[size_t(r)] = -2 - P.parent[size_t(Lb)];
          if (st == 1) part_of[size_t(Lb)] = int32_t(r);
          else part_of[size_t(Le)] = int32_t(r);
        }
      }
      std::lock_guard<std::mutex> lk(mu);
      runs.push_back(std::move(run));
    });
    if (!ok) return false;
    // the runs' programs in one list, in the order of their first cells
    std::sort(runs.begin(), runs.end(), [](const Run &a, const Run &b) { return a.k0 < b.k0; });
    std::vector<CellProg> prog;
    {
      std::unordered_multimap<uint64_t, int32_t> by_hash;
      for (size_t q = 0; q < runs.size(); ++q) {
        std::vector<int32_t> to;
        for (CellProg &C : runs[q].prog) {
          const uint64_t h = C.hash();
          int32_t t = -1;
          const auto eq = by_hash.equal_range(h);
          for (auto it = eq.first; it != eq.second && t < 0; ++it)
            if (C.same(prog[size_t(it->second)])) t = it->second;
          if (t < 0) {
            t = int32_t(prog.size());
            prog.push_back(std::move(C));
            by_hash.emplace(h, t);
          }
          to.push_back(t);
        }
        const int64_t k1 = q + 1 < runs.size() ? runs[q + 1].k0 : nc;
        for (int64_t k = runs[q].k0; k < k1; ++k) tmpl[size_t(k)] = to[size_t(tmpl[size_t(k)])];
      }
    }
    auto lds = [&](int32_t kind) {
      int32_t most = 0;
      for (const CellProg &C : prog) most = std::max(most, cell_lds(C.nl, int32_t(C.row.size()), C.xa, kind, S.block));
      return most;
    };
    S.kind = all_pairs && st == 1 ? kCellPair : kCellLayers;
    for (const CellProg &C : prog)
      if (C.wide) S.kind = kCellGen;
    if (S.kind == kCellLayers && P.max_width > 2 && lds(S.kind) > kCellLdsCap) S.kind = kCellGen;
    S.lds = lds(S.kind);
    // concatenated programs: two-row stages pack their descriptors by variable
    std::vector<int32_t> wbase, kbase, nwork, tbase;
    int64_t total_w = 0;
    for (const CellProg &C : prog) {
      wbase.push_back(int32_t(total_w));
      kbase.push_back(int32_t(S.work.size()));
      tbase.push_back(int32_t(S.row.size()));
      total_w += C.nl;
      if (total_w >= INT32_MAX / 8) return false;
      const int32_t per = S.kind == kCellPair ? 2 : 1;
      if (S.kind == kCellGen) {
        for (int32_t j = 0; j < C.nl; ++j) {
          const uint32_t o = C.own[size_t(j)];
          S.ga.insert(S.ga.end(), {(C.h[size_t(j)] & 0x7FFFu) | (o & 0xFFFFu) << 16, C.kid[size_t(j)] | C.dad[size_t(j)] << 16,
                                   (C.w1[size_t(j)] & 0xFFFFu) | (o & 0xFF0000u), 0u});
        }
        S.gb.insert(S.gb.end(), C.arc.begin(), C.arc.end());
      } else {
        for (int32_t j = 0; j < C.nl; j += per)
          S.w0.push_back(C.h[size_t(j)] | (per == 2 ? C.h[size_t(j) + 1] : C.kid[size_t(j)]) << 16);
        S.w1.insert(S.w1.end(), C.w1.begin(), C.w1.end());
      }
      for (int32_t s = 0; s < C.ns; ++s) {
        const int32_t e = int32_t(C.step[size_t(s) + 1]);
        for (int32_t j = int32_t(C.step[size_t(s)]); j < e; j += per * S.block) {
          const int32_t j1 = std::min(e, j + per * S.block);
          S.work.push_back(uint32_t(j / per) | uint32_t((j1 - j) / per) << 13 | chunk_class(C, S.kind, j, j1) |
                           (j == int32_t(C.step[size_t(s)]) ? kCellStepBegin : 0u) | (j1 == e ? kCellStepEnd : 0u));
        }
      }
      nwork.push_back(int32_t(S.work.size()) - kbase.back());
      S.row.insert(S.row.end(), C.row.begin(), C.row.end());
    }
    for (int32_t k = 0; k < nc; ++k) {
      const size_t t = size_t(tmpl[size_t(k)]);
      const CellProg &C = prog[t];
      S.rec.insert(S.rec.end(), {C.nl, nwork[t], wbase[t], kbase[t], int32_t(lbase[size_t(k)]), int32_t(rbase[size_t(k)]),
                                 C.xa, 0, int32_t(C.row.size()), tbase[t], 0, 0});
    }
    if (S.lds > kCellLdsCap) return false;
  }
  // links: an A row part that ends above a layer of B, with the B row part starting there
  for (int64_t L = 0; L < P.I; ++L) {
    const int32_t ch = P.child[size_t(L)];
    if (ch < 0 || P.var_stage[size_t(P.layer_var[size_t(ch)])] == P.var_stage[size_t(P.layer_var[size_t(L)])]) continue;
    const int32_t a = part_of[size_t(L)], b = part_of[size_t(ch)];
    P.cell[0].link[size_t(a)] = b;
    P.cell[1].link[size_t(b)] = a;
  }
  return true;
}

// Estimated time of an iteration as cells, in us (fitted to the measurements at cells_pay in plan.cpp). Per
// stage, the cells beyond those that the compute units hold at once (by LDS and by wavefronts) run in
// further rounds, each as long as the largest cell's chunks and rows take in sequence (0.35 us each for a
// wavefront by itself, 0.6 us for several, which meet at barriers, 0.15 us more on levels of up to four
// nodes); many small cells are bound by the chunks that all wavefronts issue. Two stages add their launches,
// the multipliers, and the cache lines of the messages that a cell hands on to scattered places.
double cell_time(const Plan &P) {
  double us = 1.0;
  for (const CellStage &S : P.cell) {
    if (!S.n_cells) continue;
    const int32_t step = (S.n_cells + kCellSample - 1) / kCellSample;
    double chunks = 0.0, lines = 0.0, links = 0.0, layers = 0.0;
    int32_t most = 0, rows = 0;
    std::vector<int32_t> line;
    for (int32_t k = 0; k < S.n_cells; ++k) {
      const int32_t *r = &S.rec[12 * size_t(k)];
      layers += r[0];
      chunks += r[1];
      most = std::max(most, r[1]);
      rows = std::max(rows, (r[8] + S.block - 1) / S.block);
      if (k % step) continue;
      line.clear();
      for (int32_t q = 0; q < r[8]; ++q)
        if (const int32_t to = S.link[size_t(r[5] + q)]; to >= 0) line.push_back(int32_t(int64_t(to) * S.bw / 16));
      std::sort(line.begin(), line.end());
      links += step * double(line.size());
      lines += step * double(std::unique(line.begin(), line.end()) - line.begin());
    }
    const int32_t slots = 256 * std::min(kCellLdsCap / std::max(S.lds, 1), 2048 / S.block);
    const double unit = (S.block == 64 ? 0.35 : 0.6) + (S.kind == kCellGen ? 0.15 : 0.0);
    const double chain = (2.0 * most + 2.0 * rows + 2.0) * unit * ((S.n_cells + slots - 1) / slots);
    us += std::max(chain, 0.15 / 1024.0 * 2.0 * chunks * (S.block / 64));
    if (P.cell_kind == 2) us += 2.5 + 1e-6 * layers + 17e-6 * std::max(0.0, lines - links * S.bw / 16);
  }
  return us;
}

// Checks every index the cell kernels use, and that the cells run each layer exactly once, after its
// row's previous level. Empty when sound.
std::string validate_cells(const Plan &P, const std::vector<int32_t> &ownw, const std::vector<int32_t> &childw) {
  std::vector<uint8_t> seen(size_t(P.I), 0);
  std::vector<int32_t> place(size_t(P.I), -1);
  std::atomic<int64_t> total{0};
  std::atomic<const char *> bad{nullptr};
  for (int st = 0; st < 2; ++st) {
    const CellStage &S = P.cell[st];
    if (S.rec.size() != 12 * size_t(S.n_cells) || S.w0.size() * (S.kind == kCellPair ? 2 : 1) != S.w1.size() ||
        S.ga.size() != S.gb.size() || S.link.size() != S.term.size() || S.bw < 2 ||
        (S.bw & 1) || S.bw != P.cell[1 - st].bw)
      return "cell arrays";
    // each storage layer's index in S.layer
    for (size_t q = 0; q < S.layer.size(); ++q)
      if (S.layer[q] >= 0) {
        if (S.layer[q] >= P.I) return "cell layer";
        place[size_t(S.layer[q])] = int32_t(q);
      }
    const int64_t share = cell_share(S.n_cells, int64_t(S.layer.size()));
    on_threads(S.n_cells, share, [&](int64_t k0, int64_t k1) {
      auto fail = [&](const char *w) { bad = w; };
      std::vector<int32_t> step_of, part_f, part_b, chunk_of, chunk0;
      std::vector<std::pair<int32_t, int32_t>> wide;
      for (int64_t k = k0; k < k1; ++k) {
        const int32_t *r = &S.rec[12 * size_t(k)];
        for (int q = 0; q < 12; ++q)
          if (r[q] < 0) return fail("cell record");
        const int32_t nl = r[0], nw = r[1], xa = r[6], nrow = r[8], bwp = S.bw / 2, per = S.kind == kCellPair ? 2 : 1;
        const bool gen = S.kind == kCellGen;
        if (nl < 4 || (nl & 3) || nl > 0x1FFF || nw < 1 || (r[2] & 3) || (r[4] & 3) ||
            size_t(r[2]) + size_t(nl) > (gen ? S.ga.size() / 4 : S.w1.size()) ||
            size_t(r[3]) + size_t(nw) > S.work.size() || size_t(r[4]) + size_t(nl) > S.layer.size() || nrow < 1 ||
            size_t(r[5]) + size_t(nrow) > S.link.size() || size_t(r[9]) + size_t(nrow) > S.row.size() ||
            (xa & 1) || xa < nl + nrow * bwp + (gen ? 2 : 0) || xa > 0x7FFF || cell_lds(nl, nrow, xa, S.kind, S.block) > S.lds)
          return fail("cell record");
        const uint32_t *row = S.row.data() + r[9], *work = &S.work[size_t(r[3])];
        const int32_t *lay = &S.layer[size_t(r[4])];
        auto word = [&](int32_t j, int q) { return S.ga[4 * size_t(r[2] + j) + size_t(q)]; };
        auto w1 = [&](int32_t j) { return gen ? word(j, 2) : S.w1[size_t(r[2] + j)]; };
        auto parent_area = [&](int32_t j) {  // with kCellCount in bit 15
          if (gen) return word(j, 0) & 0xFFFFu;
          if (per == 1) return S.w0[size_t(r[2] + j)] & 0xFFFFu;
          return (S.w0[size_t((r[2] + j) / 2)] >> (16 * (j & 1))) & 0xFFFFu;
        };
        auto area = [&](int32_t j) { return gen ? int32_t(word(j, 0) >> 16) : j; };  // layer j's link
        // chunks: consecutive from the first layer on, inside their steps
        step_of.assign(size_t(nl), -1);
        chunk_of.assign(size_t(nl), -1);
        chunk0.assign(size_t(nw), 0);
        int32_t at_j = 0, s = -1;
        for (int32_t q = 0; q < nw; ++q) {
          const int32_t j0 = int32_t(work[q] & 0x1FFFu) * per, c = int32_t((work[q] >> 13) & 0x3FFu) * per;
          if (j0 != at_j || c < 1 || c > per * S.block || j0 + c > nl) return fail("cell chunk");
          if (bool(work[q] & kCellStepBegin) != (q == 0 || bool(work[q - 1] & kCellStepEnd))) return fail("cell chunk");
          if (work[q] & kCellStepBegin) ++s;
          if (q + 1 == nw && !(work[q] & kCellStepEnd)) return fail("cell chunk");
          chunk0[size_t(q)] = j0;
          for (int32_t j = j0; j < j0 + c; ++j) {
            step_of[size_t(j)] = s;
            chunk_of[size_t(j)] = q;
          }
          at_j = j0 + c;
        }
        for (int32_t j = 0; j < nl; ++j) {
          if ((lay[j] >= 0) != ((w1(j) & 0x7Fu) != 0u) || lay[j] >= P.I || (lay[j] >= 0 && step_of[size_t(j)] < 0))
            return fail("cell layer");
          if (lay[j] < 0) continue;
          seen[size_t(lay[j])] = 1;
        }
        // row parts: walks along the children cover each layer once; links and terms
        part_f.assign(size_t(nl), -1);
        part_b.assign(size_t(nl), -1);
        // a storage layer's place in this cell
        auto local = [&](int32_t L) {
          const int32_t q = place[size_t(L)] - r[4];
          return q >= 0 && q < nl && lay[q] == L ? q : -1;
        };
        int64_t walked = 0, layers = 0;
        for (int32_t q = 0; q < nrow; ++q) {
          const int32_t jb = int32_t(row[q] & 0x1FFFu), je = int32_t((row[q] >> 13) & 0x1FFFu);
          if (jb >= nl || je >= nl || lay[jb] < 0 || lay[je] < 0 || part_f[size_t(jb)] >= 0 || part_b[size_t(je)] >= 0)
            return fail("cell row part");
          part_f[size_t(jb)] = part_b[size_t(je)] = q;
          int32_t j = jb;
          for (++walked; j != je; ++walked) {
            const int32_t c = P.child[size_t(lay[j])];
            j = c < 0 ? -1 : local(c);
            if (j < 0 || walked > nl) return fail("cell row part");
          }
          const int32_t pa = P.parent[size_t(lay[jb])], ch = P.child[size_t(lay[je])];
          const int32_t link = S.link[size_t(r[5] + q)], term = S.term[size_t(r[5] + q)];
          if (bool(row[q] & kCellRowRoot) != (pa <= -2) || bool(row[q] & kCellRowLast) != (ch < 0) ||
              term != (pa <= -2 ? -2 - pa : -1) || (pa >= 0 && local(pa) >= 0) || (ch >= 0 && local(ch) >= 0))
            return fail("cell row ends");
          // stage A hands on at a row part's end, stage B at its start
          const bool linked = st == 0 ? ch >= 0 : pa >= 0;
          if ((st == 0 && pa >= 0) || (st == 1 && ch >= 0) || linked != (link >= 0)) return fail("cell link");
          if (linked && (size_t(link) >= P.cell[1 - st].link.size() || P.cell[1 - st].link[size_t(link)] != r[5] + q))
            return fail("cell link");
          if (pa >= 0 && ownw[size_t(lay[jb])] > S.bw) return fail("cell boundary width");
          if (ch >= 0 && childw[size_t(lay[je])] > S.bw) return fail("cell boundary width");
        }
        wide.clear();
        for (int32_t j = 0; j < nl; ++j) {
          const int32_t L = lay[j];
          if (L < 0) continue;
          ++layers;
          const int32_t s = step_of[size_t(j)], len = int32_t(w1(j) & 0x7Fu), pos = int32_t((w1(j) >> kCellPosShift) & 0x7Fu);
          const int32_t v = P.layer_var[size_t(L)], h = j - pos;
          // a variable's layers lie in one chunk, on one wavefront
          if (len != P.var_nj[size_t(v)] || pos != L - P.var_first[size_t(v)] || h < 0 || h + len > nl ||
              chunk_of[size_t(h)] != chunk_of[size_t(j)] || chunk_of[size_t(h + len - 1)] != chunk_of[size_t(j)] ||
              lay[h] != P.var_first[size_t(v)] || lay[h + len - 1] != P.var_first[size_t(v)] + len - 1)
            return fail("cell segment");
          const int32_t c0 = chunk0[size_t(chunk_of[size_t(j)])];
          if (per == 1 && (h - c0) / 64 != (h + len - 1 - c0) / 64) return fail("cell segment");
          const int32_t ch = P.child[size_t(L)], pa = P.parent[size_t(L)], w = ownw[size_t(L)], wc = childw[size_t(L)];
          if (bool(w1(j) & kCellLast) != (ch < 0)) return fail("cell ends");
          if (!gen && (w > 2 || wc > 2)) return fail("cell kind");
          const int32_t jc = ch >= 0 ? local(ch) : -1, jp = pa >= 0 ? local(pa) : -1;
          if ((jc >= 0 && step_of[size_t(jc)] <= s) || (jp >= 0 && step_of[size_t(jp)] >= s)) return fail("cell step order");
          if ((jc < 0) != (part_b[size_t(j)] >= 0) || (jp < 0) != (part_f[size_t(j)] >= 0)) return fail("cell row ends");
          if (int32_t(parent_area(j) & 0x7FFFu) != (jp >= 0 ? area(jp) : nl + part_f[size_t(j)] * bwp)) return fail("cell parent area");
          const int32_t kid = jc >= 0 ? jc : 0xFFFF;
          if (gen) {
            const int32_t o = area(j), consts = 2 * (xa - 2);
            if (int32_t(word(j, 1) & 0xFFFFu) != kid || int32_t(word(j, 1) >> 16) != (jp >= 0 ? jp : 0xFFFF)) return fail("cell neighbours");
            if (w > 4 || wc > 4 || int32_t((word(j, 2) >> 16) & 0xFu) != w || int32_t((word(j, 2) >> 20) & 0xFu) != wc)
              return fail("cell widths");
            if ((wc <= 2) != (o == j) || o + (wc + 1) / 2 > xa - 2) return fail("cell areas");
            if (wc > 2) wide.emplace_back(o, (wc + 1) / 2);
            for (int32_t u = 0; u < 4; ++u) {
              const uint32_t a = u < w ? P.garcs[size_t(P.own_slot[size_t(L)] + u)] : kBot | kBot << 16;
              for (int hi = 0; hi < 2; ++hi) {
                const uint32_t c = hi ? a >> 16 : a & 0xFFFFu, x = S.gb[4 * size_t(r[2] + j) + size_t(u)];
                if (int32_t(hi ? x >> 16 : x & 0xFFFFu) != (c < kTop ? 2 * o + int32_t(c) : consts + (c == kTop ? 0 : 1)))
                  return fail("cell arcs");
              }
            }
            if (w - 1 > int32_t((work[chunk_of[size_t(j)]] >> 24) & 3u)) return fail("cell chunk class");
          } else if (per == 1 && int32_t(S.w0[size_t(r[2] + j)] >> 16) != kid) {
            return fail("cell child");
          }
          if (!gen) {
            // the arcs decode to the layer's, terminals through the virtual child level
            const uint32_t arcs = w1(j) >> 16;
            if (bool(parent_area(j) & kCellCount) != (arcs == kArcsCount)) return fail("cell arcs");
            for (int q = 0; q < (pa <= -2 ? 2 : 4); ++q) {
              const uint32_t c = (arcs >> (2 * q)) & 3u, o = (P.meta[size_t(L)] >> (2 * q)) & 3u;
              if (ch >= 0) {
                if (c != o) return fail("cell arcs");
              } else {
                const uint32_t rw = row[part_b[size_t(j)]];
                const bool top = c == 0u ? (rw & kCellRowTermX) != 0u : (c == 1u ? (rw & kCellRowTermY) != 0u : false);
                if (c == 3u || top != (o == kC2Top)) return fail("cell arcs");
              }
            }
            if (S.kind == kCellPair && (len != 2 || (h & 1) || (arcs != kArcsCount && arcs != kArcsTake))) return fail("cell pair");
          }
          const uint32_t cls = work[chunk_of[size_t(j)]];
          if ((cls >> 28) < std::min(uint32_t(len) - 1u, 15u)) return fail("cell chunk class");
          if (!gen) {
            const uint32_t a = w1(j) >> 16;
            if (((cls & kCellRegular) && a != kArcsCount && a != kArcsTake) || ((cls & kCellTakes) && a != kArcsTake) ||
                ((cls & kCellCounts) && a != kArcsCount))
              return fail("cell chunk class");
          }
        }
        if (walked != layers) return fail("cell row part");
        total += layers;
        std::sort(wide.begin(), wide.end());
        for (size_t q = 0; q < wide.size(); ++q)
          if (wide[q].first < nl + nrow * bwp || (q && wide[q - 1].first + wide[q - 1].second > wide[q].first))
            return fail("cell general areas");
      }
    });
    if (const char *w = bad) return w;
  }
  if (total != P.I) return "cell coverage";
  for (uint8_t s : seen)
    if (!s) return "cell coverage";
  return "";
}

}  // namespace bddmp
