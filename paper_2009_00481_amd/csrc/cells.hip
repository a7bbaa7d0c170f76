// Cell launches: an iteration's passes with every message inside a workgroup's LDS.
//
// A cell (cells.cpp) is a set of whole components of one stage: nothing it reads inside an iteration
// comes from another cell of its stage. Its workgroup loads the multipliers of its layers and the
// messages at the stage's boundary, recomputes the inner messages it starts from (they are functions
// of the multipliers alone), runs its part of the passes step by step, and stores the multipliers
// and the boundary messages. One iteration is then
//   A forward | B forward, then backward | A backward
// and over a run of iterations A's backward part is followed at once by the next forward part, so
// an iteration takes two launches and its HBM traffic is the multipliers, read and written once per
// launch, and the boundary messages, instead of every layer's record and messages in both passes.
// Every layer's operations and their order are those of the wave kernels, so results are bitwise the
// same.
//
// Bound: instruction issue and the LDS round trips along a cell's steps (about 800 cycles each for one
// wavefront alone), hidden by as many cells per compute unit as their LDS allows; everything a step
// touches is in LDS or read ahead (a global round trip per step took twice the time). Between calls of
// iterate the multipliers are in storage order; inside a run they are kept in cell order, where a
// cell's are contiguous. Measured, us per iteration against one launch per wave replayed as a graph:
// Potts 256x256x8 168 (367), 128x128x4 29 (61), 16x16x4 15 (49); Potts 8x8x3, whole in one workgroup, 11
// (38).
#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>

#include "device.h"
#include "kernels.h"

namespace bddmp {

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// float of lane l of the wavefront
__device__ __forceinline__ float lane_read(float v, int l) {
  return __int_as_float(__builtin_amdgcn_ds_bpermute(4 * l, __float_as_int(v)));
}

// minimum without the quieting of signalling NaNs that fminf adds (there are no NaNs here: a level
// whose min-marginals are both +inf is refused when the plan is built)
__device__ __forceinline__ float vmin(float a, float b) {
  float r;
  asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

// the preceding lane of the wavefront (wave_shr:1)
__device__ __forceinline__ float lane_before(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xF, 0xF, false));
}

// s / n for a row count n, with r = 1 / n rounded: one correction of s * r by the exact remainder is the
// correctly rounded quotient (checked for every mantissa and n <= 64) while nothing underflows or
// overflows; the division itself elsewhere.
__device__ __forceinline__ float over_count(float s, float n, float r) {
  const float a = fabsf(s);
  if (a != 0.0f && !(a >= 0x1p-100f && a <= 0x1p100f)) return s / n;
  const float q = s * r;
  return fmaf(fmaf(-q, n, s), r, q);
}

// A cell's LDS. X holds one message per link between a layer and its child level, in areas of pairs of
// floats: layer j's link is X[j] (a child level of more than two nodes has an area of its own). A link
// carries the forward messages of the child level or the backward ones, never both at once: a layer's
// forward step reads its link's backward messages and leaves the forward ones there, and its backward
// step reads the forward messages on its parent's link and leaves the backward ones there. That is
// half the LDS of two arrays, and LDS is what bounds the cells in flight. Behind the layers' links
// come those above the row parts' first levels (bwp pairs each).
struct Cell {
  float2 *X;
  float *lam;
  uint32_t *w0, *w1;     // descriptors (internal.h)
  const uint32_t *work;  // global: the chunks of the steps (internal.h)
  uint32_t *row;
  uint4 *grec;
  uint32_t *garc;
  int nwork, nrow, nl;
};

__device__ __forceinline__ float cell_c16(const float *b, uint32_t c) {
  return c < kTop ? b[c] : (c == kTop ? 0.0f : INFINITY);
}

// Regular levels: 0-arcs keep the node, and either node 0's 1-arc moves to node 1 (c, a counting
// level) or node 1's to node 0. These closed forms drop only terms that are +inf.
__device__ __forceinline__ float regular_m1(bool c, float2 f, float2 b, float lam) {
  return ((c ? f.x : f.y) + lam) + (c ? b.y : b.x);
}
__device__ __forceinline__ float2 regular_push(bool c, float2 f, float lam) {
  const float v = vmin((c ? f.x : f.y) + lam, c ? f.y : f.x);
  return c ? make_float2(f.x, v) : make_float2(v, f.y);
}
__device__ __forceinline__ float2 regular_bstep(bool c, float2 b, float lam) {
  const float v = vmin((c ? b.y : b.x) + lam, c ? b.x : b.y);
  return c ? make_float2(v, b.y) : make_float2(b.x, v);
}

// any narrow level, by its 2-bit child codes
__device__ __forceinline__ float2 narrow_push(uint32_t a, float2 f, float lam) {
  const uint32_t k0 = a & 3u, k1 = (a >> 2) & 3u, k2 = (a >> 4) & 3u, k3 = (a >> 6) & 3u;
  const float a0 = f.x, a1 = f.x + lam, a2 = f.y, a3 = f.y + lam;
  return make_float2(fminf(fminf(k0 == 0u ? a0 : INFINITY, k1 == 0u ? a1 : INFINITY),
                           fminf(k2 == 0u ? a2 : INFINITY, k3 == 0u ? a3 : INFINITY)),
                     fminf(fminf(k0 == 1u ? a0 : INFINITY, k1 == 1u ? a1 : INFINITY),
                           fminf(k2 == 1u ? a2 : INFINITY, k3 == 1u ? a3 : INFINITY)));
}
__device__ __forceinline__ float2 narrow_bstep(uint32_t a, float2 b, float lam) {
  return make_float2(fminf(c2val(a & 3u, b), c2val((a >> 2) & 3u, b) + lam),
                     fminf(c2val((a >> 4) & 3u, b), c2val((a >> 6) & 3u, b) + lam));
}

// levels of more than two nodes (or above one), node by node: from is the area of the forward messages
// (the parent's link), own the layer's link
__device__ __forceinline__ void general_push(const Cell &C, uint4 g, int from, float lam) {
  const float *fp = reinterpret_cast<const float *>(C.X + from);
  float *cp = reinterpret_cast<float *>(C.X + g.z);
  const uint32_t *arc = C.garc + (g.x & 0xFFFFu);
  const int w = int(g.y & 0xFu), wc = int((g.y >> 4) & 0xFu);
  for (int q = 0; q < ((wc + 1) & ~1); ++q) cp[q] = INFINITY;
  for (int u = 0; u < w; ++u) {
    const uint32_t lo = arc[u] & 0xFFFFu, hi = arc[u] >> 16;
    const float fu = fp[u];
    if (lo < kTop) cp[lo] = fminf(cp[lo], fu);
    if (hi < kTop) cp[hi] = fminf(cp[hi], fu + lam);
  }
}
__device__ __forceinline__ void general_bstep(const Cell &C, uint4 g, int to, float lam) {
  const float *bp = reinterpret_cast<const float *>(C.X + g.z);
  float *pp = reinterpret_cast<float *>(C.X + to);
  const uint32_t *arc = C.garc + (g.x & 0xFFFFu);
  const int w = int(g.y & 0xFu);
  for (int u = 0; u < w; ++u) pp[u] = fminf(cell_c16(bp, arc[u] & 0xFFFFu), cell_c16(bp, arc[u] >> 16) + lam);
  if (w & 1) pp[w] = INFINITY;
}

// Order between a step's LDS writes and the next step's reads. One wavefront's LDS accesses are
// executed in the order it issues them, so a one-wavefront workgroup only keeps the compiler from
// moving them; larger ones meet at a barrier.
template <int BLOCK>
__device__ __forceinline__ void step_sync() {
  if (BLOCK == 64) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  } else {
    __syncthreads();
  }
}

// One layer's part of a step: min-marginals, J_i exchange, update, and the message it passes on. A
// variable's layers sit on consecutive lanes of one wavefront, so the exchange is lane moves. f: the
// messages on the parent's link (area p), b: those on its own; longest: one less than the most rows of
// a variable of the chunk (-1: 16 or more); rcp: 1 / (lane + 1).
template <int DIR, bool GEN>
__device__ __forceinline__ void layer_step(const Cell &C, uint32_t d0, uint32_t d1, float lam, float2 f, float2 b, int j,
                                           bool regular, int longest, float rcp) {
  const int p = int(d0 & 0x7FFFu);
  const int len = int(d1 & 0x7Fu);
  const bool gen = GEN && (d1 & kCellGeneral) != 0u;
  const bool s = (d0 & kCellCount) != 0u;
  const uint32_t arcs = d1 >> 16;
  uint4 g = make_uint4(0u, 0u, 0u, 0u);
  float m0 = INFINITY, m1 = INFINITY;
  if (regular) {
    m0 = vmin(f.x + b.x, f.y + b.y);
    m1 = regular_m1(s, f, b, lam);
  } else if (!gen) {
    m0 = fminf(f.x + c2val(arcs & 3u, b), f.y + c2val((arcs >> 4) & 3u, b));
    m1 = fminf((f.x + lam) + c2val((arcs >> 2) & 3u, b), (f.y + lam) + c2val((arcs >> 6) & 3u, b));
  } else {
    g = C.grec[arcs];
    const float *fp = reinterpret_cast<const float *>(C.X + p);
    const float *bp = reinterpret_cast<const float *>(C.X + g.z);
    const uint32_t *arc = C.garc + (g.x & 0xFFFFu);
    const int w = int(g.y & 0xFu);
    for (int u = 0; u < w; ++u) {
      m0 = fminf(m0, fp[u] + cell_c16(bp, arc[u] & 0xFFFFu));
      m1 = fminf(m1, (fp[u] + lam) + cell_c16(bp, arc[u] >> 16));
    }
  }
  const float dd = m1 - m0;
  // J_i sum in ascending row order; rows forcing the variable (infinite difference) apart. The lanes
  // of a segment are all here, and the branch is uniform over the wavefront's active lanes.
  const int at = int((d1 >> kCellPosShift) & 0x7Fu), h = (int(threadIdx.x) & 63) - at;
  if (longest < 0 || __any(isinf(dd))) {
    float sum = 0.0f;
    int nf = 0;
    for (int q = 0; q < len; ++q) {
      const float dq = lane_read(dd, h + q);
      if (isinf(dq)) ++nf;
      else sum += dq;
    }
    lam = updated(lam, dd, nf ? sum / float(nf) : sum / float(len), nf);
  } else {
    // running sums handed from lane to lane, the last lane's to all
    float sum = dd;
    for (int t = 1; t <= longest; ++t) {
      const float x = lane_before(sum);
      if (at == t) sum = x + dd;
    }
    const float r = lane_read(rcp, len - 1);
    lam = (lam - dd) + over_count(lane_read(sum, h + len - 1), float(len), r);
  }
  C.lam[j] = lam;
  if (gen) {
    if (DIR == kFwd) general_push(C, g, p, lam);
    else general_bstep(C, g, p, lam);
  } else if (DIR == kFwd) {
    C.X[j] = regular ? regular_push(s, f, lam) : narrow_push(arcs, f, lam);
  } else {
    C.X[p] = regular ? regular_bstep(s, b, lam) : narrow_bstep(arcs, b, lam);
  }
}

// The same for a variable in two rows whose levels are regular: both layers in one lane (their links
// are neighbours, one wide LDS access), the exchange in registers. S 0: both levels take, 1: both
// count, 2: by the layers' bits.
template <int DIR, int S>
__device__ __forceinline__ void pair_step(const Cell &C, uint32_t d, float2 l, float2 f0, float2 f1, float4 own, int v) {
  const float2 b0 = make_float2(own.x, own.y), b1 = make_float2(own.z, own.w);
  const bool s0 = S == 2 ? (d & kCellCount) != 0u : S == 1, s1 = S == 2 ? (d & (kCellCount << 16)) != 0u : S == 1;
  const float d0 = regular_m1(s0, f0, b0, l.x) - vmin(f0.x + b0.x, f0.y + b0.y);
  const float d1 = regular_m1(s1, f1, b1, l.y) - vmin(f1.x + b1.x, f1.y + b1.y);
  // halving is division by two; rows forcing the variable (infinite difference) apart
  const float share = (d0 + d1) * 0.5f;
  float2 n = make_float2((l.x - d0) + share, (l.y - d1) + share);
  const bool i0 = isinf(d0), i1 = isinf(d1);
  if (i0 || i1) {
    const int nf = int(i0) + int(i1);
    const float sum = (i0 ? 0.0f : d0) + (i1 ? 0.0f : d1);
    n = make_float2(updated(l.x, d0, sum / float(nf), nf), updated(l.y, d1, sum / float(nf), nf));
  }
  reinterpret_cast<float2 *>(C.lam)[v] = n;
  if (DIR == kFwd) {
    const float2 o0 = regular_push(s0, f0, n.x), o1 = regular_push(s1, f1, n.y);
    reinterpret_cast<float4 *>(C.X)[v] = make_float4(o0.x, o0.y, o1.x, o1.y);
  } else {
    C.X[d & 0x7FFFu] = regular_bstep(s0, b0, n.x);
    C.X[(d >> 16) & 0x7FFFu] = regular_bstep(s1, b1, n.y);
  }
}

// One update pass in direction DIR over the cell's chunks (up to BLOCK layers, or variables of
// kCellPair, of one step). Reads that the chunk before does not write are issued ahead of its work:
// the descriptors two chunks ahead, the multipliers and the pass's standing messages (a forward
// pass: the own links; a backward pass: the parents') one. A lane past its chunk's end reads on
// within the cell's LDS (it ends in slack) and writes nothing.
template <int BLOCK, int DIR, int KIND>
__device__ __forceinline__ void cell_pass(const Cell &C) {
  constexpr bool kPair = KIND == kCellPair;
  using Own = std::conditional_t<kPair, float4, float2>;
  using Lam = std::conditional_t<kPair, float2, float>;
  struct Far {
    float2 a, b;
  };
  const int tid = int(threadIdx.x), nw = C.nwork;
  const float rcp = kPair ? 0.0f : 1.0f / float((tid & 63) + 1);
  // chunk records: 64 of them in a register, one per lane, so that a chunk's bounds cost a lane read
  // instead of a round trip to memory
  int base = -64;
  uint32_t win = 0u;
  auto record = [&](int i) {  // i-th chunk in pass order
    const int q = DIR == kFwd ? min(i, nw - 1) : max(nw - 1 - i, 0);
    if (uint32_t(q - base) >= 64u) {
      base = DIR == kFwd ? q : max(q - 63, 0);
      win = C.work[min(base + (tid & 63), nw - 1)];
    }
    return uint32_t(__builtin_amdgcn_readlane(int(win), q - base));
  };
  auto pos = [&](uint32_t r) { return int(r & 0x1FFFu) + tid; };
  // a descriptor leads to an area, so past the cell's end the last one is read again
  const int last = C.nl / (kPair ? 2 : 1) - 1;
  auto desc = [&](uint32_t r) { return C.w0[min(pos(r), last)]; };
  auto far = [&](uint32_t d) {
    Far x;
    x.a = C.X[d & 0x7FFFu];
    x.b = kPair ? C.X[(d >> 16) & 0x7FFFu] : x.a;
    return x;
  };
  uint32_t r0 = record(0), r1 = record(1);
  uint32_t da = desc(r0), db = desc(r1), ea = 0u;
  Lam la = reinterpret_cast<const Lam *>(C.lam)[pos(r0)];
  if (!kPair) ea = C.w1[pos(r0)];
  Own oa{};
  Far fa{};
  if (DIR == kFwd) oa = reinterpret_cast<const Own *>(C.X)[pos(r0)];
  else fa = far(da);
  for (int i = 0; i < nw; ++i) {
    const uint32_t r2 = record(i + 2);
    // what the pass itself wrote: a forward pass its parents' links, a backward pass its own
    if (DIR == kFwd) fa = far(da);
    else oa = reinterpret_cast<const Own *>(C.X)[pos(r0)];
    const uint32_t dc = desc(r2);
    const Lam lb = reinterpret_cast<const Lam *>(C.lam)[pos(r1)];
    const uint32_t eb = kPair ? 0u : C.w1[pos(r1)];
    Own ob{};
    Far fb{};
    if (DIR == kFwd) ob = reinterpret_cast<const Own *>(C.X)[pos(r1)];
    else fb = far(db);
    if (tid < int((r0 >> 13) & 0x3FFu)) {
      if constexpr (kPair) {
        if (r0 & kCellTakes) pair_step<DIR, 0>(C, da, la, fa.a, fa.b, oa, pos(r0));
        else if (r0 & kCellCounts) pair_step<DIR, 1>(C, da, la, fa.a, fa.b, oa, pos(r0));
        else pair_step<DIR, 2>(C, da, la, fa.a, fa.b, oa, pos(r0));
      } else if (ea & 0x7Fu) {  // not a pad
        layer_step<DIR, KIND == kCellGen>(C, da, ea, la, fa.a, oa, pos(r0), (r0 & kCellRegular) != 0u,
                                             int(r0 >> 28) == 15 ? -1 : int(r0 >> 28), rcp);
      }
    }
    // the next step reads what this one wrote
    if (BLOCK == 64 || (r0 & (DIR == kFwd ? kCellStepEnd : kCellStepBegin))) step_sync<BLOCK>();
    r0 = r1;
    r1 = r2;
    da = db;
    db = dc;
    ea = eb;
    la = lb;
    oa = ob;
    fa = fb;
  }
}

// The messages that direction DIR's pass leaves under the current multipliers (no update): rows are
// independent, so a lane walks a whole row part with the message in registers and no barrier, the
// next level's descriptor and multiplier in flight behind the current one's work. (A kCellPair
// descriptor names no child, so such stages sweep backward only.)
template <int BLOCK, int DIR, int KIND>
__device__ __forceinline__ void cell_sweep(const Cell &C, int bwp) {
  constexpr bool kPair = KIND == kCellPair;
  static_assert(!kPair || DIR == kBwd, "two-row stages sweep backward");
  auto w0 = [&](int j) { return kPair ? uint32_t(reinterpret_cast<const uint16_t *>(C.w0)[j]) : C.w0[j]; };
  for (int k = int(threadIdx.x); k < C.nrow; k += BLOCK) {
    const uint32_t r = C.row[k];
    int j = int(DIR == kFwd ? r & 0x1FFFu : (r >> 13) & 0x1FFFu);
    const int end = int(DIR == kFwd ? (r >> 13) & 0x1FFFu : r & 0x1FFFu);
    uint32_t d0 = w0(j), d1 = kPair ? 0u : C.w1[j];
    float lam = C.lam[j];
    float2 m = DIR == kFwd ? C.X[C.nl + k * bwp] : C.X[j];
    while (j != end) {
      const int p = int(d0 & 0x7FFFu);
      if (KIND == kCellGen && (d1 & kCellGeneral)) {
        const uint4 g = C.grec[d1 >> 16];
        if (DIR == kFwd) general_push(C, g, p, lam);
        else general_bstep(C, g, p, lam);
        const int own = int(g.z);
        j = int(DIR == kFwd ? d0 >> 16 : g.y >> 16);
        m = DIR == kFwd ? C.X[own] : C.X[j];  // used by a narrow neighbour, whose link is its index
        d0 = w0(j);
        d1 = C.w1[j];
        lam = C.lam[j];
      } else {
        const int nx = DIR == kFwd ? int(d0 >> 16) : p;  // a narrow layer's parent's link is its index
        const uint32_t n0 = w0(nx), n1 = kPair ? 0u : C.w1[nx];
        const float nlam = C.lam[nx];
        if constexpr (kPair) {
          m = regular_bstep((d0 & kCellCount) != 0u, m, lam);
        } else {
          m = DIR == kFwd ? narrow_push(d1 >> 16, m, lam) : narrow_bstep(d1 >> 16, m, lam);
        }
        C.X[DIR == kFwd ? j : p] = m;
        j = nx;
        d0 = n0;
        d1 = n1;
        lam = nlam;
      }
    }
  }
  step_sync<BLOCK>();
}

// PROG: which phases the launch runs (kernels.h). first: the multipliers come from storage order
// (and A's incoming messages from the solver's child slots) instead of the run's cell-order arrays.
// all: the launch is the stage's last of a call: multipliers and inner backward messages go back to
// storage order, where every other entry point finds the state of whole iterations.
template <int BLOCK, int PROG, int KIND>
__global__ __launch_bounds__(BLOCK) void cell_kernel(const Dev D, const CellArgs A, const int first, const int all,
                                                     const int n) {
  extern __shared__ __align__(16) char lds[];
  const int cell = xcd_tile(int(blockIdx.x), int(gridDim.x));
  const int4 r0 = A.rec[4 * cell], r1 = A.rec[4 * cell + 1], r2 = A.rec[4 * cell + 2], r3 = A.rec[4 * cell + 3];
  const int nl = r0.x, tid = int(threadIdx.x);
  const int bw = KIND == kCellGen ? A.bw : 2;  // narrow stages have narrow boundaries
  const int32_t *layer = A.layer + r1.x;
  float *lamc = A.lamc + r1.x;
  constexpr bool kPair = KIND == kCellPair;
  const int bwp = bw / 2;
  Cell C;
  C.nwork = r0.y;
  C.nrow = r2.x;
  C.nl = nl;
  C.work = A.work + r0.w;
  C.X = reinterpret_cast<float2 *>(lds);
  C.grec = reinterpret_cast<uint4 *>(C.X + r1.z);
  C.lam = reinterpret_cast<float *>(C.grec + r2.z);
  C.w0 = reinterpret_cast<uint32_t *>(C.lam + nl);
  C.w1 = C.w0 + nl;
  C.row = kPair ? C.w0 + nl / 2 : C.w1 + nl;
  C.garc = C.row + C.nrow;

  // prologue: the program (shared by cells of equal structure, so it comes from cache), the
  // multipliers, and per row part the messages it starts from; every load that needs no other is
  // issued before the first is used, the epilogue's links and terms among them
  constexpr bool kPush = PROG == kCellFirst || PROG == kCellWrap;  // the last phase is a forward one
  constexpr bool kLinked = kPush || PROG == kCellTurn;             // sends to the other stage
  constexpr bool kTerms = PROG != kCellFirst;
  const int kr = min(tid, C.nrow - 1);
  const uint32_t row0 = A.row[r2.y + kr];
  const float2 in0 = PROG == kCellWhole ? make_float2(0.0f, 0.0f)
                                        : *reinterpret_cast<const float2 *>(A.in + size_t(r1.y + kr) * size_t(bw));
  const int link0 = kLinked ? A.link[r1.y + kr] : -1;
  const int term0 = kTerms ? A.term[r1.y + kr] : -1;
  {
    // quads of layers; lanes past the end repeat the last quad (the same values to the same place)
    constexpr int Q = 4;
    const int nq = nl / 4;
    for (int q0 = tid; q0 < nq; q0 += Q * BLOCK) {
      int q[Q];
      float4 l[Q];
#pragma unroll
      for (int t = 0; t < Q; ++t) q[t] = min(q0 + t * BLOCK, nq - 1);
      if (first) {
#pragma unroll
        for (int t = 0; t < Q; ++t) {
          const int4 L = reinterpret_cast<const int4 *>(layer)[q[t]];
          // a pad's value is never used
          l[t] = make_float4(D.lam[max(L.x, 0)], D.lam[max(L.y, 0)], D.lam[max(L.z, 0)], D.lam[max(L.w, 0)]);
        }
      } else {
#pragma unroll
        for (int t = 0; t < Q; ++t) l[t] = reinterpret_cast<const float4 *>(lamc)[q[t]];
      }
      if constexpr (kPair) {
        // two layers per word
        uint2 a[Q];
#pragma unroll
        for (int t = 0; t < Q; ++t) a[t] = reinterpret_cast<const uint2 *>(A.w0 + r0.z / 2)[q[t]];
#pragma unroll
        for (int t = 0; t < Q; ++t) reinterpret_cast<uint2 *>(C.w0)[q[t]] = a[t];
      } else {
        u32x4 a[Q], c[Q];
#pragma unroll
        for (int t = 0; t < Q; ++t) {
          a[t] = reinterpret_cast<const u32x4 *>(A.w0 + r0.z)[q[t]];
          c[t] = reinterpret_cast<const u32x4 *>(A.w1 + r0.z)[q[t]];
        }
#pragma unroll
        for (int t = 0; t < Q; ++t) {
          reinterpret_cast<u32x4 *>(C.w0)[q[t]] = a[t];
          reinterpret_cast<u32x4 *>(C.w1)[q[t]] = c[t];
        }
      }
#pragma unroll
      for (int t = 0; t < Q; ++t) reinterpret_cast<float4 *>(C.lam)[q[t]] = l[t];
    }
  }
  if constexpr (KIND == kCellGen) {
    for (int q = tid; q < r2.z; q += BLOCK) C.grec[q] = A.grec[r2.w + q];
    for (int q = tid; q < r3.x; q += BLOCK) C.garc[q] = A.garc[r3.y + q];
  }
  for (int k = tid; k < C.nrow; k += BLOCK) {
    const uint32_t r = k == tid ? row0 : A.row[r2.y + k];
    C.row[k] = r;
    const int jb = int(r & 0x1FFFu), je = int((r >> 13) & 0x1FFFu);
    const float *in = A.in + size_t(r1.y + k) * size_t(bw);
    const int top = nl + k * bwp;  // the link above the first level; fw, bc: floats of it and of the last level's
    int fw = 2, ba = je, bc = 2;
    if constexpr (KIND == kCellGen) {
      const uint32_t xb = A.w1[r0.z + jb], xe = A.w1[r0.z + je];
      if (xb & kCellGeneral) fw = max(2, int(A.grec[r2.w + int(xb >> 16)].y & 0xFu));
      if (xe & kCellGeneral) {
        const uint4 g = A.grec[r2.w + int(xe >> 16)];
        ba = int(g.z);
        bc = max(2, int((g.y >> 4) & 0xFu));
      }
    }
    float2 fi = make_float2(0.0f, INFINITY);
    float2 bi = make_float2((r & kCellRowTermX) ? 0.0f : INFINITY, (r & kCellRowTermY) ? 0.0f : INFINITY);
    const float *src = in;
    if constexpr (PROG == kCellFirst) {
      if (!(r & kCellRowLast)) {
        const int L = layer[je];
        src = D.mbc + (KIND == kCellGen && D.grec ? D.grec[L].y : 2 * L);
        bi = *reinterpret_cast<const float2 *>(src);
      }
    } else if constexpr (PROG != kCellWhole) {
      const float2 m = k == tid ? in0 : *reinterpret_cast<const float2 *>(in);
      if (!(r & kCellRowRoot)) fi = m;
      if (!(r & kCellRowLast)) bi = m;
    }
    C.X[top] = fi;
    C.X[ba] = bi;
    if constexpr (KIND == kCellGen && PROG != kCellWhole) {
      if (!(r & kCellRowRoot))
        for (int q = 2; q < fw; ++q) reinterpret_cast<float *>(C.X + top)[q] = in[q];
      if (!(r & kCellRowLast))
        for (int q = 2; q < bc; ++q) reinterpret_cast<float *>(C.X + ba)[q] = src[q];
    }
  }
  __syncthreads();

  // the energies of the rows that start in the cell, left above their roots by the backward pass, to
  // the bound terms of iteration it; then a root's forward message there again
  auto energies = [&](int it) {
    float *e = A.root_e + size_t(it) * size_t(A.root_stride);
    for (int k = tid; k < C.nrow; k += BLOCK)
      if (C.row[k] & kCellRowRoot) {
        e[k == tid ? term0 : A.term[r1.y + k]] = C.X[nl + k * bwp].x;
        C.X[nl + k * bwp] = make_float2(0.0f, INFINITY);
      }
    step_sync<BLOCK>();
  };

  // a forward pass leaves pushes on the links below last levels too: their terminals' values again
  auto terminals = [&] {
    for (int k = tid; k < C.nrow; k += BLOCK) {
      const uint32_t r = C.row[k];
      if (r & kCellRowLast)
        C.X[(r >> 13) & 0x1FFFu] = make_float2((r & kCellRowTermX) ? 0.0f : INFINITY, (r & kCellRowTermY) ? 0.0f : INFINITY);
    }
    step_sync<BLOCK>();
  };

  if constexpr (PROG == kCellFirst) {
    cell_sweep<BLOCK, kBwd, KIND>(C, bwp);
    cell_pass<BLOCK, kFwd, KIND>(C);
  } else if constexpr (PROG == kCellTurn) {
    cell_sweep<BLOCK, kBwd, KIND>(C, bwp);
    cell_pass<BLOCK, kFwd, KIND>(C);
    terminals();
    cell_pass<BLOCK, kBwd, KIND>(C);
    energies(0);
  } else if constexpr (PROG == kCellWrap) {
    cell_sweep<BLOCK, kFwd, KIND>(C, bwp);
    cell_pass<BLOCK, kBwd, KIND>(C);
    energies(0);
    cell_pass<BLOCK, kFwd, KIND>(C);
  } else if constexpr (PROG == kCellFinal) {
    cell_sweep<BLOCK, kFwd, KIND>(C, bwp);
    cell_pass<BLOCK, kBwd, KIND>(C);
    energies(0);
  } else {
    cell_sweep<BLOCK, kBwd, KIND>(C, bwp);
    for (int it = 0; it < n; ++it) {
      cell_pass<BLOCK, kFwd, KIND>(C);
      terminals();
      cell_pass<BLOCK, kBwd, KIND>(C);
      energies(it);
    }
  }

  // epilogue: what the row parts send to the other stage, then the multipliers
  if (kLinked) {
    for (int k = tid; k < C.nrow; k += BLOCK) {
      const int to = k == tid ? link0 : A.link[r1.y + k];
      if (to < 0) continue;
      int from = nl + k * bwp;
      if (kPush) {
        from = int((C.row[k] >> 13) & 0x1FFFu);
        if (KIND == kCellGen && (C.w1[from] & kCellGeneral)) from = int(C.grec[C.w1[from] >> 16].z);
      }
      float2 *out = reinterpret_cast<float2 *>(A.out + size_t(to) * size_t(bw));
      out[0] = C.X[from];
      if (KIND == kCellGen)
        for (int q = 1; q < bwp; ++q) out[q] = C.X[from + q];
    }
  }
  if (!all) {
    for (int q = tid; q < nl / 4; q += BLOCK) reinterpret_cast<float4 *>(lamc)[q] = reinterpret_cast<const float4 *>(C.lam)[q];
    return;
  }
  for (int q = tid; q < nl; q += BLOCK) {
    const int L = layer[q];
    if (L < 0) continue;
    D.lam[L] = C.lam[q];
    const uint32_t d1 = A.w1[r0.z + q];
    if (d1 & kCellLast) continue;
    if (KIND == kCellGen && (d1 & kCellGeneral)) {
      const uint4 g = C.grec[d1 >> 16];
      const float *bp = reinterpret_cast<const float *>(C.X + g.z);
      float *to = D.mbc + D.grec[L].y;
      for (int u = 0; u < int((g.y >> 4) & 0xFu); ++u) to[u] = bp[u];
    } else {
      *reinterpret_cast<float2 *>(D.mbc + 2 * L) = C.X[q];
    }
  }
}

template <int BLOCK, int PROG, int KIND>
hipError_t cell_launch(const CellLaunch &c, const Dev &D, const CellArgs &A, hipStream_t s) {
  hipLaunchKernelGGL((cell_kernel<BLOCK, PROG, KIND>), dim3(c.n_cells), dim3(BLOCK), size_t(c.lds), s, D, A, c.first, c.all,
                     c.n);
  return hipGetLastError();
}

template <int BLOCK, int KIND>
hipError_t cell_prog(const CellLaunch &c, const Dev &D, const CellArgs &A, hipStream_t s) {
  switch (c.prog) {
    case kCellTurn: return cell_launch<BLOCK, kCellTurn, KIND>(c, D, A, s);
    case kCellWhole: return cell_launch<BLOCK, kCellWhole, KIND>(c, D, A, s);
    default: break;
  }
  if constexpr (KIND != kCellPair) {
    switch (c.prog) {
      case kCellFirst: return cell_launch<BLOCK, kCellFirst, KIND>(c, D, A, s);
      case kCellWrap: return cell_launch<BLOCK, kCellWrap, KIND>(c, D, A, s);
      case kCellFinal: return cell_launch<BLOCK, kCellFinal, KIND>(c, D, A, s);
      default: break;
    }
  }
  return hipErrorInvalidValue;
}

template <int BLOCK>
hipError_t cell_kind(const CellLaunch &c, const Dev &D, const CellArgs &A, hipStream_t s) {
  switch (c.kind) {
    case kCellLayers: return cell_prog<BLOCK, kCellLayers>(c, D, A, s);
    case kCellGen: return cell_prog<BLOCK, kCellGen>(c, D, A, s);
    case kCellPair: return cell_prog<BLOCK, kCellPair>(c, D, A, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_cells(const CellLaunch &c, const Dev &D, const CellArgs &A, hipStream_t s) {
  if (c.n_cells <= 0) return hipSuccess;
  if (c.lds <= 0 || c.lds > kCellLdsCap) return hipErrorInvalidValue;
  switch (c.block) {
    case 64: return cell_kind<64>(c, D, A, s);
    case 128: return cell_kind<128>(c, D, A, s);
    case 256: return cell_kind<256>(c, D, A, s);
    case 512: return cell_kind<512>(c, D, A, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace bddmp
