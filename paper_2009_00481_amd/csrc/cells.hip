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
// Potts 256x256x8 166 (366), 128x128x4 28 (61), 16x16x4 16 (48); Potts 8x8x3, whole in one workgroup, 10
// (36); a batch of 32 tracking instances of 200 to 1967 detections 132 (916). On 256x256x8 the two launches
// move 189 MB (counted) in 105 and 55 us, 1.2 TB/s; their wavefronts issue in 47% and 36% of their cycles and
// wait in 45% and 46%.
#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>

#include "device.h"
#include "kernels.h"
#include "quotient.h"

namespace bddmp {

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// float of lane l of the wavefront
__device__ __forceinline__ float lane_read(float v, int l) {
  return __int_as_float(__builtin_amdgcn_ds_bpermute(4 * l, __float_as_int(v)));
}

// minimum without the quieting of signalling NaNs that fminf adds: messages, multipliers and their sums hold
// none (a level whose min-marginals are both +inf is refused when the plan is built). Absent nodes may give a
// NaN, by an addition and so a quiet one, which the minimum drops.
__device__ __forceinline__ float vmin(float a, float b) {
  float r;
  asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

// the preceding lane of the wavefront (wave_shr:1)
__device__ __forceinline__ float lane_before(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xF, 0xF, false));
}

// the following one (wave_shl:1)
__device__ __forceinline__ float lane_after(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xF, 0xF, false));
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
  uint32_t *w0, *w1;     // descriptors (internal.h); kCellGen reads ga, gb from global memory instead
  const u32x4 *ga, *gb;
  const uint32_t *work;  // global: the chunks of the steps (internal.h)
  uint32_t *row;
  int nwork, nrow, nl;
  int consts;            // kCellGen: the float index of the constants behind terminal arcs
};

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

// Levels of up to four nodes (kCellGen). Each arc names the float of X behind it: its child's on the
// layer's own link, or one of the constants 0 (TOP) and +inf (BOT, and the arcs of absent nodes), so a
// node costs two LDS reads and no decoding. w: nodes of the level, or of the widest in the chunk.
struct Arcs {
  u32x4 a;  // per node lo | hi << 16
  __device__ __forceinline__ int lo(int u) const { return int(a[u] & 0xFFFFu); }
  __device__ __forceinline__ int hi(int u) const { return int(a[u] >> 16); }
};
template <int W>
__device__ __forceinline__ void gen_push(const Cell &C, u32x4 d, Arcs arc, const float *f, float lam) {
  float *x = reinterpret_cast<float *>(C.X);
  const int own = int(d[0] >> 16);
  // the link's messages start at +inf (one-node levels keep their second float there); a lane owns the
  // link, so the order of the minima does not matter
  C.X[own] = make_float2(INFINITY, INFINITY);
  if (((d[2] >> 20) & 7u) > 2u) C.X[own + 1] = make_float2(INFINITY, INFINITY);
#pragma unroll
  for (int u = 0; u < W; ++u) {
    if (arc.lo(u) < C.consts) __hip_atomic_fetch_min(x + arc.lo(u), f[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    if (arc.hi(u) < C.consts) __hip_atomic_fetch_min(x + arc.hi(u), f[u] + lam, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
  }
}
// lo, hi: what the arcs carry
template <int W>
__device__ __forceinline__ void gen_bstep(const Cell &C, u32x4 d, const float *lo, const float *hi, float lam) {
  const int p = int(d[0] & 0x7FFFu);
  C.X[p] = make_float2(vmin(lo[0], hi[0] + lam), vmin(lo[1], hi[1] + lam));
  if constexpr (W > 2)
    if (((d[2] >> 16) & 7u) > 2u) C.X[p + 1] = make_float2(vmin(lo[2], hi[2] + lam), vmin(lo[3], hi[3] + lam));
}

// Order between a step's LDS writes and the next step's reads. One wavefront's LDS accesses are
// executed in the order it issues them, so a one-wavefront workgroup only keeps the compiler from
// moving them; larger ones meet at a barrier once their LDS accesses are done. (__syncthreads would
// also wait for the descriptors that a pass has in flight from global memory.)
template <int BLOCK>
__device__ __forceinline__ void step_sync() {
  if (BLOCK == 64) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  } else {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
  }
}

// J_i exchange and update: the layer's new multiplier from its difference dd. A variable's layers sit
// on consecutive lanes of one wavefront (at: the layer's place among its len), so the exchange is lane
// moves; the sum runs in ascending row order, rows forcing the variable (infinite difference) apart.
// The lanes of a segment are all here, and the branch is uniform over the wavefront's active lanes.
// longest: one less than the most rows of a variable of the chunk (-1: 16 or more); rcp: 1 / (lane + 1).
__device__ __forceinline__ float exchange(float lam, float dd, int len, int at, int longest, float rcp) {
  const int h = (int(threadIdx.x) & 63) - at;
  if (longest < 0 || __any(isinf(dd))) {
    float sum = 0.0f;
    int nf = 0;
    for (int q = 0; q < len; ++q) {
      const float dq = lane_read(dd, h + q);
      if (isinf(dq)) ++nf;
      else sum += dq;
    }
    return updated(lam, dd, nf ? sum / float(nf) : sum / float(len), nf);
  }
  if (longest <= 1) {
    // one or two rows: the neighbour's difference by a register move
    const float up = lane_after(dd), dn = lane_before(dd);
    const float sum = at ? dn + dd : dd + up;
    return (lam - dd) + (len == 1 ? dd : sum * 0.5f);
  }
  // running sums handed from lane to lane, the last lane's to all
  float sum = dd;
  for (int t = 1; t <= longest; ++t) {
    const float x = lane_before(sum);
    if (at == t) sum = x + dd;
  }
  const float r = lane_read(rcp, len - 1);
  return (lam - dd) + over_count(lane_read(sum, h + len - 1), float(len), r);
}

// One narrow layer's part of a step: min-marginals, exchange, update, and the message it passes on.
// f: the messages on the parent's link (area p), b: those on its own.
template <int DIR>
__device__ __forceinline__ void layer_step(const Cell &C, uint32_t d0, uint32_t d1, float lam, float2 f, float2 b, int j,
                                           bool regular, int longest, float rcp) {
  const bool s = (d0 & kCellCount) != 0u;
  const uint32_t arcs = d1 >> 16;
  float m0, m1;
  if (regular) {
    m0 = vmin(f.x + b.x, f.y + b.y);
    m1 = regular_m1(s, f, b, lam);
  } else {
    m0 = fminf(f.x + c2val(arcs & 3u, b), f.y + c2val((arcs >> 4) & 3u, b));
    m1 = fminf((f.x + lam) + c2val((arcs >> 2) & 3u, b), (f.y + lam) + c2val((arcs >> 6) & 3u, b));
  }
  lam = exchange(lam, m1 - m0, int(d1 & 0x7Fu), int((d1 >> kCellPosShift) & 0x7Fu), longest, rcp);
  C.lam[j] = lam;
  if (DIR == kFwd) C.X[j] = regular ? regular_push(s, f, lam) : narrow_push(arcs, f, lam);
  else C.X[d0 & 0x7FFFu] = regular ? regular_bstep(s, b, lam) : narrow_bstep(arcs, b, lam);
}

// The same for a layer of any kind in a cell with levels of up to four nodes (W: 2 or 4, the chunk's
// widest). f: its own forward messages; lo, hi: what its arcs carry. Absent nodes take what happens to
// lie behind their messages: their arcs are +inf, and a minimum drops the NaN that some bit patterns give.
template <int DIR, int W>
__device__ __forceinline__ void gen_step(const Cell &C, u32x4 d, Arcs arc, float lam, const float *f, const float *lo,
                                         const float *hi, int j, int longest, float rcp) {
  float m0 = vmin(f[0] + lo[0], f[1] + lo[1]), m1 = vmin((f[0] + lam) + hi[0], (f[1] + lam) + hi[1]);
  if constexpr (W > 2) {
    m0 = vmin(vmin(m0, f[2] + lo[2]), f[3] + lo[3]);
    m1 = vmin(vmin(m1, (f[2] + lam) + hi[2]), (f[3] + lam) + hi[3]);
  }
  lam = exchange(lam, m1 - m0, int(d[2] & 0x7Fu), int((d[2] >> kCellPosShift) & 0x7Fu), longest, rcp);
  C.lam[j] = lam;
  if constexpr (DIR == kFwd) gen_push<W>(C, d, arc, f, lam);
  else gen_bstep<W>(C, d, lo, hi, lam);
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

// The cell's chunk records, 64 of them in a register, one per lane, so that a chunk's bounds cost a
// lane read instead of a round trip to memory.
template <int DIR>
struct Work {
  const uint32_t *work;
  int nw, lane, base = -64;
  uint32_t win = 0u;
  __device__ __forceinline__ uint32_t at(int i) {  // i-th chunk in pass order
    const int q = DIR == kFwd ? min(i, nw - 1) : max(nw - 1 - i, 0);
    if (uint32_t(q - base) >= 64u) {
      base = DIR == kFwd ? q : max(q - 63, 0);
      win = work[min(base + lane, nw - 1)];
      // waits here: where the paths meet again the compiler would wait for every load in flight
      asm volatile("" : "+v"(win));
    }
    return uint32_t(__builtin_amdgcn_readlane(int(win), q - base));
  }
};
__device__ __forceinline__ int chunk_count(uint32_t r) { return int((r >> 13) & 0x3FFu); }
__device__ __forceinline__ int chunk_longest(uint32_t r) { return int(r >> 28) == 15 ? -1 : int(r >> 28); }

// A layer's messages in a kCellGen cell: its own nodes' forward ones, and what their arcs carry. wide:
// more than two nodes.
__device__ __forceinline__ void take_f(const Cell &C, u32x4 d, bool wide, float *f) {
  const int p = int(d[0] & 0x7FFFu);
  const float2 a = C.X[p];
  f[0] = a.x;
  f[1] = a.y;
  if (wide) {
    const float2 b = C.X[p + 1];
    f[2] = b.x;
    f[3] = b.y;
  }
}
__device__ __forceinline__ void take_arcs(const Cell &C, Arcs arc, bool wide, float *lo, float *hi) {
  const float *x = reinterpret_cast<const float *>(C.X);
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    lo[u] = x[arc.lo(u)];
    hi[u] = x[arc.hi(u)];
  }
  if (wide) {
#pragma unroll
    for (int u = 2; u < 4; ++u) {
      lo[u] = x[arc.lo(u)];
      hi[u] = x[arc.hi(u)];
    }
  }
}

// One update pass of a kCellGen cell. Its descriptors stay in global memory (the cells are large and
// few, so LDS goes to messages): read two chunks ahead. The multipliers and the pass's standing messages
// (forward: behind the arcs, backward: the own nodes') are read one chunk ahead, as in cell_pass. Two
// slots take turns, so that nothing in flight is moved between registers (a move waits for the load).
template <int BLOCK, int DIR>
__device__ __forceinline__ void gen_pass(const Cell &C) {
  const int tid = int(threadIdx.x), nw = C.nwork;
  const float rcp = 1.0f / float((tid & 63) + 1);
  Work<DIR> work{C.work, nw, tid & 63};
  struct Slot {
    uint32_t r;
    u32x4 d;
    Arcs arc;
    float lam, f[4], lo[4], hi[4];
  };
  auto pos = [&](uint32_t r) { return min(int(r & 0x1FFFu) + tid, C.nl - 1); };
  auto wide = [](uint32_t r) { return ((r >> 24) & 3u) > 1u; };
  auto fetch = [&](Slot &s, int i) {
    s.r = work.at(i);
    s.d = C.ga[pos(s.r)];
    s.arc.a = C.gb[pos(s.r)];
  };
  auto standing = [&](Slot &s) {
    s.lam = C.lam[pos(s.r)];
    if (DIR == kFwd) take_arcs(C, s.arc, wide(s.r), s.lo, s.hi);
    else take_f(C, s.d, wide(s.r), s.f);
  };
  auto step = [&](Slot &s, Slot &next, int i) {
    if (DIR == kFwd) take_f(C, s.d, wide(s.r), s.f);
    else take_arcs(C, s.arc, wide(s.r), s.lo, s.hi);
    standing(next);
    if (tid < chunk_count(s.r) && (s.d[2] & 0x7Fu)) {
      const int j = pos(s.r);
      if (wide(s.r)) gen_step<DIR, 4>(C, s.d, s.arc, s.lam, s.f, s.lo, s.hi, j, chunk_longest(s.r), rcp);
      else gen_step<DIR, 2>(C, s.d, s.arc, s.lam, s.f, s.lo, s.hi, j, chunk_longest(s.r), rcp);
    }
    const bool ends = BLOCK == 64 || (s.r & (DIR == kFwd ? kCellStepEnd : kCellStepBegin));
    fetch(s, i + 2);
    if (ends) step_sync<BLOCK>();
  };
  Slot a, b;
  fetch(a, 0);
  fetch(b, 1);
  standing(a);
  for (int i = 0; i < nw; i += 2) {
    step(a, b, i);
    if (i + 1 < nw) step(b, a, i + 1);
  }
}

// One update pass in direction DIR over the cell's chunks (up to BLOCK layers, or variables of
// kCellPair, of one step). Reads that the chunk before does not write are issued ahead of its work:
// the descriptors two chunks ahead, the multipliers and the pass's standing messages (a forward
// pass: the own links; a backward pass: the parents') one. A lane past its chunk's end reads on
// within the cell's LDS (it ends in slack) and writes nothing.
template <int BLOCK, int DIR, int KIND>
__device__ __forceinline__ void cell_pass(const Cell &C) {
  if constexpr (KIND == kCellGen) {
    gen_pass<BLOCK, DIR>(C);
    return;
  } else {
  constexpr bool kPair = KIND == kCellPair;
  using Own = std::conditional_t<kPair, float4, float2>;
  using Lam = std::conditional_t<kPair, float2, float>;
  struct Far {
    float2 a, b;
  };
  const int tid = int(threadIdx.x), nw = C.nwork;
  const float rcp = kPair ? 0.0f : 1.0f / float((tid & 63) + 1);
  Work<DIR> work{C.work, nw, tid & 63};
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
  uint32_t r0 = work.at(0), r1 = work.at(1);
  uint32_t da = desc(r0), db = desc(r1), ea = 0u;
  Lam la = reinterpret_cast<const Lam *>(C.lam)[pos(r0)];
  if (!kPair) ea = C.w1[pos(r0)];
  Own oa{};
  Far fa{};
  if (DIR == kFwd) oa = reinterpret_cast<const Own *>(C.X)[pos(r0)];
  else fa = far(da);
  for (int i = 0; i < nw; ++i) {
    const uint32_t r2 = work.at(i + 2);
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
    if (tid < chunk_count(r0)) {
      if constexpr (kPair) {
        if (r0 & kCellTakes) pair_step<DIR, 0>(C, da, la, fa.a, fa.b, oa, pos(r0));
        else if (r0 & kCellCounts) pair_step<DIR, 1>(C, da, la, fa.a, fa.b, oa, pos(r0));
        else pair_step<DIR, 2>(C, da, la, fa.a, fa.b, oa, pos(r0));
      } else if (ea & 0x7Fu) {  // not a pad
        layer_step<DIR>(C, da, ea, la, fa.a, oa, pos(r0), (r0 & kCellRegular) != 0u, chunk_longest(r0), rcp);
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
}

// The messages that direction DIR's pass leaves under the current multipliers (no update): rows are
// independent, so a lane walks a whole row part with the message in registers and no barrier, the
// next level's descriptor and multiplier in flight behind the current one's work. (A kCellPair
// descriptor names no child, so such stages sweep backward only.)
template <int BLOCK, int DIR, int KIND>
__device__ __forceinline__ void cell_sweep(const Cell &C, int bwp) {
  constexpr bool kPair = KIND == kCellPair;
  static_assert(!kPair || DIR == kBwd, "two-row stages sweep backward");
  for (int k = int(threadIdx.x); k < C.nrow; k += BLOCK) {
    const uint32_t r = C.row[k];
    int j = int(DIR == kFwd ? r & 0x1FFFu : (r >> 13) & 0x1FFFu);
    const int end = int(DIR == kFwd ? (r >> 13) & 0x1FFFu : r & 0x1FFFu);
    if constexpr (KIND == kCellGen) {
      u32x4 d = C.ga[j];
      Arcs arc{C.gb[j]};
      while (j != end) {
        const int nx = int(DIR == kFwd ? d[1] & 0xFFFFu : d[1] >> 16);
        const u32x4 nd = C.ga[nx];
        const Arcs na{C.gb[nx]};
        const float lam = C.lam[j];
        const bool wide = ((d[2] >> 16) & 7u) > 2u;
        if (DIR == kFwd) {
          float f[4];
          take_f(C, d, wide, f);
          if (wide) gen_push<4>(C, d, arc, f, lam);
          else gen_push<2>(C, d, arc, f, lam);
        } else {
          float lo[4], hi[4];
          take_arcs(C, arc, wide, lo, hi);
          if (wide) gen_bstep<4>(C, d, lo, hi, lam);
          else gen_bstep<2>(C, d, lo, hi, lam);
        }
        j = nx;
        d = nd;
        arc = na;
      }
    } else {
      auto w0 = [&](int q) { return kPair ? uint32_t(reinterpret_cast<const uint16_t *>(C.w0)[q]) : C.w0[q]; };
      uint32_t d0 = w0(j), d1 = kPair ? 0u : C.w1[j];
      float lam = C.lam[j];
      float2 m = DIR == kFwd ? C.X[C.nl + k * bwp] : C.X[j];
      while (j != end) {
        const int p = int(d0 & 0x7FFFu);
        const int nx = DIR == kFwd ? int(d0 >> 16) : p;  // the parent's link is the parent's index
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
  const int4 r0 = A.rec[3 * cell], r1 = A.rec[3 * cell + 1], r2 = A.rec[3 * cell + 2];
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
  C.lam = reinterpret_cast<float *>(C.X + r1.z);
  C.w0 = reinterpret_cast<uint32_t *>(C.lam + nl);
  C.w1 = C.w0 + nl;
  C.row = kPair ? C.w0 + nl / 2 : (KIND == kCellGen ? C.w0 : C.w1 + nl);
  C.ga = A.ga + r0.z;
  C.gb = A.gb + r0.z;
  C.consts = 2 * (r1.z - 2);  // the last areas are the constants' (and one to keep the count even)

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
      } else if constexpr (KIND == kCellLayers) {
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
  if (KIND == kCellGen && tid == 0) C.X[r1.z - 2] = make_float2(0.0f, INFINITY);
  for (int k = tid; k < C.nrow; k += BLOCK) {
    const uint32_t r = k == tid ? row0 : A.row[r2.y + k];
    C.row[k] = r;
    const int jb = int(r & 0x1FFFu), je = int((r >> 13) & 0x1FFFu);
    const float *in = A.in + size_t(r1.y + k) * size_t(bw);
    const int top = nl + k * bwp;  // the link above the first level; fw, bc: floats of it and of the last level's
    int fw = 2, ba = je, bc = 2;
    if constexpr (KIND == kCellGen) {
      const u32x4 xb = C.ga[jb], xe = C.ga[je];
      fw = max(2, int((xb[2] >> 16) & 7u));
      ba = int(xe[0] >> 16);
      bc = max(2, int((xe[2] >> 20) & 7u));
    }
    float2 fi = make_float2(0.0f, INFINITY);
    float2 bi = make_float2((r & kCellRowTermX) ? 0.0f : INFINITY, (r & kCellRowTermY) ? 0.0f : INFINITY);
    const float *src = in;
    if constexpr (PROG == kCellFirst) {
      if (!(r & kCellRowLast)) {
        const int L = layer[je];
        src = D.mbc + (KIND == kCellGen && D.grec ? D.grec[L].y : 2 * L);
        // (areas of wide levels may start at any float)
        if (KIND == kCellGen) bi = make_float2(src[0], src[1]);
        else bi = *reinterpret_cast<const float2 *>(src);
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
    if (KIND == kCellGen) return;
    for (int k = tid; k < C.nrow; k += BLOCK) {
      const uint32_t r = C.row[k];
      // (kCellGen: its arcs name the terminals themselves)
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
        if (KIND == kCellGen) from = int(C.ga[from][0] >> 16);
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
    if constexpr (KIND == kCellGen) {
      const u32x4 d = C.ga[q];
      if (d[2] & kCellLast) continue;
      const float *bp = reinterpret_cast<const float *>(C.X + (d[0] >> 16));
      float *to = D.mbc + (D.grec ? D.grec[L].y : 2 * L);
      for (int u = 0; u < int((d[2] >> 20) & 7u); ++u) to[u] = bp[u];
    } else {
      if (!(A.w1[r0.z + q] & kCellLast)) *reinterpret_cast<float2 *>(D.mbc + 2 * L) = C.X[q];
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
