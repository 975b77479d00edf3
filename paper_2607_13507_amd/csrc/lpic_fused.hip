// The fused particle kernel of the PIC hot path (gfx950, wave64): gather + relativistic
// Boris push + Esirkepov deposit in one pass over a tile-sorted particle stream, with the
// field tile staged in LDS and the tile's current accumulated in LDS (64-bit fixed point on
// the FP32 path, FP64 on the FP64 path) before one global atomic flush per non-zero entry;
// the particles whose stencils have left the staged region of their tile are pushed through
// global memory by the workgroup that met them, or, re-binned, by a second pass.
#include <algorithm>

#include "lpic_internal.hpp"

namespace lpic {

// =======================================================================================
// Fused gather + push + deposit (unified pusher).  Persistent workgroups walk the chunk
// table; for each tile the field region (tile + halo) is staged in LDS once, the current
// accumulates in LDS and is flushed when the tile changes.  Workgroups are mapped to chunks
// so that each XCD (every 8th workgroup) walks a contiguous range of chunks: neighbouring
// tiles share that XCD's L2.
// =======================================================================================
// Region geometries compiled with constant strides: (tile x, y, z, halo, z-layer pad).
// Geometry 0 is the runtime-stride kernel used for every other tiling.  The 3D pads put
// consecutive z layers 4 (8 x 4 x 4 tiles: a 16 x 12 layer is 192 entries, 3 x 64) or 8
// (8 x 8 x 4 tiles: 256 entries) banks apart; the 8 x 4 x 4 pad is also the largest whose
// region, charge planes included, still fits the LDS.  Geometry 7 (8 x 4 x 4 tiles, halo 3)
// runs 512-thread workgroups, two per CU: it is also the second pass of the re-binned
// escape path for 8 x 4 x 4 tilings with halo 4 (its particles lie inside their present
// tile, so a halo of 3 always holds their stencils).  Geometry 8 is the same region without
// the layer pad, for the FP32 steps that carry one charge plane (chained charge, see
// k_fused): it still fits two 512-thread workgroups per CU (81.5 KB each, of 163.8).  Geometry 9 is
// the padded region with 1024-thread workgroups, for FP32 steps with both charge planes:
// they leave room for one workgroup per CU, which then brings all sixteen waves by itself.
struct GeoFix { int tx, ty, tz, halo, pz; };
__host__ __device__ constexpr GeoFix geo_table(int g) {
  return g == 1 ? GeoFix{16, 16, 1, 5, 0} : g == 2 ? GeoFix{8, 8, 1, 5, 0}
       : g == 3 ? GeoFix{32, 32, 1, 5, 0} : g == 4 ? GeoFix{16, 16, 1, 4, 0}
       : g == 5 ? GeoFix{8, 4, 4, 4, 4} : g == 6 ? GeoFix{8, 8, 4, 4, 8}
       : g == 7 ? GeoFix{8, 4, 4, 3, 8} : g == 8 ? GeoFix{8, 4, 4, 3, 0}
       : g == 9 ? GeoFix{8, 4, 4, 3, 8} : GeoFix{0, 0, 0, 0, 0};
}
constexpr int NUM_GEO = 10;   // fused_geometry() returns the first match: 7, never 8 or 9

template <int DIM, int G>
struct GeoStrides {
  static constexpr GeoFix f = geo_table(G);
  using type = FixStrides<f.tx + 2 * f.halo, f.ty + 2 * f.halo, DIM == 3 ? f.tz + 2 * f.halo : 1,
                          DIM == 3 ? f.pz : 0>;
};
template <int DIM>
struct GeoStrides<DIM, 0> {
  using type = DynStrides;
};

// One staged region: the home tile of a run plus `halo` cells, in LDS.
struct Region {
  int r0[3];     // global origin (may be negative: periodic)
  int rw[3];     // extent
};

template <int DIM>
__device__ __forceinline__ Region region_of(const RunDesc& r, const SegDesc& s, int tile,
                                            int halo) {
  Region g;
  const int TXs[3] = {1 << s.lx, 1 << s.ly, DIM == 3 ? (1 << s.lz) : 1};
  int tc[3];
  tc[0] = tile % r.ntx; tile /= r.ntx;
  tc[1] = tile % r.nty;
  tc[2] = tile / r.nty;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    if (d < DIM) { g.r0[d] = tc[d] * TXs[d] - halo; g.rw[d] = TXs[d] + 2 * halo; }
    else { g.r0[d] = 0; g.rw[d] = 1; }
  }
  return g;
}

// The periodic wrap of a staged region (uniform per tile): the wrapped origin per axis,
// and whether some extent exceeds its box's (then a full modulo per cell, else one
// conditional subtraction).
struct RegionWrap {
  int o[3], n[3];
  bool wide;
};

__device__ __forceinline__ RegionWrap region_wrap(const RunDesc& r, const Region& g) {
  RegionWrap w;
  w.n[0] = r.nx; w.n[1] = r.ny; w.n[2] = r.nz;
  w.wide = false;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    w.o[d] = wrapm(g.r0[d], w.n[d]);
    w.wide = w.wide || g.rw[d] > w.n[d];
  }
  return w;
}

// Region cell e (x fastest over the region's extents): its global index, and its LDS entry
// li under the strides S (which may pad the z layers).  With the extents of a fixed
// geometry the decomposition divides by constants.
template <class S>
__device__ __forceinline__ int64_t region_cell(const RegionWrap& w, const S& st, int e,
                                               int& li) {
  const int lx = e % st.ex();
  const int rest = e / st.ex();
  const int ly = rest % st.ey();
  const int lz = rest / st.ey();
  li = lx + ly * st.sy() + lz * st.sz();
  int gx = w.o[0] + lx, gy = w.o[1] + ly, gz = w.o[2] + lz;
  if (w.wide) {
    gx %= w.n[0]; gy %= w.n[1]; gz %= w.n[2];
  } else {
    gx -= gx >= w.n[0] ? w.n[0] : 0;
    gy -= gy >= w.n[1] ? w.n[1] : 0;
    gz -= gz >= w.n[2] ? w.n[2] : 0;
  }
  return ((int64_t)gz * w.n[1] + gy) * w.n[0] + gx;
}

// Stage E and B of the region, clear its current (and charge) planes.  Each thread takes
// up to STAGE_BATCH region cells per pass and issues all their loads before the first LDS
// write, so a tile change costs about one memory latency rather than one per cell (a 3D
// region of 2304 cells is 2.25 cells per thread of a 1024-thread workgroup).
constexpr int STAGE_BATCH = 4;

template <typename R, class S>
__device__ __forceinline__ void stage_region(const RunDesc& r, const Region& g, const S& st,
                                             int njplanes, R* sm, double* jm, bool paired) {
  gptr<R> F[6];
#pragma unroll
  for (int c = 0; c < 6; ++c) F[c] = gp((R*)r.f[c]);
  const int bd = (int)blockDim.x;
  const int plane = st.plane();
  const int ncell = g.rw[0] * g.rw[1] * g.rw[2];
  const RegionWrap w = region_wrap(r, g);
  for (int e0 = threadIdx.x; e0 < ncell; e0 += STAGE_BATCH * bd) {
    R v[STAGE_BATCH][6];
    int li[STAGE_BATCH];
#pragma unroll
    for (int k = 0; k < STAGE_BATCH; ++k) {
      const int e = e0 + k * bd;
      if (e < ncell) {
        const int64_t gi = region_cell(w, st, e, li[k]);
#pragma unroll
        for (int c = 0; c < 6; ++c) v[k][c] = F[c][gi];
      }
    }
#pragma unroll
    for (int k = 0; k < STAGE_BATCH; ++k) {
      if (e0 + k * bd < ncell) {
        const int e = li[k];
        if (paired) {   // 2D: (Ex,By) pairs, (Ey,Bx) pairs, Ez, Bz
          sm[2 * e] = v[k][F_EX];
          sm[2 * e + 1] = v[k][F_BY];
          sm[2 * (plane + e)] = v[k][F_EY];
          sm[2 * (plane + e) + 1] = v[k][F_BX];
          sm[4 * plane + e] = v[k][F_EZ];
          sm[5 * plane + e] = v[k][F_BZ];
        } else {
#pragma unroll
          for (int c = 0; c < 6; ++c) sm[c * plane + e] = v[k][c];
        }
        for (int c = 0; c < njplanes; ++c) jm[c * plane + e] = 0.0;
      }
    }
  }
}

// Add the region's current (and charge) into the global arrays: one atomic per non-zero
// entry, converted to the field precision (FP32 path: from fixed point, times 2^-S).  With
// a single charge plane (with_rho 2 or 3) it goes to rho0 or rho1.
template <typename R, class S>
__device__ __forceinline__ void flush_region(const RunDesc& r, const Region& g, const S& st,
                                             int njplanes, const double* jm, double unscale,
                                             int with_rho) {
  gptr<R> F[5];
#pragma unroll
  for (int c = 0; c < 5; ++c) F[c] = gp((R*)r.f[F_JX + c]);
  if (with_rho == 3) F[3] = gp((R*)r.f[F_R1]);
  const int plane = st.plane();
  const int ncell = g.rw[0] * g.rw[1] * g.rw[2];
  const RegionWrap w = region_wrap(r, g);
  for (int i = threadIdx.x; i < ncell; i += blockDim.x) {
    int e;
    const int64_t gi = region_cell(w, st, i, e);
    for (int c = 0; c < njplanes; ++c) {
      double v;
      if constexpr (sizeof(R) == 4) v = (double)((const long long*)jm)[c * plane + e] * unscale;
      else v = jm[c * plane + e];
      if (v != 0.0) atomic_add_global(F[c] + gi, R(v));
    }
  }
}

// The second pass of the re-binned escape path: its chunk ranges index `list` (entries
// segment << 32 | slot) and, when set, `rec` (the same particles' escape records in the same
// order, read contiguously instead of the particles' scattered slots).
struct PassList {
  const unsigned long long* list;
  const void* rec;
};

// An escaped particle: the same push through global memory, and the path it deposits.
template <typename R>
struct EscPath {
  int c[3];
  R o[3], e[3];
  R w, vz;
  int rho;
};

template <typename R, int DIM, int ORDER>
__device__ __forceinline__ bool escape_push(const RunDesc& r, const SegDesc& s, int64_t p,
                                            const PushConst<R>& k, int with_rho, EscPath<R>& d,
                                            double& ke) {
  PState<R> ps;
  load_particle<R, DIM>(s, r, p, ps);
  if (!ps.alive) return false;
  const GlobalAcc<R> G = global_acc<R>(r);
  R x1[3], g1;
  push<DIM, ORDER>(G, ps.c, ps, k, d.c, d.o, d.e, x1, d.vz, g1);
  const int n[3] = {r.nx, r.ny, r.nz};
#pragma unroll
  for (int i = 0; i < DIM; ++i) {
    d.c[i] = wrapi(d.c[i], n[i]);
    advance_cell<R>(ps.c[i], ps.o[i], x1[i], n[i]);
  }
  if (leaves_box(r, ps.c[0])) ps.alive = false;
  store_particle<R, DIM>(s, r, p, ps);
  d.w = ps.w;
  d.rho = with_rho == 2 && !ps.alive ? 0 : with_rho;
  if (ps.alive) {
    const double u2 = (double)ps.u[0] * ps.u[0] + (double)ps.u[1] * ps.u[1] + (double)ps.u[2] * ps.u[2];
    ke += (double)ps.w * s.m * u2 / (1.0 + (double)g1);
  }
  return true;
}

// Where a workgroup's escaped particles go.
//   KEEP (2D simulations of up to FUSED_KEEP slots, without the re-binned path): the
//     workgroup keeps them itself, at items[base ...] -- the list positions of the particles
//     it is pushing, so no other workgroup writes there and there is room for all of them --
//     and pushes them when its tile or species changes (drain_escapes).  A launch over a
//     list takes 6 us with its gap, whatever it holds: 20 steps of 65,536 FP64 particles
//     765 us with one and 703 without.
//   Otherwise the shared list; in 2D through one in LDS (list, cap entries), so that the
//     particles of a tile reach it side by side and share a deposit box in k_escape.  Where a
//     tile loses most of its particles (a wake's bubble) the workgroup that meets them is no
//     place to push them: the last one ends long after the others.
//   The line between the two (FUSED_KEEP) goes by the slots of the simulation, which bound that
//   tail, not by the escapes per tile, which cause it.  With the list and with every workgroup
//   pushing its own, above the line: 8192 x 512 wakefield box, 15.2M FP32 particles, 12.92 and
//   13.74 ms per 20 steps; laser slab of 16.8M FP32 particles 9.83 and 9.91, 64 slabs of 180M
//   70.1 and 71.4; but a hot slab of 1.5M FP64 particles late in the run 4.00 and 3.71.
struct EscapeOut {
  EscapeList list;
  int32_t* count;              // LDS: entries kept, or in the LDS list
  unsigned long long* lds;     // the LDS list (2D without KEEP): segment << 32 | slot
  int cap;                     // entries the LDS list holds (3D: waiting slots of the rounds)
  int64_t base;                // KEEP
};

// Entry k of the escape list: the particle's record and the bin of the tile it is in.
template <typename R, int DIM>
__device__ __forceinline__ void escape_record(const EscapeList& esc, int64_t k,
                                              const RunDesc& r, const SegDesc& s,
                                              const PartPtrs<R>& q, int32_t p) {
  const PWords<R> x = load_words<R, DIM>(q, p);
  store_rec<R>(esc.rec, k, rec_of(x));
  if (!esc.keys) return;   // (the list may carry records without keys)
  int c[3];
  esc.keys[k] = decode_cell<R, DIM>(q, x.cell, x.pos, c)
                    ? s.bin_base + (((c[2] >> s.lz) * r.nty) + (c[1] >> s.ly)) * r.ntx + (c[0] >> s.lx)
                    : s.bin_base + r.ntiles;
}

// Append the lanes that want it to the workgroup's list or the shared one (one reservation per
// wave), there with their escape records when the list keeps them (3D only: the 2D body has no
// registers to spare for the record's words, and 2D particles rarely leave their regions).
template <typename R, int DIM, bool KEEP>
__device__ __forceinline__ void escape_append(const EscapeOut& out, bool want, int seg,
                                              int32_t p, const PartPtrs<R>& q,
                                              const RunDesc& r, const SegDesc& s) {
  uint64_t mask = __ballot(want);
  if (!mask) return;
  const EscapeList& esc = out.list;
  const int lane = __lane_id();
  int leader = __ffsll((unsigned long long)mask) - 1;
  if constexpr (DIM == 2) {
    int k = 0;
    if (lane == leader) k = atomicAdd(out.count, __popcll(mask));
    k = __shfl(k, leader, 64) + __popcll(mask & ((1ull << lane) - 1ull));
    if constexpr (KEEP) {
      if (want) gp(esc.items)[out.base + k] = (unsigned long long)(uint32_t)p;
      return;
    }
    if (want && k < out.cap) out.lds[k] = ((unsigned long long)seg << 32) | (unsigned long long)p;
    want = want && k >= out.cap;   // a full LDS list: straight to the shared one
    mask = __ballot(want);
    if (!mask) return;
    leader = __ffsll((unsigned long long)mask) - 1;
  }
  unsigned int base = 0;
  if (lane == leader) base = atomicAdd(esc.count, (unsigned int)__popcll(mask));
  base = __shfl(base, leader, 64);
  if (want) {
    const unsigned int k = base + (unsigned int)__popcll(mask & ((1ull << lane) - 1ull));
    if ((int64_t)k < esc.capacity) {
      esc.items[k] = ((unsigned long long)seg << 32) | (unsigned long long)p;
      if constexpr (DIM == 3)
        if (esc.rec) escape_record<R, DIM>(esc, k, r, s, q, p);
    }
  }
}

// The particles of one chunk against the staged region, in rounds: each thread first
// issues the loads of BATCH particles (a workgroup apart, so every load instruction reads 64
// consecutive particles) and then pushes them one by one, so HBM latency is paid once per
// round rather than once per particle.  Returns the summed w m u^2/(1+gamma).
// In 3D one particle per thread per round: the unrolled body of four 3D particles is too
// large for the compiler to keep their states in registers (it put them in scratch memory,
// read and written for every particle), and a 3D workgroup brings 16 waves per CU anyway.
// In 2D FP64 one as well: a second FP64 state takes the registers of a third wave per SIMD
// (169 VGPRs with two, two waves; 154 with one, three waves and a 10% faster launch).
template <typename R, int DIM>
constexpr int batch_of() { return DIM == 3 ? 1 : (sizeof(R) == 4 ? 4 : 1); }
// Waves per SIMD the fused kernel's register budget is set for: 2D FP32 and the two-per-CU
// 3D FP32 geometry fit 4 (at most 128 VGPRs), the others keep the compiler's choice.
template <typename R, int DIM, int G>
constexpr int fused_waves() {
  return (sizeof(R) == 4 && (DIM == 2 || G >= 7)) ? 4 : 1;
}

// Threads per workgroup: a 3D region (tile + halo on three axes) fills most of a CU's LDS,
// so one workgroup per CU must bring enough waves by itself: 16 (four per SIMD) in FP32, whose
// quadratic particle loop fits 128 VGPRs; 8 in FP64, which needs more registers per lane.
// The smaller regions of geometries 7 and 8 let two 512-thread workgroups share a CU.
template <typename R, int DIM, int G>
constexpr int fused_block() {
  return DIM == 2 ? 256 : (sizeof(R) == 8 || G == 7 || G == 8 ? 512 : 1024);
}

// pl.list != NULL (the second pass of the re-binned escape path): the chunk's range indexes
// pl.list, whose entries name the particles (segment << 32 | slot), and pl.rec when set.
// Local start cell a of a particle in the staged region, and whether it can be on chip: a
// particle that stays in its cell for the half push and keeps its nearest node reads and
// adds cells [a-1, a+2] per axis, so a must lie in [1, rw-3].  The exact test follows once
// the particle's own half-step position and path are known (gather_fits, deposit_fits): a
// fast particle near the edge of the region may still need the cells beyond.
template <int DIM>
__device__ __forceinline__ bool on_chip(const int c[3], const Region& g, const int n[3],
                                        int a[3]) {
  bool inside = true;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    if (d < DIM) {
      int v = c[d] - g.r0[d];
      v = v < 0 ? v + n[d] : (v >= n[d] ? v - n[d] : v);
      a[d] = v;
      inside = inside && v >= 1 && v <= g.rw[d] - 3;
    } else {
      a[d] = 0;
    }
  }
  return inside;
}

// Whether start cell a lies at least two cells inside the staged region on every axis:
// then, whatever the particle's momentum, its gather stencil and deposit window fit (with
// dt below the CFL step a particle moves less than half a cell per axis in a half push, so
// the stencil lies in [a-2, a+2] and the window in [a-2, a+3]), and the exact tests can be
// skipped for a wave whose particles all start there.
template <int DIM>
__device__ __forceinline__ bool deep_inside(const int a[3], const Region& g) {
  bool deep = true;
#pragma unroll
  for (int d = 0; d < DIM; ++d) deep = deep && a[d] >= 2 && a[d] <= g.rw[d] - 4;
  return deep;
}

// Push and deposit one particle against the staged region if its gather stencil and its
// deposit window both lie inside it (the particle is stored); false otherwise (nothing is
// written and the particle's stored state is unchanged: it escapes to a later pass).
// check: false when every particle of the wave starts deep inside the region (a uniform
// value, so the tests are branched over rather than evaluated).
template <typename R, int DIM, int ORDER, class LA>
__device__ __forceinline__ bool push_on_chip(const RunDesc& r, const Region& g, const LA& L,
                                             const int n[3], const int a[3], PState<R>& ps,
                                             const PushConst<R>& k, const PartPtrs<R>& q,
                                             int32_t slot, int with_rho, bool want_ke,
                                             double& ke, bool check) {
  const int lim[3] = {g.rw[0] - 1, g.rw[1] - 1, g.rw[2] - 1};
  int pcell[3];
  R po[3], xh[3];
  half_push<DIM>(a, ps, k, pcell, po, xh);
  bool fit = true;
  if (check) fit = gather_fits<DIM, ORDER>(pcell, po, lim);
  if (!fit) return false;
  R pe[3], x1[3], vz1, g1;
  push_rest<DIM, ORDER>(L, pcell, po, xh, ps, k, pe, x1, vz1, g1);
  if (check) fit = deposit_fits<DIM, ORDER>(pcell, po, pe, lim);
  if (!fit) return false;
#pragma unroll
  for (int d = 0; d < DIM; ++d) advance_cell<R>(ps.c[d], ps.o[d], x1[d], n[d]);
  if (leaves_box(r, ps.c[0])) ps.alive = false;
  // (with_rho 2: the charge where the next step's paths start; a particle leaving the box
  // has none there)
  deposit<DIM, ORDER>(L, pcell, po, pe, ps.w, vz1, k, with_rho == 2 && !ps.alive ? 0 : with_rho);
  store_particle<R, DIM>(q, slot, ps);
  if (want_ke && ps.alive) {   // diagnostic steps only
    const double u2 = (double)ps.u[0] * ps.u[0] + (double)ps.u[1] * ps.u[1] +
                      (double)ps.u[2] * ps.u[2];
    ke += (double)ps.w * u2 / (1.0 + (double)g1);
  }
  return true;
}

// 3D rounds with compaction (one particle per thread per round): each thread first reads
// only its particle's cell and classifies it (on chip / escaped / none); the places of the
// on-chip ones go into a ring in LDS, and as soon as it holds one for every thread they are
// pushed, so no lane idles for escaped particles however many there are.  One barrier per
// round: its counts (three sets, taken in turn) and its places in the ring are not written
// again before every wave has passed the next barrier.  The cells of the next round are loaded
// while this one is pushed.  Escaped particles wait in LDS and go to the escape list by the
// hundred: a reservation per round kept every round waiting for a global atomic and for the
// loads of a few records.  What bounds it now is the body itself: over a sort interval LDS 61%
// and the vector units 60% of the busy cycles, over half of the LDS cycles bank conflicts of
// random positions.
// 20 steps of 256^3 FP32, 134M particles: three barriers and a reservation per round 369 ms,
// one barrier 355, with the ring instead of a push per round 347 (100 x 84 x 60 FP64, 10
// steps: 9.76, 9.74, 9.54 ms).  768 instead of 512 threads in FP64 (three waves per SIMD, 168
// VGPRs): 9.37 ms, but 9.8 instead of 9.2 right after a sort, where the 1024 particles of a
// tile make two full rounds of 512.
constexpr int ROUND_ESC = 256;
constexpr int ROUNDS = 64;   // of up to 1024 threads: places of 16 bits

// LDS of the rounds, in words, for a workgroup of bd threads and `wait` waiting particles:
// ROUND_ESC in the fixed geometries (all fit), with runtime strides what the planes leave, at
// least 56.
constexpr int ROUND_ESC_MIN = 56;
__host__ __device__ constexpr int round_words(int bd, int wait) { return bd + wait + 8; }

// The waiting escaped particles to the escape list (every thread calls it).
template <typename R, int DIM>
__device__ __forceinline__ void flush_waiting(const EscapeList& esc, const int32_t* wait, int m,
                                              int32_t* gbase, int seg, const PartPtrs<R>& q,
                                              const RunDesc& r, const SegDesc& s) {
  if (threadIdx.x == 0) *gbase = (int32_t)atomicAdd(esc.count, (unsigned int)m);
  __syncthreads();
  const int64_t base = (int64_t)(uint32_t)*gbase;
  for (int e = (int)threadIdx.x; e < m; e += (int)blockDim.x)
    if (base + e < esc.capacity) {
      const int32_t es = wait[e];
      esc.items[base + e] = ((unsigned long long)seg << 32) | (unsigned long long)(uint32_t)es;
      if (esc.rec) escape_record<R, DIM>(esc, base + e, r, s, q, es);
    }
  __syncthreads();                     // the list and gbase may be written again
}

template <typename R, int DIM, int ORDER, int BD, class LA>
__device__ __forceinline__ double process_chunk_compact(
    const RunDesc& r, const SegDesc& s, int seg, const Chunk& ch, const Region& g, const LA& L,
    int with_rho, bool want_ke, const EscapeOut& out, const PassList& pl, int32_t* cbuf) {
  const EscapeList& esc = out.list;
  const int n[3] = {r.nx, r.ny, r.nz};
  const PushConst<R> k = push_const<R>(r, s);
  const PartPtrs<R> q = part_ptrs<R>(s, r);
  const int tid = (int)threadIdx.x;
  const int lane = __lane_id();
  const uint64_t below = (1ull << lane) - 1ull;
  uint16_t* list = (uint16_t*)cbuf;    // a ring of 2 BD places in the present ROUNDS rounds
  const int room = out.cap;            // escaped slots that may wait
  int32_t* cnt = cbuf + BD;            // [0..2] on chip, [3..5] escaped, by round modulo 3
  int32_t* gbase = cnt + 6;
  int32_t* wait = cnt + 8;
  if (tid < 6) cnt[tid] = 0;
  __syncthreads();
  double ke = 0.0;
  int pend = 0;                        // escaped particles waiting (uniform)
  int turn = 0;
  int head = 0, tot = 0;               // the ring: first place taken and how many (uniform)
  int32_t from = ch.beg;               // what its places count from
  auto place = [](int i) {             // (i < 4 BD)
    return (BD & (BD - 1)) == 0 ? i & (2 * BD - 1) : (i < 2 * BD ? i : i - 2 * BD);
  };
  // the cell word (FP32) or positions (FP64) of this thread's next particle
  int32_t ncell = -1;
  R npos[3] = {R(-1), R(-1), R(-1)};
  auto prefetch = [&](int32_t lp) {
    if (pl.list || lp >= ch.end) return;
    if constexpr (sizeof(R) == 4) {
      ncell = *at_byte(q.cell, (uint32_t)lp * 4u);
    } else {
#pragma unroll
      for (int d = 0; d < DIM; ++d) npos[d] = *at_byte(q.pos[d], (uint32_t)lp * 8u);
    }
  };
  prefetch(ch.beg + tid);
  for (int32_t base = ch.beg; base < ch.end; base += BD) {
    const int32_t lp = base + tid;
    const bool ok = lp < ch.end;
    const int next = turn == 2 ? 0 : turn + 1;
    int32_t slot = lp;
    bool alive = false;
    int c[3] = {0, 0, 0};
    if (ok) {
      if (pl.list) {
        slot = (int32_t)(gp(pl.list)[lp] & 0xffffffffull);
        alive = pl.rec ? rec_cell<R, DIM>(q, pl.rec, lp, c) : load_cell<R, DIM>(q, slot, c);
      } else {
        alive = decode_cell<R, DIM>(q, ncell, npos, c);
      }
    }
    prefetch(lp + BD);
    int a[3];
    const bool inside = alive && on_chip<DIM>(c, g, n, a);
    const bool gone = alive && !inside;
    const uint64_t mi = __ballot(inside), me = __ballot(gone);
    int bi = 0, be = 0;
    if (lane == 0) {
      if (mi) bi = atomicAdd(&cnt[turn], __popcll(mi));
      if (me) be = atomicAdd(&cnt[3 + turn], __popcll(me));
    }
    bi = uniform(bi);
    be = uniform(be) + pend + __popcll(me & below);
    if (inside) list[place(head + tot + bi + __popcll(mi & below))] = (uint16_t)(lp - from);
    if (gone && be < room) wait[be] = slot;
    escape_append<R, DIM, false>(out, gone && be >= room, seg, slot, q, r, s);
    if (tid < 2) cnt[3 * tid + next] = 0;
    __syncthreads();
    tot += uniform(cnt[turn]);
    pend += uniform(cnt[3 + turn]);
    if (pend >= room / 2) {
      flush_waiting<R, DIM>(esc, wait, min(pend, room), gbase, seg, q, r, s);
      pend = 0;
    }
    const bool last = base + BD >= ch.end || base + BD - from >= ROUNDS * BD;
    while (tot >= BD || (last && tot > 0)) {
      const int m = min(tot, BD);
      int32_t src = 0;
      if (tid < m) src = from + (int32_t)list[place(head + tid)];
      // more than BD taken: the next round's places may be these
      if (tot > BD) __syncthreads();
      head = place(head + m);
      tot -= m;
      bool late = false;               // on chip by its cell, not by its own path
      int32_t p = src;
      if (tid < m) {
        PState<R> ps;
        if (pl.list) {
          p = (int32_t)(gp(pl.list)[src] & 0xffffffffull);
          if (pl.rec) decode_particle<R, DIM>(q, words_of(load_rec<R>(pl.rec, src)), ps);
          else load_particle<R, DIM>(q, p, ps);
        } else {
          load_particle<R, DIM>(q, p, ps);
        }
        int b[3];
        (void)on_chip<DIM>(ps.c, g, n, b);
        // always tested: skipping the tests for deep waves costs the 3D body a spilled
        // register
        late = !push_on_chip<R, DIM, ORDER>(r, g, L, n, b, ps, k, q, p, with_rho, want_ke, ke,
                                            true);
      }
      // late ones wait too, counted with the next round
      const uint64_t ml = __ballot(late);
      if (ml) {
        int bl = 0;
        if (lane == 0) bl = atomicAdd(&cnt[3 + next], __popcll(ml));
        bl = uniform(bl) + pend + __popcll(ml & below);
        if (late && bl < room) wait[bl] = p;
        escape_append<R, DIM, false>(out, late && bl >= room, seg, p, q, r, s);
      }
    }
    if (last) from = base + BD;
    turn = next;
  }
  __syncthreads();
  pend += uniform(cnt[3 + turn]);
  if (pend) flush_waiting<R, DIM>(esc, wait, min(pend, room), gbase, seg, q, r, s);
  return ke * s.m;
}

template <typename R, int DIM, int ORDER, int BD, bool DIRECT, bool KEEP, class LA>
__device__ __forceinline__ double process_chunk(const RunDesc& r, const SegDesc& s, int seg,
                                                const Chunk& ch, const Region& g,
                                                const LA& L, int with_rho,
                                                bool want_ke, const EscapeOut& out,
                                                const PassList& pl, int32_t* cbuf,
                                                bool by_four) {
  // 3D: compacted rounds, except for the second pass of the re-binned path on the two-per-CU
  // geometry (DIRECT), whose particles lie inside their present tile (nearly all on chip):
  // there the records are loaded directly, one memory latency and no barriers per round
  if constexpr (DIM == 3)
    if (!(DIRECT && pl.rec))
      return process_chunk_compact<R, DIM, ORDER, BD>(r, s, seg, ch, g, L, with_rho, want_ke, out,
                                                  pl, cbuf);
  (void)cbuf;
  const int n[3] = {r.nx, r.ny, r.nz};
  const PushConst<R> k = push_const<R>(r, s);
  const PartPtrs<R> q = part_ptrs<R>(s, r);
  double ke = 0.0;
  constexpr int BATCH = batch_of<R, DIM>();
  const int32_t span = (int32_t)blockDim.x * BATCH;
  // the particle of a thread in a batch of blockDim: 2D by_four, neighbours go to the four
  // waves of the workgroup (cell_order)
  const int32_t at = DIM == 2 && by_four ? (int32_t)(4 * (threadIdx.x & 63) + (threadIdx.x >> 6))
                                         : (int32_t)threadIdx.x;
  for (int32_t base = ch.beg; base < ch.end; base += span) {
    PState<R> ps[BATCH];
    int32_t pi[BATCH];
    bool ok[BATCH];
#pragma unroll
    for (int b = 0; b < BATCH; ++b) {
      const int32_t lp = base + b * (int32_t)blockDim.x + at;
      ok[b] = lp < ch.end;
      pi[b] = lp;
      if (pl.list && ok[b]) pi[b] = (int32_t)(gp(pl.list)[lp] & 0xffffffffull);
      if (ok[b]) {
        if constexpr (DIM == 3) {
          if (pl.rec) decode_particle<R, DIM>(q, words_of(load_rec<R>(pl.rec, lp)), ps[b]);
          else load_particle<R, DIM>(q, pi[b], ps[b]);
        } else {
          load_particle<R, DIM>(q, pi[b], ps[b]);   // 2D lists carry no records
        }
      }
    }
#pragma unroll
    for (int b = 0; b < BATCH; ++b) {
      int a[3];
      const bool live = ok[b] && ps[b].alive;
      const bool in = live && on_chip<DIM>(ps[b].c, g, n, a);
      const bool check = __ballot(in && !deep_inside<DIM>(a, g)) != 0;
      bool done = false;
      if (in)
        done = push_on_chip<R, DIM, ORDER>(r, g, L, n, a, ps[b], k, q, pi[b], with_rho,
                                           want_ke, ke, check);
      escape_append<R, DIM, KEEP>(out, live && !done, seg, pi[b], q, r, s);
    }
  }
  return ke * s.m;
}

// Empties the workgroup's list at the end of a tile (KEEP: of a tile's species): KEEP pushes
// the particles (their kinetic energy is returned), otherwise they move to the shared list in
// one piece.
// Every thread calls it; the first barrier stands whatever the count.  Between the read of the
// count and the next append lies a barrier on every way out: on the early return the one of
// the next tile's staging or, for KEEP, whose species may change within a tile (nothing is
// staged then), the one right after the read; otherwise the last one here.
template <typename R, int DIM, bool KEEP>
__device__ __forceinline__ double drain_escapes(const Tables& T, int seg, const EscapeOut& out,
                                                int with_rho) {
  __syncthreads();
  if constexpr (DIM == 3) return 0.0;
  const int n = *out.count;
  if constexpr (KEEP) __syncthreads();
  if (n == 0) return 0.0;
  double ke = 0.0;
  if constexpr (KEEP) {
    const SegDesc& s = seg_of(T, seg);
    const RunDesc& r = run_of(T, s.run);
    const PushConst<R> k = push_const<R>(r, s);
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
      const int64_t p = (int64_t)gp(out.list.items)[out.base + i];
      EscPath<R> d;
      const bool live = s.order == 1 ? escape_push<R, DIM, 1>(r, s, p, k, with_rho, d, ke)
                                     : escape_push<R, DIM, 2>(r, s, p, k, with_rho, d, ke);
      if (!live) continue;
      const GlobalAcc<R> G = global_acc<R>(r);
      if (s.order == 1) deposit<DIM, 1>(G, d.c, d.o, d.e, d.w, d.vz, k, d.rho);
      else deposit<DIM, 2>(G, d.c, d.o, d.e, d.w, d.vz, k, d.rho);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      *out.count = 0;
      atomicAdd(out.list.total, (unsigned long long)n);
    }
  } else {
    const int m = min(n, out.cap);
    __syncthreads();
    if (threadIdx.x == 0) *out.count = (int32_t)atomicAdd(out.list.count, (unsigned int)m);
    __syncthreads();
    const int64_t base = (int64_t)(uint32_t)*out.count;
    for (int i = threadIdx.x; i < m; i += blockDim.x)
      if (base + i < out.list.capacity)
        gp(out.list.items)[base + i] = out.lds[i];
    __syncthreads();
    if (threadIdx.x == 0) *out.count = 0;
  }
  __syncthreads();
  return ke;
}

template <typename T>
__device__ __forceinline__ T block_sum(T v, T* red) {
  v = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  T t = T(0);
  if (threadIdx.x == 0)
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += red[w];
  return t;
}

// Whether particles that share a cell lie side by side in the stream from slot p on: at
// least CELL_PAIRS pairs of its first 64 that are up to 7 apart (two a cell in cell order give
// 32, eight 224 or, after a cell's worth of drift, about 70; a mixed order of 256 cells 2).
// Adds of one wave to one address serialise, so such a stream is dealt to the workgroup's
// waves in turn (by_four).  1000 x 750 cells with charge, a stateless step, in slot order and
// dealt out: 8 a cell FP64 530 and 442 us, FP32 356 and 288; 4 a cell FP32 189 and 176; 1 or
// 2 a cell within 1%.  A mixed stream would only lose (four times the lines per load: 3% in
// FP64, 9% in FP32), so lpic_step, whose first sort spreads every tile, does not ask.
constexpr int CELL_PAIRS = 16;

template <typename R>
__device__ __forceinline__ bool cell_order(const PartPtrs<R>& q, int32_t p, int32_t end) {
  const int lane = __lane_id();
  int c[3] = {-1, -1, 0};
  const bool ok = p + lane < end && load_cell<R, 2>(q, p + lane, c);
  const int key = ok ? c[1] * q.nx + c[0] : -1 - lane;
  int pairs = 0;
#pragma unroll
  for (int d = 1; d < 8; ++d) pairs += __popcll(__ballot(key == __shfl_up(key, d, 64) && lane >= d));
  return pairs >= CELL_PAIRS;
}

// A descriptor copied into wavefront-uniform registers word by word.  Every lane holds the
// same descriptor, but loaded through a generic reference (the device table, or the copy in
// the kernel arguments) its words land in vector registers; with the particle loop's
// registers at the limit of four waves per SIMD they were spilled to scratch memory around
// every chunk, which raised the kernel's memory traffic about 40% above the bytes its
// particles and fields need.
template <typename D>
__device__ __forceinline__ D uniform_copy(const D& src) {
  static_assert(sizeof(D) % 4 == 0, "descriptor of whole words");
  D out;
  const uint32_t* w = (const uint32_t*)&src;
  uint32_t* o = (uint32_t*)&out;
#pragma unroll
  for (int i = 0; i < (int)(sizeof(D) / 4); ++i) o[i] = __builtin_amdgcn_readfirstlane(w[i]);
  return out;
}

// Fused gather + push + deposit over the chunk table, persistent: the grid is a multiple of
// 8 and XCD x (workgroups x, x+8, ...) owns the contiguous chunk range [x*per, (x+1)*per),
// split into equal contiguous slices per workgroup.  Consecutive chunks of one tile (and of
// the other species of the same box, which follow in the table) reuse the staged region;
// the region is flushed when the tile changes.
template <typename R, int DIM, int G, bool KEEP>
__global__ __launch_bounds__((fused_block<R, DIM, G>())) __attribute__((amdgpu_waves_per_eu(fused_waves<R, DIM, G>()))) void k_fused(Tables T, const Chunk* chunks,
                                               const int32_t* nchunks, int with_rho,
                                               double* kinetic, int ke_to_diag,
                                               EscapeList esc, int list_end, int probe,
                                               const int32_t* jshift, PassList pl) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ double red[fused_block<R, DIM, G>() / 64];
  __shared__ int32_t kept;   // escaped particles of the present tile and species (2D)
  R* sm = (R*)smem_raw;
  const int nch = uniform(*nchunks);
  const int nb8 = gridDim.x >> 3;
  const int per = (nch + 7) >> 3;
  const int q = (per + nb8 - 1) / nb8;
  const int xcd = blockIdx.x & 7, j = blockIdx.x >> 3;
  const int lo = xcd * per + j * q;
  const int hi = min(min(lo + q, (xcd + 1) * per), nch);
  if (lo >= hi) return;

  using ST = typename GeoStrides<DIM, G>::type;
  const SegDesc& s0 = seg_of(T, uniform(chunks[lo].seg));
  ST st;
  if constexpr (G == 0) {
    const int rw = (1 << s0.lx) + 2 * s0.halo, rh = (1 << s0.ly) + 2 * s0.halo;
    const int rd = DIM == 3 ? (1 << s0.lz) + 2 * s0.halo : 1;
    st.sy_ = rw;
    st.sz_ = rw * rh;
    st.plane_ = rw * rh * rd;
    st.ey_ = rh;
  }
  const int plane = st.plane();
  const int njplanes = 3 + charge_planes(with_rho);
  // the current planes follow the six field planes; 6 plane values of 4 or 8 bytes end on an
  // 8-byte boundary, as the 64-bit LDS atomics need
  double* jm = (double*)(sm + 6 * plane);
  // after the current (and charge) planes: 3D the round compaction's slot list, 2D the
  // list of escaped particles
  int32_t* cbuf = (int32_t*)(jm + (size_t)njplanes * plane);
  LdsAcc<R, ST, DIM == 2> L;
  L.fbase = sm;
  L.jbase = jm;
  L.st = st;
  L.jfold = 1.0f;

  // (the lists take the launch's LDS after the current planes, up to list_end)
  const int left = list_end - (int)((unsigned char*)cbuf - smem_raw);
  EscapeOut out{esc, &kept, (unsigned long long*)cbuf,
                left / 8, 0};
  if constexpr (DIM == 3)
    out.cap = G ? ROUND_ESC : min(ROUND_ESC, left / 4 - round_words(fused_block<R, DIM, G>(), 0));
  if (threadIdx.x == 0) kept = 0;   // (staging's barrier comes before the first append)
  bool by_four = false;
  if constexpr (DIM == 2) {
    if (probe) {
      const int32_t beg = uniform(chunks[lo].beg), end = uniform(chunks[lo].end);
      by_four = cell_order<R>(part_ptrs<R>(s0, run_of(T, s0.run)), beg, end);
    }
  }
  int cur_run = -1, cur_tile = -1, cur_seg = -1;
  Region g;
  double ke = 0.0;
  double unscale = 1.0;
  for (int c = lo; c < hi; ++c) {
    Chunk ch = chunks[c];
    ch.seg = uniform(ch.seg);
    ch.tile = uniform(ch.tile);
    ch.beg = uniform(ch.beg);
    ch.end = uniform(ch.end);
    const SegDesc s = uniform_copy(seg_of(T, ch.seg));
    const bool new_tile = s.run != cur_run || ch.tile != cur_tile;
    if (new_tile || (KEEP && ch.seg != cur_seg)) {
      if (cur_run >= 0) ke += drain_escapes<R, DIM, KEEP>(T, cur_seg, out, with_rho);
      if (KEEP) out.base = s.pbase + ch.beg;
      cur_seg = ch.seg;
    }
    if (new_tile) {
      if (cur_run >= 0) {
        const RunDesc& rp = run_of(T, cur_run);
        flush_region<R>(rp, g, st, njplanes, jm, unscale, with_rho);
        if (kinetic || ke_to_diag) {
          const double t = block_sum(ke, red);
          if (threadIdx.x == 0) atomic_add_global(ke_to_diag ? rp.diag + DIAG_UKIN : kinetic, t);
          ke = 0.0;
        }
      }
      if constexpr (sizeof(R) == 4) {
        const int sh = uniform(jshift[s.run]);
        L.jfold = ldexpf(1.0f, sh);
        unscale = ldexp(1.0, -sh);
      }
      const RunDesc rn = run_of(T, s.run);
      g = region_of<DIM>(rn, s, ch.tile, G ? geo_table(G).halo : s.halo);
      __syncthreads();
      stage_region<R>(rn, g, st, njplanes, sm, jm, DIM == 2);
      __syncthreads();
      cur_run = s.run;
      cur_tile = ch.tile;
    }
    const RunDesc r = run_of(T, s.run);
    const bool want_ke = kinetic || ke_to_diag;
    ke += s.order == 1
              ? process_chunk<R, DIM, 1, fused_block<R, DIM, G>(), (G >= 7), KEEP>(r, s, ch.seg, ch, g, L, with_rho, want_ke, out, pl, cbuf, by_four)
              : process_chunk<R, DIM, 2, fused_block<R, DIM, G>(), (G >= 7), KEEP>(r, s, ch.seg, ch, g, L, with_rho, want_ke, out, pl, cbuf, by_four);
  }
  const RunDesc& rl = run_of(T, cur_run);
  ke += drain_escapes<R, DIM, KEEP>(T, cur_seg, out, with_rho);
  flush_region<R>(rl, g, st, njplanes, jm, unscale, with_rho);
  if (kinetic || ke_to_diag) {
    const double t = block_sum(ke, red);
    if (threadIdx.x == 0) atomic_add_global(ke_to_diag ? rl.diag + DIAG_UKIN : kinetic, t);
  }
}

// Escaped particles of a shared list.  Entries that lie side by side come from one tile and
// its neighbourhood (escape_append), so a workgroup adds the windows of 256 of them in a box
// in LDS (pick_box) and flushes it once: with an atomic per window entry the atomics were
// what a launch took, whatever the number of workgroups (hot slab of 1.5M FP64 particles,
// 20 steps late in the run: 5.0 ms with 128 workgroups and 5.2 with 1024, 3.8 with boxes).
// Each workgroup takes a contiguous share of the list.  BOX false: every entry straight into
// memory, for the two lists of a re-binned step, which are short or empty (the boxes' code and
// LDS are then all that a launch takes).  skip_at: a list of at least this many entries was
// taken by the re-binned path; only the clearing is left to do.
template <typename R, int DIM, bool BOX>
__global__ __launch_bounds__(256) void k_escape(Tables T, int with_rho, double* kinetic,
                                                int ke_to_diag, EscapeList esc, int skip_at,
                                                int cap) {
  extern __shared__ double jm[];
  __shared__ int red[BOX ? 4 : 1][13];
  __shared__ int wrun[4];
  int64_t cnt = min((int64_t)esc.count[0], esc.capacity);
  if ((int)min(esc.count[0], 0x7fffffffu) >= skip_at) cnt = 0;
  const int lane = (int)__lane_id(), wave = (int)(threadIdx.x >> 6);
  const int planes = 3 + charge_planes(with_rho);
  // a short list is dealt out to all workgroups one entry at a time and deposits straight
  // into memory: a box's clearing, bounds and flush would be most of its time
  const bool few = !BOX || cnt <= (int64_t)gridDim.x * ESCAPE_FEW;
  const int64_t passes = (cnt + 255) / 256, per = (passes + gridDim.x - 1) / gridDim.x;
  const int64_t it0 = few ? 0 : blockIdx.x * per, it1 = few ? per : min(it0 + per, passes);
  NodeBox box;
#pragma unroll
  for (int d = 0; d < 3; ++d) { box.at[d] = 0; box.lo[d] = 0; box.ext[d] = 1; }
  int brun = -1;                  // the box's run
  for (int64_t it = it0; it < it1; ++it) {
    const int64_t i = few ? blockIdx.x + (int64_t)gridDim.x * (it * 256 + threadIdx.x)
                          : it * 256 + 4 * lane + wave;
    int seg = 0, run = 0;
    bool live = false;
    EscPath<R> d;
    double ke = 0.0;
    if (i < cnt) {
      const unsigned long long v = esc.items[i];
      seg = (int)(v >> 32);
      const int64_t p = (int64_t)(v & 0xffffffffull);
      const SegDesc& s = seg_of(T, seg);
      run = s.run;
      const RunDesc& r = run_of(T, run);
      const PushConst<R> k = push_const<R>(r, s);
      live = s.order == 1 ? escape_push<R, DIM, 1>(r, s, p, k, with_rho, d, ke)
                          : escape_push<R, DIM, 2>(r, s, p, k, with_rho, d, ke);
    }
    if (kinetic || ke_to_diag) {
      const int first = uniform(run);   // (the first lane's run; the others may differ)
      if (kinetic || __ballot(run != first) == 0) {
        ke = wave_sum(ke);
        if (lane == 0) atomic_add_global(kinetic ? kinetic : run_of(T, first).diag + DIAG_UKIN, ke);
      } else if (live) {
        atomic_add_global(run_of(T, run).diag + DIAG_UKIN, ke);
      }
    }
    int lo[3] = {0, 0, 0}, hi[3] = {0, 0, 0}, v[3] = {0, 0, 0};
    bool in = BOX && live && run == brun;
    if constexpr (BOX) {
      if (live) {
        const RunDesc& r = run_of(T, run);
        const int n[3] = {r.nx, r.ny, r.nz};
        const bool cic = seg_of(T, seg).order == 1;
#pragma unroll
        for (int x = 0; x < DIM; ++x) {
          if (cic) path_nodes<1>(d.o[x], d.e[x], lo[x], hi[x]);
          else path_nodes<2>(d.o[x], d.e[x], lo[x], hi[x]);
          v[x] = wrap_near(d.c[x] - box.at[x], n[x]) - box.lo[x];
          in = in && v[x] + lo[x] >= 0 && v[x] + hi[x] < box.ext[x];
        }
      }
      const int stray = few ? 0 : __syncthreads_count(live && !in);
      if (stray > (brun >= 0 ? DEPOSIT_STRAY : 0)) {
        if (brun >= 0) flush_box<R, DIM>(run_of(T, brun), box, planes, jm, with_rho == 3);
        else
          for (int q = threadIdx.x; q < cap * planes; q += 256) jm[q] = 0.0;
        const uint64_t m = __ballot(live);
        const int lead = m ? __ffsll((unsigned long long)m) - 1 : 0;
        const int lr = __shfl(run, lead, 64);
        if (lane == 0) wrun[wave] = m ? lr : -1;
        __syncthreads();
        brun = uniform(wrun[0] >= 0 ? wrun[0] : (wrun[1] >= 0 ? wrun[1] : (wrun[2] >= 0 ? wrun[2] : wrun[3])));
        const RunDesc& r = run_of(T, brun);
        const int n[3] = {r.nx, r.ny, r.nz};
        const bool here = live && run == brun;
        box = pick_box<DIM>(here, d.c, lo, hi, n, cap, red);
        in = here;
        if (here) {
#pragma unroll
          for (int x = 0; x < DIM; ++x) {
            v[x] = wrap_near(d.c[x] - box.at[x], n[x]) - box.lo[x];
            in = in && v[x] + lo[x] >= 0 && v[x] + hi[x] < box.ext[x];
          }
        }
        __syncthreads();
      }
    }
    if (live) {
      const SegDesc& s = seg_of(T, seg);
      const RunDesc& r = run_of(T, run);
      const PushConst<R> k = push_const<R>(r, s);
      if (BOX && in) {
        const BoxAcc<R> B{jm, box.ext[0], box.ext[0] * box.ext[1],
                          box.ext[0] * box.ext[1] * box.ext[2]};
        if (s.order == 1) deposit<DIM, 1>(B, v, d.o, d.e, d.w, d.vz, k, d.rho);
        else deposit<DIM, 2>(B, v, d.o, d.e, d.w, d.vz, k, d.rho);
      } else {
        const GlobalAcc<R> G = global_acc<R>(r);
        if (s.order == 1) deposit<DIM, 1>(G, d.c, d.o, d.e, d.w, d.vz, k, d.rho);
        else deposit<DIM, 2>(G, d.c, d.o, d.e, d.w, d.vz, k, d.rho);
      }
    }
  }
  __syncthreads();
  if (BOX && brun >= 0) flush_box<R, DIM>(run_of(T, brun), box, planes, jm, with_rho == 3);
  // the last workgroup to finish clears the list (every workgroup has read the count by
  // then; no fence: nothing this launch wrote is read before the launch ends)
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned int done = atomicAdd(esc.count + 1, 1u);
    if (done == gridDim.x - 1) {
      atomicAdd(esc.total, (unsigned long long)esc.count[0]);
      atomicExch(esc.count, 0u);
      atomicExch(esc.count + 1, 0u);
    }
  }
}

// ---------------------------------------------------------------------------------------
// Host-side launchers
// ---------------------------------------------------------------------------------------
int fused_geometry(int dim, int tx, int ty, int tz, int halo) {
  for (int g = 1; g < NUM_GEO; ++g) {
    const GeoFix f = geo_table(g);
    if (dim == 2 && f.tz == 1 && f.tx == tx && f.ty == ty && f.halo == halo) return g;
    if (dim == 3 && f.tz > 1 && f.tx == tx && f.ty == ty && f.tz == tz && f.halo == halo) return g;
  }
  return 0;
}

template <typename R, int D, int G>
static void launch_fused_g(const Tables& T, int nblocks, size_t smem, const Chunk* chunks,
                           const int32_t* nchunks, int with_rho, double* kinetic, int ke_to_diag,
                           const EscapeList& esc, bool keep, int probe, const int32_t* jshift,
                           PassList pl, hipStream_t st) {
  if constexpr (D == 2)
    if (keep) {
      k_fused<R, D, G, true><<<nblocks, fused_block<R, D, G>(), smem, st>>>(
          T, chunks, nchunks, with_rho, kinetic, ke_to_diag, esc, (int)smem, probe, jshift, pl);
      return;
    }
  k_fused<R, D, G, false><<<nblocks, fused_block<R, D, G>(), smem, st>>>(
      T, chunks, nchunks, with_rho, kinetic, ke_to_diag, esc, (int)smem, probe, jshift, pl);
}

template <typename R, int D>
static void launch_fused_d(int geo, const Tables& T, int nblocks, size_t smem,
                           const Chunk* chunks, const int32_t* nchunks, int with_rho,
                           double* kinetic, int ke_to_diag, const EscapeList& esc, bool keep, int probe,
                           const int32_t* jshift, PassList pl, hipStream_t st) {
#define LPIC_GEO(g) launch_fused_g<R, D, g>(T, nblocks, smem, chunks, nchunks, with_rho, kinetic, ke_to_diag, esc, keep, probe, jshift, pl, st)
  if constexpr (D == 2) {
    switch (geo) {
      case 1: LPIC_GEO(1); return;
      case 2: LPIC_GEO(2); return;
      case 3: LPIC_GEO(3); return;
      case 4: LPIC_GEO(4); return;
      default: LPIC_GEO(0); return;
    }
  } else {
    switch (geo) {
      case 5: LPIC_GEO(5); return;
      case 6: LPIC_GEO(6); return;
      case 7: LPIC_GEO(7); return;
      case 8: LPIC_GEO(8); return;
      case 9: LPIC_GEO(9); return;
      default: LPIC_GEO(0); return;
    }
  }
#undef LPIC_GEO
}

// LDS of an escape workgroup: 2D three a CU.  3D one: 256 escaped particles of a few 8 x 4 x 4
// tiles need about 18 nodes per axis, and a box of 13 (52 KB) leaves most of them to global
// atomics.  62 x 73 x 51 FP32, 5 a cell, one step: 52 KB and 128 workgroups 623 us, 150 KB 622,
// with 256 workgroups 565, 75 KB and 256 577 (99 x 75 x 15, 8 a cell, 10 steps: 2809, 2815,
// 2656, 2671).  Below 128K slots 128, for the empty lists of short steps.
static int escape_smem(int dim) { return (dim == 3 ? 150 : 52) * 1024; }
static int escape_blocks(int dim, int64_t slots) {
  if (dim == 3 && slots > 131072) return 2 * ESCAPE_BLOCKS;
  return (int)std::min<int64_t>(ESCAPE_BLOCKS, (slots + 255) / 256);
}

template <typename R, int D, bool BOX>
static void launch_escape(const Tables& T, int with_rho, double* kinetic, int ke_to_diag,
                          const EscapeList& esc, int skip_at, int blocks, hipStream_t st) {
  const int smem = BOX ? escape_smem(D) : 0;
  k_escape<R, D, BOX><<<blocks, 256, smem, st>>>(T, with_rho, kinetic, ke_to_diag, esc, skip_at,
                                                 smem / 8 / (3 + charge_planes(with_rho)));
}

void launch_fused(const Tables& T, int prec, int dim, int geo, int nblocks, size_t smem,
                  const Chunk* chunks, const int32_t* nchunks, int with_rho, double* kinetic,
                  int ke_to_diag, const EscapeList& esc, const int32_t* jshift,
                  hipStream_t st, const Rebin* rb, bool probe) {
  const bool keep = dim == 2 && !rb && esc.capacity <= FUSED_KEEP;
  LPIC_PD(prec, dim, (launch_fused_d<R, D>(geo, T, nblocks, smem, chunks, nchunks, with_rho,
                                           kinetic, ke_to_diag, esc, keep, probe ? 1 : 0, jshift,
                                           PassList{nullptr, nullptr}, st)));
  if (keep) return;
  if (rb) {
    // escapees by present tile, a second pass over them, then whatever that pass could not
    // place (normally nothing) and a list below the threshold through global memory
    launch_rebin(T, prec, dim, esc, *rb, st);
    const int k = with_rho == 0 ? 0 : (with_rho == 1 ? 1 : 2);
    LPIC_PD(prec, dim, (launch_fused_d<R, D>(rb->geo[k], T, rb->grid[k], rb->smem[k], rb->chunks,
                                             rb->nchunks, with_rho, kinetic, ke_to_diag,
                                             rb->esc2, false, 0, jshift,
                                             PassList{rb->items, esc.rec ? rb->rec : nullptr},
                                             st)));
    // (a list below the threshold is a short one for as many workgroups, and the second pass's
    // list is normally empty: without boxes for either.  128 workgroups with their boxes of LDS
    // cost a step of 2D or 3D some 4 us)
    const int few = (rb->threshold + ESCAPE_FEW - 1) / ESCAPE_FEW;
    LPIC_PD(prec, dim, (launch_escape<R, D, false>(T, with_rho, kinetic, ke_to_diag, esc,
                                                   rb->threshold, few, st)));
    LPIC_PD(prec, dim, (launch_escape<R, D, false>(T, with_rho, kinetic, ke_to_diag, rb->esc2,
                                                   0x7fffffff, few, st)));
  } else {
    const int blocks = escape_blocks(dim, esc.capacity);
    LPIC_PD(prec, dim, (launch_escape<R, D, true>(T, with_rho, kinetic, ke_to_diag, esc,
                                                  0x7fffffff, blocks, st)));
  }
}

template <typename R, int D, int G>
static hipError_t set_smem(size_t smem, size_t smem_occ, int* blocks_per_cu) {
  hipError_t e = hipFuncSetAttribute((const void*)k_fused<R, D, G, false>,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if constexpr (D == 2)
    if (e == hipSuccess)
      e = hipFuncSetAttribute((const void*)k_fused<R, D, G, true>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if constexpr (D == 3)
    if (e == hipSuccess)
      e = hipFuncSetAttribute((const void*)k_escape<R, D, true>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, escape_smem(D));
  if (e != hipSuccess) return e;
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, k_fused<R, D, G, false>,
                                                      fused_block<R, D, G>(),
                                                      smem_occ);
}

hipError_t prepare_fused(int prec, int dim, int geo, size_t smem, size_t smem_occ,
                         int* blocks_per_cu) {
  hipError_t e = hipSuccess;
  int* b = blocks_per_cu;
  if (dim == 2) {
    switch (geo) {
      case 1: e = prec == 0 ? set_smem<float, 2, 1>(smem, smem_occ, b) : set_smem<double, 2, 1>(smem, smem_occ, b); break;
      case 2: e = prec == 0 ? set_smem<float, 2, 2>(smem, smem_occ, b) : set_smem<double, 2, 2>(smem, smem_occ, b); break;
      case 3: e = prec == 0 ? set_smem<float, 2, 3>(smem, smem_occ, b) : set_smem<double, 2, 3>(smem, smem_occ, b); break;
      case 4: e = prec == 0 ? set_smem<float, 2, 4>(smem, smem_occ, b) : set_smem<double, 2, 4>(smem, smem_occ, b); break;
      default: e = prec == 0 ? set_smem<float, 2, 0>(smem, smem_occ, b) : set_smem<double, 2, 0>(smem, smem_occ, b); break;
    }
  } else {
    switch (geo) {
      case 5: e = prec == 0 ? set_smem<float, 3, 5>(smem, smem_occ, b) : set_smem<double, 3, 5>(smem, smem_occ, b); break;
      case 6: e = prec == 0 ? set_smem<float, 3, 6>(smem, smem_occ, b) : set_smem<double, 3, 6>(smem, smem_occ, b); break;
      case 7: e = prec == 0 ? set_smem<float, 3, 7>(smem, smem_occ, b) : set_smem<double, 3, 7>(smem, smem_occ, b); break;
      case 8: e = prec == 0 ? set_smem<float, 3, 8>(smem, smem_occ, b) : set_smem<double, 3, 8>(smem, smem_occ, b); break;
      case 9: e = prec == 0 ? set_smem<float, 3, 9>(smem, smem_occ, b) : set_smem<double, 3, 9>(smem, smem_occ, b); break;
      default: e = prec == 0 ? set_smem<float, 3, 0>(smem, smem_occ, b) : set_smem<double, 3, 0>(smem, smem_occ, b); break;
    }
  }
  return e;
}

size_t fused_smem_bytes(int prec, int dim, int tx, int ty, int tz, int halo, int with_rho,
                        int geo) {
  // the z layers of a fixed 3D geometry are padded (GeoFix::pz)
  if (geo < 0) geo = fused_geometry(dim, tx, ty, tz, halo);
  const int pz = dim == 3 ? geo_table(geo).pz : 0;
  const size_t plane = ((size_t)(tx + 2 * halo) * (ty + 2 * halo) + pz) *
                       (dim == 3 ? (tz + 2 * halo) : 1);
  // six field planes in the kernel precision (24 or 48 bytes per cell: the current planes
  // after them start 8-byte aligned), then 8-byte current planes (and, on diagnostic steps,
  // two charge planes)
  const int jplanes = 3 + charge_planes(with_rho);
  static_assert((6 * sizeof(float)) % 8 == 0, "current planes must start 8-byte aligned");
  // 3D: the lists of the compacted rounds (process_chunk_compact), sized for the workgroup of
  // this precision and geometry
  const int block = geo == 7 || geo == 8
                        ? (prec == 0 ? fused_block<float, 3, 7>() : fused_block<double, 3, 7>())
                        : (prec == 0 ? fused_block<float, 3, 0>() : fused_block<double, 3, 0>());
  const size_t planes = plane * 6 * (prec == 0 ? 4 : 8) + plane * jplanes * 8;
  // the lists of escaped particles (2D of the tile, 3D of the rounds) take what the planes
  // leave, up to their size
  constexpr size_t room = 160 * 1024 - 512;
  const size_t least = planes + (dim == 3 ? (size_t)round_words(block, geo ? ROUND_ESC : ROUND_ESC_MIN) * 4 : 0);
  const size_t most = planes + (dim == 3 ? (size_t)round_words(block, ROUND_ESC) * 4 : 8 * FUSED_LIST);
  return std::max(least, std::min(most, room) / 8 * 8);
}

}  // namespace lpic
