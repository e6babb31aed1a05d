// Resolution of the contact clusters in LDS, patch of cells by patch of cells
// (Eqs. 17-18).
//
// A workgroup takes the particles of one patch that have contacts (the contact
// kernel's sorted rows and degrees), one per thread, and turns every row entry
// into the partner's place among them.  The pairs are applied in rounds: each
// particle names its next partner in index order, and a pair fires in the
// round in which its two particles name each other.  Then every earlier pair
// of both is done, so each particle meets its partners in ascending index
// order, which is the sequential sweep over the pairs (i, j) in lexicographic
// order bit for bit.  A particle is in at most one pair per round, so a round
// is one barrier, and no lane walks a cluster alone.
//
// The velocities change in LDS only.  A particle with a partner outside the
// patch is marked, and so is everything connected to it; when nothing fires any
// more, the unmarked particles, who form whole clusters, take their wall pass,
// go back to memory and leave the stage (degree 0).  The marked ones are as if
// nothing had happened.
//
// A second pass with larger patches, moved against the first's, leaves the few
// clusters that cross an edge in both (of the particles with contacts on a
// 512 x 4096 riser 4 % after one pass, 0.1 % after two); one workgroup takes those
// of the whole bed at once.  Where it could not hold them, because the patches
// were too full or the clusters span many of them, the particles left are taken
// cluster by cluster before it (k_rest), wherever they lie.  A bed whose particles
// seldom touch, or whose clusters no patch holds, goes by clusters from the start
// (k_clusters).
//
// The first pass is bound by its chain of dependent loads, barriers and rounds:
// on the 2 M-sphere riser it issues for 17 of its 46 us, eight patches of 400
// particles per CU.  Hence the single range check per row entry (the entry
// carries the partner's row of cells), and the rounds of one wavefront once at
// most 64 particles have partners left, while the others wait at the barrier.
// Measured there, FP32: 47 us for the first pass, 16 us for the second, 19 us for
// the final workgroup, against 145 us (88 us in its best launch shape) and 5 us
// for one lane per cluster and the ordered sweep; 310 + 129 + 30 against 1 034 us
// at 16 M spheres.  The later kernels are such chains too.  A counter all patches
// add to costs 7 ns each, one after the other, so a pass lists what it leaves only
// where it may be the last one of its bed (34 us more for the first pass of the
// riser, had it listed).
#pragma once

#include "kernels.hpp"

namespace lbdps {

// The patches of cells of one pass: patch (i, j) covers the cells
// [i tw - ox, (i + 1) tw - ox) x [j th - oy, (j + 1) th - oy) of the lattice.
struct PatchGrid {
  int tw, th, ox, oy, ntx, nty;
  __host__ __device__ int count() const { return ntx * nty; }
};

// How the row stage resolves a bed: all of it in the final workgroup, by one or
// two passes of patches, or by clusters; or the tile stage.
enum { PLAN_TILES = -1, PLAN_WHOLE = 0, PLAN_ONE_PASS = 1, PLAN_TWO_PASSES = 2, PLAN_CLUSTERS };
constexpr int PATCH_PASSES = 2;      // most passes
constexpr int PATCH_ROWS = 64;       // most rows of cells in a patch
constexpr int PATCH_NB = 8;          // partners' places kept in registers
constexpr int PATCH_NONE = 0xffff;   // no partner, or one outside
// Bands of rows a patch of the first pass is taken in, before the rest of it is
// left, and the share (one in PATCH_FLOOD) of the bed that may be left so before
// the second pass only lists: its patches would be as full.  Beds laid out about
// right take two bands at most.  The collision stage of 1 M spheres in the bottom
// 40 % of a periodic 1000 x 1600 lattice takes 590, 320 and 250 us with 3, 4 and 6
// bands, and as long with 12; of 100 000 in a quarter of 400 x 400 cells 272 us
// with 6, 302 with 12.
constexpr int PATCH_BANDS = 6, PATCH_FLOOD = 16;
// Particles a patch's workgroup looks at together: of the first pass, where about
// half of them have contacts, and of the second, where few are left.
constexpr int PATCH_HELD0 = 2 * BLOCK, PATCH_HELD1 = 8 * BLOCK;
// The final workgroup: threads, and particles it holds.
constexpr int FINAL_THREADS = 1024, FINAL_PT = 4, FINAL_CAP = FINAL_THREADS * FINAL_PT;
// Cell of a particle relative to the patch, for the separation in the cell +
// offset modes: partners are at most one cell apart after the periodic wrap.
template <int P>
__device__ __forceinline__ void patch_sep(const Consts<typename Prec<P>::T> &k, int ca, typename Prec<P>::T xa,
                                          typename Prec<P>::T ya, int cb, typename Prec<P>::T xb,
                                          typename Prec<P>::T yb, typename Prec<P>::T &dx, typename Prec<P>::T &dy) {
  using T = typename Prec<P>::T;
  if constexpr (Pos<P>::G) {
    Pos<P>::sep(k, 0, xa, ya, 0, xb, yb, dx, dy);
  } else {
    int dcx = (ca & 0xffff) - (cb & 0xffff), dcy = (ca >> 16) - (cb >> 16);
    dcx = dcx > 1 ? -1 : (dcx < -1 ? 1 : dcx);
    dcy = dcy > 1 ? -1 : (dcy < -1 ? 1 : dcy);
    const T ox = xa - xb, oy = ya - yb;
    dx = (T)dcx + ox;
    dy = (T)dcy + oy;
  }
}

// Places of a particle's first PATCH_NB partners, 16 bits each, in registers
// (selected, never indexed, which would put them in scratch or LDS).
struct alignas(16) Partners {
  unsigned w0, w1, w2, w3;
  __device__ __forceinline__ void set(int a, int q) {  // a known at compile time
    unsigned &w = a < 4 ? (a < 2 ? w0 : w1) : (a < 6 ? w2 : w3);
    w = a & 1 ? ((w & 0xffffu) | ((unsigned)q << 16)) : ((w & 0xffff0000u) | (unsigned)q);
  }
  __device__ __forceinline__ int get(int a) const {
    const unsigned lo = a < 2 ? w0 : w1, hi = a < 6 ? w2 : w3, v = a < 4 ? lo : hi;
    return (int)(a & 1 ? v >> 16 : v & 0xffffu);
  }
};
static_assert(PATCH_NB == 8, "Partners holds eight places");

template <class T, int HELD> struct PatchLds {
  static constexpr int NT = BLOCK;
  T x[NT], y[NT], vx[NT], vy[NT];
  Partners nb[NT];
  int cell[NT], slot[NT], ext[NT], hits[NT];
  int st[NT];                 // next entry | degree << 8 | partners of lower index left << 16
  unsigned short nxt[2][NT];  // place of the next partner, double-buffered over the rounds
  unsigned short row[NT], list[NT], work[NT];
  unsigned short loc[HELD];   // particle of the band -> its place among those with contacts
  int rlo[PATCH_ROWS + 1], rbase[PATCH_ROWS + 1];
  int np, nleft, base, nlist, nwork, busy[3], alive[3], ncoll, nwall;
};

// The first pass left so many particles of patches too full for it that they are
// for the rest to take cluster by cluster; full counts them.
__device__ __forceinline__ bool patches_flooded(int full, int npart) { return full > npart / PATCH_FLOOD; }

template <int P, int HELD, bool FIRST>
__device__ __forceinline__ void patches_body(PatchLds<typename Prec<P>::T, HELD> &S, const int bidx,
    Parts<typename Prec<P>::T> pt, const int32_t *__restrict__ cs, const Consts<typename Prec<P>::T> &k, Adj adj,
    int32_t *__restrict__ deg, const PatchGrid g, const bool last, int32_t *__restrict__ left,
    int32_t *__restrict__ place_of, int32_t *__restrict__ nleft, int32_t *__restrict__ full, int32_t *__restrict__ coll_part,
    int32_t *__restrict__ wall_part) {
  using T = typename Prec<P>::T;
  constexpr int NT = BLOCK;
  const bool flooded = !FIRST && patches_flooded(*full, k.npart);
  const int tid = (int)threadIdx.x, lane = tid & 63;
  const int bx = bidx % g.ntx, by = bidx / g.ntx;
  const int x0 = max(bx * g.tw - g.ox, 0), x1 = min((bx + 1) * g.tw - g.ox, k.nx);
  const int y0 = max(by * g.th - g.oy, 0), y1 = min((by + 1) * g.th - g.oy, k.ny);
  const int H = y1 - y0;
  // an overflowed contact row leaves the graph incomplete: nothing is resolved
  const bool overflow = __hip_atomic_load(&k.flags[FLAG_CAPACITY], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
  // particles of this patch can touch a wall
  const bool walls = (!k.per_x && (x0 == 0 || x1 == k.nx)) || (!k.per_y && (y0 == 0 || y1 == k.ny));
  if (tid < 64) {  // first slot and length of each row of the patch, and the running total
    int lo = 0, len = 0;
    if (tid < H) {
      lo = ldu(cs, (y0 + tid) * k.nx + x0);
      len = ldu(cs, (y0 + tid) * k.nx + x1) - lo;
    }
    int inc = len;
    for (int o = 1; o < 64; o <<= 1) {
      const int u = __shfl_up(inc, o, 64);
      if (lane >= o) inc += u;
    }
    S.rlo[tid] = lo;
    S.rbase[tid + 1] = inc;
    if (tid == 0) {
      S.rbase[0] = 0;
      S.ncoll = S.nwall = 0;
    }
  }
  __syncthreads();
  int ncoll = 0, nwall = 0;
  // Leaves the particle in slot s to the final workgroup, at place `to`.
  auto leave = [&](int s, int to) {
    left[to] = s;
    place_of[s] = to;
  };
  // Slot of particle l of the rows from r0 on, and its row (rbase[row] <= base0 + l
  // < rbase[row + 1], row < r1).
  auto slot_of = [&](int l, int r0, int r1, int base0, int &row) {
    int r = r0, hi = r1;
    while (hi - r > 1) {
      const int mid = (r + hi) >> 1;
      if (S.rbase[mid] - base0 <= l) r = mid;
      else hi = mid;
    }
    row = r;
    return S.rlo[r] + (base0 + l - S.rbase[r]);
  };
  // Leaves the particles with contacts of rows [a, b) of the patch: counts them,
  // takes their places by one addition to the bed's counter, lists them.
  auto leave_rows = [&](int a, int b) {
    if (!last) return;
    const int base0 = S.rbase[a], total = S.rbase[b] - base0;
    for (int listing = 0; listing < 2; ++listing) {
      __syncthreads();
      if (tid == 0) S.nleft = 0;
      __syncthreads();
      for (int l0 = 0; l0 < total; l0 += NT) {
        int row, s = 0;
        bool has = false;
        if (l0 + tid < total) {
          s = slot_of(l0 + tid, a, b, base0, row);
          has = ldu(deg, s) > 0;
        }
        const unsigned long long m = __ballot(has);
        int at = 0;
        if (lane == 0 && m) at = atomicAdd(&S.nleft, __popcll(m));
        at = __shfl(at, 0, 64) + __popcll(m & ((1ull << lane) - 1));
        if (has && listing) leave(s, S.base + at);
      }
      __syncthreads();
      if (tid == 0 && !listing) S.base = atomicAdd(nleft, S.nleft);
    }
  };
  // Bands of rows, one after the other; usually the patch is one.  A band holds
  // at most HELD particles, NT of them with contacts.
  int want = H;  // rows to try
  int bands = 0;
  for (int r0 = 0, r1; r0 < H && !overflow; r0 = r1) {
    if (FIRST && bands == PATCH_BANDS) {  // far too full
      if (tid == 0) atomicAdd(full, S.rbase[H] - S.rbase[r0]);
      leave_rows(r0, H);
      break;
    }
    if (!FIRST && flooded) {
      leave_rows(0, H);
      break;
    }
    const int base0 = S.rbase[r0];
    r1 = min(H, r0 + want);
    while (r1 > r0 + 1 && S.rbase[r1] - base0 > HELD) r1 = r0 + (r1 - r0 + 1) / 2;
    const int held = S.rbase[r1] - base0;
    want = H;
    if (held == 0) continue;
    if (held > HELD) {  // one crowded row
      leave_rows(r0, r1);
      continue;
    }
    __syncthreads();  // the previous band's LDS is free
    if (tid == 0) {
      S.np = S.nleft = S.nlist = S.nwork = 0;
      S.busy[0] = S.alive[0] = 0;
    }
    // the particles with contacts, compacted; every degree is requested first
    constexpr int PT = HELD / NT;
    int ps[PT], pd[PT], pr[PT];
#pragma unroll
    for (int j = 0; j < PT; ++j) {
      const int l = tid + j * NT;
      ps[j] = pd[j] = pr[j] = 0;
      if (l < held) {
        ps[j] = slot_of(l, r0, r1, base0, pr[j]);
        pd[j] = ldu(deg, ps[j]);
      }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PT; ++j) {
      if (j > 0 && j * NT >= held) break;  // uniform
      const unsigned long long m = __ballot(pd[j] > 0);
      int b = 0;
      if (lane == 0 && m) b = atomicAdd(&S.np, __popcll(m));
      b = __shfl(b, 0, 64);
      if (pd[j] > 0) {
        const int c = b + __popcll(m & ((1ull << lane) - 1));
        S.loc[tid + j * NT] = (unsigned short)c;
        if (c < NT) {
          S.slot[c] = ps[j];
          S.row[c] = (unsigned short)pr[j];
        }
      }
    }
    __syncthreads();
    const int n = S.np;
    if (n == 0) continue;
    if (n > NT) {
      // Too many with contacts: fewer rows at a time.  Many too many after the
      // first pass are of clusters that span many patches, which no patch resolves.
      if ((FIRST || n <= 2 * NT) && r1 > r0 + 1) {
        want = (r1 - r0) / 2;
        r1 = r0;
      } else {
        leave_rows(r0, r1);
      }
      continue;
    }
    ++bands;
    // place of the partner of an entry of a particle in row `row_of`, or
    // PATCH_NONE if it is outside the band.  Contacts are mutual, so a partner in
    // the band has its place in loc; the test against n keeps the access inside
    // the LDS whatever a row holds.
    auto place = [&](long long e, int row_of) -> int {
      const int rr = row_of + adj_dy(e);
      if (rr < r0 || rr >= r1) return PATCH_NONE;
      const int q = adj_slot(e) - S.rlo[rr], b = S.rbase[rr];
      if (q < 0 || q >= S.rbase[rr + 1] - b) return PATCH_NONE;
      const int c = S.loc[b - base0 + q];
      return c < n ? c : PATCH_NONE;
    };
    // this thread's particle
    const bool act = tid < n;
    int s = -1, dg = 0, low = 0;
    bool out = false;
    Partners nb{~0u, ~0u, ~0u, ~0u};
    if (act) {
      s = S.slot[tid];
      const int row_of = S.row[tid];
      const AdjRow row = adj.row(s);
      const Dense4 e4(row.a);
      dg = min(ldu(deg, s), KMAX);
      const int id = ldu(pt.pid, s);
      S.x[tid] = ldu(pt.px, s);
      S.y[tid] = ldu(pt.py, s);
      S.vx[tid] = ldu(pt.vx, s);
      S.vy[tid] = ldu(pt.vy, s);
      if constexpr (!Pos<P>::G) S.cell[tid] = (ldu(pt.key, s) - (y0 + row_of) * k.nx - x0) | (row_of << 16);
#pragma unroll
      for (int a = 0; a < PATCH_NB; ++a)
        if (a < dg) {
          const long long e = a < ADJ_IN ? e4.get(a) : row[a];
          const int q = place(e, row_of);
          out |= q == PATCH_NONE;
          low += (int)(e >> 32) < id;
          nb.set(a, q);
        }
      for (int a = PATCH_NB; a < dg; ++a) {
        out |= place(row[a], row_of) == PATCH_NONE;
        low += (int)(row[a] >> 32) < id;
      }
      S.nb[tid] = nb;
      S.ext[tid] = out;
      S.hits[tid] = 0;
      S.st[tid] = dg << 8 | low << 16;
      if (out) S.work[atomicAdd(&S.nwork, 1)] = (unsigned short)tid;
    }
    int nx = act ? nb.get(0) : PATCH_NONE, st = dg << 8 | low << 16;
    if (act) S.nxt[0][tid] = (unsigned short)nx;
    // the pair of the particle at place c with its next partner q, both naming
    // each other; then its next entry
    auto fire = [&](int c, int &st_, int &q_, const Partners &nb_) {
      if (st_ >> 16 == 0) {  // it has the lower index: it applies the pair
        T dx, dy, vix = S.vx[c], viy = S.vy[c], vjx = S.vx[q_], vjy = S.vy[q_];
        patch_sep<P>(k, S.cell[c], S.x[c], S.y[c], S.cell[q_], S.x[q_], S.y[q_], dx, dy);
        if (pair_core<P>(k, dx, dy, vix, viy, vjx, vjy)) {
          S.vx[c] = vix;
          S.vy[c] = viy;
          S.vx[q_] = vjx;
          S.vy[q_] = vjy;
          S.hits[c] += 1;
        }
      } else {
        st_ -= 1 << 16;
      }
      ++st_;
      const int at = st_ & 0xff;
      q_ = at >= ((st_ >> 8) & 0xff) ? PATCH_NONE
                                      : (at < PATCH_NB ? nb_.get(at) : place(adj.row(S.slot[c])[at], S.row[c]));
    };
    __syncthreads();
    // Rounds of the whole workgroup while more than a wavefront of particles has
    // partners left ...
    int cur = 0;
    bool any = true;
    for (int rd = 0, alive = n; alive > WAVE; rd = rd == 2 ? 0 : rd + 1) {
      const bool pair = nx != PATCH_NONE && S.nxt[cur][nx] == tid;
      if (pair) fire(tid, st, nx, nb);
      if (act) S.nxt[cur ^ 1][tid] = (unsigned short)nx;
      const unsigned long long m = __ballot(nx != PATCH_NONE);
      if (lane == 0 && m) atomicAdd(&S.alive[rd], __popcll(m));
      if (pair) S.busy[rd] = 1;
      if (tid == 0) S.busy[rd == 2 ? 0 : rd + 1] = S.alive[rd == 2 ? 0 : rd + 1] = 0;
      __syncthreads();
      cur ^= 1;
      alive = S.alive[rd];
      if (!S.busy[rd]) {  // the rest waits for partners outside
        any = false;
        break;
      }
    }
    if (any && nx != PATCH_NONE) {
      S.st[tid] = st;
      S.list[atomicAdd(&S.nlist, 1)] = (unsigned short)tid;
    }
    __syncthreads();
    // ... then the first wavefront goes on alone, while the last one spreads the
    // marks through the clusters of the marked.
    if (tid < WAVE) {
      if (any) {
        const bool on = lane < S.nlist;
        int c = 0, st1 = 0, q = PATCH_NONE;
        Partners nb1{~0u, ~0u, ~0u, ~0u};
        if (on) {
          c = S.list[lane];
          st1 = S.st[c];
          nb1 = S.nb[c];
          q = S.nxt[cur][c];
        }
        for (;;) {
          const bool pair = q != PATCH_NONE && S.nxt[cur][q] == c;
          if (!__any(pair)) break;
          Group<WAVE>::sync();
          if (pair) {
            fire(c, st1, q, nb1);
            S.nxt[cur][c] = (unsigned short)q;
          }
          Group<WAVE>::sync();
        }
      }
    } else if (tid >= NT - WAVE) {
      for (int w0 = 0;;) {
        const int w1 = S.nwork;
        Group<WAVE>::sync();
        if (w0 >= w1) break;
        for (int w = w0 + lane; w < w1; w += WAVE) {
          const int c = S.work[w], d = (S.st[c] >> 8) & 0xff;
          const Partners p = S.nb[c];
          for (int a = 0; a < d; ++a) {
            const int q = a < PATCH_NB ? p.get(a) : place(adj.row(S.slot[c])[a], S.row[c]);
            if (q != PATCH_NONE && atomicExch(&S.ext[q], 1) == 0) S.work[atomicAdd(&S.nwork, 1)] = (unsigned short)q;
          }
        }
        Group<WAVE>::sync();
        w0 = w1;
      }
    }
    __syncthreads();
    int mine = -1;
    if (act) {
      if (!S.ext[tid]) {
        T vx = S.vx[tid], vy = S.vy[tid];
        if (walls) nwall += Pos<P>::walls_key(k, ldu(pt.key, s), S.x[tid], S.y[tid], vx, vy);
        ncoll += S.hits[tid];
        pt.vx[s] = vx;
        pt.vy[s] = vy;
        deg[s] = 0;
      } else if (last) {
        mine = atomicAdd(&S.nleft, 1);
      }
    }
    if (last) {
      __syncthreads();
      const int nl = S.nleft;
      if (nl > 0) {
        if (tid == 0) S.base = atomicAdd(nleft, nl);
        __syncthreads();
        if (mine >= 0) leave(s, S.base + mine);
      }
    }
  }
  if (ncoll) atomicAdd(&S.ncoll, ncoll);
  if (nwall) atomicAdd(&S.nwall, nwall);
  __syncthreads();
  if (tid == 0) {
    coll_part[bidx] = S.ncoll;
    wall_part[bidx] = S.nwall;
  }
}

template <int P, int HELD, bool FIRST>
__global__ __launch_bounds__(BLOCK) void k_patches(Parts<typename Prec<P>::T> pt, const int32_t *__restrict__ cs,
                                                   Consts<typename Prec<P>::T> k, Adj adj, int32_t *__restrict__ deg,
                                                PatchGrid g, int last, int32_t *__restrict__ left,
                                                int32_t *__restrict__ place_of, int32_t *__restrict__ nleft,
                                                int32_t *__restrict__ full, int32_t *__restrict__ coll_part,
                                                int32_t *__restrict__ wall_part) {
  __shared__ PatchLds<typename Prec<P>::T, HELD> S;
  patches_body<P, HELD, FIRST>(S, xcd_block<XCD_RUN_PATCHES>(blockIdx.x, gridDim.x), pt, cs, k, adj, deg, g,
                                   last != 0, left, place_of, nleft, full, coll_part, wall_part);
}

constexpr int CLUSTERS_SL = 4;  // slots per lane of the cluster kernel over many particles

// The whole bed by clusters, one from each candidate root: a particle whose
// partners all have higher indices.  A workgroup takes SL BLOCK slots.  A resolved
// particle is marked DONE_WHOLE in its degree, not cleared, since other candidates
// of its cluster may still be gathering.  Bound by the chain of dependent loads
// from a root through its cluster, in the lanes' cluster size at a time: on the
// 2 M-sphere riser, FP32, 82 us with four slots per lane, whose candidates fill
// the lanes, against 143 from candidate lists of one slot per lane.
template <int P, int SL> struct RootsLds {
  ClustersLds<P, BLOCK, SL * BIG_LIST> cl;
  long long cand[SL * BLOCK];
  long long sh[BLOCK / 64];
  int n;
};
template <int P, int SL>
__device__ __forceinline__ void clusters_body(RootsLds<P, SL> &S, const int bidx, Parts<typename Prec<P>::T> pt,
    const Consts<typename Prec<P>::T> &k, Adj adj, int32_t *deg, int32_t *sweep, long long *coll_part,
    long long *wall_part) {
  const int tid = (int)threadIdx.x, lane = tid & 63, s0 = bidx * SL * BLOCK + tid;
  // an overflowed contact row leaves the graph incomplete: nothing is resolved
  const bool overflow = __hip_atomic_load(&k.flags[FLAG_CAPACITY], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
  if (tid == 0) S.n = 0;
  int d[SL], id[SL];
  long long e[SL];
#pragma unroll
  for (int j = 0; j < SL; ++j) d[j] = s0 + j * BLOCK < k.npart ? ldu(deg, s0 + j * BLOCK) : 0;
#pragma unroll
  for (int j = 0; j < SL; ++j)
    if (d[j] > 0) {
      id[j] = ldu(pt.pid, s0 + j * BLOCK);
      e[j] = adj.row(s0 + j * BLOCK).a[0];
    }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < SL; ++j) {
    const bool c = d[j] > 0 && (int)(e[j] >> 32) > id[j];
    const unsigned long long m = __ballot(c);
    int b = 0;
    if (lane == 0 && m) b = atomicAdd(&S.n, __popcll(m));
    b = __shfl(b, 0, 64);
    if (c) S.cand[b + __popcll(m & ((1ull << lane) - 1))] = ((long long)id[j] << 32) | (unsigned)(s0 + j * BLOCK);
  }
  __syncthreads();
  const int tot = overflow ? 0 : S.n;
  if (tot == 0) {  // uniform
    if (tid == 0) coll_part[bidx] = wall_part[bidx] = 0;
    return;
  }
  long long ncoll = 0, nwall = 0, tc, tw;
  resolve_candidates<P>(S.cl, tot, [&](int f) { return S.cand[f]; }, pt, adj, deg, deg, k, &sweep[SW_MORE], ncoll,
                        nwall);
  block_sum2(ncoll, nwall, S.sh, tc, tw);
  if (tid == 0) {
    coll_part[bidx] = tc;
    wall_part[bidx] = tw;
  }
}
template <int P, int SL>
__global__ __launch_bounds__(BLOCK) void k_clusters(Parts<typename Prec<P>::T> pt,
                                                         Consts<typename Prec<P>::T> k, Adj adj, int32_t *deg,
                                                         int32_t *sweep, long long *coll_part, long long *wall_part) {
  __shared__ RootsLds<P, SL> S;
  clusters_body<P, SL>(S, xcd_block<XCD_RUN_CLUSTERS>(blockIdx.x, gridDim.x), pt, k, adj, deg, sweep, coll_part,
                            wall_part);
}

// The clusters that are left, of the whole bed in one workgroup, by the same
// firing rule.  left lists them; place_of maps a slot to its place among them.  A pair can only become
// ready when one of the two has just gone on to it, so a particle that goes on
// wakes itself and its new partner, and a round looks at the awake alone: most
// wavefronts read one word and meet at the barriers.  Bound by the longest chain of
// pairs: 131 links in a settled bed of 15 000 spheres of d = 0.2, whose largest
// cluster has 3 100, take 237 us in FP64, 1.8 us a link.
template <int P> struct FinalLds {
  using T = typename Prec<P>::T;
  T x[FINAL_CAP], y[FINAL_CAP], vx[FINAL_CAP], vy[FINAL_CAP];
  int key[Prec<P>::global_pos ? 1 : FINAL_CAP];
  unsigned short nxt[FINAL_CAP];
  alignas(4) unsigned char wake[FINAL_CAP];
  unsigned ready[FINAL_CAP / 2];  // the round's pairs: lower index's place | the other's << 16
};
static_assert(FINAL_PT == 4, "a thread's marks are one 32-bit word");
// Place of an entry's partner: contacts are mutual and whole clusters are left,
// so it has one; the mask keeps the access inside the LDS whatever a row holds.
__device__ __forceinline__ int final_place(const int32_t *place_of, long long e) {
  static_assert((FINAL_CAP & (FINAL_CAP - 1)) == 0 && FINAL_CAP < PATCH_NONE, "a mask of the places");
  return place_of[adj_slot(e)] & (FINAL_CAP - 1);
}

// n <= FINAL_CAP particles in LDS, places tid, tid + FINAL_THREADS, ... per thread; the
// marks of a thread's particles are one word.
template <int P>
__device__ __forceinline__ void final_lds(FinalLds<P> &S, Parts<typename Prec<P>::T> pt,
    const Consts<typename Prec<P>::T> &k, Adj adj, const int32_t *deg, const int32_t *left, const int32_t *place_of,
    const int n, int *busy, int &ncoll, int &nwall) {
  using T = typename Prec<P>::T;
  constexpr int PT = FINAL_PT;
  const int tid = (int)threadIdx.x;
  auto at_place = [&](int j) { return tid + j * FINAL_THREADS; };
  auto mark = [&](int c) { S.wake[(c % FINAL_THREADS) * PT + c / FINAL_THREADS] = 1; };
  int sl[PT], dg[PT], low[PT], at[PT], nx[PT];
  Partners nb[PT];
#pragma unroll
  for (int j = 0; j < PT; ++j) {
    sl[j] = at_place(j) < n ? left[at_place(j)] : -1;
    dg[j] = low[j] = at[j] = 0;
    nx[j] = PATCH_NONE;
    nb[j] = Partners{~0u, ~0u, ~0u, ~0u};
  }
  // every load a particle needs before its partners' places goes out at once
  long long e0[PT], e1[PT];
  int id[PT];
#pragma unroll
  for (int j = 0; j < PT; ++j)
    if (sl[j] >= 0) {
      const long long *const in = adj.row(sl[j]).a;
      dg[j] = min(deg[sl[j]], KMAX);
      e0[j] = in[0];
      e1[j] = in[1];
      id[j] = ldu(pt.pid, sl[j]);
      S.x[at_place(j)] = ldu(pt.px, sl[j]);
      S.y[at_place(j)] = ldu(pt.py, sl[j]);
      S.vx[at_place(j)] = ldu(pt.vx, sl[j]);
      S.vy[at_place(j)] = ldu(pt.vy, sl[j]);
      if constexpr (!Pos<P>::G) S.key[at_place(j)] = ldu(pt.key, sl[j]);
    }
  if (tid == 0) busy[0] = 0;
#pragma unroll
  for (int j = 0; j < PT; ++j)
    if (sl[j] >= 0) {
      const AdjRow row = adj.row(sl[j]);
#pragma unroll
      for (int a = 0; a < PATCH_NB; ++a)
        if (a < dg[j]) {
          const long long e = a == 0 ? e0[j] : (a == 1 ? e1[j] : row[a]);
          nb[j].set(a, final_place(place_of, e));
          low[j] += (int)(e >> 32) < id[j];
        }
      for (int a = PATCH_NB; a < dg[j]; ++a) {  // later partners: their places go into the row itself
        const long long e = row[a];
        low[j] += (int)(e >> 32) < id[j];
        row[a] = final_place(place_of, e);
      }
      nx[j] = nb[j].get(0);
      S.nxt[at_place(j)] = (unsigned short)nx[j];
    }
  unsigned *const mine = reinterpret_cast<unsigned *>(S.wake + tid * PT);
  *mine = 0x01010101u;
  __syncthreads();
  // busy[rd]: the round's pairs.  They are dealt to the threads densely, while
  // each particle of a pair goes on to its next partner in its own thread.
  for (int rd = 0;; rd = rd == 2 ? 0 : rd + 1) {
    const unsigned awake = *mine;
    unsigned pairs = 0;
    if (awake) {
      *mine = 0;
#pragma unroll
      for (int j = 0; j < PT; ++j)
        if ((awake >> (8 * j) & 1u) && nx[j] != PATCH_NONE && S.nxt[nx[j]] == at_place(j)) {
          pairs |= 1u << j;
          if (low[j] == 0) S.ready[atomicAdd(&busy[rd], 1)] = (unsigned)at_place(j) | (unsigned)nx[j] << 16;
        }
    }
    if (tid == 0) busy[rd == 2 ? 0 : rd + 1] = 0;
    __syncthreads();
    const int np = busy[rd];
    if (np == 0) break;
    for (int i = tid; i < np; i += FINAL_THREADS) {
      const int c = (int)(S.ready[i] & 0xffffu), q = (int)(S.ready[i] >> 16);
      T dx, dy, vix = S.vx[c], viy = S.vy[c], vjx = S.vx[q], vjy = S.vy[q];
      int kc = 0, kq = 0;
      if constexpr (!Pos<P>::G) {
        kc = S.key[c];
        kq = S.key[q];
      }
      Pos<P>::sep(k, kc, S.x[c], S.y[c], kq, S.x[q], S.y[q], dx, dy);
      if (pair_core<P>(k, dx, dy, vix, viy, vjx, vjy)) {
        S.vx[c] = vix;
        S.vy[c] = viy;
        S.vx[q] = vjx;
        S.vy[q] = vjy;
        ++ncoll;
      }
    }
    if (pairs) {
#pragma unroll
      for (int j = 0; j < PT; ++j)
        if (pairs >> j & 1u) {
          low[j] = max(low[j] - 1, 0);
          ++at[j];
          nx[j] = at[j] >= dg[j] ? PATCH_NONE
                                 : (at[j] < PATCH_NB ? nb[j].get(at[j]) : (int)(adj.row(sl[j])[at[j]] & 0xffffll));
          S.nxt[at_place(j)] = (unsigned short)nx[j];
          if (nx[j] != PATCH_NONE) {
            mark(at_place(j));
            mark(nx[j]);
          }
        }
    }
    __syncthreads();
  }
#pragma unroll
  for (int j = 0; j < PT; ++j)
    if (sl[j] >= 0) {
      T vx = S.vx[at_place(j)], vy = S.vy[at_place(j)];
      nwall += Pos<P>::walls_key(k, ldu(pt.key, sl[j]), S.x[at_place(j)], S.y[at_place(j)], vx, vy);
      pt.vx[sl[j]] = vx;
      pt.vy[sl[j]] = vy;
    }
}

// More particles than that (the contacts of a large settled bed percolate): the
// same in memory, by particles listed for the round instead of marks.  state:
// next entry | degree << 8 | partners of lower index left << 16.
struct FinalMem {  // by place, each [N]
  int32_t *next, *state, *list[2];
};
template <int P>
__device__ __forceinline__ void final_mem(const FinalMem M, Parts<typename Prec<P>::T> pt,
    const Consts<typename Prec<P>::T> &k, Adj adj, const int32_t *deg, const int32_t *left, const int32_t *place_of,
    const int n, int *cnt,
    int &ncoll, int &nwall) {
  constexpr int NT = FINAL_THREADS;
  constexpr int READY = 1 << 30;  // a listed place whose pair this entry fires
  const int tid = (int)threadIdx.x, lane = tid & 63;
  if (tid == 0) {
    cnt[0] = n;
    cnt[1] = 0;
  }
  for (int c = tid; c < n; c += NT) {
    const int s = left[c], id = pt.pid[s], dg = min(deg[s], KMAX);
    const AdjRow row = adj.row(s);
    int low = 0;
    for (int a = 0; a < dg; ++a) {
      const long long e = row[a];
      low += (int)(e >> 32) < id;
      const int c1 = place_of[adj_slot(e)];
      row[a] = (unsigned)c1 < (unsigned)n ? c1 : -1;  // the row now holds places
    }
    M.state[c] = dg << 8 | low << 16;
    M.next[c] = (int)row[0];
    M.list[0][c] = c;
  }
  __syncthreads();
  for (int b = 0, m = n; m > 0;) {  // uniform
    // A pair is fired through its lower index, which is listed whichever of the
    // two went on to the other.
    for (int i = tid; i < m; i += NT) {
      const int c = M.list[b][i], q = M.next[c];
      if (q >= 0 && M.next[q] == c && M.state[c] >> 16 == 0) M.list[b][i] = c | READY;
    }
    __syncthreads();
    for (int i0 = 0; i0 < m; i0 += NT) {
      const int i = i0 + tid;
      int on[2] = {-1, -1};  // the lower index of each new pair named
      if (i < m) {
        const int v = M.list[b][i], c = v & ~READY;
        // listed twice in a round: the first to take the pair fires it
        if (v != c && atomicOr(&M.state[c], READY) < READY) {
          const int q = M.next[c], s = left[c], t = left[q];
          ncoll += pair_collide<P>(k, pt, s, t);
          const int sc = (M.state[c] & ~READY) + 1, sq = M.state[q] + 1 - (1 << 16);
          const int nc = (sc & 0xff) < ((sc >> 8) & 0xff) ? (int)adj.row(s)[sc & 0xff] : -1;
          const int nq = (sq & 0xff) < ((sq >> 8) & 0xff) ? (int)adj.row(t)[sq & 0xff] : -1;
          M.next[c] = nc;
          M.next[q] = nq;
          M.state[c] = sc | READY;  // until the round ends
          M.state[q] = sq;
          on[0] = nc >= 0 && sc >> 16 == 0 ? c : nc;
          on[1] = nq >= 0 && sq >> 16 == 0 ? q : nq;
        }
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const unsigned long long f = __ballot(on[u] >= 0);
        int to = 0;
        if (lane == 0 && f) to = atomicAdd(&cnt[b ^ 1], __popcll(f));
        to = __shfl(to, 0, 64);
        if (on[u] >= 0) M.list[b ^ 1][to + __popcll(f & ((1ull << lane) - 1))] = on[u];
      }
    }
    __syncthreads();
    for (int i = tid; i < m; i += NT) {
      const int v = M.list[b][i];
      if (v & READY) M.state[v & ~READY] &= ~READY;
    }
    if (tid == 0) cnt[b] = 0;
    b ^= 1;
    __syncthreads();
    m = cnt[b];
  }
  for (int c = tid; c < n; c += NT) nwall += wall_pass<P>(k, pt, left[c]);
}

// What is left, for the final workgroup: of a bed of few particles everything
// (PLAN_WHOLE); after the patches what the last pass listed, where it is more than
// the final workgroup holds only what is left once the lanes and wavefronts of
// all workgroups have taken its clusters; of a bed resolved by clusters those too
// large for a workgroup.  The final workgroup is then the one that ends last; if
// there is nothing to do before it, the others end at once.  At most one
// workgroup per CU, since each has the LDS of the final one.  The collision stage
// of 100 000 spheres in the bottom quarter of 400 x 400 cells takes 272 us, against
// 531 with a pass of wider patches and the final workgroup in memory.
constexpr int REST_BLOCKS = 256, REST_BIG = 512;
struct RestBuffers {
  int32_t *left, *left2, *place_of;
  int32_t *sweep;        // SW_LEFT to SW_ENDED
  int32_t *coll, *wall;  // by workgroup
  FinalMem mem;
};
template <int P> union RestLds {
  FinalLds<P> fin;
  struct {
    ClustersLds<P, FINAL_THREADS, REST_BIG> cl;
    long long cand[FINAL_THREADS];
    int n;
  };
};
// A value that is the same in every lane, in a scalar register.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
// LISTS: the bed may have come by patches, or whole; CLUSTERS: by clusters.
template <int P, bool LISTS, bool CLUSTERS>
__device__ __forceinline__ void rest_body(const int bidx, const int gdim, const int plan, const bool listed,
    Parts<typename Prec<P>::T> pt, const Consts<typename Prec<P>::T> &k, Adj adj, int32_t *deg, const RestBuffers R) {
  __shared__ RestLds<P> U;
  __shared__ int cnt[3], tot[2], np, base, ended;
  const int tid = (int)threadIdx.x, lane = tid & 63;
  // an overflowed contact row leaves the graph incomplete: nothing is resolved
  const bool overflow =
      uniform(__hip_atomic_load(&k.flags[FLAG_CAPACITY], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) != 0;
  int n = 0;
  bool second = false;  // the list is left2
  bool first = false;  // work for all workgroups before the final one
  const bool clusters = CLUSTERS && (!LISTS || plan == PLAN_CLUSTERS), whole = LISTS && plan == PLAN_WHOLE;
  if (clusters) {
    first = uniform(R.sweep[SW_MORE]) != 0;
  } else if (!whole) {
    n = uniform(R.sweep[SW_LEFT]);
    if (listed && n > FINAL_CAP) {  // the second pass was needed
      n = uniform(R.sweep[SW_LEFT2]);
      second = true;
    }
    first = n > FINAL_CAP;
  }
  if (overflow) {
    first = false;
    n = 0;
  }
  if (!first && bidx != 0) {  // nothing to do but for the final workgroup
    if (tid == 0) R.coll[bidx] = R.wall[bidx] = 0;
    return;
  }
  // Appends the particle in slot l, where `has`, to the list `to`, whose length is
  // np; with count, *count is the length and the others append to it too.
  auto append = [&](bool has, int l, int32_t *to, int32_t *count) {
    const unsigned long long m = __ballot(has);
    int at = 0;
    if (lane == 0 && m) at = atomicAdd(&np, __popcll(m));
    at = __shfl(at, 0, 64) + __popcll(m & ((1ull << lane) - 1));
    if (count) {
      __syncthreads();
      if (tid == 0) {
        base = np > 0 ? atomicAdd(count, np) : 0;
        np = 0;
      }
      __syncthreads();
      at += base;
    }
    if (has) {
      to[at] = l;
      R.place_of[l] = at;
    }
  };
  int ncoll = 0, nwall = 0;
  // The final workgroup's n particles in `left`, and the sums.
  auto finish = [&](const int32_t *left) {
    if (n > 0) {
      if (n <= FINAL_CAP) final_lds<P>(U.fin, pt, k, adj, deg, left, R.place_of, n, cnt, ncoll, nwall);
      else final_mem<P>(R.mem, pt, k, adj, deg, left, R.place_of, n, cnt, ncoll, nwall);
    }
    if (ncoll) atomicAdd(&tot[0], ncoll);
    if (nwall) atomicAdd(&tot[1], nwall);
    __syncthreads();
    if (tid == 0) {
      R.coll[bidx] = tot[0];
      R.wall[bidx] = tot[1];
    }
  };
  if (tid < 2) tot[tid] = 0;
  if (tid == 0) np = 0;
  __syncthreads();
  if (!first) {
    if (whole) {
      for (int l0 = 0; l0 < k.npart && !overflow; l0 += FINAL_THREADS)
        append(l0 + tid < k.npart && ldu(deg, l0 + tid) > 0, l0 + tid, R.left, nullptr);
      __syncthreads();
      n = uniform(np);
    }
    finish(second ? R.left2 : R.left);
  } else {  // (the final workgroup's code again: its registers are its own so)
    if (clusters) {
      for (int l0 = bidx * FINAL_THREADS; l0 < k.npart; l0 += gdim * FINAL_THREADS) {
        const int d = l0 + tid < k.npart ? ldu(deg, l0 + tid) : 0;
        append(d > 0 && d < DONE_WHOLE, l0 + tid, R.left, &R.sweep[SW_LISTED]);
      }
    } else if constexpr (LISTS) {
      // runs of the list, so many that every workgroup has one
      const int32_t *left = second ? R.left2 : R.left;
      const int run = min(max((n + gdim - 1) / gdim, WAVE), FINAL_THREADS);
      long long nc = 0, nw = 0;
      for (int i0 = bidx * run; i0 < n; i0 += gdim * run) {
        if (tid == 0) U.n = 0;
        __syncthreads();
        bool c = false;
        long long r = 0;
        if (tid < run && i0 + tid < n) {
          const int s = left[i0 + tid], id = pt.pid[s];
          c = (int)(adj.row(s).a[0] >> 32) > id;
          r = ((long long)id << 32) | (unsigned)s;
        }
        const unsigned long long m = __ballot(c);
        int at = 0;
        if (lane == 0 && m) at = atomicAdd(&U.n, __popcll(m));
        at = __shfl(at, 0, 64);
        if (c) U.cand[at + __popcll(m & ((1ull << lane) - 1))] = r;
        __syncthreads();
        resolve_candidates<P>(U.cl, U.n, [&](int f) { return U.cand[f]; }, pt, adj, deg, deg, k, &R.sweep[SW_MORE],
                              nc, nw);
        __syncthreads();
      }
      ncoll = (int)nc;
      nwall = (int)nw;
    }
    __threadfence();
    __syncthreads();
    if (tid == 0) ended = atomicAdd(&R.sweep[SW_ENDED], 1);
    __syncthreads();
    const int listed_n = n;
    n = 0;
    if (uniform(ended) == gdim - 1) {
      __threadfence();
      if (clusters) {
        n = uniform(__hip_atomic_load(&R.sweep[SW_LISTED], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
      } else if (__hip_atomic_load(&R.sweep[SW_MORE], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
        for (int i0 = 0; i0 < listed_n; i0 += FINAL_THREADS) {
          const int l = i0 + tid < listed_n ? (second ? R.left2 : R.left)[i0 + tid] : -1;
          append(l >= 0 && deg[l] < DONE_WHOLE, l, second ? R.left : R.left2, nullptr);
        }
        __syncthreads();
        n = uniform(np);
        second = !second;
      }
    }
    finish(second ? R.left2 : R.left);
  }
}
template <int P, int PLAN>
__global__ __launch_bounds__(FINAL_THREADS) void k_rest(Parts<typename Prec<P>::T> pt,
                                                        Consts<typename Prec<P>::T> k, Adj adj, int32_t *deg,
                                                        RestBuffers R) {
  constexpr bool CLUSTERS = PLAN == PLAN_CLUSTERS;
  rest_body<P, !CLUSTERS, CLUSTERS>(blockIdx.x, gridDim.x, PLAN, false, pt, k, adj, deg, R);
}

}  // namespace lbdps
