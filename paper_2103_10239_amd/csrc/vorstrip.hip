// vorstrip.hip -- Voronoi (Delaunay) rows from strips of cells staged in LDS:
// the fast path of the Voronoi lists (voronoi.hip holds the general one).
//
// A workgroup stages a strip of cells with its halo (strip.h), as the k-NN
// kernel does, and each lane builds one particle's row from its block, one
// contiguous LDS range of candidates, by wrapping the Delaunay star:
//   - the nearest particle a_0 is always a neighbour (the disc on the segment
//     to it holds no other particle);
//   - the neighbour after a, counter-clockwise, is the particle c on the left
//     of a whose circle through 0, a and c is empty.  The circumcentre is
//     (a + t perp(a)) / 2 with t(c) = c.(c - a) / (a x c), and a smaller t is
//     a circle that holds less on the left: the neighbour has the smallest t;
//   - the star closes when a_0 comes round again.
// Every step is one uniform pass over the block (two packed subtracts, two
// 16-bit dot products, a reciprocal and a running minimum per candidate), so
// the lanes of a wavefront stay together, where clipping a cell candidate by
// candidate is a serial chain of exact predicates with its own path per lane.
//
// Exactness.  c.(c - a) and a x c are exact integers (16-bit offsets) or
// within 2^-23 of them; t is their fp32 quotient, within 2^-20.4 of itself.
// Where the two smallest quotients lie within 2^-19 of each other the step is
// decided again in exact integers (cross-multiplied); equal values are
// co-circular particles, of which the last counter-clockwise is the neighbour
// (the others' cells only touch), or particles that share a site, which the row
// then lists by index.  A row is written only when every circle of its star lies
// inside the block (with a margin above the rounding of its centre and radius)
// and its centre within L/8: no particle outside the block can then change it.
// Everything else -- circles that reach out of the block, stars of more than 16
// sites, rows longer than dmax, strips that could not be staged -- is listed for
// k_vor_wave, which takes a wavefront per row, and what that leaves is flagged
// for the general kernel.
//
// Bound by VALU issue: about 17 instructions per candidate and step, 56
// candidates and 6 steps per particle at the mean (the longest row of a
// wavefront, 9 to 10, sets its steps): 12,700 instructions a wave, 51% of the
// lanes active.  Offsets of more than 16 bits (sparse systems) take fp32 sums of
// products with their rounding put back (60,000 particles, 256 queries a strip:
// 106 us, 115 with fp64 products and their conversions).  Rows of 2^20 uniform
// particles, four a cell: 1.83 ms by clipping alone, 0.74 the strips and 0.03 the
// rows they leave, one a cell 0.44; of 250,000: 633 us, now 150 + 27.
#include "strip.h"

namespace nm {

namespace {

constexpr int kVsCap = 16;         // longest row
// Candidates of a block above which a row goes to the general kernel at once: a
// star costs its candidates times its steps, clipping each candidate about once,
// but has a cell's latency.  Rows of 2^20 particles, half of them in 64 clusters,
// with 900, without a limit, by clipping alone: 16 particles a cell 10.5, 14.1
// and 11.1 ms, four a cell 2.5, 2.5 and 5.1 (4.2 with a limit of 400 or 600).
constexpr int kVsCands = 900;
constexpr int kVsTwin = 1 << 16;   // flag of a site with several particles
constexpr double kVsReach = 2.6;   // block half side, in mean spacings

// Dot product of two packed pairs of 16-bit values (below 2^31), with a zero
// accumulator operand so that no register is cleared first.
__device__ __forceinline__ int dot2(int a, int b) {
  int r;
  asm("v_dot2_i32_i16 %0, %1, %2, 0" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

// t of candidate c in the step from neighbour a, within 2^-20.4 of itself;
// infinite where c is not on the left of a.  (pq, pqy), (pa, pay): packed
// positions of the query and of a (narrow, with perp = perp(a)), or x, y.
// Wide: fp32 offsets are exact (below 2^24); a sum or difference of two products
// with the rounding of one put back is within 2^-23 of itself, and zero only
// where it is zero.
template <bool kWide>
struct PivotStep {
  int pq, pqy, pa, perp;
  float axf, ayf;
  __device__ __forceinline__ PivotStep(int pq_, int pqy_, int pa_, int ax, int ay)
      : pq(pq_), pqy(pqy_), pa(pa_), perp(pack_rel(-ay, ax)), axf(static_cast<float>(ax)), ayf(static_cast<float>(ay)) {}
  __device__ __forceinline__ float t(int2 c) const {
    const float cx = static_cast<float>(c.x - pq), cy = static_cast<float>(c.y - pqy);
    const float ex = cx - axf, ey = cy - ayf;
    const float p = cy * ey, q = ayf * cx;
    const float num = fmaf(cx, ex, p) + fmaf(cy, ey, -p);
    const float den = fmaf(axf, cy, -q) - fmaf(ayf, cx, -q);
    const float v = num * __builtin_amdgcn_rcpf(den);
    return den > 0.0f ? v : INFINITY;
  }
  __device__ __forceinline__ float t(int c) const {
    const short2v d = __builtin_bit_cast(short2v, c) - __builtin_bit_cast(short2v, pq);
    const short2v f = __builtin_bit_cast(short2v, c) - __builtin_bit_cast(short2v, pa);
    const int num = dot2(__builtin_bit_cast(int, d), __builtin_bit_cast(int, f));
    const int den = dot2(__builtin_bit_cast(int, d), perp);
    const float q = static_cast<float>(num) * __builtin_amdgcn_rcpf(static_cast<float>(den));
    return den > 0 ? q : INFINITY;
  }
};

// The step from neighbour (ax, ay) in exact integers: of the candidates [b, e),
// those whose t is not above `lim` (twice the error above the smallest) decide.
// They are collected by a pass like the step's own, over the rows of cells that
// the circle found meets, and then compared, the lanes' first, second, ... ones
// together: 2^20 particles on a square lattice 254 us (375 with every candidate
// of the block compared in integers, 249 by clipping alone), 2^18 on one a few
// units out of place 264 (500, 362).
// Returns the neighbour's LDS index (the first of its site), with kVsTwin where
// others share its position; -1: none.
template <bool kWide>
__device__ __noinline__ int vor_pivot_exact(const int* lpos, int b, int e, int pq, int pqy, int pa, int ax, int ay,
                                            float lim) {
  using I = std::conditional_t<kWide, __int128, long long>;
  using P = std::conditional_t<kWide, int2, int>;
  const P* pos = reinterpret_cast<const P*>(lpos);
  const PivotStep<kWide> step(pq, pqy, pa, ax, ay);
  int best = -1;
  bool twin = false;
  long long bn = 0, bd = 1, bx = 0, by = 0;
  auto compare = [&](int i) {
    long long cx, cy;
    if constexpr (kWide) {
      cx = pos[i].x - pq;
      cy = pos[i].y - pqy;
    } else {
      const short2v d = __builtin_bit_cast(short2v, pos[i]) - __builtin_bit_cast(short2v, pq);
      cx = d[0];
      cy = d[1];
    }
    const long long den = ax * cy - ay * cx;
    if (den <= 0) return;
    const long long num = cx * (cx - ax) + cy * (cy - ay);
    const I diff = static_cast<I>(num) * bd - static_cast<I>(bn) * den;
    bool take = best < 0 || diff < 0;
    if (take) twin = false;
    if (best >= 0 && diff == 0) {
      const long long turn = bx * cy - by * cx;
      take = turn > 0;
      if (take) twin = false;
      if (turn == 0) twin = true;  // the same position twice
    }
    if (take) {
      best = i;
      bn = num;
      bd = den;
      bx = cx;
      by = cy;
    }
  };
  unsigned long long near = 0ull;
  int count = 0;
  for (int i0 = b; i0 < e; i0 += kUnroll) {
    P c[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) c[u] = pos[i0 + u];  // (buffer padded by kUnroll)
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      if (i0 + u < e && step.t(c[u]) <= lim) {
        if (count < 4) near |= static_cast<unsigned long long>(i0 + u) << (16 * count);
        ++count;
      }
    }
  }
  if (count <= 4) {
    for (int j = 0; j < count; ++j) compare(static_cast<int>(near >> (16 * j)) & 0xFFFF);
  } else {
    for (int i = b; i < e; ++i) compare(i);
  }
  return twin ? best | kVsTwin : best;
}

// The star of staged particle `self` over the candidates of its block, whose rows
// of cells start at rows[0], rows[1], ... and whose outside lies at offsets
// <= -gl or >= gr in x, <= -gd or >= gu in y.
// Writes the neighbours' LDS indices to col[0 .. m) (stride kBlock),
// counter-clockwise from the nearest; first: the entry to start the row at
// (counter-clockwise from +x); shared: particles share the own position or a
// neighbour's.  Returns m, or 0 when the row is not certain.
template <bool kWide>
__device__ __forceinline__ int vor_star(const int* lpos, const int* rows, int lw, int self, int gl, int gr, int gd,
                                        int gu, int cap, float domain, uint16_t* col, int& first,
                                        bool& shared) {
  const int b = rows[0], e = rows[(gd + gu - 1) >> lw];
  const int2* lpos2 = reinterpret_cast<const int2*>(lpos);
  int pq, pqy = 0;
  if (kWide) {
    pq = lpos2[self].x;
    pqy = lpos2[self].y;
  } else {
    pq = lpos[self];
  }
  // the nearest other site, and how many particles are at the particle's own
  int start = -1, own = 0;
  if (kWide) {
    unsigned long long best = ~0ull;
    for (int i = b; i < e; ++i) {
      const int2 c = lpos2[i];
      const long long dx = c.x - pq, dy = c.y - pqy;
      const unsigned long long d2 = static_cast<unsigned long long>(dx * dx + dy * dy);
      own += d2 == 0ull ? 1 : 0;
      if (d2 - 1ull < best) {  // (0: the largest)
        best = d2 - 1ull;
        start = i;
      }
    }
  } else {
    uint32_t best = ~0u;
    auto round = [&](int i, bool tail) {
      int c[kUnroll];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) c[u] = lpos[i + u];  // (buffer padded by kUnroll)
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        uint32_t d2 = rel_d2_u(c[u], pq) - 1u;  // (0: the largest)
        if (tail && i + u >= e) d2 = ~0u - 1u;
        own += d2 == ~0u ? 1 : 0;
        start = d2 < best ? i + u : start;
        best = min(best, d2);
      }
    };
    const int full = b + ((e - b) & ~(kUnroll - 1));
    for (int i = b; i < full; i += kUnroll) round(i, false);
    if (full < e) round(full, true);
  }
  if (start < 0 || start >= e) return 0;
  shared = own > 1;
  int cur = start, m = 0;
  first = -1;
  for (;;) {
    if (m >= cap) return 0;
    col[m * kBlock] = static_cast<uint16_t>(cur);
    ++m;
    int pa, ax, ay;
    if (kWide) {
      pa = lpos2[cur].x;
      ax = pa - pq;
      ay = lpos2[cur].y - pqy;
    } else {
      pa = lpos[cur];
      const short2v d = __builtin_bit_cast(short2v, pa) - __builtin_bit_cast(short2v, pq);
      ax = d[0];
      ay = d[1];
    }
    float t0 = INFINITY, t1 = INFINITY;  // the two smallest t
    int next = -1;
    const PivotStep<kWide> step(pq, pqy, pa, ax, ay);
    auto round = [&](int i, bool tail) {
      float t[kUnroll];
      std::conditional_t<kWide, int2, int> c[kUnroll];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        if constexpr (kWide)
          c[u] = lpos2[i + u];
        else
          c[u] = lpos[i + u];
      }
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) t[u] = step.t(c[u]);
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const float v = tail && i + u >= e ? INFINITY : t[u];
        next = v < t0 ? i + u : next;
        t1 = __builtin_amdgcn_fmed3f(t0, t1, v);
        t0 = fminf(t0, v);
      }
    };
    const int full = b + ((e - b) & ~(kUnroll - 1));
    for (int i = b; i < full; i += kUnroll) round(i, false);
    if (full < e) round(full, true);
    if (next < 0) return 0;
    // the circle through 0, a and the neighbour lies inside the block, its
    // centre inside the domain (fp32: a few 2^-22 of the radius, well under
    // the margin)
    const float fx = static_cast<float>(ax), fy = static_cast<float>(ay);
    const float hx = 0.5f * (fx - t0 * fy), hy = 0.5f * (fy + t0 * fx);
    const float r = sqrtf(hx * hx + hy * hy) * 1.001f + 1.0f;
    if (!(r < domain && hx - r > static_cast<float>(-gl) && hx + r < static_cast<float>(gr) &&
          hy - r > static_cast<float>(-gd) && hy + r < static_cast<float>(gu)))
      return 0;
    if (t1 - t0 <= (fabsf(t0) + fabsf(t1)) * 0x1p-19f) {
      // what may be nearer lies on that circle: in the rows of cells that it meets
      const int top = ((gd + gu - 1) >> lw) - 1;
      const int lo = max(static_cast<int>(hy - r + static_cast<float>(gd - 1)) >> lw, 0);
      const int hi = min(static_cast<int>(hy + r + static_cast<float>(gd)) >> lw, top);
      next = vor_pivot_exact<kWide>(lpos, rows[lo], rows[hi + 1], pq, pqy, pa, ax, ay, t0 + fabsf(t0) * 0x1p-19f);
      if (next < 0) return 0;
      if (next & kVsTwin) {
        shared = true;
        next &= ~kVsTwin;
      }
    }
    int bx, by;
    if (kWide) {
      bx = lpos2[next].x - pq;
      by = lpos2[next].y - pqy;
    } else {
      const short2v d = __builtin_bit_cast(short2v, lpos[next]) - __builtin_bit_cast(short2v, pq);
      bx = d[0];
      by = d[1];
    }
    // the turn from the lower half plane into the upper one passes +x: the
    // row starts with the neighbour after it
    const bool la = !(ay > 0 || (ay == 0 && ax > 0)), lb = !(by > 0 || (by == 0 && bx > 0));
    if (la && !lb) first = next == start ? 0 : m;
    if (next == start) break;
    cur = next;
  }
  return first < 0 ? 0 : m;
}

// The row of a star with shared sites: the other particles of the own site by
// index, then each neighbour site's.  A site lies in one cell, so its particles
// are among the staged ones of its halo row.  Returns the row's length, or 0,
// with nothing written, where it exceeds dmax.  (2^20 particles in pairs: 2.3 ms,
// as by clipping; 21 with a wavefront for each of their rows.)
template <bool kWide>
__device__ __noinline__ int vor_write_shared(const int* lpos, const int* lidx, const uint8_t* rowid, const int* rbase,
                                             const uint16_t* col, int self, int m, int first, int dmax,
                                             int32_t* __restrict__ row) {
  using P = std::conditional_t<kWide, int2, int>;
  const P* pos = reinterpret_cast<const P*>(lpos);
  auto same = [&](int i, int j) {
    if constexpr (kWide)
      return pos[i].x == pos[j].x && pos[i].y == pos[j].y;
    else
      return pos[i] == pos[j];
  };
  const int who = lidx[self];
  int len = 0;
  for (int write = 0; write < 2; ++write) {
    int at = 0;
    for (int t = -1; t < m; ++t) {
      int u = first + t;
      u = u >= m ? u - m : u;
      const int p = t < 0 ? self : col[u * kBlock];
      const int b = rbase[rowid[p]], e = rbase[rowid[p] + 1];
      if (write) {
        for (int prev = -1;;) {
          int next = 0x7FFFFFFF, left = 0;  // the next index, and how many remain
          for (int i = b; i < e; ++i) {
            const int j = lidx[i];
            if (same(i, p) && j > prev && j != who) {
              ++left;
              next = min(next, j);
            }
          }
          if (left == 0) break;
          row[at++] = next;
          if (left == 1) break;
          prev = next;
        }
      } else {
        for (int i = b; i < e; ++i) at += same(i, p) && i != self ? 1 : 0;
      }
    }
    len = at;
    if (len > dmax) return 0;
  }
  for (int u = len; u < dmax; ++u) row[u] = -1;
  return len;
}

// Append slot s to the wave kernel's list (one atomic per wavefront).
__device__ __forceinline__ void vor_list(const DevWs& w, bool go, int s) {
  const unsigned long long b = __ballot(go);
  if (b == 0ull) return;
  const int lane = threadIdx.x & 63;
  const int leader = __ffsll(static_cast<long long>(b)) - 1;
  uint32_t base = 0u;
  if (lane == leader) base = atomicAdd(&w.hdr->nvstale, static_cast<uint32_t>(__popcll(b)));
  base = __shfl(base, leader, 64);
  const uint32_t at = base + static_cast<uint32_t>(__popcll(b & ((1ull << lane) - 1ull)));
  if (go && at < static_cast<uint32_t>(w.n)) w.rank[at] = s;
}

// Half side, in cells, of a block at density rho particles per cell.
__device__ __host__ __forceinline__ int vor_half(float rho) {
  return static_cast<int>(ceilf(static_cast<float>(kVsReach) / sqrtf(rho)));
}

// kStale: only the rows marked in `stale` (by particle) unless the header's
// nvfull asks for all, else every row.
// Nothing runs when `gate` is given and *gate is 0.
template <bool kStale, bool kWide>
__global__ __launch_bounds__(kBlock) void k_vor_strip(DevWs w, TileCfg tc, int dmax, int32_t* __restrict__ ring,
                                                      int32_t* __restrict__ deg,
                                                      const uint8_t* __restrict__ stale,
                                                      const uint32_t* __restrict__ gate) {
  __shared__ int2 lpos_store[kStripPts / 2 + kUnroll];
  __shared__ int lidx[kStripPts];
  __shared__ int s_rbase[kStripRows + 1];
  __shared__ int s_ga0[kStripRows];
  __shared__ int s_n0[kStripRows];
  __shared__ int s_ga1[kStripRows];
  __shared__ int s_qoff[kStripRows + 1];
  __shared__ int s_tself[kStripRows];
  __shared__ int s_wsum[kBlock / 64];
  __shared__ uint8_t s_rowid[kStripPts];
  __shared__ uint16_t s_qmap[kStripPts];
  __shared__ int s_nsel;
  __shared__ uint16_t s_col[kVsCap * kBlock];
  __shared__ int s_sub[kStripRows + 1];  // sub-strips: first row, bit 30 when it cannot be staged
  __shared__ int s_nsub;
  int* lpos = reinterpret_cast<int*>(lpos_store);
  const WsHeader* hd = w.hdr;
  const int tile = xcd_run(blockIdx.x, gridDim.x);
  if (!cells_built(w)) {
    if (tile == 0 && threadIdx.x == 0) set_err(w.hdr, NM_E_INVAL);
    return;
  }
  if (gate && *gate == 0u) return;
  const bool all = !kStale || hd->nvfull != 0u;
  const int total = min(w.start[w.C], w.n);
  const int G = w.G, lw = w.log2_w;
  const int tyi = tile / tc.ntx, txi = tile - tyi * tc.ntx;
  const int x0 = txi * tc.tw, y0 = tyi * tc.th, ty = min(tc.th, G - y0);
  const int tw = tc.tw, hy = tc.hy;
  constexpr bool wide = kWide;
  const float domain = static_cast<float>(w.box >> 3);
  const int cap = min(kVsCap, dmax);
  // the halo's width from the strip's own density, never wider than the grid's
  int hx = tc.hx;
  {
    int q = 0;
    if (static_cast<int>(threadIdx.x) < ty) {
      const int64_t prow = static_cast<int64_t>(y0 + threadIdx.x) * G;
      q = max(min(w.start[prow + x0 + tw], total) - w.start[prow + x0], 0);
    }
    int nqs;
    (void)block_exclusive_scan(q, s_wsum, &nqs);
    if (nqs == 0) return;
    hx = max(1, min(vor_half(static_cast<float>(nqs) / static_cast<float>(tw * ty)), tc.hx));
  }
  const int W = tw + 2 * hx;
  StripGeo geo{x0, y0, ty, tw, hx, hy, wide};
  int next = -1, nsub = 0;  // the sub-strip to stage next (-1: the whole strip)
  for (;;) {
    int npts, nq;
    __builtin_amdgcn_s_setprio(3);
    const bool staged = strip_stage<true>(
        w, geo, StripLds{lpos_store, lidx, s_rbase, s_ga0, s_n0, s_ga1, s_qoff, s_tself, s_wsum, s_rowid, s_qmap},
        total, npts, nq);
    __builtin_amdgcn_s_setprio(0);
    nq = __builtin_amdgcn_readfirstlane(nq);
    if (next < 0 && !staged && nq > 0) {
      // the halo does not fit: sub-strips of whole rows, each as tall as fits
      const int room = wide ? kStripPts / 2 : kStripPts;
      if (threadIdx.x == 0) {
        int ns = 0;
        for (int r0 = 0; r0 < ty;) {
          const bool fits = s_rbase[r0 + 2 * hy + 1] - s_rbase[r0] <= room;
          int r1 = r0 + 1;
          if (fits)
            while (r1 < ty && s_rbase[r1 + 2 * hy + 1] - s_rbase[r0] <= room) ++r1;
          s_sub[ns++] = r0 | (fits ? 0 : 1 << 30);
          r0 = r1;
        }
        s_sub[ns] = ty;
        s_nsub = ns;
      }
      __syncthreads();
      nsub = __builtin_amdgcn_readfirstlane(s_nsub);
      next = 0;
    } else {
      int run = nq;
      if (kStale && staged && !all) {
        // the stale queries to the front of the query map: a round's entries
        // are read before any is written, and go to places read before
        if (threadIdx.x == 0) s_nsel = 0;
        __syncthreads();
        for (int q0 = 0; q0 < nq; q0 += kBlock) {
          const int qi = q0 + threadIdx.x;
          const int self = qi < nq ? s_qmap[qi] : 0;
          const bool go = qi < nq && stale[lidx[self]] != 0;
          const unsigned long long bal = __ballot(go);
          const int lane = threadIdx.x & 63;
          int base = 0;
          if (lane == 0 && bal != 0ull) base = atomicAdd(&s_nsel, __popcll(bal));
          base = __shfl(base, 0, 64);
          __syncthreads();
          if (go) s_qmap[base + __popcll(bal & ((1ull << lane) - 1ull))] = static_cast<uint16_t>(self);
        }
        __syncthreads();
        run = __builtin_amdgcn_readfirstlane(s_nsel);
      }
      for (int q0 = 0; q0 < run; q0 += kBlock) {
        const int qi = q0 + threadIdx.x;
        bool defer = false;
        int s = 0;
        if (qi < run) {
          if (staged) {
            const int self = s_qmap[qi];
            const int cy = s_rowid[self];
            int rx, oy;
            if (wide) {
              const int2 p = lpos_store[self];
              rx = p.x;
              oy = p.y & ((1 << lw) - 1);
            } else {
              rx = lpos[self] & 0xFFFF;
              oy = (lpos[self] >> 16) & ((1 << lw) - 1);
            }
            const int n3 = s_rbase[cy + 2] - s_rbase[cy - 1];
            const float rho = fmaxf(static_cast<float>(n3), 0.5f) / static_cast<float>(3 * W);
            const int half = max(1, min(vor_half(rho), hy));
            const int cw = 1 << lw;
            const int gl = rx + 1, gr = W * cw - rx;
            const int gd = oy + half * cw + 1, gu = (half + 1) * cw - oy;
            int first = 0;
            bool shared = false;
            uint16_t* col = s_col + threadIdx.x;
            const int* rows = s_rbase + cy - half;
            const bool dense = rows[2 * half + 1] - rows[0] > kVsCands;
            int m = 0;
            if (!dense) m = vor_star<kWide>(lpos, rows, lw, self, gl, gr, gd, gu, cap, domain, col, first, shared);
            if (shared && m > 0) {
              m = vor_write_shared<kWide>(lpos, lidx, s_rowid, s_rbase, col, self, m, first, dmax,
                                          ring + static_cast<int64_t>(lidx[self]) * dmax);
              if (m > 0) deg[lidx[self]] = m;
            } else if (m > 0) {
              const int who = lidx[self];
              int32_t* row = ring + static_cast<int64_t>(who) * dmax;
              // four entries a store (rows start on any 4-byte boundary)
              for (int u = 0; u + 4 <= dmax; u += 4) {
                int v[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                  int p = first + u + c;
                  p = p >= m ? p - m : p;
                  v[c] = u + c < m ? lidx[col[(p < m ? p : 0) * kBlock]] : -1;
                }
                *reinterpret_cast<nm_int4u*>(row + u) = nm_int4u{v[0], v[1], v[2], v[3]};
              }
              for (int u = dmax & ~3; u < dmax; ++u) {
                int p = first + u;
                p = p >= m ? p - m : p;
                row[u] = u < m ? lidx[col[(p < m ? p : 0) * kBlock]] : -1;
              }
              deg[who] = m;
            }
            if (m == 0) {
              defer = !dense;
              s = strip_slot(StripLds{lpos_store, lidx, s_rbase, s_ga0, s_n0, s_ga1, s_qoff, s_tself, s_wsum,
                                      s_rowid, s_qmap},
                             self);
              if (dense) {
                w.dflag[s] = 1;
                w.hdr->nvflag = 1u;
              }
            }
          } else {
            int r = 0;
#pragma unroll
            for (int step = kRowStep; step > 0; step >>= 1)
              if (r + step < geo.ty && s_qoff[r + step] <= qi) r += step;
            s = w.start[static_cast<int64_t>(geo.y0 + r) * G + x0] + (qi - s_qoff[r]);
            defer = !kStale || all || stale[w.sorted[s].z] != 0;
          }
        }
        vor_list(w, defer, s);
      }
      if (next < 0 || next >= nsub) break;
      __syncthreads();  // this sub-strip's queries are done with LDS
    }
    const int e = __builtin_amdgcn_readfirstlane(s_sub[next]);
    const int r0 = e & 0xFFFF, r1 = __builtin_amdgcn_readfirstlane(s_sub[next + 1]) & 0xFFFF;
    geo = StripGeo{x0, y0 + r0, r1 - r0, tw, (e >> 30) == 0 ? hx : 0, hy, wide};
    ++next;
  }
}

// ---------------------------------------------------------------------------
// The rows that the strips leave, a wavefront each.  The wave gathers a block
// of cells around the particle from the cell-ordered copy into LDS (up to
// kVwCands candidates; the block grows until it holds the star), its lanes
// evaluate 64 candidates a round and the step is the smallest t over the
// wave.  Offsets are int32 and the products fp64 (exact below 2^53), ambiguous
// steps are decided in exact integers, and coincident particles are expanded
// site by site, so only rows whose circles leave every block that fits (or
// the domain), or that do not fit their row, remain: they are flagged for the
// general kernel.
//
// A lane alone took 0.9 ms for such a row (its ring walk and its clipping are
// one serial chain), whatever their number: at 250,000 uniform particles the
// 0.3% that the strips leave took longer than clipping every cell did.
// ---------------------------------------------------------------------------
constexpr int kVwCands = 512;     // candidates a wave holds
constexpr int kVwWant = 128;      // candidates the first block should hold
constexpr int kVwWaves = 4;       // waves per workgroup
constexpr int kVwSites = 64;      // neighbour sites a wave can list (one per lane)
constexpr int kVwGridMax = 2048;  // workgroups

__device__ __forceinline__ long long shfl_ll(long long v, int src) {
  const int lo = __shfl(static_cast<int>(v), src, 64);
  const int hi = __shfl(static_cast<int>(v >> 32), src, 64);
  return static_cast<long long>((static_cast<uint64_t>(static_cast<uint32_t>(hi)) << 32) | static_cast<uint32_t>(lo));
}

// The step from neighbour (ax, ay) in exact integers over the wave's n
// candidates ((0, 0): the start, the smallest circle that touches the y axis
// at the particle from the right).  Every lane gets the neighbour's index.
__device__ __noinline__ int vor_wave_exact(const int2* c, int n, int ax, int ay) {
  const int lane = threadIdx.x & 63;
  const bool begin = ax == 0 && ay == 0;
  long long bn = 0, bd = 0;  // bd == 0: none yet
  int bx = 0, by = 0, best = -1;
  // does (n1, d1, x1, y1) come before the best so far: smaller t, or the same
  // circle and farther counter-clockwise
  auto before = [](long long n1, long long d1, int x1, int y1, long long n0, long long d0, int x0, int y0) {
    if (d1 == 0) return false;
    if (d0 == 0) return true;
    const __int128 diff = static_cast<__int128>(n1) * d0 - static_cast<__int128>(n0) * d1;
    if (diff != 0) return diff < 0;
    return static_cast<long long>(x0) * y1 - static_cast<long long>(y0) * x1 > 0;
  };
  for (int i = lane; i < n; i += 64) {
    const long long cx = c[i].x, cy = c[i].y;
    const long long den = begin ? cx : ax * cy - ay * cx;
    if (den <= 0) continue;
    const long long num = cx * (cx - ax) + cy * (cy - ay);
    if (before(num, den, c[i].x, c[i].y, bn, bd, bx, by)) {
      bn = num;
      bd = den;
      bx = c[i].x;
      by = c[i].y;
      best = i;
    }
  }
  for (int off = 32; off > 0; off >>= 1) {
    const int src = lane ^ off;
    const long long on = shfl_ll(bn, src), od = shfl_ll(bd, src);
    const int ox = __shfl(bx, src, 64), oy = __shfl(by, src, 64), oi = __shfl(best, src, 64);
    // (the two lanes of a pair have to agree: twins go to the lower index)
    const bool theirs = before(on, od, ox, oy, bn, bd, bx, by);
    const bool ours = before(bn, bd, bx, by, on, od, ox, oy);
    if (theirs || (!ours && oi >= 0 && oi < best)) {
      bn = on;
      bd = od;
      bx = ox;
      by = oy;
      best = oi;
    }
  }
  return best;
}

__global__ __launch_bounds__(64 * kVwWaves) void k_vor_wave(DevWs w, int dmax, int32_t* __restrict__ ring,
                                                            int32_t* __restrict__ deg) {
  __shared__ int2 s_off[kVwWaves][kVwCands];
  __shared__ int s_idx[kVwWaves][kVwCands];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int2* off = s_off[wave];
  int* idx = s_idx[wave];
  if (!cells_built(w)) return;  // (reported by the strip kernel; the list may hold anything)
  const int total = min(w.start[w.C], w.n);
  const int nl = static_cast<int>(min<uint32_t>(w.hdr->nvstale, static_cast<uint32_t>(w.n)));
  const int sh = 32 - w.log2_box, cw = 1 << w.log2_w, gm = w.G - 1;
  const float domain = static_cast<float>(w.box >> 3);
  const float rho = static_cast<float>(w.n) / static_cast<float>(w.C);
  const int guess = max(1, min(min(15, (w.G - 2) / 2), static_cast<int>(0.5f * (sqrtf(kVwWant / rho) - 1.0f))));
  for (int k = blockIdx.x * kVwWaves + wave; k < nl; k += gridDim.x * kVwWaves) {
    const int s = w.rank[k];
    const int4 q = w.sorted[s];
    const int hx = q.x >> w.log2_w, hy = q.y >> w.log2_w;
    const int ox = q.x & (cw - 1), oy = q.y & (cw - 1);
    bool done = false;
    int had = 0;
    // from the block that should hold enough at the mean density (a block too
    // dense for it: from the smallest)
    bool smaller = guess > 1;
    for (int half = guess; half <= 15 && 2 * half + 2 <= w.G && !done; ++half) {
      // row l / 2 of the block, the part before (0) or after (1) the box edge
      int beg = 0, cnt = 0;
      {
        const int r = (lane >> 1) - half, part = lane & 1;
        if (r <= half) {
          const int64_t row = static_cast<int64_t>((hy + r) & gm) * w.G;
          const int c0 = hx - half, c1 = hx + half;
          int a = c0, b = c1;  // columns, inclusive
          if (c0 < 0) {
            a = part == 0 ? c0 + w.G : 0;
            b = part == 0 ? gm : c1;
          } else if (c1 > gm) {
            a = part == 0 ? c0 : 0;
            b = part == 0 ? gm : c1 - w.G;
          } else if (part == 1) {
            b = a - 1;
          }
          if (b >= a) {
            beg = w.start[row + a];
            cnt = max(min(w.start[row + b + 1], total) - beg, 0);
          }
        }
      }
      int incl = cnt;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
      }
      const int n = __shfl(incl, 63, 64);
      if (n > kVwCands && smaller) {
        smaller = false;
        half = 0;
        continue;
      }
      if (n > kVwCands) break;  // too dense for larger blocks
      smaller = false;
      // blocks too sparse to hold a star are passed over, unless they are the last
      const bool last = half == 15 || 2 * half + 4 > w.G;
      if (n < kVwWant && !last) continue;
      if (had == n && !last) continue;
      had = n;
      const int excl = incl - cnt;
      for (int j0 = 0; j0 < n; j0 += 64) {
        const int j = j0 + lane;
        int lo = 0;  // owner lane of flattened candidate j: the last with excl <= j
#pragma unroll
        for (int step = 32; step > 0; step >>= 1) {
          const int e = __shfl(excl, lo + step, 64);
          if (e <= j) lo += step;
        }
        const int ob = __shfl(beg, lo, 64), oe = __shfl(excl, lo, 64);
        if (j < n) {
          const int4 e = w.sorted[ob + (j - oe)];
          off[j] = make_int2(wrap_axis(e.x - q.x, sh), wrap_axis(e.y - q.y, sh));
          idx[j] = e.z;
        }
      }
      __builtin_amdgcn_wave_barrier();
      __threadfence_block();
      const int gl = ox + half * cw + 1, gr = (half + 1) * cw - ox;
      const int gd = oy + half * cw + 1, gu = (half + 1) * cw - oy;
      // the star, from the particle of the smallest circle touching the y axis
      int ax = 0, ay = 0, m = 0, first = -1, start = -1;
      int site = -1;  // lane t: the t-th neighbour
      bool ok = true;
      for (;;) {
        const bool begin = start < 0;
        float t0 = INFINITY, t1 = INFINITY;
        int next = -1;
        const double axd = ax, ayd = ay;
        for (int i = lane; i < n; i += 64) {
          const double cx = off[i].x, cy = off[i].y;
          const double num = cx * (cx - axd) + cy * (cy - ayd), den = begin ? cx : axd * cy - ayd * cx;
          const float v = den > 0.0 ? static_cast<float>(num) * __builtin_amdgcn_rcpf(static_cast<float>(den)) : INFINITY;
          next = v < t0 ? i : next;
          t1 = __builtin_amdgcn_fmed3f(t0, t1, v);
          t0 = fminf(t0, v);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
          const float u0 = __shfl_xor(t0, o, 64), u1 = __shfl_xor(t1, o, 64);
          const int un = __shfl_xor(next, o, 64);
          t1 = fminf(fminf(t1, u1), fmaxf(t0, u0));
          next = u0 < t0 || (u0 == t0 && un < next) ? un : next;
          t0 = fminf(t0, u0);
        }
        if (next < 0) {
          ok = false;
          break;
        }
        if (!(t1 - t0 > (fabsf(t0) + fabsf(t1)) * 0x1p-19f)) next = vor_wave_exact(off, n, ax, ay);
        const float fx = static_cast<float>(ax), fy = static_cast<float>(ay);
        // centre (a + t perp(a)) / 2; the start's circle has its centre at (t, 0) / 2
        const float vx = begin ? 0.5f * t0 : 0.5f * (fx - t0 * fy), vy = begin ? 0.0f : 0.5f * (fy + t0 * fx);
        const float r = sqrtf(vx * vx + vy * vy) * 1.001f + 1.0f;
        const bool inside = vx - r > static_cast<float>(-gl) && vx + r < static_cast<float>(gr) &&
                            vy - r > static_cast<float>(-gd) && vy + r < static_cast<float>(gu);
        if (!inside || (!begin && !(r < domain))) {
          ok = false;
          break;
        }
        const int bx = off[next].x, by = off[next].y;
        if (begin) {
          start = next;
        } else {
          const bool la = !(ay > 0 || (ay == 0 && ax > 0)), lb = !(by > 0 || (by == 0 && bx > 0));
          const bool closed = bx == off[start].x && by == off[start].y;
          if (la && !lb) first = closed ? 0 : m;
          if (closed) break;
        }
        if (m >= kVwSites) {
          ok = false;
          break;
        }
        if (lane == m) site = next;
        ++m;
        ax = bx;
        ay = by;
      }
      if (!ok || first < 0) continue;
      // particles per site: lane t < m counts its own, lane 0 also the row's own site
      int row_len = 0;
      bool plain = true;
      for (int t = -1; t < m; ++t) {
        const int p = t < 0 ? 0 : __shfl(site, t, 64);
        const int px = t < 0 ? 0 : off[p].x, py = t < 0 ? 0 : off[p].y;
        int c = 0;
        for (int i0 = 0; i0 < n; i0 += 64) {
          const int i = i0 + lane;
          c += __popcll(__ballot(i < n && off[i].x == px && off[i].y == py));
        }
        if (t < 0) --c;  // the particle itself
        plain = plain && c == (t < 0 ? 0 : 1);
        row_len += c;
      }
      if (row_len > dmax) break;  // the general kernel reports it
      int32_t* row = ring + static_cast<int64_t>(q.z) * dmax;
      if (plain) {
        int p = first + lane;
        p = p >= m ? p - m : p;
        const int src = __shfl(site, p < m ? p : 0, 64);
        if (lane < dmax) row[lane] = lane < m ? idx[src] : -1;
      } else {
        int at = 0;
        for (int t = -1; t < m; ++t) {
          int u = first + max(t, 0);
          u = u >= m ? u - m : u;
          const int p = __shfl(site, u, 64);
          const int px = t < 0 ? 0 : off[p].x, py = t < 0 ? 0 : off[p].y;
          int prev = -1;
          for (;;) {  // the site's particles by index
            int best = 0x7FFFFFFF;
            for (int i = lane; i < n; i += 64)
              if (off[i].x == px && off[i].y == py && idx[i] > prev && idx[i] != q.z) best = min(best, idx[i]);
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) best = min(best, __shfl_xor(best, o, 64));
            if (best == 0x7FFFFFFF) break;
            if (lane == 0) row[at] = best;
            ++at;
            prev = best;
          }
        }
        for (int u = at + lane; u < dmax; u += 64) row[u] = -1;
      }
      if (lane == 0) deg[q.z] = row_len;
      done = true;
    }
    if (!done && lane == 0) {  // for the general kernel
      w.dflag[s] = 1;
      w.hdr->nvflag = 1u;
    }
    __builtin_amdgcn_wave_barrier();
  }
}

// Strip geometry: blocks of vor_half cells around the query's cell, about 256
// queries a strip, or 128 where 256 would leave CUs with one strip or none
// (60,000 particles: 106 -> 83 us, 120,000: 114 -> 91, 250,000: 173 and 174,
// 2^20: 476 -> 549), one column where offsets take 32 bits (4096 particles: 78
// -> 62 us); halo within the staging buffer; false where a block would
// meet itself around the box (the general kernel takes such grids).
bool vor_cfg(const DevWs& w, TileCfg& t) {
  const double rho = static_cast<double>(w.n) / static_cast<double>(w.C);
  if (rho < 1e-6) return false;
  const int half = vor_half(static_cast<float>(rho));
  const int hx = max(1, min(half, 15)), hy = max(1, min(half + 1, 15));  // (rows: sparser than the mean)
  int tw = hx >= 3 && (static_cast<long long>(2 + 2 * hx) << w.log2_w) < 32768 ? 2 : 1;
  while (tw < 16 && 2 * tw <= w.G && 256.0 / (tw * rho) > 1.1 * (kTwRows - 2 * hy)) tw *= 2;
  if (half > 15 || tw + 2 * hx > w.G || 2 * hy + 1 > w.G) return false;
  const int W = tw + 2 * hx;
  const bool narrow = (static_cast<long long>(W) << w.log2_w) < 32768 &&
                      (static_cast<long long>(2 * hy + 1) << w.log2_w) < 32768;
  const int room = narrow ? kStripPts : kStripPts / 2;
  const double queries = w.n < 200000 ? 128.0 : 256.0;
  int th = max(1, min(static_cast<int>(ceil(queries / (tw * rho))), w.G));
  while (th > 1 && (th + 2 * hy > kStripRows || (th + 2 * hy) * W * rho > 0.75 * room)) --th;
  if (th + 2 * hy > kStripRows) return false;
  t = TileCfg{tw, th, hx, hy, w.G / tw, (w.G + th - 1) / th, 2 * hy + 1, narrow ? 0 : 1};
  return true;
}

}  // namespace

bool vor_strips_fit(const DevWs& w) {
  TileCfg tc;
  return vor_cfg(w, tc);
}

bool launch_vor_strips(const DevWs& w, int dmax, int32_t* ring, int32_t* deg, const uint8_t* stale,
                       const uint32_t* gate, hipStream_t s) {
  TileCfg tc;
  if (!vor_cfg(w, tc)) return false;
  const dim3 grid(tc.ntx * tc.nty), block(kBlock);
  if (stale && tc.wide)
    hipLaunchKernelGGL((k_vor_strip<true, true>), grid, block, 0, s, w, tc, dmax, ring, deg, stale, gate);
  else if (stale)
    hipLaunchKernelGGL((k_vor_strip<true, false>), grid, block, 0, s, w, tc, dmax, ring, deg, stale, gate);
  else if (tc.wide)
    hipLaunchKernelGGL((k_vor_strip<false, true>), grid, block, 0, s, w, tc, dmax, ring, deg, stale, gate);
  else
    hipLaunchKernelGGL((k_vor_strip<false, false>), grid, block, 0, s, w, tc, dmax, ring, deg, stale, gate);
  const int nb = (w.n + kVwWaves - 1) / kVwWaves;
  hipLaunchKernelGGL(k_vor_wave, dim3(min(nb, kVwGridMax)), dim3(64 * kVwWaves), 0, s, w, dmax, ring, deg);
  return true;
}

}  // namespace nm
