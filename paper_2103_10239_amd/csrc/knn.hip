// knn.hip -- topological neighbour lists (Sec. III: each particle interacts
// with its k nearest neighbours), the fused step kernel and the field-of-view
// lists.
//
// The kernels work on strips of cells staged in LDS (see "Strips" below);
// queries that a strip cannot serve from LDS run the global-memory paths
// here, one lane per query, queries taken in cell order so that a
// wavefront's queries are spatial neighbours and read the same cached cells.
//
// Fast path: the lane scans a B x B block of cells around the query (a few
// contiguous slot ranges) and pushes every candidate through a branch-free
// insertion network of 32-bit keys (v_med3_u32), which keeps the k+1 best.
// The result is certified exact when the k+1 best have distinct distances
// and the k-th distance is strictly inside the block (no point outside can
// be as near); this holds for the great majority of queries.
//
// Exact path (the rest): rings of cells outward from the home cell, skipping
// cells whose nearest point is already farther than the current k-th
// neighbour, with 64-bit (d^2, index) keys.  It stops after ring r once the
// k-th squared distance is strictly below the squared distance to the edge of
// the scanned block: an equal distance in the next ring could still carry a
// smaller index, so equality does not stop the walk.
//
// The fused kernel then evaluates Eq. (2) and Eq. (1) for the query from the
// fp64 unit vectors stored beside the cell-ordered copy (the neighbours'
// entries sit in the cells just scanned, so they are cache hits) and writes
// the list, the new position and the new heading at the particle's index.
#include "fov.h"
#include "strip.h"

namespace nm {

namespace {

// Exact ring search (64-bit keys), filling `slot` with the k nearest.
template <int KMAX>
__device__ __forceinline__ bool knn_exact(const DevWs& w, int s, int qx, int qy, int k, int total,
                                          int (&slot)[KMAX]) {
  const int sh = 32 - w.log2_box;
  const int cw = 1 << w.log2_w;
  const int gm = w.G - 1;
  const QueryGeom q(qx, qy, w);
  TopK<KMAX, true> top;
  top.init(k);
  for (int r = 0; r <= q.rmax; ++r) {
    for_ring(r, q.lo, q.hi, [&](int dx, int dy) {
      const long long gx = axis_gap(dx, q.ox, cw, sh);
      const long long gy = axis_gap(dy, q.oy, cw, sh);
      if (gx * gx + gy * gy > key_bound_d2(top.worst())) return;
      const int64_t c = static_cast<int64_t>((q.hy + dy) & gm) * w.G + ((q.hx + dx) & gm);
      const int beg = w.start[c];
      const int end = min(w.start[c + 1], total);
      for (int t = beg; t < end; ++t) {
        if (t == s) continue;
        const int4 e = w.sorted[t];
        const int ex = wrap_axis(e.x - qx, sh);
        const int ey = wrap_axis(e.y - qy, sh);
        const long long d2 = static_cast<long long>(ex) * ex + static_cast<long long>(ey) * ey;
        const unsigned long long kk = pack_key(d2, e.z);
        if (kk < top.worst()) top.push(kk, t);
      }
    });
    if (key_bound_d2(top.worst()) < q.ring_bound(r, cw)) break;
  }
#pragma unroll
  for (int t = 0; t < KMAX; ++t) slot[t] = top.slot[t];
  return top.worst() != ~0ull;
}

// Ascending order of eight keys and what they carry (Batcher's network of 19).
__device__ __forceinline__ bool sort_eight(unsigned long long (&key)[8], int (&v)[8]) {
  constexpr int net[19][2] = {{0, 1}, {2, 3}, {4, 5}, {6, 7}, {0, 2}, {1, 3}, {4, 6}, {5, 7}, {1, 2}, {5, 6},
                              {0, 4}, {1, 5}, {2, 6}, {3, 7}, {2, 4}, {3, 5}, {1, 2}, {3, 4}, {5, 6}};
  bool moved = false;
#pragma unroll
  for (int c = 0; c < 19; ++c) {
    const int i = net[c][0], j = net[c][1];
    const bool swap = key[j] < key[i];
    const unsigned long long ki = key[i], kj = key[j];
    const int vi = v[i], vj = v[j];
    key[i] = swap ? kj : ki;
    key[j] = swap ? ki : kj;
    v[i] = swap ? vj : vi;
    v[j] = swap ? vi : vj;
    moved = moved || swap;
  }
  return moved;
}

// Reorder neighbours whose distance fields tie (or lie too close for their
// order to be certain) by the exact (d^2, index): bit t of `link` says that
// entries t and t + 1 do.  exact(v) gives an entry's 64-bit key; entries before
// `first` are unused.  Windows of eight entries, four apart, that hold a link
// are sorted by their exact keys, which agree with the fields' order everywhere
// else; runs of up to five lie within one window, longer ones take passes until
// nothing moves.  (All entries sorted at once held 64 registers at k = 32; each
// linked pair compared in turn, passes until nothing moved, is a chain of LDS
// reads: lists on a square lattice of 1024, k = 24 48 us, 25 so; k = 8 16 and 11;
// of 2^16, k = 24 74 and 49.  The longest lists keep those pairs: the windows
// take registers that their network needs, lists of 31 on 200,003 clustered
// particles 461 and 471 us, and gain lattices 3%.)
template <int KMAX, class Exact>
__device__ __forceinline__ void sort_linked(uint32_t link, int first, int (&v)[KMAX], Exact&& exact) {
  if constexpr (KMAX > 24) {
    bool again = true;
    while (again) {
      again = false;
#pragma unroll
      for (int t = 0; t + 1 < KMAX; ++t) {
        if ((link >> t) & 1u) {
          if (exact(v[t + 1]) < exact(v[t])) {
            const int s = v[t];
            v[t] = v[t + 1];
            v[t + 1] = s;
            again = true;
          }
        }
      }
    }
    return;
  }
  const bool longer = (link & (link >> 1) & (link >> 2) & (link >> 3) & (link >> 4)) != 0u;
  auto key_of = [&](int t) { return t >= KMAX ? ~0ull : (t < first ? 0ull : exact(v[t < KMAX ? t : 0])); };
  bool again = true;
  while (again) {
    again = false;
    unsigned long long key[8] = {};
    bool carried = false;  // key[4 .. 7] are those of this window's first four
#pragma unroll
    for (int t0 = 0; t0 == 0 || t0 + 4 < KMAX; t0 += 4) {
      if ((link >> t0) & 0x7Fu) {
        int w[8];
#pragma unroll
        for (int u = 0; u < 4; ++u) key[u] = key[u + 4];
        if (!carried) {
#pragma unroll
          for (int u = 0; u < 4; ++u) key[u] = key_of(t0 + u);
        }
#pragma unroll
        for (int u = 4; u < 8; ++u) key[u] = key_of(t0 + u);
#pragma unroll
        for (int u = 0; u < 8; ++u) w[u] = v[t0 + u < KMAX ? t0 + u : KMAX - 1];
        const bool moved = sort_eight(key, w);
        again = again || (longer && moved);
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (t0 + u < KMAX) v[t0 + u < KMAX ? t0 + u : 0] = w[u];
        carried = true;
      } else {
        carried = false;
      }
    }
  }
}

// Sorted batches for long lists.  An insertion costs an operation per list
// entry; a batch of kNetBatch costs 114 operations to sort and 106 (22 entries)
// or 182 (34) to merge, that is 14 and 19 a candidate.  Insertions and batches:
// lists of 20 on 2^22 clustered particles 2.00 and 1.83 ms, of 31 on 200,003
// clustered 456-480 and 399 us.  Lists under kNetBatch entries gain nothing.
constexpr int kNetBatch = 16;

__device__ __forceinline__ void cmp_swap(uint32_t& a, uint32_t& b) {
  const uint32_t lo = min(a, b);
  b = max(a, b);
  a = lo;
}

// Batcher's odd-even merge of the sorted halves of v[LO .. LO + N), stride R.
template <int LO, int N, int R, int M>
__device__ __forceinline__ void oe_merge(uint32_t (&v)[M]) {
  if constexpr (2 * R < N) {
    oe_merge<LO, N, 2 * R>(v);
    oe_merge<LO + R, N, 2 * R>(v);
#pragma unroll
    for (int i = LO + R; i + R < LO + N; i += 2 * R) cmp_swap(v[i], v[i + R]);
  } else {
    cmp_swap(v[LO], v[LO + R]);
  }
}

// Ascending order: groups of four by median-of-three insertion, then merges.
__device__ __forceinline__ void sort_batch(uint32_t (&v)[kNetBatch]) {
#pragma unroll
  for (int g = 0; g < kNetBatch; g += 4) {
    const uint32_t a = v[g], b = v[g + 1], c = v[g + 2], e = v[g + 3];
    const uint32_t lo = min(min(a, b), c), mid = umed3(a, b, c), hi = max(max(a, b), c);
    v[g] = min(lo, e);
    v[g + 1] = umed3(lo, mid, e);
    v[g + 2] = umed3(mid, hi, e);
    v[g + 3] = max(hi, e);
  }
  oe_merge<0, 8, 1>(v);
  oe_merge<8, 8, 1>(v);
  oe_merge<0, 16, 1>(v);
}

// The KS smallest of an ascending list (whose first entries may be the
// sentinel 0) and an ascending batch, ascending: the minimum of the list's
// last entries and the reversed batch leaves them as a bitonic sequence,
// sorted as the last KS places of a power of two whose first are zeros.
template <int KS>
__device__ __forceinline__ void merge_batch(uint32_t (&kl)[KS], const uint32_t (&v)[kNetBatch]) {
  static_assert(KS >= kNetBatch, "the batch meets the list's last entries");
#pragma unroll
  for (int j = 0; j < kNetBatch; ++j) kl[KS - 1 - j] = min(kl[KS - 1 - j], v[j]);
  constexpr int P = KS > 32 ? 64 : (KS > 16 ? 32 : 16);
  constexpr int off = P - KS;
#pragma unroll
  for (int st = P / 2; st > 0; st >>= 1) {
#pragma unroll
    for (int i = off; i < P; ++i)
      if ((i & st) == 0 && i + st < P) cmp_swap(kl[i - off], kl[i + st - off]);
  }
}

// Candidates per round of a staged block's loop.
template <int KS>
constexpr int kRound = KS >= kNetBatch ? kNetBatch : kUnroll;

// Exact squared distance from a staged query (packed position pq, or x and
// y) to staged particle i: the 16-bit differences are exact inside a block.
template <bool kWide>
__device__ __forceinline__ long long staged_d2(const int* lpos, int i, int pq, int pqy) {
  if (kWide) {
    const int2 c = reinterpret_cast<const int2*>(lpos)[i];
    const long long dx = c.x - pq, dy = c.y - pqy;
    return dx * dx + dy * dy;
  }
  return rel_d2(lpos[i], pq);
}

// Block side for a query: its edge should sit `reach` mean k-th-neighbour
// radii away, r_k^2 = k / (pi rho), with the density rho estimated from the
// occupancy of the (up to) 3 x 3 cells around the home cell.
__device__ __forceinline__ int pick_block(const DevWs& w, const FastCfg& f, int k, int qx, int qy) {
  if (f.bfix > 0) return f.bfix;
  const int G = w.G;
  const int hx = qx >> w.log2_w, hy = qy >> w.log2_w;
  const int c0 = max(hx - 1, 0), c1 = min(hx + 1, G - 1);
  int n9 = 0;
#pragma unroll
  for (int dy = -1; dy <= 1; ++dy) {
    const int64_t row = static_cast<int64_t>((hy + dy) & (G - 1)) * G;
    n9 += w.start[row + c1 + 1] - w.start[row + c0];
  }
  const float cells = 3.0f * static_cast<float>(c1 - c0 + 1);
  const float rk = sqrtf(static_cast<float>(k) * cells / (3.14159265f * fmaxf(static_cast<float>(n9), 0.5f)));
  const int B = static_cast<int>(ceilf(2.0f * f.reach * rk)) + 1;
  return min(max(B, 3), f.bmax);
}

// Fast block search; true (and `slot` filled) only when certified exact.
template <int KMAX>
__device__ __forceinline__ bool knn_fast(const DevWs& w, const FastCfg& f, int s, int qx, int qy,
                                         int k, int total, int (&slot)[KMAX]) {
  constexpr int KT = KMAX + 1;
  if (f.bmax == 0) return false;
  int B = pick_block(w, f, k, qx, qy);
  for (int attempt = 0; attempt < 2; ++attempt) {
    const QBlock b = make_qblock(w, qx, qy, B);
    uint32_t key[KT];
#pragma unroll
    for (int t = 0; t < KT; ++t) key[t] = (t < KT - (k + 1)) ? 0u : kKey32Inf;
    const uint32_t clampd = static_cast<uint32_t>(b.bound);
    const int sh = b.sh;
    const bool ok = walk_block(w, b, s, qx, qy, total,
                               [&](int x, int y, int qxi, int qyi, int tag, bool valid) {
                                 const int dx = x - qxi, dy = y - qyi;
                                 const uint32_t d2 = static_cast<uint32_t>(__mul24(dx, dx)) +
                                                     static_cast<uint32_t>(__mul24(dy, dy));
                                 const uint32_t kk = ((min(d2, clampd) >> sh) << 13) | static_cast<uint32_t>(tag);
                                 net_insert(key, valid ? kk : kKey32Inf);
                               });
    if (!ok) return false;
    const uint32_t kth = key[KT - 2];
    const long long dmax = (static_cast<long long>(key32_d(kth) + 1) << sh) - 1;
    if (kth == kKey32Inf || dmax >= b.bound) {  // the k-th may lie outside: widen once
      if (attempt == 0 && B < f.bmax) {
        B = min(B + 2, f.bmax);
        continue;
      }
      return false;
    }
    // The k nearest form the set {d^2 >> sh <= that of the k-th} only if the
    // (k+1)-th has a larger distance field; otherwise the exact search decides.
    if (key32_d(kth) >= key32_d(key[KT - 1])) return false;
    uint32_t link = 0u;
#pragma unroll
    for (int t = 0; t < KT - 2; ++t)
      if (t >= KT - (k + 1) && key32_d(key[t]) == key32_d(key[t + 1])) link |= 1u << t;
    bool mapped = true;
#pragma unroll
    for (int t = 0; t < KMAX; ++t) {
      if (t >= KMAX - k) {
        slot[t] = tag_slot(w, b, key[t] & 0x1FFFu, qx, qy);
        mapped = mapped && static_cast<uint32_t>(slot[t]) < static_cast<uint32_t>(total);
      }
    }
    if (mapped && link != 0u) {
      const int shx = 32 - w.log2_box;
      sort_linked<KMAX>(link, KMAX - k, slot, [&](int q) {
        const int4 e = w.sorted[q];
        const long long ex = wrap_axis(e.x - qx, shx), ey = wrap_axis(e.y - qy, shx);
        return pack_key(ex * ex + ey * ey, e.z);
      });
    }
    return mapped;
  }
  return false;
}

__device__ __forceinline__ bool ws_ready(const DevWs& w) {
  const WsHeader* h = w.hdr;
  return h->built == kBuilt && h->n == w.n && h->box == w.box && h->cell_w == w.cell_w;
}

// Outputs of one query from the slots of its k neighbours: the list row (and
// squared distances), and for the fused step Eq. (2) and Eq. (1).
template <int KMAX, bool kAlign>
__device__ __forceinline__ void finish_query(const DevWs& w, int s, const int4& q, const int (&slot)[KMAX],
                                             int k, int32_t* __restrict__ nbr,
                                             long long* __restrict__ d2out, const AlignArgs& a) {
  int32_t* row = nbr + static_cast<int64_t>(q.z) * k;
  const int sh = 32 - w.log2_box;
  double sx = 0.0, sy = 0.0;
  int rv[KMAX];
#pragma unroll
  for (int t = 0; t < KMAX; ++t) {
    rv[t] = 0;
    if (t >= KMAX - k) {
      const int4 e = w.sorted[slot[t]];
      if constexpr (kRowVec<KMAX>)
        rv[t] = e.z;
      else
        row[t - (KMAX - k)] = e.z;
      if (!kAlign && d2out) {
        const int ex = wrap_axis(e.x - q.x, sh), ey = wrap_axis(e.y - q.y, sh);
        d2out[static_cast<int64_t>(q.z) * k + t - (KMAX - k)] =
            static_cast<long long>(ex) * ex + static_cast<long long>(ey) * ey;
      }
      if (kAlign) {
        const double2 u = w.cs[2 * slot[t]];
        sx += u.x;
        sy += u.y;
      }
    }
  }
  if constexpr (kRowVec<KMAX>) store_row<KMAX>(row, rv, k);
  if (!kAlign) return;

  // Eq. (2): average of the neighbours' unit vectors (plus the particle's own),
  // vectorial noise, normalisation (only the direction is kept).
  const double2 own = w.cs[2 * s];
  const double2 xi = w.cs[2 * s + 1];
  if (a.include_self) {
    sx += own.x;
    sy += own.y;
  }
  const double m = static_cast<double>(k + (a.include_self ? 1 : 0));
  const double ax = sx / m, ay = sy / m;
  const float th = heading_update(ax, ay, xi.x, xi.y, noise_angle(static_cast<uint32_t>(q.w)), a.eta,
                                  a.theta + q.z, a.variant);

  // Eq. (1): move with the heading at time t (or the new one), rounded to the grid.
  int ddx, ddy;
  move_step(a.v0, own.x, own.y, th, a.variant, ddx, ddy);
  const int mask = w.box - 1;
  a.x_out[q.z] = (q.x + ddx) & mask;
  a.y_out[q.z] = (q.y + ddy) & mask;
  a.theta_out[q.z] = th;
}

// ---------------------------------------------------------------------------
// Strips.  A workgroup owns a strip of tw x th cells (tw = 1 to 16 columns,
// about 256 queries) and stages the halo of W = tw + 2 hx columns by
// R = th + 2 hy rows into LDS: the LDS offset of each halo row, and every
// particle's position in the strip's periodic image relative to the halo
// corner, with its particle index.  A query's block is all W columns of
// Bq consecutive halo rows around its own, so its candidates are one
// contiguous LDS range, read several at a time.  Positions are a packed pair
// of 16-bit offsets whose differences are taken in 16-bit wrap-around
// arithmetic (exact: every block spans under 2^15 units), so that a squared
// distance is one packed subtract and one 16-bit dot product; where a block
// spans more (sparse systems) they are int32 pairs with 64-bit distances.
// A strip whose halo holds more particles than fit searches global memory,
// or, in the sub-strip kernel, runs as sub-strips staged in turn.
// Uncertified queries are finished at the end of the strip by the exact
// search.
// ---------------------------------------------------------------------------
constexpr int kDeferCap = 128;    // uncertified queries listed in LDS per strip
constexpr double kReachX = 1.25;  // strip half width, in mean k-th-neighbour radii
// A system stepped by itself with few strips waits for its last uncertified
// query (9 of 25 us at 1000 particles), so its blocks cover more of the k-th
// distance's tail where 1.25 radii round to a halo just as wide: n = 1000 and
// 4000 at k = 7 26 -> 16 us, 16,000 27 -> 24; at 50,000 the candidates cost
// more (32 -> 34 us), at 10^6 173 -> 185.
constexpr double kReachXSmall = 1.5;
constexpr float kReachSmall = 1.6f;
constexpr int kSmallN = 1 << 14;
constexpr double kStripQ = 256.0;  // queries per strip
// Share of the staging buffer that a sparse ("wide") strip of a served job
// fills at the mean density.  No tuner picks those grids, and a strip over the
// buffer searches global memory, which the whole iteration waits for: 16 jobs
// of 1024 to 131,072 particles, half clustered, up to 20 steps: 4.6-15.9 ms at
// 0.75 (by the clusters), 4.0-4.6 at 0.5, all uniform 3.54 and 3.52, all
// clustered 9.6 and 5.5.  (Tuned batches keep 0.75: 512 systems of up to 8192
// particles 303 us against 329.)
constexpr double kFillServed = 0.5;
constexpr double kReachY = 1.2;   // halo height over the expected block height


// Block height for a staged query: fixed, or such that the block edge sits
// `reach` mean k-th-neighbour radii away, the density taken from the three
// halo rows around the query's (3 W cells).
__device__ __forceinline__ int strip_block_rows(const FastCfg& f, const int* rbase, int W, int cy,
                                                int k) {
  if (f.bfix > 0) return f.bfix;
  const int n3 = rbase[cy + 2] - rbase[cy - 1];
  const float rk = sqrtf(static_cast<float>(k) * static_cast<float>(3 * W) /
                         (3.14159265f * fmaxf(static_cast<float>(n3), 0.5f)));
  return max(static_cast<int>(ceilf(2.0f * f.reach * rk)) + 1, 1);
}

// Geometry of a query's block in a strip: halo rows [r0, r0 + Bq), all W
// columns; squared distance to the nearest point outside it, and the shift
// that fits that bound in the distance field of a 32-bit key.
struct StripBlock {
  int r0;
  long long bound;
  int sh;
};

__device__ __forceinline__ StripBlock strip_block(int rx, int oy, int cy, int Bq, int W, int lw) {
  const int cw = 1 << lw;
  const int half = Bq >> 1;
  const int lo = (Bq & 1) ? -half : -half + (oy >= (cw >> 1) ? 1 : 0);
  StripBlock b;
  b.r0 = cy + lo;
  const int gl = rx + 1, gr = W * cw - rx;
  const int gd = oy - lo * cw + 1, gu = (lo + Bq) * cw - oy;
  const long long m = min(min(gl, gr), min(gd, gu));
  b.bound = m * m;
  const int bits = 64 - __clzll(b.bound);
  b.sh = bits > kDBits ? bits - kDBits : 0;
  return b;
}

// Candidate filters of the strip search: every staged particle, or those
// inside the query's field of view.
struct NoFilter {
  static constexpr bool kActive = false;
};

struct FovFilter {
  static constexpr bool kActive = true;
  FovHeading h;
  __device__ bool visible_short(int dx, int dy, int d2) const { return fov_visible_short(dx, dy, d2, h); }
  __device__ bool visible(long long dx, long long dy) const { return fov_visible(dx, dy, h); }
};

// Certified search of one staged query over LDS.  self: the query's LDS
// index; (pq, pqy): its relative position (narrow: packed pair in pq);
// (rx, oy): its x offset from the halo corner and y offset in its cell; cy:
// its halo row.  True with `lds` filled (LDS indices of the k nearest that
// pass `filt`, in order) when they are certified.  Anything outside the
// block is farther than its edge whatever the filter, so the certificate
// holds for the filtered lists too.
template <int KMAX, bool kWide, class Filter>
__device__ __forceinline__ bool strip_search(const DevWs& w, const TileCfg& tc, const int* rbase,
                                             const int* lpos, const int* lidx, int W, int self,
                                             int pq, int pqy, int rx, int oy, int cy, int k, int Bq,
                                             const Filter& filt, int (&lds)[KMAX]) {
  constexpr int KT = KMAX + 1;
  // Without a filter the query's own key (distance 0, its LDS index) goes
  // through the network with the others, one more list entry, and is taken
  // out at the end: cheaper than masking every candidate against it.
  constexpr bool kWithSelf = !Filter::kActive;
  constexpr int KS = kWithSelf ? KT + 1 : KT;
  constexpr int RN = kRound<KS>;
  const int2* lpos2 = reinterpret_cast<const int2*>(lpos);
  if (Bq > tc.bmax) return false;
  for (int attempt = 0; attempt < 2; ++attempt) {
    const StripBlock b = strip_block(rx, oy, cy, Bq, W, w.log2_w);
    uint32_t kl[KS];
#pragma unroll
    for (int t = 0; t < KS; ++t) kl[t] = (t < KS - (k + 1 + (kWithSelf ? 1 : 0))) ? 0u : kKey32Inf;
    const int sh = b.sh;
    // wide strips: the bound rounded down to fp32 (so that a clamped field
    // stays below 2^19) and the exact scale 2^-sh
    float boundf = static_cast<float>(b.bound);
    if (static_cast<long long>(boundf) > b.bound) boundf = nextafterf(boundf, 0.0f);
    const float scale = ldexpf(1.0f, -sh);
    const int a = rbase[b.r0], e = rbase[b.r0 + Bq];
    // One round: candidates i .. i + RN - 1.  Only the last round of a
    // block (tail) can pass its end; it masks what lies beyond.
    auto round = [&](int i, bool tail) {
      uint32_t kk[RN];
      if (kWide) {
        // fp32 squared distances: the offsets are exact (below 2^24), the
        // square and the sum round twice (relative error below 2^-23, an
        // eighth of a distance-field unit), so every field is within one of
        // the exact one; the certificate below widens its margins to match.
        int2 pc[RN];
#pragma unroll
        for (int u = 0; u < RN; ++u) pc[u] = lpos2[i + u];  // (buffer padded by RN)
#pragma unroll
        for (int u = 0; u < RN; ++u) {
          const int dxi = pc[u].x - pq, dyi = pc[u].y - pqy;
          const float dx = static_cast<float>(dxi), dy = static_cast<float>(dyi);
          const float d2 = fmaf(dy, dy, dx * dx);
          kk[u] = (static_cast<uint32_t>(fminf(d2, boundf) * scale) << 13) | static_cast<uint32_t>(i + u);
          if constexpr (Filter::kActive)
            if (!filt.visible(static_cast<long long>(dxi), static_cast<long long>(dyi))) kk[u] = kKey32Inf;
        }
      } else {
        int pc[RN];
#pragma unroll
        for (int u = 0; u < RN; ++u) pc[u] = lpos[i + u];  // (buffer padded by RN)
        const uint32_t clampd = static_cast<uint32_t>(b.bound);
#pragma unroll
        for (int u = 0; u < RN; ++u) {
          const uint32_t d2 = rel_d2_u(pc[u], pq);
          kk[u] = ((min(d2, clampd) >> sh) << 13) | static_cast<uint32_t>(i + u);
          if constexpr (Filter::kActive) {
            const short2v dd = __builtin_bit_cast(short2v, pc[u]) - __builtin_bit_cast(short2v, pq);
            if (!filt.visible_short(dd[0], dd[1], static_cast<int>(d2))) kk[u] = kKey32Inf;
          }
        }
      }
#pragma unroll
      for (int u = 0; u < RN; ++u)
        if (!kWithSelf && i + u == self) kk[u] = kKey32Inf;
      if (tail) {
#pragma unroll
        for (int u = 0; u < RN; ++u)
          if (i + u >= e) kk[u] = kKey32Inf;
      }
      if constexpr (RN == kNetBatch) {
        sort_batch(kk);
        merge_batch(kl, kk);
      } else {
#pragma unroll
        for (int u = 0; u < RN; ++u) net_insert(kl, kk[u]);
      }
    };
    if constexpr (RN == kNetBatch) {  // (one copy of the networks: 431 -> 399 us for lists of 31)
      for (int i = a; i < e; i += RN) round(i, i + RN > e);
    } else {
      const int full = a + ((e - a) & ~(RN - 1));
      for (int i = a; i < full; i += RN) round(i, false);
      if (full < e) round(full, true);
    }
    uint32_t key[KT];
    if constexpr (kWithSelf) {
      // the first entry not below the query's own key is that key (it is in
      // the list unless more than KS duplicates of lower index precede it)
      const uint32_t selfkey = static_cast<uint32_t>(self);
#pragma unroll
      for (int t = 0; t < KT; ++t) key[t] = kl[t] < selfkey ? kl[t] : kl[t + 1];
    } else {
#pragma unroll
      for (int t = 0; t < KT; ++t) key[t] = kl[t];
    }
    // Certificate (fields exact, or within one of exact on wide strips: M = 2):
    // the k-th lies inside the block, the (k+1)-th is strictly farther than
    // the k-th, and fields closer than M + 1 inside the k are re-sorted by
    // the exact (d^2, index).
    constexpr uint32_t M = kWide ? 2u : 0u;
    const uint32_t kth = key[KT - 2];
    const long long dmax = (static_cast<long long>(key32_d(kth) + 1 + M / 2) << sh) - 1;
    if (kth == kKey32Inf || dmax >= b.bound) {
      if (attempt == 0 && Bq + 2 <= tc.bmax) {
        Bq += 2;
        continue;
      }
      return false;
    }
    if (key32_d(kth) + M >= key32_d(key[KT - 1])) return false;
    uint32_t link = 0u;
#pragma unroll
    for (int t = 0; t < KT - 2; ++t)
      if (t >= KT - (k + 1) && key32_d(key[t + 1]) - key32_d(key[t]) <= M) link |= 1u << t;
#pragma unroll
    for (int t = 0; t < KMAX; ++t)
      if (t >= KMAX - k) lds[t] = static_cast<int>(key[t] & 0x1FFFu);
    if (link != 0u)
      sort_linked<KMAX>(link, KMAX - k, lds, [&](int i) { return pack_key(staged_d2<kWide>(lpos, i, pq, pqy), lidx[i]); });
    return true;
  }
  return false;
}

// Cell (dx, dy) number q of ring r (q < 8r; the single cell of ring 0),
// walking the perimeter from (-r, -r) as the exact lane search does.
__device__ __forceinline__ void ring_cell(int r, int q, int& dx, int& dy) {
  if (r == 0) {
    dx = dy = 0;
    return;
  }
  const int side = q / (2 * r), p = q - side * 2 * r;
  dx = side == 0 ? -r + p : (side == 1 ? r : (side == 2 ? r - p : -r));
  dy = side == 0 ? -r : (side == 1 ? -r + p : (side == 2 ? r : r - p));
}

// LDS of a wavefront's search: where its list's entries change places.
struct WaveScratch {
  unsigned long long key[32];
  int slot[32];
};

__device__ __forceinline__ unsigned long long read_lane64(unsigned long long v, int l) {
  const uint32_t lo = __builtin_amdgcn_readlane(static_cast<int>(v), l);
  const uint32_t hi = __builtin_amdgcn_readlane(static_cast<int>(v >> 32), l);
  return static_cast<unsigned long long>(hi) << 32 | lo;
}

// One deferred query searched by a whole wavefront.  The 49 cells of rings 0
// to 3 are looked up at once, one a lane, and searched from the inside: first
// the rings that hold k others, then the rest; each further ring 64 cells at
// a time.  Cells whose nearest point is farther than the current k-th
// neighbour are skipped, and the candidates of the others flattened across
// the lanes, 64 per round.  Same stop rule as the lane search; candidates
// that fail `filt` are skipped.  Lane t < k returns the t-th nearest's slot in
// `mslot`.
//
// A search is a chain of memory round trips and of merges.  The list is spread
// over the wave (lane t holds the t-th nearest so far), and a round's
// candidates below the current k-th take their places at once: each is
// broadcast and counted against every lane's entry and candidate, which
// gives the new ranks, and the entries move through LDS (scratch).
template <class Filter = NoFilter>
__device__ __forceinline__ bool knn_wave(const DevWs& w, WaveScratch* scratch, int s, const int4& q, int k,
                                         int total, int& mslot, const Filter& filt = Filter{}) {
  const int lane = threadIdx.x & 63;
  const int sh = 32 - w.log2_box;
  const int cw = 1 << w.log2_w;
  const int gm = w.G - 1;
  const QueryGeom g(q.x, q.y, w);
  unsigned long long mine = ~0ull;
  mslot = -1;
  int have = 0;                       // entries of the list
  unsigned long long worst = ~0ull;  // the k-th entry (uniform)
  // this lane's cell: slots [beg, beg + cnt) and the squared distance to it
  int beg = 0, cnt = 0;
  long long gap2 = 0;
  auto cell = [&](int r, int p) {
    int dx, dy;
    ring_cell(r, p, dx, dy);
    beg = cnt = 0;
    if (dx >= g.lo && dx <= g.hi && dy >= g.lo && dy <= g.hi) {
      const long long gx = axis_gap(dx, g.ox, cw, sh), gy = axis_gap(dy, g.oy, cw, sh);
      gap2 = gx * gx + gy * gy;
      if (gap2 <= key_bound_d2(worst)) {
        const int64_t c = static_cast<int64_t>((g.hy + dy) & gm) * w.G + ((g.hx + dx) & gm);
        beg = w.start[c];
        cnt = max(min(w.start[c + 1], total) - beg, 0);
      }
    }
  };
  auto prefix = [&]() {  // candidates of the lanes up to this one
    int incl = cnt;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int t = __shfl_up(incl, off, 64);
      if (lane >= off) incl += t;
    }
    return incl;
  };
  auto search = [&](int incl, int ntot) {  // the first ntot of the lanes' candidates
    const int excl = incl - cnt;
    for (int j0 = 0; j0 < ntot; j0 += 64) {
      const int j = j0 + lane;
      int lo = 0;  // owner lane of flattened candidate j: last lane with excl <= j
#pragma unroll
      for (int step = 32; step > 0; step >>= 1) {
        const int probe = lo + step;
        const int e = __shfl(excl, probe < 64 ? probe : 63, 64);
        if (probe < 64 && e <= j) lo = probe;
      }
      const int ob = __shfl(beg, lo, 64), oe = __shfl(excl, lo, 64);
      unsigned long long kk = ~0ull;
      const int t = ob + (j - oe);
      if (j < ntot && t != s) {
        const int4 e = w.sorted[t];
        const int ex = wrap_axis(e.x - q.x, sh), ey = wrap_axis(e.y - q.y, sh);
        bool keep = true;
        if constexpr (Filter::kActive) keep = filt.visible(ex, ey);
        if (keep) kk = pack_key(static_cast<long long>(ex) * ex + static_cast<long long>(ey) * ey, e.z);
      }
      const unsigned long long better = __ballot(kk < worst);
      if (better == 0ull) continue;
      int rc = 0, rl = lane;  // new ranks of this lane's candidate and entry (keys are distinct)
      for (unsigned long long m = better; m != 0ull; m &= m - 1) {
        const int l = __ffsll(static_cast<long long>(m)) - 1;
        const unsigned long long bk = read_lane64(kk, l);
        const bool before = bk < mine;
        rc += bk < kk ? 1 : 0;
        rl += before ? 1 : 0;
        const int above = have - __popcll(__ballot(lane < have && before));  // entries before the candidate
        rc += lane == l ? above : 0;
      }
      if (lane < have && rl < k) {
        scratch->key[rl] = mine;
        scratch->slot[rl] = mslot;
      }
      if (kk < worst && rc < k) {
        scratch->key[rc] = kk;
        scratch->slot[rc] = t;
      }
      have = min(k, have + static_cast<int>(__popcll(better)));
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      if (lane < have) {
        mine = scratch->key[lane];
        mslot = scratch->slot[lane];
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      if (have == k) worst = read_lane64(mine, k - 1);
    }
  };
  {  // rings 0 to 3, whose lanes begin at 0, 1, 9 and 25
    const int r = lane == 0 ? 0 : (lane < 9 ? 1 : (lane < 25 ? 2 : 3));
    if (lane < 49) cell(r, lane - (2 * r - 1) * (2 * r - 1) * (r > 0 ? 1 : 0));
    const int incl = prefix();
    int inner = 3;  // the rings that hold k others than the query
    for (int t = 2; t >= 0; --t)
      if (__builtin_amdgcn_readlane(incl, (2 * t + 1) * (2 * t + 1) - 1) > k) inner = t;
    search(incl, __builtin_amdgcn_readlane(incl, (2 * inner + 1) * (2 * inner + 1) - 1));
    if (key_bound_d2(worst) < g.ring_bound(inner, cw)) return true;
    if (inner < 3) {
      if (r <= inner || gap2 > key_bound_d2(worst)) cnt = 0;
      const int rest = prefix();
      search(rest, __builtin_amdgcn_readlane(rest, 63));
      if (key_bound_d2(worst) < g.ring_bound(3, cw)) return true;
    }
  }
  for (int r = 4; r <= g.rmax; ++r) {
    const int ncell = 8 * r;
    for (int c0 = 0; c0 < ncell; c0 += 64) {
      beg = cnt = 0;
      if (c0 + lane < ncell) cell(r, c0 + lane);
      const int incl = prefix();
      search(incl, __builtin_amdgcn_readlane(incl, 63));
    }
    if (key_bound_d2(worst) < g.ring_bound(r, cw)) break;
  }
  return worst != ~0ull;
}

// One uncertified query searched by its own lane (exact ring search).
template <int KMAX, bool kAlign>
__device__ __forceinline__ void exact_lane(const DevWs& w, int s, int k, int total,
                                           int32_t* __restrict__ nbr, long long* __restrict__ d2out,
                                           const AlignArgs& a) {
  const int4 q = w.sorted[s];
  int slot[KMAX];
  if (knn_exact<KMAX>(w, s, q.x, q.y, k, total, slot))
    finish_query<KMAX, kAlign>(w, s, q, slot, k, nbr, d2out, a);
  else
    set_err(w.hdr, NM_E_RANGE);  // fewer than k other particles were binned
}

// Cells of strip `tile`: columns [x0, x0 + tw), rows [y0, y0 + ty).
struct StripBox {
  int x0, y0, ty;
};

__device__ __forceinline__ StripBox strip_box(const DevWs& w, const TileCfg& tc, int tile) {
  StripBox b;
  const int tyi = tile / tc.ntx, txi = tile - tyi * tc.ntx;
  b.x0 = txi * tc.tw;
  b.y0 = tyi * tc.th;
  b.ty = min(tc.th, w.G - b.y0);
  return b;
}


// What a strip does when its halo holds more particles than LDS.  The two
// are compiled as separate kernels: the sub-strip loop costs the common
// (fitting) strips some 10% when it shares their kernel, so the choice is a
// grid parameter that the autotuner weighs like the cell width.
enum StripMode {
  kOverflowGlobal = 0,  // search its queries in global memory (fast block search)
  kOverflowSplit = 1,   // run it as sub-strips of whole rows, each staged in turn
  kFieldOfView = 2,     // field-of-view lists (a.theta, a.cone); such a strip's
                        // queries and the uncertified ones take the exact search
};

template <int KMAX, bool kAlign, int kMode, int kPts>
__device__ __forceinline__ void knn_tile_body(const DevWs& w, const FastCfg& f, const TileCfg& tc,
                                              int k, int32_t* __restrict__ nbr,
                                              long long* __restrict__ d2out, const AlignArgs& a,
                                              int tile) {
  // packed 16-bit pairs, or int32 pairs (wide); padded so that a round of
  // candidates read past a block's last one stays inside the buffer
  __shared__ int2 lpos_store[kPts / 2 + kRound<KMAX + 1>];
  __shared__ int lidx[kPts];               // particle index of each staged particle
  __shared__ int s_rbase[kStripRows + 1];  // LDS offset of each halo row
  __shared__ int s_ga0[kStripRows];        // first slot of the row's first piece
  __shared__ int s_n0[kStripRows];         // particles in the row's first piece
  __shared__ int s_ga1[kStripRows];        // first slot of its second piece (x wrap)
  __shared__ int s_qoff[kStripRows + 1];   // query prefix over the strip's rows
  __shared__ int s_tself[kStripRows];      // LDS index of each strip row's first query
  __shared__ int s_wsum[kBlock / 64];
  __shared__ int s_defer;
  __shared__ int s_dq[kDeferCap];  // slots of the strip's uncertified queries
  __shared__ uint8_t s_rowid[kPts];        // halo row of each staged particle
  __shared__ uint16_t s_qmap[kPts];        // LDS index of each of the strip's queries
  __shared__ int s_sub[kStripRows + 1];    // sub-strip rows (kOverflowSplit)
  __shared__ int s_nsub;
  int* lpos = reinterpret_cast<int*>(lpos_store);
  if (!ws_ready(w)) {
    if (tile == 0 && threadIdx.x == 0) set_err(w.hdr, NM_E_INVAL);
    return;
  }
  const StripBox tb = strip_box(w, tc, tile);
  const int G = w.G, lw = w.log2_w;
  const int total = min(w.start[w.C], w.n);
  const int tw = tc.tw, hy = tc.hy;
  // The sub-strip kernel (chosen for clustered systems) takes each strip's
  // halo width from the strip's own density, never wider than the grid's:
  // dense strips get narrower blocks (6% less time at k = 20 on the clustered
  // state; the extra pass over the strip's rows costs the default kernel 7%
  // on uniform systems, which keep the grid's width).
  int hx = tc.hx;
  if (kMode == kOverflowSplit && hx > 1) {
    int q = 0;
    if (static_cast<int>(threadIdx.x) < tb.ty) {
      const int64_t prow = static_cast<int64_t>(tb.y0 + threadIdx.x) * G;
      q = max(min(w.start[prow + tb.x0 + tw], total) - w.start[prow + tb.x0], 0);
    }
    int nqs;
    (void)block_exclusive_scan(q, s_wsum, &nqs);
    if (nqs > 0) {
      const float rho = static_cast<float>(nqs) / static_cast<float>(tw * tb.ty);
      int hs = static_cast<int>(
          ceilf(static_cast<float>(kReachX) * sqrtf(static_cast<float>(k) / (3.14159265f * rho))));
      if (f.bfix > 0) hs = max(hs, f.bfix / 2);
      hx = max(1, min(hs, tc.hx));
    }
  }
  const int W = tw + 2 * hx;
  const int uL = tb.x0 - hx;
  const int lane = threadIdx.x & 63;
  const int ox0 = uL << lw;  // halo corner x (strip image)
  // the (sub-)strip being run: first row, rows, halo corner y (strip image)
  int y0_cur = tb.y0, ty_cur = tb.ty, oy0 = (tb.y0 - hy) << lw;
  const bool wide = tc.wide != 0;

  StripGeo geo{tb.x0, tb.y0, tb.ty, tw, hx, hy, wide};
  // built at each use: an aggregate of LDS addresses shared by the lambdas
  // below would become a constant global, which the target cannot express
  auto strip_lds = [&]() {
    return StripLds{lpos_store, lidx, s_rbase, s_ga0, s_n0, s_ga1, s_qoff, s_tself, s_wsum, s_rowid, s_qmap};
  };
  if (threadIdx.x == 0) s_defer = 0;

  auto defer = [&](int slot_s) {
    const int pos = atomicAdd(&s_defer, 1);
    if (pos < kDeferCap)
      s_dq[pos] = slot_s;
    else
      w.dflag[slot_s] = 1;  // overflow of the list: found again below by its flag
  };
  auto row_of = [&](int qi) {  // strip row of query qi
    int r = 0;
#pragma unroll
    for (int step = kRowStep; step > 0; step >>= 1)
      if (r + step < ty_cur && s_qoff[r + step] <= qi) r += step;
    return r;
  };
  // One staged query (LDS index self, halo row cy): the certified search over
  // LDS, then its outputs with the neighbours' indices from LDS and their
  // unit vectors gathered by slot; otherwise it is deferred to the exact search.
  auto staged_query = [&](int self, int cy) {
    int rx, oy, pq, pqy;
    if (wide) {
      const int2 p2 = lpos_store[self];
      pq = p2.x;
      pqy = p2.y;
      rx = p2.x;
      oy = p2.y & ((1 << lw) - 1);
    } else {
      pq = lpos[self];
      pqy = 0;
      rx = pq & 0xFFFF;
      oy = (pq >> 16) & ((1 << lw) - 1);
    }
    const int Bq = strip_block_rows(f, s_rbase, W, cy, k);
    int nb[KMAX];
    bool ok;
    if constexpr (kMode == kFieldOfView) {
      const FovFilter filt{fov_heading(a.theta[lidx[self]], a.cone)};
      ok = wide ? strip_search<KMAX, true>(w, tc, s_rbase, lpos, lidx, W, self, pq, pqy, rx, oy, cy, k, Bq,
                                           filt, nb)
                : strip_search<KMAX, false>(w, tc, s_rbase, lpos, lidx, W, self, pq, pqy, rx, oy, cy, k, Bq,
                                            filt, nb);
    } else {
      ok = wide ? strip_search<KMAX, true>(w, tc, s_rbase, lpos, lidx, W, self, pq, pqy, rx, oy, cy, k, Bq,
                                           NoFilter{}, nb)
                : strip_search<KMAX, false>(w, tc, s_rbase, lpos, lidx, W, self, pq, pqy, rx, oy, cy, k, Bq,
                                            NoFilter{}, nb);
    }
    const int s = strip_slot(strip_lds(), self);
    if (!ok) {
      defer(s);
      return;
    }
    const int qi = lidx[self];
    int32_t* row = nbr + static_cast<int64_t>(qi) * k;
    double sx = 0.0, sy = 0.0;
    int rv[KMAX];
#pragma unroll
    for (int t = 0; t < KMAX; ++t) {
      rv[t] = 0;
      if (t >= KMAX - k) {
        const int i = nb[t];
        if constexpr (kRowVec<KMAX>)
          rv[t] = lidx[i];
        else
          row[t - (KMAX - k)] = lidx[i];
        if (!kAlign && d2out)
          d2out[static_cast<int64_t>(qi) * k + t - (KMAX - k)] =
              wide ? staged_d2<true>(lpos, i, pq, pqy) : staged_d2<false>(lpos, i, pq, pqy);
        if (kAlign) {
          const double2 u = w.cs[2 * strip_slot(strip_lds(), i)];
          sx += u.x;
          sy += u.y;
        }
      }
    }
    if constexpr (kRowVec<KMAX>) store_row<KMAX>(row, rv, k);
    if (kAlign) {
      // Eq. (2) and Eq. (1) as in finish_query, the position from the staged copy
      const double2 own = w.cs[2 * s];
      const double2 xi = w.cs[2 * s + 1];
      if (a.include_self) {
        sx += own.x;
        sy += own.y;
      }
      const double m = static_cast<double>(k + (a.include_self ? 1 : 0));
      const double phi = (a.variant & NM_NOISE_SCALAR) ? noise_angle(static_cast<uint32_t>(w.sorted[s].w)) : 0.0;
      const float th = heading_update(sx / m, sy / m, xi.x, xi.y, phi, a.eta, a.theta + qi, a.variant);
      int ddx, ddy;
      move_step(a.v0, own.x, own.y, th, a.variant, ddx, ddy);
      const int qx = rx + ox0, qy = ((cy << lw) | oy) + oy0;  // strip-image coordinates
      const int mask = w.box - 1;
      a.x_out[qi] = (qx + ddx) & mask;
      a.y_out[qi] = (qy + ddy) & mask;
      a.theta_out[qi] = th;
    }
  };

  // The queries of the (sub-)strip just staged, or searched in global memory
  // (the fast block search) when its halo could not be staged.
  auto global_query = [&](int qi, int r) {
    int slot[KMAX];
    const int s = w.start[static_cast<int64_t>(y0_cur + r) * G + tb.x0] + (qi - s_qoff[r]);
    const int4 q = w.sorted[s];
    if constexpr (kMode == kFieldOfView) {
      fov_exact<KMAX>(w, s, q, fov_heading(a.theta[q.z], a.cone), k, total, nbr);
      return;
    }
    if (knn_fast<KMAX>(w, f, s, q.x, q.y, k, total, slot))
      finish_query<KMAX, kAlign>(w, s, q, slot, k, nbr, d2out, a);
    else
      defer(s);
  };
  if constexpr (kMode != kOverflowSplit) {
    int npts, nq;
    // Staging is a chain of global reads and barriers: its waves issue first
    // (wave priority), so that other strips' searches fill the gaps.
    __builtin_amdgcn_s_setprio(3);
    const bool staged = strip_stage<true, kPts>(w, geo, strip_lds(), total, npts, nq);
    __builtin_amdgcn_s_setprio(0);
    if (nq == 0) return;
    for (int qi = threadIdx.x; qi < nq; qi += kBlock) {
      if (staged) {
        const int self = s_qmap[qi];
        staged_query(self, s_rowid[self]);
      } else {
        global_query(qi, row_of(qi));
      }
    }
  } else {
    // The strip is staged whole when its halo fits LDS.  Otherwise it runs
    // as sub-strips of whole rows, each as tall as fits, staged one after
    // another; a row whose own halo does not fit (bit 30) is searched in
    // global memory.  One staging site keeps a single copy of that code.
    int next = -1, nsub = 0;  // the sub-strip to stage next (-1: none planned)
    for (;;) {
      int np_cur, nq_cur;
      __builtin_amdgcn_s_setprio(3);
      const bool st = strip_stage<true, kPts>(w, geo, strip_lds(), total, np_cur, nq_cur);
      __builtin_amdgcn_s_setprio(0);
      nq_cur = __builtin_amdgcn_readfirstlane(nq_cur);  // block-uniform: keep it scalar
      bool plan = false;
      if (next < 0) {
        if (nq_cur == 0) return;
        plan = !st && hx > 0;
      }
      if (plan) {
        const int cap = wide ? kPts / 2 : kPts;
        if (threadIdx.x == 0) {
          int ns = 0;
          for (int r0 = 0; r0 < tb.ty;) {
            const bool fits = s_rbase[r0 + 2 * hy + 1] - s_rbase[r0] <= cap;
            int r1 = r0 + 1;
            if (fits)
              while (r1 < tb.ty && s_rbase[r1 + 2 * hy + 1] - s_rbase[r0] <= cap) ++r1;
            s_sub[ns++] = r0 | (fits ? 0 : 1 << 30);
            r0 = r1;
          }
          s_sub[ns] = tb.ty;
          s_nsub = ns;
        }
        __syncthreads();
        nsub = __builtin_amdgcn_readfirstlane(s_nsub);
        next = 0;
      } else {
        if (st) {
          for (int qi = threadIdx.x; qi < nq_cur; qi += kBlock) {
            const int self = s_qmap[qi];
            staged_query(self, s_rowid[self]);
          }
        } else {
          for (int qi = threadIdx.x; qi < nq_cur; qi += kBlock) global_query(qi, row_of(qi));
        }
        if (next < 0 || next >= nsub) break;
        __syncthreads();  // this sub-strip's queries are done with LDS
      }
      const int e = __builtin_amdgcn_readfirstlane(s_sub[next]);
      const int r0 = e & 0xFFFF, r1 = __builtin_amdgcn_readfirstlane(s_sub[next + 1]) & 0xFFFF;
      y0_cur = tb.y0 + r0;
      ty_cur = r1 - r0;
      oy0 = (y0_cur - hy) << lw;
      geo = StripGeo{tb.x0, y0_cur, ty_cur, tw, (e >> 30) == 0 ? hx : 0, hy, wide};
      ++next;
    }
  }
  __syncthreads();
  const int nd = s_defer;
  if (nd == 0) return;

  // The strip's uncertified queries, by the exact ring search.  With many
  // (over 48), each lane searches its own; otherwise a wavefront searches one
  // at a time, so that a single long search is not one lane's serial chain
  // (on the clustered 2^22 state, from 16 to 48: 3-8% faster; wavefronts for
  // any number: 2.03-2.07 -> 2.10 ms at k = 20).
  const int nl = min(nd, kDeferCap);
  if (kMode == kFieldOfView && nl > 16) {
    for (int j = threadIdx.x; j < nl; j += kBlock) {
      const int sq = s_dq[j];
      const int4 q = w.sorted[sq];
      fov_exact<KMAX>(w, sq, q, fov_heading(a.theta[q.z], a.cone), k, total, nbr);
    }
  } else if (kMode != kFieldOfView && nl > 48) {
    for (int j = threadIdx.x; j < nl; j += kBlock) exact_lane<KMAX, kAlign>(w, s_dq[j], k, total, nbr, d2out, a);
  } else {
    // Lane c of a wavefront keeps the list of its c-th query, and the lanes
    // finish their queries together.
    static_assert(kDeferCap <= 64 * (kBlock / 64), "a lane for each of a wavefront's queries");
    WaveScratch* scratch = reinterpret_cast<WaveScratch*>(lpos_store) + (threadIdx.x >> 6);  // (staging is over)
    int slot[KMAX];
#pragma unroll
    for (int t = 0; t < KMAX; ++t) slot[t] = 0;
    int mine = -1;
    bool found = false;
    int c = 0;
    for (int j = threadIdx.x >> 6; j < nl; j += kBlock / 64, ++c) {
      const int sq = __builtin_amdgcn_readfirstlane(s_dq[j]);
      const int4 q = w.sorted[sq];
      int ms;
      bool ok;
      if constexpr (kMode == kFieldOfView)
        ok = knn_wave(w, scratch, sq, q, k, total, ms, FovFilter{fov_heading(a.theta[q.z], a.cone)});
      else
        ok = knn_wave(w, scratch, sq, q, k, total, ms);
#pragma unroll
      for (int t = 0; t < KMAX; ++t) {
        const int v = __builtin_amdgcn_readlane(ms, max(t - (KMAX - k), 0));
        if (lane == c) slot[t] = v;
      }
      if (lane == c) {
        mine = sq;
        found = ok;
      }
    }
    if (mine >= 0) {
      if (found)
        finish_query<KMAX, kAlign>(w, mine, w.sorted[mine], slot, k, nbr, d2out, a);
      else
        set_err(w.hdr, NM_E_RANGE);  // fewer than k other (visible) particles were binned
    }
  }
  if (nd > kDeferCap) {
    for (int r = 0; r < tb.ty; ++r) {
      const int64_t row = static_cast<int64_t>(tb.y0 + r) * G;
      const int a0 = w.start[row + tb.x0];
      const int a1 = max(min(w.start[row + tb.x0 + tw], total), a0);
      for (int sq = a0 + threadIdx.x; sq < a1; sq += kBlock) {
        if (w.dflag[sq]) {
          w.dflag[sq] = 0;
          if constexpr (kMode == kFieldOfView) {
            const int4 q = w.sorted[sq];
            fov_exact<KMAX>(w, sq, q, fov_heading(a.theta[q.z], a.cone), k, total, nbr);
          } else {
            exact_lane<KMAX, kAlign>(w, sq, k, total, nbr, d2out, a);
          }
        }
      }
    }
  }
}

// Waves per SIMD asked of the compiler: five for the short lists (96 VGPRs,
// which the LDS of a strip also allows), four for KMAX 12-20, whose insertion
// networks would otherwise take the kernel to three or two, three for KMAX 24
// and 32 (k = 31, 200,000 uniform particles: 250 us at the one wave it would
// take, 184 at two, 165 at three, 204 at four); the spills these limits add
// lie outside the search loops and cost less than the waves they gain.  The
// batched kernel, which also holds its system's descriptors, spills at five
// and takes four.
template <int KMAX>
constexpr int kKnnWaves = (KMAX >= 12 && KMAX <= 20) ? 4 : (KMAX <= 8 ? 5 : 3);
template <int KMAX>
constexpr int kBatchKnnWaves = KMAX <= 8 ? 4 : kKnnWaves<KMAX>;

// Particles a strip stages: what the LDS of a CU holds for that many strips
// (kStripPts for all: 2^22 clustered particles, k = 20 2035 -> 2016 us; 200,003
// clustered, k = 31 484 -> 471; 512 batched systems of 256 to 65,536, k = 7
// 1.60-1.74 -> 1.54 ms; 16 served jobs 4.5 -> 4.3 ms).
constexpr int strip_pts(int waves) { return waves >= 5 ? kStripPts : (waves == 4 ? 3328 : 4480); }
template <int KMAX>
constexpr int kKnnPts = strip_pts(kKnnWaves<KMAX>);
template <int KMAX>
constexpr int kBatchKnnPts = strip_pts(kBatchKnnWaves<KMAX>);

template <int KMAX, bool kAlign, int kMode>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(kKnnWaves<KMAX>))) void k_knn(DevWs w, FastCfg f, TileCfg tc, int k,
                                                int32_t* __restrict__ nbr,
                                                long long* __restrict__ d2out, AlignArgs a) {
  knn_tile_body<KMAX, kAlign, kMode, kKnnPts<KMAX>>(w, f, tc, k, nbr, d2out, a, xcd_run(blockIdx.x, gridDim.x));
}

// Field-of-view lists over the same strips (a.theta: headings, a.cone: the
// cone's cos(half angle) * 4096).
// Two waves per SIMD asked of the compiler for the long lists, three for up to 12,
// four for up to 4: left to itself it takes 256 registers, and one wave, for lists
// of 20 (2^20 uniform particles, every direction: 290 us at two waves, 402 at one,
// 358 at three, which spill; half plane 640 and 1070).
template <int KMAX>
constexpr int kFovWaves = KMAX <= 4 ? 4 : (KMAX <= 12 ? 3 : 2);

template <int KMAX>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(kFovWaves<KMAX>))) void k_knn_fov_strip(DevWs w, FastCfg f, TileCfg tc, int k,
                                                          int32_t* __restrict__ nbr, AlignArgs a) {
  knn_tile_body<KMAX, false, kFieldOfView, kStripPts>(w, f, tc, k, nbr, nullptr, a, xcd_run(blockIdx.x, gridDim.x));
}

template <int KMAX>
hipError_t launch_fov_strip_t(const DevWs& w, const FastCfg& f, const TileCfg& tc, int k, int32_t* nbr,
                              const AlignArgs& a, hipStream_t s) {
  const int ntiles = tc.ntx * tc.nty;
  hipLaunchKernelGGL(k_knn_fov_strip<KMAX>, dim3(ntiles), dim3(kBlock), 0, s, w, f, tc, k, nbr, a);
  return hipGetLastError();
}

// Batched k-NN + alignment.  Items of the tile stage are (system, tile); the
// hardware item order is remapped so that each XCD walks one contiguous run of
// items (consecutive tiles of a system share halo cells in that XCD's L2).
template <class T>
__device__ __forceinline__ T* uniform_ptr(T* p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v >> 32));
  return reinterpret_cast<T*>((static_cast<uint64_t>(hi) << 32) | lo);
}

__device__ __forceinline__ AlignArgs uniform_load_align(const BatchSys* d) {
  const int p = __builtin_amdgcn_readfirstlane(d->parity);
  AlignArgs a;
  a.v0 = __builtin_amdgcn_readfirstlane(d->v0);
  a.eta = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, d->eta)));
  a.include_self = __builtin_amdgcn_readfirstlane(d->include_self);
  a.variant = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(d->variant)));
  a.theta = uniform_ptr(d->th[p]);
  a.x_out = uniform_ptr(d->x[1 - p]);
  a.y_out = uniform_ptr(d->y[1 - p]);
  a.theta_out = uniform_ptr(d->th[1 - p]);
  return a;
}

template <int KMAX, int kMode>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(kBatchKnnWaves<KMAX>))) void k_bb_knn(BatchRef b, int k) {
  constexpr int kSt = kMode == kOverflowSplit ? kStKnnSplit : kStKnn;
  const int ni = b.begin[kSt + 1] - b.begin[kSt];
  const int per = gridDim.x & ~7;  // whole rounds of the 8 XCDs
  for (int hw = blockIdx.x; hw < ni; hw += gridDim.x) {
    // Neighbouring strips on one XCD (one L2): over all items when each
    // workgroup takes one, else within the rounds that every workgroup of a
    // multiple-of-8 grid takes.
    int it = hw;
    const int round_base = (hw / gridDim.x) * gridDim.x;
    if (static_cast<int>(gridDim.x) == ni)
      it = xcd_tile(hw, ni);
    else if (per == static_cast<int>(gridDim.x) && round_base + per <= ni)
      it = round_base + xcd_tile(hw - round_base, per);
    const BatchSys* g = b.sys + b.items[b.begin[kSt] + it];
    const DevWs w = uniform_load(&g->w);
    const FastCfg f = uniform_load(&g->f);
    const TileCfg tc = uniform_load(&g->tc);
    const AlignArgs a = uniform_load_align(g);
    const int li = it - __builtin_amdgcn_readfirstlane(g->base[kSt]);
    knn_tile_body<KMAX, true, kMode, kBatchKnnPts<KMAX>>(w, f, tc, k, uniform_ptr(g->nbr), nullptr, a, li);
    __syncthreads();
  }
}

// Queries per strip of a system run by itself: fewer where 256 would leave
// CUs without a strip (n = 16,000, k = 7: 32 us with 256, 26 with 64; 50,000,
// k = 12: 41 and 32; 130,000: 49 with 256, 41 with 128, 58 with 64; larger
// systems fill the device and stage less with 256, and up to some 4000
// particles the few strips take one strip's latency whatever their size).
// Uniform systems alone would do with larger strips from half of these limits on
// (lists of 85,000, k = 12: 30 us with 64, 24 with 128 or 256; of 210,000, k = 1:
// 16.5 with 128, 14.4 with 256), but smaller strips overflow the staging buffer
// less often where particles cluster: 99,999, k = 20, 82 us with 64, 167 with 128;
// 262,143, k = 7, 72 with 128, 189 with 256.
inline double solo_strip_queries(int n) {
  return n < 4096 ? kStripQ : (n < 100000 ? 64.0 : (n < 262144 ? 128.0 : kStripQ));
}

// Strip geometry.  Block rows: up to the expected block height plus one
// widening step (hy); block width: all W = tw + 2 hx columns, hx the expected
// half width.  The strip height aims at about 256 queries; the halo must fit
// the staging buffer and the row table, W <= G (a block never meets itself
// around the box), and narrow strips keep every block under 2^15 units.
// `reach_x`: half width in mean k-th-neighbour radii; `pts`: particles staged.
TileCfg tile_cfg_impl(const DevWs& w, const FastCfg& f, int k, bool narrow_strips, int pts, StripUse use = kUseBatch,
                      double reach_x = kReachX) {
  const bool solo = use == kUseSolo || use == kUseSoloFov;
  const double queries = solo ? solo_strip_queries(w.n) : kStripQ;
  TileCfg t{1, 1, 0, 0, w.G, w.G, 0, 0};
  const double rho = static_cast<double>(w.n) / static_cast<double>(w.C);  // particles per cell
  const double rr = rho > 1e-12 ? rho : 1e-12;
  const double rk = sqrt(static_cast<double>(k) / (3.141592653589793 * rr));
  const int bmax_all = max(f.bmax, f.bmax_w);
  auto plain = [&]() {  // no staging: one row of queries per strip, global search
    t.tw = 1;
    t.hx = t.hy = 0;
    t.th = max(1, min(w.G, static_cast<int>(lround(256.0 / (rr * 1.0)))));
    t.th = min(t.th, kStripRows);
    t.ntx = w.G;
    t.nty = (w.G + t.th - 1) / t.th;
    t.bmax = 0;
    return t;
  };
  if (bmax_all < 1) return plain();
  // Halo rows: for a block kReachY times the expected height (queries in
  // sparse rows choose taller blocks; 1 with `narrow_strips`), plus one
  // widening step.
  const double ry = narrow_strips ? 1.0 : kReachY;
  const int bq = f.bfix > 0 ? f.bfix : static_cast<int>(ceil(2.0 * ry * f.reach * rk)) + 1;
  int hy = min((bq + 2) / 2, 15);  // (hy <= 15: block heights fit 5 bits)
  // The block width is fixed per strip, so it covers the tail of the k-th
  // neighbour distance, not only its mean.
  int hx = min(max(1, static_cast<int>(ceil(reach_x * rk))), 15);
  if (f.bfix > 0) hx = min(max(hx, f.bfix / 2), 15);
  // Strip width: wider as the halo widens (hx 2: two columns, hx >= 3: four,
  // or two for lists of up to 8, where a block's candidates (its rows times
  // W = tw + 2 hx) cost more than the extra staging: 93 -> 88 us for k = 7 at
  // w = 1024, block 6, while k = 12 loses 4%), and at least the narrowest
  // power of two whose strips reach ~256 queries within the row limit.  Wider
  // strips stage each particle fewer times and leave fewer queries near a
  // strip's side.  `narrow_strips` (two columns
  // only from hx 3, and halo rows for the expected block height) serves the
  // sub-strip kernel, whose larger halos overflow LDS more often, and the
  // field-of-view lists, whose blocks span every column of the strip.
  int tw = narrow_strips ? (hx >= 3 ? 2 : 1) : (hx >= 3 ? (k <= 8 ? 2 : 4) : (hx >= 2 ? 2 : 1));
  auto widen = [&]() {
    while (tw < 16 && 2 * tw <= w.G && kStripQ / (tw * rr) > 1.1 * (kTwRows - 2 * hy)) tw *= 2;
  };
  widen();
  // Sparse systems, whose blocks would span 2^15 units, take one column where
  // the rows allow: their buffer holds half the particles, and one column may
  // bring the block under the limit (k = 31, 200,000 particles: 626 -> 490 us
  // clustered, 170 -> 163 uniform; k = 12, 50,000: 41 -> 33).  Not the wide halos of
  // field-of-view lists on systems that fill the device anyway, which one column
  // stages for few queries (300,000 uniform particles, k = 20, 43 degrees: 1.28 ms
  // with one column, 1.01 with two; 20,000, k = 16: 139 us and 161).
  const bool one = use == kUseSolo || (use == kUseSoloFov && (hx <= 4 || w.n < 65536));
  if (one && (static_cast<long long>(tw + 2 * hx) << w.log2_w) >= 32768) {
    tw = 1;
    widen();
  }
  while (hx > 1 && tw + 2 * hx > w.G) --hx;
  while (hy > 1 && 2 * hy + 1 > w.G) --hy;
  if (tw + 2 * hx > w.G || 2 * hy + 1 > w.G) return plain();
  const int W = tw + 2 * hx;
  const bool narrow = (static_cast<long long>(W) << w.log2_w) < 32768 &&
                      (static_cast<long long>(2 * hy + 1) << w.log2_w) < 32768;
  const int cap = narrow ? pts : pts / 2;
  int th = static_cast<int>(ceil(queries / (tw * rr)));
  th = max(1, min(th, w.G));
  const double fill = use == kUseServed && !narrow ? kFillServed : 0.75;
  while (th > 1 && (th + 2 * hy > kStripRows || (th + 2 * hy) * W * rho > fill * cap)) --th;
  if (th + 2 * hy > kStripRows) return plain();
  t.tw = tw;
  t.th = th;
  t.hx = hx;
  t.hy = hy;
  t.ntx = w.G / tw;
  t.nty = (w.G + th - 1) / th;
  t.bmax = min(2 * hy + 1, w.G);
  t.wide = narrow ? 0 : 1;
  return t;
}

// Register list sizes compiled; a request for k uses the smallest KMAX >= k.
template <class F>
hipError_t dispatch_k(int k, F&& f) {
  if (k <= 1) return f(std::integral_constant<int, 1>{});
  if (k <= 2) return f(std::integral_constant<int, 2>{});
  if (k <= 4) return f(std::integral_constant<int, 4>{});
  if (k <= 6) return f(std::integral_constant<int, 6>{});
  if (k <= 7) return f(std::integral_constant<int, 7>{});
  if (k <= 8) return f(std::integral_constant<int, 8>{});
  if (k <= 12) return f(std::integral_constant<int, 12>{});
  if (k <= 16) return f(std::integral_constant<int, 16>{});
  if (k <= 20) return f(std::integral_constant<int, 20>{});
  if (k <= 24) return f(std::integral_constant<int, 24>{});
  return f(std::integral_constant<int, 32>{});
}

int solo_pts(int k) {
  int pts = kStripPts;
  (void)dispatch_k(k, [&](auto km) {
    pts = kKnnPts<decltype(km)::value>;
    return hipSuccess;
  });
  return pts;
}

// The strips of a system run by itself (f.reach too may grow for small ones).
TileCfg solo_cfg(const DevWs& w, FastCfg& f, int k) {
  const TileCfg t = tile_cfg_impl(w, f, k, f.split != 0, solo_pts(k), kUseSolo);
  // (the sub-strip kernel takes each strip's halo from its own density)
  if (w.n > kSmallN || f.bfix > 0 || f.split != 0 || t.hx == 0) return t;
  const TileCfg wider = tile_cfg_impl(w, f, k, f.split != 0, solo_pts(k), kUseSolo, kReachXSmall);
  if (wider.hx <= t.hx) return t;
  f.reach = kReachSmall;
  return tile_cfg_impl(w, f, k, f.split != 0, solo_pts(k), kUseSolo, kReachXSmall);
}

template <int KMAX, bool kAlign>
hipError_t launch_t(const DevWs& w, FastCfg f, int k, int32_t* nbr, long long* d2,
                    const AlignArgs& a, hipStream_t s) {
  const TileCfg tc = solo_cfg(w, f, k);
  const int ntiles = tc.ntx * tc.nty;
  if (f.split && tc.hx > 0)
    hipLaunchKernelGGL((k_knn<KMAX, kAlign, kOverflowSplit>), dim3(ntiles), dim3(kBlock), 0, s, w, f,
                       tc, k, nbr, d2, a);
  else
    hipLaunchKernelGGL((k_knn<KMAX, kAlign, kOverflowGlobal>), dim3(ntiles), dim3(kBlock), 0, s, w, f,
                       tc, k, nbr, d2, a);
  return hipGetLastError();
}

}  // namespace

TileCfg tile_cfg(const DevWs& w, const FastCfg& f, int k, StripUse use) {
  int pts = kStripPts;
  (void)dispatch_k(k, [&](auto km) {
    pts = kBatchKnnPts<decltype(km)::value>;
    return hipSuccess;
  });
  return tile_cfg_impl(w, f, k, f.split != 0, pts, use);
}

// The tiles of the plain-strip systems, then those of the sub-strip systems
// (each launch only when it has items).
hipError_t launch_batch_knn(const BatchRef& b, int k, hipStream_t s) {
  const int nt = b.begin[kStKnn + 1] - b.begin[kStKnn];
  const int ns = b.begin[kStKnnSplit + 1] - b.begin[kStKnnSplit];
  return dispatch_k(k, [&](auto km) {
    constexpr int KM = decltype(km)::value;
    if (nt > 0) {
      const int g = nt;  // one workgroup per strip: uneven strips balance over the CUs
      hipLaunchKernelGGL((k_bb_knn<KM, kOverflowGlobal>), dim3(g), dim3(kBlock), 0, s, b, k);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    if (ns > 0) {
      const int g = ns;
      hipLaunchKernelGGL((k_bb_knn<KM, kOverflowSplit>), dim3(g), dim3(kBlock), 0, s, b, k);
      return hipGetLastError();
    }
    return hipSuccess;
  });
}

// Fast-path limits for a grid: block sides up to the largest B whose
// offsets keep 32-bit squared distances exact ((B / 2 + 1) w < 2^15) and whose
// block cannot meet itself around the box (B + 2 <= G).  `block` > 0 fixes the
// side, 0 picks it per query, < 0 disables the fast path; NM_BLOCK_SUBSTRIPS
// in it selects the sub-strip kernel.
FastCfg fast_cfg(const DevWs& w, int k, int block) {
  (void)k;
  FastCfg f{0, 0, 1.25f, 0, 0};
  if (block < 0) return f;
  f.split = (block & NM_BLOCK_SUBSTRIPS) ? 1 : 0;
  block &= ~NM_BLOCK_SUBSTRIPS;
  int bw = kMaxB;  // any span (64-bit distances): the block must not meet itself
  while (bw >= 3 && bw + 2 > w.G) --bw;
  if (bw < 3) return f;
  int bmax = bw;
  while (bmax >= 3 && (static_cast<long long>((bmax >> 1) + 1) << w.log2_w) >= 32768) --bmax;
  if (bmax < 3) bmax = 0;
  if (block > 0) {
    if (block > bw) return f;
    f.bfix = block;
    if (block > bmax) bmax = 0;
  }
  f.bmax = bmax;
  f.bmax_w = bw;
  return f;
}

// A cone of half angle alpha sees the fraction alpha / pi of the directions,
// so its k nearest visible lie about as far as the k / (alpha / pi) nearest
// of all: the strips and blocks are sized for that many.
hipError_t launch_knn_fov_strips(const DevWs& w, int block, const float* theta, int k, int c,
                                 int32_t* nbr, hipStream_t s) {
  FastCfg f = fast_cfg(w, k, block);
  const double alpha = acos(fmax(-1.0, fmin(1.0, c / 4096.0)));
  const double frac = fmax(alpha / 3.141592653589793, 1.0 / 64.0);
  const int ks = static_cast<int>(ceil(k / frac));
  const TileCfg tc = tile_cfg_impl(w, f, ks, true, kStripPts, kUseSoloFov);
  f.reach = static_cast<float>(f.reach * sqrt(static_cast<double>(ks) / k));
  AlignArgs a{};
  a.theta = theta;
  a.cone = c;
  if (k <= 4) return launch_fov_strip_t<4>(w, f, tc, k, nbr, a, s);
  if (k <= 8) return launch_fov_strip_t<8>(w, f, tc, k, nbr, a, s);
  if (k <= 12) return launch_fov_strip_t<12>(w, f, tc, k, nbr, a, s);
  if (k <= 16) return launch_fov_strip_t<16>(w, f, tc, k, nbr, a, s);
  if (k <= 24) return launch_fov_strip_t<24>(w, f, tc, k, nbr, a, s);
  return launch_fov_strip_t<32>(w, f, tc, k, nbr, a, s);
}

void knn_layout(const DevWs& w, int k, int block, int32_t out[10]) {
  FastCfg f = fast_cfg(w, k, block);
  const TileCfg tc = solo_cfg(w, f, k);
  // kernel: 0 = one row of queries per strip, searched in global memory;
  // 1 = staged strips (default kernel); 2 = staged strips, sub-strip kernel
  out[0] = tc.hx == 0 ? 0 : (f.split ? 2 : 1);
  out[1] = tc.tw;
  out[2] = tc.th;
  out[3] = tc.hx;
  out[4] = tc.hy;
  out[5] = f.bfix;
  out[6] = tc.wide;
  out[7] = tc.bmax;
  out[8] = tc.ntx;
  out[9] = tc.nty;
}

hipError_t launch_knn(const DevWs& w, int k, int block, int32_t* nbr, long long* d2, hipStream_t s) {
  const FastCfg f = fast_cfg(w, k, block);
  AlignArgs a{};
  return dispatch_k(k, [&](auto km) { return launch_t<decltype(km)::value, false>(w, f, k, nbr, d2, a, s); });
}

hipError_t launch_knn_align(const DevWs& w, int k, int block, const nm_params* p, const float* theta,
                            int32_t* nbr, int32_t* x_out, int32_t* y_out, float* theta_out,
                            hipStream_t s) {
  const FastCfg f = fast_cfg(w, k, block);
  AlignArgs a{p->v0, p->eta, p->include_self, p->variant, theta, x_out, y_out, theta_out};
  return dispatch_k(k, [&](auto km) {
    return launch_t<decltype(km)::value, true>(w, f, k, nbr, nullptr, a, s);
  });
}

}  // namespace nm
