// vmodel.hip -- the Voronoi model of dense tissue (Sec. V): each particle
// owns its Voronoi cell, the energy is Eq. (3),
//   E = sum_i K_A (A_i - A_0)^2 + K_P (P_i - P_0)^2,
// and the force on particle i is -dE/dr_i (Eq. 9), by the chain rule through
// the cell vertices (Eqs. 10-19); the vertex forces -dE/dh of the vertex
// model (Eqs. 5-8) are a by-product.
//
// Input: the Voronoi rows of nm_voronoi (counter-clockwise; consecutive
// entries a_t, a_{t+1} of row i are the Delaunay triangle (i, a_t, a_{t+1})
// whose circumcentre h_t is vertex t of cell i).  Eight lanes per particle, lane
// t for vertex t (vertices 8 and on in further rounds, rows of up to eight
// entries, 95%, exchanging offsets and vertices between their lanes), in two
// passes:
//   1. the vertices h_t (relative to the particle), the area (shoelace) and
//      the perimeter of every cell;
//   2. for every vertex h_t of cell i, dE/dh_t summed over the three cells
//      that share it (cell i, cell a_t and cell a_{t+1}; each needs h_t's two
//      neighbours in its own polygon: h_{t-1}, h_{t+1} and the vertex across
//      the edge between a_t and a_{t+1}, found in a_t's row), then
//      F_i -= (dh_t/dr_i)^T dE/dh_t.
// Vectors r_ab point from a to b.  Readings of the printed formulas (they
// are the gradient of Eq. 3 only so; finite differences of the energy decide):
// Eq. (8) dP/dh = t_ij/|t_ij| - t_ik/|t_ik|; c = r_ij x r_jk in Eqs. (15) and
// (19); Eq. (18) ends in -|r_ij|^2 r_jk.
// Everything is fp64 from exact integer minimum-image offsets.
//
// With a lane per particle the dependent gathers of each vertex (the
// neighbour's row, the position across) stood one after another, behind a walk
// by index through rows in registers or memory: forces 200 us at 250,000
// particles and 1.30 ms at 2^20, cells 30 and 140 us.  With eight lanes the
// vertices' gathers are in flight together: 90 and 350 us, 27 and 107 us.  At
// 2^20 the force pass moves 1.4 GB from the memory-side cache into the L2s (10
// lines of 128 bytes a particle) and issues VALU instructions for 40% of its
// time.  Errors against 80-bit arithmetic, 60,000 particles, relative to the root
// mean square force: mean 1.9e-16 and 99.9% below 4.3e-15, as with a lane per
// particle (1.9e-16, 4.7e-15).
#include "nm_internal.h"

namespace nm {
namespace {

struct V2 {
  double x, y;
};
__device__ __forceinline__ V2 operator+(V2 a, V2 b) { return {a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ V2 operator-(V2 a, V2 b) { return {a.x - b.x, a.y - b.y}; }
__device__ __forceinline__ V2 operator*(V2 a, double s) { return {a.x * s, a.y * s}; }
__device__ __forceinline__ double dot(V2 a, V2 b) { return fma(a.x, b.x, a.y * b.y); }
__device__ __forceinline__ double cross(V2 a, V2 b) { return fma(a.x, b.y, -(a.y * b.x)); }
__device__ __forceinline__ V2 add_scaled(V2 v, V2 a, double s) { return {fma(a.x, s, v.x), fma(a.y, s, v.y)}; }

struct VmArgs {
  double ka, kp, a0, p0;
};

// minimum-image offset from i to j, as an exact fp64 vector
__device__ __forceinline__ V2 offset(const int32_t* __restrict__ x, const int32_t* __restrict__ y, int sh,
                                     int i, int j) {
  return {static_cast<double>(wrap_axis(x[j] - x[i], sh)), static_cast<double>(wrap_axis(y[j] - y[i], sh))};
}

// Circumcentre of (i, j, k) relative to i from r_ij, r_ik (Eqs. 15-16), with
// the reciprocal cross product that its derivative needs again.
struct Circum {
  V2 h;
  double inv_c;
};
__device__ __forceinline__ Circum circumcentre(V2 rij, V2 rik) {
  const V2 rjk = rik - rij;
  const double c = cross(rij, rjk);
  const double d = 2.0 * c * c;
  const double bd = -dot(rik, rik) * dot(rij, rjk);
  const double gd = dot(rij, rij) * dot(rik, rjk);
  const double inv_c = 1.0 / c, inv_d = 0.5 * inv_c * inv_c;
  // (rij bd + rik gd) / d, with the first product's rounding and the
  // quotient's remainder put back: short edges are differences of vertices
  auto part = [&](double a, double b) {
    const double p = b * gd, e = fma(b, gd, -p);
    const double z = fma(a, bd, p), h = z * inv_d;
    return fma(fma(-h, d, z) + e, inv_d, h);
  };
  return {{part(rij.x, rik.x), part(rij.y, rik.y)}, inv_c};
}

// g^T (dh/dr_i) for the circumcentre h of (i, j, k) (Eqs. 16-19).  The sums
// of integers come first (exact up to 2^53), their large parts cancel there.
__device__ __forceinline__ V2 pull_back(V2 rij, V2 rik, const Circum& v, V2 g) {
  const V2 rjk = rik - rij;
  const double jj = dot(rij, rij), kk = dot(rik, rik), jd = dot(rij, rjk), kd = dot(rik, rjk);
  const double same = kk * jd - jj * kd;  // -(beta d + gamma d)
  const V2 dbd = add_scaled(rjk * kk, rik, 2.0 * jd);    // Eq. 17
  const V2 dgd = add_scaled(rjk * -jj, rij, -2.0 * kd);  // Eq. 18
  const V2 dd = V2{-rjk.y, rjk.x} * (2.0 * v.inv_c);      // Eq. 19
  const double inv_d = 0.5 * v.inv_c * v.inv_c;
  const double nxx = fma(rij.x, dbd.x, fma(rik.x, dgd.x, same)), nyx = fma(rij.y, dbd.x, rik.y * dgd.x);
  const double nxy = fma(rij.x, dbd.y, rik.x * dgd.y), nyy = fma(rij.y, dbd.y, fma(rik.y, dgd.y, same));
  const double jxx = fma(nxx, inv_d, fma(-v.h.x, dd.x, 1.0)), jyx = fma(nyx, inv_d, -v.h.y * dd.x);
  const double jxy = fma(nxy, inv_d, -v.h.x * dd.y), jyy = fma(nyy, inv_d, fma(-v.h.y, dd.y, 1.0));
  return {fma(g.x, jxx, g.y * jyx), fma(g.x, jxy, g.y * jyy)};
}

// 1 / sqrt(x): the hardware's estimate and two Newton steps (each squares the
// relative error), the second with the rounding of x y added back.
__device__ __forceinline__ double inv_sqrt(double x) {
  double y = __builtin_amdgcn_rsq(x);
  y = fma(0.5 * y, fma(-x * y, y, 1.0), y);
  const double p = x * y, r = fma(x, y, -p);
  return fma(0.5 * y, fma(-r, y, fma(-p, y, 1.0)), y);
}

__device__ __forceinline__ V2 unit(V2 v) { return v * inv_sqrt(dot(v, v)); }

// The order to take n particles in: the cells of the workspace whose header is
// given, if they hold all n, else nullptr (the caller's order).
__device__ __forceinline__ const int4* cell_order(const WsHeader* h, int n) {
  if (h == nullptr || h->magic != kMagic || h->built != kBuilt || h->n != n) return nullptr;
  const char* base = reinterpret_cast<const char*>(h);
  const int64_t G = h->box / h->cell_w;
  if (reinterpret_cast<const int32_t*>(base + h->off_start)[G * G] != n) return nullptr;
  return reinterpret_cast<const int4*>(base + h->off_sorted);
}

constexpr int kVmLanes = 8;                    // lanes per particle
constexpr int kVmPer = kBlock / kVmLanes;      // particles per workgroup
// The first pass gathers only positions: while those stay in an XCD's L2 (4 MB)
// the caller's order is faster, since a cell's own row, length and outputs are
// then whole lines (cells' order against caller's: 44 and 39 us at 400,000
// particles, 74 and 72 at 700,000, 107 and 136 at 2^20).
constexpr int kVmOrderCells = 3 << 18;

// This group's particle (n: none), in the order of the cells of the workspace
// `h`, or the caller's.
__device__ __forceinline__ int my_particle(const WsHeader* h, int n) {
  const int4* order = cell_order(h, n);
  const int at = (order ? xcd_tile(blockIdx.x, gridDim.x) : static_cast<int>(blockIdx.x)) * kVmPer +
                 static_cast<int>(threadIdx.x) / kVmLanes;
  if (at >= n) return n;
  if (!order) return at;
  const int i = order[at].z;
  return static_cast<unsigned>(i) < static_cast<unsigned>(n) ? i : n;
}

// Any lane of this group of kVmLanes.
__device__ __forceinline__ bool group_any(bool v) {
  const int base = threadIdx.x & 63 & ~(kVmLanes - 1);
  return ((__ballot(v) >> base) & ((1ull << kVmLanes) - 1ull)) != 0ull;
}

// Sum over the group, in a fixed order.
__device__ __forceinline__ double group_sum(double v) {
#pragma unroll
  for (int o = 1; o < kVmLanes; o <<= 1) v += __shfl_xor(v, o, 64);
  return v;
}

__device__ __forceinline__ V2 group_get(V2 v, int t) {
  return {__shfl(v.x, t, kVmLanes), __shfl(v.y, t, kVmLanes)};
}

enum : int { kRowOk = 0, kRowBad = 1, kRowCoincident = 2 };

// State of row i's m entries over the group: bad (an index outside [0, n)),
// coincident (a particle at i's own position) or in order; j and (ox, oy):
// entry l of this lane and its offset (l < m).
__device__ __forceinline__ int row_state(const int32_t* __restrict__ x, const int32_t* __restrict__ y, int n, int sh,
                                         const int32_t* __restrict__ row, int m, int i, int l, int& j, V2& off) {
  const int xi = x[i], yi = y[i];
  bool bad = false, coincident = false;
  j = -1;
  off = {1.0, 0.0};
  for (int t = l; t < m; t += kVmLanes) {
    const int q = row[t];
    if (static_cast<unsigned>(q) >= static_cast<unsigned>(n)) {
      bad = true;
      continue;
    }
    const int dx = wrap_axis(x[q] - xi, sh), dy = wrap_axis(y[q] - yi, sh);
    coincident = coincident || (dx == 0 && dy == 0);
    if (t == l) {
      j = q;
      off = {static_cast<double>(dx), static_cast<double>(dy)};
    }
  }
  if (group_any(bad)) return kRowBad;
  return group_any(coincident) ? kRowCoincident : kRowOk;
}

// Pass 1: area and perimeter of every cell (and its vertices, if asked).
__global__ __launch_bounds__(kBlock) void k_vm_cells(const int32_t* __restrict__ x,
                                                     const int32_t* __restrict__ y, int n, int log2_box,
                                                     int dmax, const int32_t* __restrict__ ring,
                                                     const int32_t* __restrict__ deg, double* __restrict__ area,
                                                     double* __restrict__ perim, double* __restrict__ vert,
                                                     WsHeader* err) {
  const int i = my_particle(n >= kVmOrderCells ? err : nullptr, n);
  if (i >= n) return;
  const int l = threadIdx.x & (kVmLanes - 1);
  const int sh = 32 - log2_box;
  const int m = deg[i];
  const int32_t* row = ring + static_cast<long long>(i) * dmax;
  int state = kRowBad, j = -1;
  V2 mine;
  if (m >= 3 && m <= dmax) state = row_state(x, y, n, sh, row, m, i, l, j, mine);
  double a2 = 0.0, per = 0.0;
  if (state != kRowOk) {
    // the model gives each particle its own cell: coincident particles have none
    if (l == 0) set_err(err, state == kRowBad ? NM_E_INVAL : NM_E_RANGE);
  } else {
    double* v = vert ? vert + static_cast<long long>(i) * dmax * 4 : nullptr;
    if (m <= kVmLanes) {
      const int tn = l + 1 < m ? l + 1 : 0;
      const V2 h = circumcentre(mine, group_get(mine, tn)).h;
      const V2 hn = group_get(h, tn);
      if (l < m) {
        if (v) {
          v[4 * l] = h.x;
          v[4 * l + 1] = h.y;
        }
        a2 = cross(h, hn);
        per = sqrt(dot(hn - h, hn - h));
      }
    } else {
      for (int t = l; t < m; t += kVmLanes) {
        const int t1 = t + 1 < m ? t + 1 : 0, t2 = t1 + 1 < m ? t1 + 1 : 0;
        const V2 ra = offset(x, y, sh, i, row[t]), rb = offset(x, y, sh, i, row[t1]), rc = offset(x, y, sh, i, row[t2]);
        const V2 h = circumcentre(ra, rb).h, hn = circumcentre(rb, rc).h;
        if (v) {
          v[4 * t] = h.x;
          v[4 * t + 1] = h.y;
        }
        a2 += cross(h, hn);
        per += sqrt(dot(hn - h, hn - h));
      }
    }
    a2 = group_sum(a2);
    per = group_sum(per);
  }
  if (l == 0) {
    area[i] = 0.5 * a2;
    perim[i] = per;
  }
}

// Pass 2: the force on every particle, and the vertex forces if asked.
// Vertex t of cell i lies between entries j = a_t and k = a_{t+1}; the cells
// i, j and k share it, and it has three edges: to h_{t-1}, to h_{t+1} and to
// the vertex across the edge between j and k, the circumcentre of (j, mm, k)
// with mm the entry before k in j's row (i follows k there).  With u_p, u_n,
// u_x the unit vectors from those three to h, Eqs. (6)-(8) over the three
// cells are
//   dE/dh = T_i (u_p + u_n) + T_j (u_p + u_x) + T_k (u_n + u_x)
//         + rot(S_i (h_n - h_p) + S_j (h_p - h_x) + S_k (h_x - h_n)) / 2,
// rot(v) = (v_y, -v_x), S = 2 K_A (A - A_0), T = 2 K_P (P - P_0) of each cell
// (the three differences add up to zero, so S_k is taken from S_i and S_j and
// its term left out).
__global__ __launch_bounds__(kBlock) void k_vm_forces(const int32_t* __restrict__ x,
                                                      const int32_t* __restrict__ y, int n, int log2_box,
                                                      int dmax, const int32_t* __restrict__ ring,
                                                      const int32_t* __restrict__ deg,
                                                      const double* __restrict__ area,
                                                      const double* __restrict__ perim, VmArgs va,
                                                      double* __restrict__ fx, double* __restrict__ fy,
                                                      double* __restrict__ vert, WsHeader* err) {
  // In the order of the cells that `err`'s workspace holds, where it holds
  // them for n particles (the same results in any order): neighbouring groups
  // then gather the same rows, positions, areas and perimeters.
  const int i = my_particle(err, n);
  if (i >= n) return;
  const int l = threadIdx.x & (kVmLanes - 1);
  const int sh = 32 - log2_box;
  const int m = deg[i];
  const int32_t* row = ring + static_cast<long long>(i) * dmax;
  int state = kRowBad, mine_j = -1;
  V2 mine;
  if (m >= 3 && m <= dmax) state = row_state(x, y, n, sh, row, m, i, l, mine_j, mine);
  V2 F = {0.0, 0.0};
  bool lost = false;  // the rows are not one triangulation
  if (state == kRowOk) {
    const bool whole = m <= kVmLanes;
    const double Si = 2.0 * va.ka * (area[i] - va.a0), Ti = 2.0 * va.kp * (perim[i] - va.p0);
    const int xi = x[i], yi = y[i];
    for (int r = 0; r < m; r += kVmLanes) {
      const int t = r + l;
      const bool act = t < m;
      const int tc = act ? t : 0;
      const int tn = tc + 1 < m ? tc + 1 : 0, tp = tc > 0 ? tc - 1 : m - 1;
      V2 rj, rk, hp, hn;
      Circum c;
      int j, k;
      double Sj, Tj, Sk, Tk;
      auto cell_coeff = [&](int q, double& S, double& T) {
        S = 2.0 * va.ka * (area[q] - va.a0);
        T = 2.0 * va.kp * (perim[q] - va.p0);
      };
      if (whole) {
        j = act ? mine_j : i;
        rj = mine;
        cell_coeff(j, Sj, Tj);
        k = __shfl(j, tn, kVmLanes);
      } else {
        j = row[tc];
        k = row[tn];
        rj = offset(x, y, sh, i, j);
        cell_coeff(j, Sj, Tj);
      }
      // the particle across the edge between j and k, from j's row
      const int mj = deg[j];
      const int32_t* rowj = ring + static_cast<long long>(j) * dmax;
      int mm = -1, after = -1;
      if (mj >= 3 && mj <= 8 && dmax >= 8) {
        int q[8];
#pragma unroll
        for (int u = 0; u < 8; u += 4) {
          const nm_int4u v = *reinterpret_cast<const nm_int4u*>(rowj + u);
          q[u] = v[0];
          q[u + 1] = v[1];
          q[u + 2] = v[2];
          q[u + 3] = v[3];
        }
        int sk = -1;
#pragma unroll
        for (int u = 7; u >= 0; --u)
          if (u < mj && q[u] == k) sk = u;
        const int ua = sk + 1 < mj ? sk + 1 : 0, um = sk > 0 ? sk - 1 : mj - 1;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          if (sk >= 0 && u == ua) after = q[u];
          if (sk >= 0 && u == um) mm = q[u];
        }
      } else if (mj >= 3 && mj <= dmax) {
        int sk = -1;
        for (int u = 0; u < mj && sk < 0; ++u)
          if (rowj[u] == k) sk = u;
        if (sk >= 0) {
          after = rowj[sk + 1 < mj ? sk + 1 : 0];
          mm = rowj[sk > 0 ? sk - 1 : mj - 1];
        }
      }
      const bool found = after == i && static_cast<unsigned>(mm) < static_cast<unsigned>(n);
      if (act && !found) lost = true;
      const int mx = found ? x[mm] : 0, my = found ? y[mm] : 0;
      if (whole) {
        rk = group_get(rj, tn);
        c = circumcentre(rj, rk);
        hp = group_get(c.h, tp);
        hn = group_get(c.h, tn);
        Sk = __shfl(Sj, tn, kVmLanes);
        Tk = __shfl(Tj, tn, kVmLanes);
      } else {
        const int t2 = tn + 1 < m ? tn + 1 : 0;
        rk = offset(x, y, sh, i, k);
        c = circumcentre(rj, rk);
        hp = circumcentre(offset(x, y, sh, i, row[tp]), rj).h;
        hn = circumcentre(rk, offset(x, y, sh, i, row[t2])).h;
        cell_coeff(k, Sk, Tk);
      }
      // offsets from j of the particle across and of k
      const int xj = xi + static_cast<int>(rj.x), yj = yi + static_cast<int>(rj.y);
      const V2 rjm = {static_cast<double>(wrap_axis(mx - xj, sh)), static_cast<double>(wrap_axis(my - yj, sh))};
      const V2 rjk = {static_cast<double>(wrap_axis(static_cast<int>(rk.x - rj.x), sh)),
                      static_cast<double>(wrap_axis(static_cast<int>(rk.y - rj.y), sh))};
      const V2 hx = rj + circumcentre(rjm, rjk).h;
      const V2 up = unit(c.h - hp), un = unit(c.h - hn), ux = unit(c.h - hx);
      const V2 e = add_scaled((hn - hp) * (Si - Sk), hp - hx, Sj - Sk);
      const V2 g = add_scaled(add_scaled(add_scaled(V2{0.5 * e.y, -0.5 * e.x}, up, Ti + Tj), un, Ti + Tk), ux, Tj + Tk);
      if (act && found) {
        if (vert) {
          double* v = vert + (static_cast<long long>(i) * dmax + t) * 4;
          v[2] = -g.x;
          v[3] = -g.y;
        }
        F = F - pull_back(rj, rk, c, g);
      }
    }
    if (group_any(lost)) {
      if (l == 0) set_err(err, NM_E_INVAL);
      F = {0.0, 0.0};
    }
    F = {group_sum(F.x), group_sum(F.y)};
  }
  if (l == 0) {
    fx[i] = F.x;
    fy[i] = F.y;
  }
}

// Eq. (3) over many workgroups, still in a fixed order: workgroup g sums
// the cells of its contiguous share (lanes, then a fixed tree) into part[g];
// one workgroup then sums the parts in a fixed tree.  The parts go into the
// force array before the force pass overwrites it.
constexpr int kEParts = 256;
__global__ __launch_bounds__(kBlock) void k_vm_energy_part(const double* __restrict__ area,
                                                           const double* __restrict__ perim, int n, VmArgs va,
                                                           double* __restrict__ part) {
  __shared__ double red[kBlock];
  const int chunk = (n + gridDim.x - 1) / gridDim.x;
  const int b = blockIdx.x * chunk, e = min(n, b + chunk);
  double acc = 0.0;
  for (int i = b + threadIdx.x; i < e; i += kBlock) {
    const double da = area[i] - va.a0, dp = perim[i] - va.p0;
    acc += va.ka * da * da + va.kp * dp * dp;
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int h = kBlock / 2; h > 0; h >>= 1) {
    if (threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

__global__ __launch_bounds__(kEParts) void k_vm_energy_sum(const double* __restrict__ part, int np,
                                                           double* __restrict__ energy) {
  __shared__ double red[kEParts];
  red[threadIdx.x] = static_cast<int>(threadIdx.x) < np ? part[threadIdx.x] : 0.0;
  __syncthreads();
  for (int h = kEParts / 2; h > 0; h >>= 1) {
    if (threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) *energy = red[0];
}

}  // namespace

hipError_t launch_voronoi_forces(const int32_t* x, const int32_t* y, int32_t n, int log2_box, int dmax,
                                 const int32_t* ring, const int32_t* deg, const nm_vm_params* p,
                                 double* area, double* perim, double* fx, double* fy, double* energy,
                                 double* vert, WsHeader* err, hipStream_t s) {
  const VmArgs va{p->ka, p->kp, p->a0, p->p0};
  const int nb = (n + kVmPer - 1) / kVmPer;
  hipLaunchKernelGGL(k_vm_cells, dim3(nb), dim3(kBlock), 0, s, x, y, n, log2_box, dmax, ring, deg, area,
                     perim, vert, err);
  if (energy) {
    // (one workgroup alone read the cells at one CU's bandwidth: 0.25 ms at 2^20)
    const int np = n < kEParts ? n : kEParts;
    hipLaunchKernelGGL(k_vm_energy_part, dim3(np), dim3(kBlock), 0, s, area, perim, n, va, fx);
    hipLaunchKernelGGL(k_vm_energy_sum, dim3(1), dim3(kEParts), 0, s, fx, np, energy);
  }
  hipLaunchKernelGGL(k_vm_forces, dim3(nb), dim3(kBlock), 0, s, x, y, n, log2_box, dmax, ring, deg, area,
                     perim, va, fx, fy, vert, err);
  return hipGetLastError();
}

}  // namespace nm
