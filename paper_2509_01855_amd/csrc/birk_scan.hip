// P^{-1} y and P^{-T} y for n_x <= 8 (gfx950): block substitution as a scan of affine maps.
//
// Forward (see birk_solve.hip): with H_k = w_k J_k K_k^{-1} = K_k^{-1} (w_k J_k),
// K_k = I - w_k J_k / 2, node k takes the carried sum S to (I + H_k) S + H_k y_k and emits
//     u = y_k + S,  v = H_k u,  xi_k = u + v / 2,  J_k xi_k = v / w_k.
// Backward (P^{-T}, from the last node down, G_k = H_k^T formed from J_k^T): T goes to
// (I + G_k) T + (I + G_k / 2) y_k and x_k = y_k + G_k (T + y_k / 2).
//
// A wave works a tile of 64 R consecutive nodes (positions p; node p, or N_n - 1 - p
// backwards) in R rounds of 64, four chunks of sixteen nodes each.  In every round
//   * each lane loads its node's J, y and w, factors K_k and leaves H_k in the node's LDS
//     record: all 64 lanes on different nodes, whole 512-byte runs of every field, and no
//     table of H in memory;
//   * reduce: lanes 16 g + c and 16 g + 8 + c carry the two row halves of column c of chunk
//     g's map (column n_x: the constant) through its sixteen nodes, H_k broadcast from the
//     records, the halves exchanged by DPP; the four chunk maps are scanned, stored, and
//     the last of them carries the tile's map on;
//   * apply: the sixteen lanes of a chunk (one state component each, states exchanged with
//     DPP row_newbcast) take their start state from the round's and the stored chunk map,
//     and replay the nodes; outputs go back through the records and are stored one node per
//     lane.
// Launches: reduce, tiles (one wave scans 64 tile maps), apply (start state: the chain over
// earlier groups of 64 tiles, then the tile's map).  Instances short enough that every
// wave's records stay in one workgroup's LDS take one launch instead (k_scan_small), which
// forms each H_k once.
//
// Bound: HBM, J twice (2 x 37 + 3 x 6 doubles per node at n_x = 6: 735 MB and 141 us at
// N = 2^20).  The former kernels (four consecutive nodes per lane through LDS tiles, 16 of 64
// lanes on each factorisation) took 365 us there with per-node J, 195 with one J, 102 at
// 65537 nodes, 39 at 257 (one J); these 227, 162, 36 and 13.  n_x = 8, 3e5 nodes: 394 -> 196.
// Tried and slower at N = 2^20, per-node J: chunks of 16 R nodes each whose rounds take 8 or
// 16 nodes of every chunk (a run of 64 or 128 bytes per field and load; no scan per round) 358
// and 247; the next round's J loaded ahead (256 registers and spills) 417.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>
#include <vector>

#include "birk_dense.h"
#include "birk_internal.h"

namespace birk {
namespace {

// Where H_k comes from: one J per instance, J per node, or (float plans in a solve with
// per-node J) H_k kept in float by scan_prepare, half the bytes of J.
constexpr int kConst = 0, kPerNode = 1, kCachedH = 2;

constexpr int kG = 16;   // nodes of a chunk, and lanes that work it
constexpr int kC = 4;    // chunks of a round
constexpr int kLaneNx = 3;   // n_x up to here: one node's map per lane

template <int NX>
struct Lay {
  static constexpr int F = NX * NX + NX;           // a map: columns 0..NX-1 of A, then b
  static constexpr int RL = F + (F & 1);           // a node's record: H row-major, then NX values
  static constexpr int REC = 64 * RL + 16;         // a wave's records: 16 bytes of skew per 8 nodes
  static constexpr int SIZE = REC + kC * F;        // and its chunk maps
};

template <int NX>
__device__ __forceinline__ double* record(double* sm, int n) {
  return sm + n * Lay<NX>::RL + (n >> 3) * 2;
}

// One node's inputs, loaded ahead of use.
template <int NX, int MODE>
struct Node {
  using JV = std::conditional_t<MODE == kCachedH, float, double>;
  JV j[MODE == kConst ? 1 : NX * NX];
  double y[NX];
  double w;
  bool ok;

  template <bool BACK, typename T>
  __device__ __forceinline__ void load(const ScanDesc& d, const double* __restrict__ J, const float* __restrict__ htab,
                                       const T* __restrict__ yv, int64_t pos) {
    const int64_t Nn = d.Nn;
    ok = pos < Nn;
    const int64_t p = ok ? pos : 0;
    const uint32_t k = (uint32_t)(BACK ? Nn - 1 - p : p);   // uniform bases, one offset
    if constexpr (MODE == kPerNode) {
#pragma unroll
      for (int e = 0; e < NX * NX; ++e) j[e] = (J + d.joff + e * Nn)[k];
    } else if constexpr (MODE == kCachedH) {
#pragma unroll
      for (int e = 0; e < NX * NX; ++e) j[e] = (htab + d.hoff + e * Nn)[k];
    }
#pragma unroll
    for (int r = 0; r < NX; ++r) y[r] = (double)(yv + d.off + r * Nn)[k];
    w = d.w[k];
  }
};

// H_k (G_k backwards) into the node's record, zero past the instance; g (when asked for):
// H_k y_k, or y_k + G_k y_k / 2 backwards.  A pivot that is non-finite or not above 1e-13
// (1 + |w_k / 2| max |J_k|) sets *flag when given.
template <int NX, int MODE, bool BACK>
__device__ __forceinline__ void form_h(const Node<NX, MODE>& nd, const double* __restrict__ Jc, double* __restrict__ rec,
                                       double (&g)[NX], int* flag) {
#pragma unroll
  for (int r = 0; r < NX; ++r) g[r] = 0.0;
  if constexpr (MODE == kCachedH) {
#pragma unroll
    for (int r = 0; r < NX; ++r)
#pragma unroll
      for (int q = 0; q < NX; ++q) {
        const double h = nd.ok ? (double)nd.j[r * NX + q] : 0.0;
        rec[r * NX + q] = h;
        g[r] += h * nd.y[q];
      }
  } else {
    const double wk = nd.ok ? nd.w : 0.0;   // past the instance: H = 0
    // w J and then H: in registers up to n_x = 6, in the record above
    constexpr bool kReg = NX <= 6;
    double K[NX][NX], X[kReg ? NX : 1][kReg ? NX : 1], rp[NX], jmax = 0.0;
#pragma unroll
    for (int r = 0; r < NX; ++r)
#pragma unroll
      for (int q = 0; q < NX; ++q) {
        const int e = BACK ? q * NX + r : r * NX + q;
        double jv;
        if constexpr (MODE == kConst) jv = Jc[e];
        else jv = nd.j[e];
        if (flag) jmax = fmax(jmax, fabs(jv));
        if constexpr (kReg) X[r][q] = wk * jv;
        else rec[r * NX + q] = wk * jv;
        K[r][q] = (r == q ? 1.0 : 0.0) - 0.5 * wk * jv;
      }
    lu_kmat<NX>(K, rp, nd.ok ? flag : nullptr, 1.0 + 0.5 * fabs(wk) * jmax);
#pragma unroll
    for (int c = 0; c < NX; ++c) {
      double x[NX];
#pragma unroll
      for (int r = 0; r < NX; ++r) {
        if constexpr (kReg) x[r] = X[r][c];
        else x[r] = rec[r * NX + c];
      }
      lu_solve<NX>(K, rp, x);
#pragma unroll
      for (int r = 0; r < NX; ++r) {
        if constexpr (kReg) X[r][c] = x[r];
        else rec[r * NX + c] = x[r];
        g[r] += x[r] * nd.y[c];
      }
    }
    if constexpr (kReg) {
#pragma unroll
      for (int r = 0; r < NX; ++r)
#pragma unroll
        for (int q = 0; q < NX; ++q) rec[r * NX + q] = X[r][q];
    }
  }
#pragma unroll
  for (int r = 0; r < NX; ++r) g[r] = nd.ok ? (BACK ? nd.y[r] + 0.5 * g[r] : g[r]) : 0.0;
}

// v of the lane eight away in the row of sixteen (DPP row_ror:8).
__device__ __forceinline__ double swap8(double v) {
  const unsigned long long x = __builtin_bit_cast(unsigned long long, v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)x, 0x128, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(x >> 32), 0x128, 0xF, 0xF, false);
  return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}

// A column of a chunk's map in two lanes: own rows and the other lane's.  NH rows in the
// first half, NX - NH in the second, whose last is a zero when NX is odd.
template <int NX>
struct Col {
  static constexpr int NH = (NX + 1) / 2;
  double own[NH], oth[NH];
  double bc;   // NX = 8: component c of the constant, in lane 16 g + c (its column has no lanes)
  __device__ __forceinline__ void identity() {
    const int c = (int)threadIdx.x & 7, half = ((int)threadIdx.x >> 3) & 1;
#pragma unroll
    for (int r = 0; r < NH; ++r) {
      own[r] = half * NH + r == c && c < NX ? 1.0 : 0.0;
      oth[r] = (1 - half) * NH + r == c && c < NX ? 1.0 : 0.0;
    }
    bc = 0.0;
  }
};

// Every chunk's columns through the round's sixteen nodes: a <- a + H a, and the constant
// (column NX) b <- b + H b + g.
template <int NX>
__device__ __forceinline__ void compose_nodes(double* sm, Col<NX>& a) {
  constexpr int NH = Col<NX>::NH;
  const int l = (int)(threadIdx.x & 63), g = l >> 4, c = l & 7, half = (l >> 3) & 1;
  const int r0 = half * NH, q0 = half * NH, q1 = (1 - half) * NH;
#pragma unroll 2
  for (int i = 0; i < kG; ++i) {
    const double* p = record<NX>(sm, kG * g + i);
    double t[NH];
#pragma unroll
    for (int r = 0; r < NH; ++r) {
      // the missing row of an odd NX reads the values after H, and is zeroed
      double acc = (NX < 8 && c == NX) ? p[NX * NX + r0 + (r0 + r < NX ? r : 0)] : 0.0;
#pragma unroll
      for (int q = 0; q < NH; ++q) acc += p[(r0 + r) * NX + q0 + q] * a.own[q];
#pragma unroll
      for (int q = 0; q < NH; ++q) acc += p[(r0 + r) * NX + q1 + q] * a.oth[q];
      t[r] = (NX % 2 && r0 + r >= NX) ? 0.0 : acc;
    }
    if constexpr (NX == 8) {
      double acc = p[NX * NX + c];
#pragma unroll
      for (int q = 0; q < NX; ++q) acc += p[c * NX + q] * __shfl(a.bc, 16 * g + q, 64);
      a.bc += acc;
    }
#pragma unroll
    for (int r = 0; r < NH; ++r) {
      a.own[r] += t[r];
      a.oth[r] = swap8(a.own[r]);
    }
  }
}

// Chunk maps of the wave to their inclusive products M_g o ... o M_0 in
// mp[g F + c NX + r] (column c; column NX: the constant), by two doubling steps.
template <int NX>
__device__ __forceinline__ void scan_chunks(double* mp, const Col<NX>& a) {
  constexpr int F = Lay<NX>::F, NH = Col<NX>::NH;
  const int l = (int)(threadIdx.x & 63), g = l >> 4, i = l & 15, c = i & 7, half = i >> 3;
  double* mine = mp + g * F;
  if (c <= NX) {
#pragma unroll
    for (int r = 0; r < NH; ++r)
      if (half * NH + r < NX) mine[c * NX + half * NH + r] = a.own[r];
  }
  if (NX == 8 && i < 8) mine[NX * NX + i] = a.bc;
  wave_sync();
#pragma unroll
  for (int d = 1; d < kC; d <<= 1) {
    // lane i of the group: column i of M_g o M_{g-d}
    double n[NX];
    const bool work = g >= d && i <= NX;
    if (work) {
      const double* lo = mine - d * F;
#pragma unroll
      for (int r = 0; r < NX; ++r) n[r] = i == NX ? mine[NX * NX + r] : 0.0;
#pragma unroll
      for (int q = 0; q < NX; ++q) {
        const double x = lo[i * NX + q];
#pragma unroll
        for (int r = 0; r < NX; ++r) n[r] += mine[q * NX + r] * x;
      }
    }
    wave_sync();
    if (work) {
#pragma unroll
      for (int r = 0; r < NX; ++r) mine[i * NX + r] = n[r];
    }
    wave_sync();
  }
}

// Replay of the round's nodes from the records (H, then y): row of lanes g replays chunk g
// from state s.  xi (x) replaces y; with keep_v, v goes to the first NX entries.
template <int NX, bool BACK>
__device__ __forceinline__ void replay_nodes(double* sm, double& s, bool keep_v) {
  const int l = (int)(threadIdx.x & 63), g = l >> 4, r = l & 15;
  const bool act = r < NX;
  const int rr = act ? r : NX - 1;
  double xo[kG], vo[kG];
#pragma unroll
  for (int i = 0; i < kG; ++i) {
    const double* p = record<NX>(sm, kG * g + i);
    const double y = p[NX * NX + rr];
    double row[NX], v[2] = {0.0, 0.0};
#pragma unroll
    for (int q = 0; q < NX; ++q) row[q] = p[rr * NX + q];
    const double u = BACK ? s + 0.5 * y : s + y;
    static_for<0, NX>([&](auto qc) {
      constexpr int q = decltype(qc)::value;
      v[q & 1] += row[q] * row_bcast<q>(u);
    });
    const double vs = v[0] + v[1];
    const double x = BACK ? y + vs : u + 0.5 * vs;
    s += BACK ? x : vs;
    xo[i] = x;
    vo[i] = vs;
  }
  wave_sync();
  if (act) {
#pragma unroll
    for (int i = 0; i < kG; ++i) {
      double* p = record<NX>(sm, kG * g + i);
      p[NX * NX + r] = xo[i];
      if (keep_v) p[r] = vo[i];
    }
  }
  wave_sync();
}

// The lane's node after the replay: xi (x) to out, J xi = v / w to jout.
template <int NX, bool BACK, typename T>
__device__ __forceinline__ void store_node(const double* __restrict__ rec, const ScanDesc& d, int64_t pos, double w,
                                           T* __restrict__ out, T* __restrict__ jout) {
  if (pos >= d.Nn) return;
  const int64_t k = BACK ? d.Nn - 1 - pos : pos;
#pragma unroll
  for (int r = 0; r < NX; ++r) out[d.off + (int64_t)r * d.Nn + k] = (T)rec[NX * NX + r];
  if (!BACK && jout) {
    const double iw = 1.0 / w;
#pragma unroll
    for (int r = 0; r < NX; ++r) jout[d.off + (int64_t)r * d.Nn + k] = (T)(rec[r] * iw);
  }
}

// Tile = (instance, tile): chunk maps scanned within each round to d.cmap, the tile's map
// to d.tmap (field-major over the tiles).
template <int NX, int MODE, bool BACK, typename T>
__global__ __launch_bounds__(64, 2) void k_scan_reduce(const double* __restrict__ J, const float* __restrict__ htab,
                                                       const T* __restrict__ y, const ScanDesc* __restrict__ sd,
                                                       const int2* __restrict__ tiles, double* __restrict__ scan) {
  constexpr int F = Lay<NX>::F;
  __shared__ __align__(16) double sm[Lay<NX>::SIZE];
  double* mp = sm + Lay<NX>::REC;
  const int2 t = tiles[blockIdx.x];
  const ScanDesc& d = sd[t.x];
  const int R = d.rounds, l = (int)threadIdx.x;
  const int64_t base = (int64_t)t.y * 64 * R + l;
  // lane 16 g + c, every g alike: column c of the tile's map
  const int c = min(l & 15, NX);
  double tm[NX];
#pragma unroll
  for (int r = 0; r < NX; ++r) tm[r] = r == c ? 1.0 : 0.0;
#pragma unroll 1
  for (int j = 0; j < R; ++j) {
    Node<NX, MODE> nd;
    nd.template load<BACK, T>(d, J, htab, y, base + 64 * j);
    double* rec = record<NX>(sm, l);
    {
      double gv[NX];
      form_h<NX, MODE, BACK>(nd, J + d.jcoff, rec, gv, nullptr);
#pragma unroll
      for (int r = 0; r < NX; ++r) rec[NX * NX + r] = gv[r];
    }
    wave_sync();
    {
      Col<NX> a;
      a.identity();
      compose_nodes<NX>(sm, a);
      scan_chunks<NX>(mp, a);
    }
    double* cm = scan + d.cmap + ((int64_t)t.y * R + j) * kC * F;
#pragma unroll
    for (int e = 0; e < (kC * F + 63) / 64; ++e)
      if (l + 64 * e < kC * F) cm[l + 64 * e] = mp[l + 64 * e];
    const double* m = mp + (kC - 1) * F;
    double n[NX];
#pragma unroll
    for (int r = 0; r < NX; ++r) n[r] = c == NX ? m[NX * NX + r] : 0.0;
#pragma unroll
    for (int q = 0; q < NX; ++q)
#pragma unroll
      for (int r = 0; r < NX; ++r) n[r] += m[q * NX + r] * tm[q];
#pragma unroll
    for (int r = 0; r < NX; ++r) tm[r] = n[r];
    wave_sync();
  }
  if (t.y + 1 < d.ntile && l <= NX) {
    double* o = scan + d.tmap + t.y;
#pragma unroll
    for (int r = 0; r < NX; ++r) o[(int64_t)(l * NX + r) * d.ntile] = tm[r];
  }
}

// 64 tiles of an instance per wave: inclusive maps within the group, in place, and the
// group's own map to d.gmap.  tile = (instance, group).
template <int NX>
__global__ __launch_bounds__(64) void k_scan_tiles(double* __restrict__ scan, const ScanDesc* __restrict__ sd,
                                                   const int2* __restrict__ groups) {
  constexpr int F = Lay<NX>::F;
  const int2 t = groups[blockIdx.x];
  const ScanDesc& d = sd[t.x];
  const int64_t tile = (int64_t)t.y * 64 + threadIdx.x;
  const bool in = tile + 1 < d.ntile;   // the last tile's map is not needed
  double* tm = scan + d.tmap + (in ? tile : 0);
  Aff<NX> m;
#pragma unroll
  for (int c = 0; c < NX; ++c)
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      const double v = tm[(int64_t)(c * NX + r) * d.ntile];
      m.A[r][c] = in ? v : (r == c ? 1.0 : 0.0);
    }
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    const double v = tm[(int64_t)(NX * NX + r) * d.ntile];
    m.b[r] = in ? v : 0.0;
  }
  wave_scan<NX>(m);
  if (in) {
#pragma unroll
    for (int c = 0; c < NX; ++c)
#pragma unroll
      for (int r = 0; r < NX; ++r) tm[(int64_t)(c * NX + r) * d.ntile] = m.A[r][c];
#pragma unroll
    for (int r = 0; r < NX; ++r) tm[(int64_t)(NX * NX + r) * d.ntile] = m.b[r];
  }
  if (threadIdx.x == 63) {
    double* gm = scan + d.gmap + (int64_t)t.y * F;
#pragma unroll
    for (int c = 0; c < NX; ++c)
#pragma unroll
      for (int r = 0; r < NX; ++r) gm[c * NX + r] = m.A[r][c];
#pragma unroll
    for (int r = 0; r < NX; ++r) gm[NX * NX + r] = m.b[r];
  }
}

template <int NX, int MODE, bool BACK, typename T>
__global__ __launch_bounds__(64, 2) void k_scan_apply(const double* __restrict__ J, const float* __restrict__ htab,
                                                      const T* __restrict__ y, const ScanDesc* __restrict__ sd,
                                                      const int2* __restrict__ tiles, const double* __restrict__ scan,
                                                      T* __restrict__ out, T* __restrict__ jout, int* flag) {
  constexpr int F = Lay<NX>::F, NM = (kC * F + 63) / 64;
  __shared__ __align__(16) double sm[Lay<NX>::SIZE];
  double* mp = sm + Lay<NX>::REC;
  const int2 t = tiles[blockIdx.x];
  const ScanDesc& d = sd[t.x];
  const int R = d.rounds, l = (int)threadIdx.x, g = l >> 4;
  const int64_t base = (int64_t)t.y * 64 * R + l;
  const double* cm = scan + d.cmap + (int64_t)t.y * R * kC * F;
  // the tile's start state: the groups before its own, then its predecessors' map
  double s = 0.0;
  const int ng = t.y >> 6;
#pragma unroll 4
  for (int q = 0; q < ng; ++q) s = advance<NX>(scan + d.gmap + (int64_t)q * F, 1, s);
  if (t.y & 63) s = advance<NX>(scan + d.tmap + t.y - 1, d.ntile, s);
#pragma unroll 1
  for (int j = 0; j < R; ++j) {
    Node<NX, MODE> nd;
    nd.template load<BACK, T>(d, J, htab, y, base + 64 * j);
    double cv[NM];   // the round's chunk maps
#pragma unroll
    for (int e = 0; e < NM; ++e) cv[e] = cm[(int64_t)j * kC * F + min(l + 64 * e, kC * F - 1)];
    double* rec = record<NX>(sm, l);
    {
      double gv[NX];
      form_h<NX, MODE, BACK>(nd, J + d.jcoff, rec, gv, flag);
    }
#pragma unroll
    for (int r = 0; r < NX; ++r) rec[NX * NX + r] = nd.ok ? nd.y[r] : 0.0;
#pragma unroll
    for (int e = 0; e < NM; ++e)
      if (l + 64 * e < kC * F) mp[l + 64 * e] = cv[e];
    const double w = nd.w;
    wave_sync();
    double sc = advance<NX>(mp + max(g - 1, 0) * F, 1, s);
    if (g == 0) sc = s;
    s = advance<NX>(mp + (kC - 1) * F, 1, s);
    replay_nodes<NX, BACK>(sm, sc, !BACK && jout);
    store_node<NX, BACK, T>(rec, d, base + 64 * j, w, out, jout);
    wave_sync();
  }
}

// n_x <= 3: the maps are small enough that each lane holds its own node's, and a round is one
// scan of 64 maps by DPP; no records, no chunk maps, the next round's loads in flight.  Bound:
// memory at N = 2^20 (n_x = 1, 2, 3 with per-node J: 19, 40, 77 us, for 67, 134, 235 MB).  The
// kernels above took 33, 51 and 78 there, leaving most of a chunk's lanes idle; at n_x = 4 the
// scan's 1512 FMAs a lane make it the slower way (131 against 109).
template <int NX, int MODE, bool BACK, typename T>
__device__ __forceinline__ void node_map(const Node<NX, MODE>& nd, const double* __restrict__ Jc, double (&h)[NX * NX],
                                         Aff<NX>& m, int* flag) {
  double gv[NX];
  form_h<NX, MODE, BACK>(nd, Jc, h, gv, flag);
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    m.b[r] = gv[r];
#pragma unroll
    for (int q = 0; q < NX; ++q) m.A[r][q] = (r == q ? 1.0 : 0.0) + h[r * NX + q];
  }
  wave_scan<NX>(m);
}

template <int NX, int MODE, bool BACK, typename T>
__global__ __launch_bounds__(64) void k_lane_reduce(const double* __restrict__ J, const float* __restrict__ htab,
                                                    const T* __restrict__ y, const ScanDesc* __restrict__ sd,
                                                    const int2* __restrict__ tiles, double* __restrict__ scan) {
  const int2 t = tiles[blockIdx.x];
  const ScanDesc& d = sd[t.x];
  const int R = d.rounds, l = (int)threadIdx.x;
  const int64_t base = (int64_t)t.y * 64 * R + l;
  if (t.y + 1 >= d.ntile) return;   // the last tile's map is not needed
  Aff<NX> tm;
  Node<NX, MODE> nd;
  nd.template load<BACK, T>(d, J, htab, y, base);
#pragma unroll 1
  for (int j = 0; j < R; ++j) {
    const Node<NX, MODE> cur = nd;
    if (j + 1 < R) nd.template load<BACK, T>(d, J, htab, y, base + 64 * (j + 1));
    Aff<NX> m;
    double h[NX * NX];
    node_map<NX, MODE, BACK, T>(cur, J + d.jcoff, h, m, nullptr);
    if (j == 0) {
      tm = m;
      continue;
    }
    Aff<NX> n = m;   // of interest in lane 63 only, as tm is
#pragma unroll
    for (int r = 0; r < NX; ++r) {
#pragma unroll
      for (int q = 0; q < NX; ++q) n.b[r] += m.A[r][q] * tm.b[q];
#pragma unroll
      for (int c = 0; c < NX; ++c) {
        double acc = 0.0;
#pragma unroll
        for (int q = 0; q < NX; ++q) acc += m.A[r][q] * tm.A[q][c];
        n.A[r][c] = acc;
      }
    }
    tm = n;
  }
  if (l == 63) {
    double* o = scan + d.tmap + t.y;
#pragma unroll
    for (int r = 0; r < NX; ++r) {
#pragma unroll
      for (int c = 0; c < NX; ++c) o[(int64_t)(c * NX + r) * d.ntile] = tm.A[r][c];
      o[(int64_t)(NX * NX + r) * d.ntile] = tm.b[r];
    }
  }
}

template <int NX, int MODE, bool BACK, typename T>
__global__ __launch_bounds__(64) void k_lane_apply(const double* __restrict__ J, const float* __restrict__ htab,
                                                   const T* __restrict__ y, const ScanDesc* __restrict__ sd,
                                                   const int2* __restrict__ tiles, const double* __restrict__ scan,
                                                   T* __restrict__ out, T* __restrict__ jout, int* flag) {
  constexpr int F = Lay<NX>::F;
  const int2 t = tiles[blockIdx.x];
  const ScanDesc& d = sd[t.x];
  const int R = d.rounds, l = (int)threadIdx.x;
  const int64_t base = (int64_t)t.y * 64 * R + l;
  Node<NX, MODE> nd;
  nd.template load<BACK, T>(d, J, htab, y, base);
  double s[NX];   // the tile's start state, in every lane
#pragma unroll
  for (int r = 0; r < NX; ++r) s[r] = 0.0;
  auto step = [&](const double* __restrict__ m, int64_t fs) {
    double n[NX];
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      n[r] = m[(NX * NX + r) * fs];
#pragma unroll
      for (int q = 0; q < NX; ++q) n[r] += m[(q * NX + r) * fs] * s[q];
    }
#pragma unroll
    for (int r = 0; r < NX; ++r) s[r] = n[r];
  };
  const int ng = t.y >> 6;
#pragma unroll 8
  for (int q = 0; q < ng; ++q) step(scan + d.gmap + (int64_t)q * F, 1);
  if (t.y & 63) step(scan + d.tmap + t.y - 1, d.ntile);
#pragma unroll 1
  for (int j = 0; j < R; ++j) {
    const Node<NX, MODE> cur = nd;
    if (j + 1 < R) nd.template load<BACK, T>(d, J, htab, y, base + 64 * (j + 1));
    Aff<NX> m;
    double h[NX * NX], u[NX], x[NX], v[NX];
    node_map<NX, MODE, BACK, T>(cur, J + d.jcoff, h, m, flag);
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      double e = m.b[r];   // the state after this lane's node
#pragma unroll
      for (int q = 0; q < NX; ++q) e += m.A[r][q] * s[q];
      x[r] = e;
      const double before = __shfl_up(e, 1, 64);
      u[r] = (l == 0 ? s[r] : before) + (BACK ? 0.5 * cur.y[r] : cur.y[r]);
    }
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      s[r] = lane63(x[r]);
      v[r] = 0.0;
#pragma unroll
      for (int q = 0; q < NX; ++q) v[r] += h[r * NX + q] * u[q];
    }
    const int64_t pos = base + 64 * j;
    if (pos < d.Nn) {
      const int64_t k = BACK ? d.Nn - 1 - pos : pos;
      const double iw = 1.0 / cur.w;
#pragma unroll
      for (int r = 0; r < NX; ++r) {
        out[d.off + (int64_t)r * d.Nn + k] = (T)(BACK ? cur.y[r] + v[r] : u[r] + 0.5 * v[r]);
        if (!BACK && jout) jout[d.off + (int64_t)r * d.Nn + k] = (T)(v[r] * iw);
      }
    }
  }
}

// One J per instance, n_x = 2 to 5, from 10^5 nodes on: nothing but y and w comes from memory, and
// the scan of 64 maps is most of the arithmetic above.  Here a lane carries four consecutive
// nodes: it composes their maps itself, the wave scans once for 256 nodes and keeps the scanned
// maps (F doubles per four nodes) for the second pass, which only replays; y, w and the outputs
// pass through LDS, so that global accesses stay whole runs.  Bound: FP64 VALU.  n_x = 2, 3, 4, 5:
// 300001 nodes 17.5, 28.5, 37.3, 52.5 us with the kernels above (a node per lane, or chunks of
// sixteen) and 15.2, 21.4, 30.6, 44.1 here; 2^20 + 1 nodes 34.9, 60.5, 75.7, 120 and 28.7, 43.5,
// 65.4, 94.3; 65537 nodes 13.8, 15.9, 19.6, 24.7 and 13.7, 15.2, 19.8, 27.3.  n_x = 1: 17 us either
// way at 2^20 + 1.
constexpr int kFour = 4;           // nodes of a lane
constexpr int kFourNx = 5;
constexpr bool four_nx(int nx) { return nx >= 2 && nx <= kFourNx; }
constexpr int kFourRound = 64 * kFour;
template <int NX>
struct FourLds {
  static constexpr int LD = kFourRound + kFourRound / kFour;   // a row, one place of skew per lane
  double v[NX + 1][LD];                                        // y (then the output), w
};
__device__ __forceinline__ int four_at(int p) { return p + p / kFour; }

// The round's y and w, zero past the instance.
template <int NX, bool BACK, typename T>
__device__ __forceinline__ void four_load(const ScanDesc& d, const T* __restrict__ yv, int64_t first, FourLds<NX>& sm) {
  const int l = (int)threadIdx.x;
  const int64_t Nn = d.Nn;
  double y[kFour][NX], w[kFour];
#pragma unroll
  for (int i = 0; i < kFour; ++i) {
    const int64_t pos = first + l + 64 * i;
    const bool ok = pos < Nn;
    const int64_t p = ok ? pos : 0;
    const uint32_t k = (uint32_t)(BACK ? Nn - 1 - p : p);
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      const double x = (double)(yv + d.off + r * Nn)[k];
      y[i][r] = ok ? x : 0.0;
    }
    const double x = d.w[k];
    w[i] = ok ? x : 0.0;
  }
#pragma unroll
  for (int i = 0; i < kFour; ++i) {
    const int a = four_at(l + 64 * i);
#pragma unroll
    for (int r = 0; r < NX; ++r) sm.v[r][a] = y[i][r];
    sm.v[NX][a] = w[i];
  }
}

// Node i of the lane: H_k, y_k and g (see form_h); left: nodes from the round's first on.
template <int NX, bool BACK>
__device__ __forceinline__ void four_node(const FourLds<NX>& sm, int i, int64_t left, const double* __restrict__ Jc,
                                          double (&h)[NX * NX], double (&y)[NX], double (&g)[NX], int* flag) {
  Node<NX, kConst> nd;
  const int a = four_at((int)threadIdx.x * kFour + i);
#pragma unroll
  for (int r = 0; r < NX; ++r) nd.y[r] = y[r] = sm.v[r][a];
  nd.w = sm.v[NX][a];
  nd.ok = (int)threadIdx.x * kFour + i < left;
  form_h<NX, kConst, BACK>(nd, Jc, h, g, flag);
}

// A round's scanned maps in the scratch: field e of lane l's at 64 e + l.
template <int NX, typename P>
__device__ __forceinline__ P* four_maps(P* scan, const ScanDesc& d, int tile, int round) {
  return scan + d.cmap + ((int64_t)tile * d.rounds + round) * 64 * Lay<NX>::F + threadIdx.x;
}

// The lane's four nodes as one map, scanned over the wave.
template <int NX, bool BACK>
__device__ __forceinline__ void four_map(const FourLds<NX>& sm, int64_t left, const double* __restrict__ Jc, Aff<NX>& m) {
#pragma unroll 1
  for (int i = 0; i < kFour; ++i) {
    double h[NX * NX], y[NX], g[NX];
    four_node<NX, BACK>(sm, i, left, Jc, h, y, g, nullptr);
    if (i == 0) {
#pragma unroll
      for (int r = 0; r < NX; ++r) {
        m.b[r] = g[r];
#pragma unroll
        for (int c = 0; c < NX; ++c) m.A[r][c] = (r == c ? 1.0 : 0.0) + h[r * NX + c];
      }
      continue;
    }
    Aff<NX> n = m;   // m <- m + H m, and the constant + g
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      n.b[r] += g[r];
#pragma unroll
      for (int q = 0; q < NX; ++q) {
        n.b[r] += h[r * NX + q] * m.b[q];
#pragma unroll
        for (int c = 0; c < NX; ++c) n.A[r][c] += h[r * NX + q] * m.A[q][c];
      }
    }
    m = n;
  }
  wave_scan<NX>(m);
}

template <int NX, bool BACK, typename T>
__global__ __launch_bounds__(64) void k_four_reduce(const double* __restrict__ J, const T* __restrict__ y,
                                                    const ScanDesc* __restrict__ sd, const int2* __restrict__ tiles,
                                                    double* __restrict__ scan) {
  __shared__ FourLds<NX> sm;
  const int2 t = tiles[blockIdx.x];
  const ScanDesc& d = sd[t.x];
  const int R = d.rounds;
  Aff<NX> tm;
#pragma unroll 1
  for (int j = 0; j < R; ++j) {
    const int64_t first = ((int64_t)t.y * R + j) * kFourRound;
    four_load<NX, BACK, T>(d, y, first, sm);
    wave_sync();
    Aff<NX> m;
    four_map<NX, BACK>(sm, d.Nn - first, J + d.jcoff, m);
    wave_sync();
    double* o = four_maps<NX>(scan, d, t.y, j);
#pragma unroll
    for (int r = 0; r < NX; ++r) {
#pragma unroll
      for (int c = 0; c < NX; ++c) o[64 * (c * NX + r)] = m.A[r][c];
      o[64 * (NX * NX + r)] = m.b[r];
    }
    if (j == 0) {
      tm = m;
      continue;
    }
    Aff<NX> n = m;   // of interest in lane 63 only, as tm is
#pragma unroll
    for (int r = 0; r < NX; ++r) {
#pragma unroll
      for (int q = 0; q < NX; ++q) n.b[r] += m.A[r][q] * tm.b[q];
#pragma unroll
      for (int c = 0; c < NX; ++c) {
        double acc = 0.0;
#pragma unroll
        for (int q = 0; q < NX; ++q) acc += m.A[r][q] * tm.A[q][c];
        n.A[r][c] = acc;
      }
    }
    tm = n;
  }
  if (threadIdx.x == 63 && t.y + 1 < d.ntile) {   // the last tile's map is not needed
    double* o = scan + d.tmap + t.y;
#pragma unroll
    for (int r = 0; r < NX; ++r) {
#pragma unroll
      for (int c = 0; c < NX; ++c) o[(int64_t)(c * NX + r) * d.ntile] = tm.A[r][c];
      o[(int64_t)(NX * NX + r) * d.ntile] = tm.b[r];
    }
  }
}

template <int NX, bool BACK, typename T>
__global__ __launch_bounds__(64) void k_four_apply(const double* __restrict__ J, const T* __restrict__ y,
                                                   const ScanDesc* __restrict__ sd, const int2* __restrict__ tiles,
                                                   const double* __restrict__ scan, T* __restrict__ out,
                                                   T* __restrict__ jout, int* flag) {
  constexpr int F = Lay<NX>::F;
  __shared__ FourLds<NX> sm;
  const int2 t = tiles[blockIdx.x];
  const ScanDesc& d = sd[t.x];
  const int R = d.rounds, l = (int)threadIdx.x;
  double s[NX];   // the tile's start state, in every lane
#pragma unroll
  for (int r = 0; r < NX; ++r) s[r] = 0.0;
  auto step = [&](const double* __restrict__ m, int64_t fs) {
    double n[NX];
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      n[r] = m[(NX * NX + r) * fs];
#pragma unroll
      for (int q = 0; q < NX; ++q) n[r] += m[(q * NX + r) * fs] * s[q];
    }
#pragma unroll
    for (int r = 0; r < NX; ++r) s[r] = n[r];
  };
  const int ng = t.y >> 6;
#pragma unroll 4
  for (int q = 0; q < ng; ++q) step(scan + d.gmap + (int64_t)q * F, 1);
  if (t.y & 63) step(scan + d.tmap + t.y - 1, d.ntile);
  const bool keep_v = !BACK && jout;
#pragma unroll 1
  for (int j = 0; j < R; ++j) {
    const int64_t first = ((int64_t)t.y * R + j) * kFourRound;
    four_load<NX, BACK, T>(d, y, first, sm);
    wave_sync();
    double S[NX], e[NX];   // the states before the lane's nodes and after them
    {
      const double* o = four_maps<NX>(scan, d, t.y, j);
#pragma unroll
      for (int r = 0; r < NX; ++r) {
        e[r] = o[64 * (NX * NX + r)];
#pragma unroll
        for (int q = 0; q < NX; ++q) e[r] += o[64 * (q * NX + r)] * s[q];
      }
    }
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      const double before = __shfl_up(e[r], 1, 64);
      S[r] = l == 0 ? s[r] : before;
    }
#pragma unroll
    for (int r = 0; r < NX; ++r) s[r] = lane63(e[r]);
    double vo[kFour][NX];
#pragma unroll
    for (int i = 0; i < kFour; ++i) {
      double h[NX * NX], yn[NX], g[NX], u[NX];
      four_node<NX, BACK>(sm, i, d.Nn - first, J + d.jcoff, h, yn, g, flag);
#pragma unroll
      for (int r = 0; r < NX; ++r) u[r] = S[r] + (BACK ? 0.5 * yn[r] : yn[r]);
      const int a = four_at(l * kFour + i);
#pragma unroll
      for (int r = 0; r < NX; ++r) {
        double v = 0.0;
#pragma unroll
        for (int q = 0; q < NX; ++q) v += h[r * NX + q] * u[q];
        const double x = BACK ? yn[r] + v : u[r] + 0.5 * v;
        S[r] += BACK ? x : v;
        vo[i][r] = v;
        sm.v[r][a] = x;   // xi (x) in place of the lane's own y
      }
    }
    wave_sync();
    auto put = [&](T* __restrict__ o) {
#pragma unroll
      for (int i = 0; i < kFour; ++i) {
        const int64_t pos = first + l + 64 * i;
        if (pos >= d.Nn) continue;
        const int64_t k = BACK ? d.Nn - 1 - pos : pos;
#pragma unroll
        for (int r = 0; r < NX; ++r) o[d.off + (int64_t)r * d.Nn + k] = (T)sm.v[r][four_at(l + 64 * i)];
      }
    };
    put(out);
    wave_sync();
    if (keep_v) {   // J xi = v / w
#pragma unroll
      for (int i = 0; i < kFour; ++i) {
        const int a = four_at(l * kFour + i);
        const double iw = 1.0 / sm.v[NX][a];
#pragma unroll
        for (int r = 0; r < NX; ++r) sm.v[r][a] = vo[i][r] * iw;
      }
      wave_sync();
      put(jout);
      wave_sync();
    }
  }
}

// Instances of at most 64 nodes per wave of the workgroup (d.ntile waves, R = 1): reduce and
// apply in one launch, H_k formed once and kept in LDS.
template <int NX, int MODE, bool BACK, typename T>
__global__ __launch_bounds__(512) void k_scan_small(const double* __restrict__ J, const float* __restrict__ htab,
                                                   const T* __restrict__ y, const ScanDesc* __restrict__ sd,
                                                   const int* __restrict__ list, T* __restrict__ out,
                                                   T* __restrict__ jout, int* flag) {
  constexpr int F = Lay<NX>::F;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const ScanDesc& d = sd[list[blockIdx.x]];
  const int wv = (int)(threadIdx.x >> 6), l = (int)(threadIdx.x & 63), g = l >> 4;
  double* all = reinterpret_cast<double*>(smem_raw);
  double* sm = all + wv * Lay<NX>::SIZE;
  double* mp = sm + Lay<NX>::REC;
  const bool on = wv < d.ntile;
  const int64_t pos = (int64_t)wv * 64 + l;
  Node<NX, MODE> nd;
  double* rec = record<NX>(sm, l);
  if (on) {
    nd.template load<BACK, T>(d, J, htab, y, pos);
    double gv[NX];
    Col<NX> a;
    a.identity();
    form_h<NX, MODE, BACK>(nd, J + d.jcoff, rec, gv, flag);
#pragma unroll
    for (int r = 0; r < NX; ++r) rec[NX * NX + r] = gv[r];
    wave_sync();
    compose_nodes<NX>(sm, a);
    wave_sync();
    scan_chunks<NX>(mp, a);
#pragma unroll
    for (int r = 0; r < NX; ++r) rec[NX * NX + r] = nd.ok ? nd.y[r] : 0.0;
  }
  __syncthreads();
  if (!on) return;
  double s = 0.0;
  for (int q = 0; q < wv; ++q) s = advance<NX>(all + q * Lay<NX>::SIZE + Lay<NX>::REC + (kC - 1) * F, 1, s);
  {
    const double adv = advance<NX>(mp + max(g - 1, 0) * F, 1, s);
    if (g > 0) s = adv;
  }
  replay_nodes<NX, BACK>(sm, s, !BACK && jout);
  store_node<NX, BACK, T>(rec, d, pos, nd.w, out, jout);
}

// H_k of every node in float, H[e][k] as J, for solves of float plans with per-node J.
template <int NX>
__global__ __launch_bounds__(256) void k_make_h(const double* __restrict__ J, float* __restrict__ htab,
                                               const ScanDesc* __restrict__ sd, const int2* __restrict__ tiles, int* flag) {
  const int2 t = tiles[blockIdx.x];
  const ScanDesc& d = sd[t.x];
  const int64_t k = (int64_t)t.y * 256 + threadIdx.x, Nn = d.Nn;
  if (k >= Nn) return;
  const double wk = d.w[k];
  double Jk[NX][NX], K[NX][NX], rp[NX], jmax = 0.0;
#pragma unroll
  for (int r = 0; r < NX; ++r)
#pragma unroll
    for (int q = 0; q < NX; ++q) {
      const double jv = J[d.joff + (int64_t)(r * NX + q) * Nn + k];
      Jk[r][q] = jv;
      jmax = fmax(jmax, fabs(jv));
      K[r][q] = (r == q ? 1.0 : 0.0) - 0.5 * wk * jv;
    }
  lu_kmat<NX>(K, rp, flag, 1.0 + 0.5 * fabs(wk) * jmax);
#pragma unroll
  for (int c = 0; c < NX; ++c) {
    double x[NX];
#pragma unroll
    for (int r = 0; r < NX; ++r) x[r] = wk * Jk[r][c];
    lu_solve<NX>(K, rp, x);
#pragma unroll
    for (int r = 0; r < NX; ++r) htab[d.hoff + (int64_t)(r * NX + c) * Nn + k] = (float)x[r];
  }
}

template <int NX>
int small_waves() {   // waves whose records fit one workgroup
  constexpr int lds = 160 * 1024;
  return std::min(8, lds / (Lay<NX>::SIZE * (int)sizeof(double)));
}

template <int NX, int MODE, bool BACK, typename T>
void launch(birk_plan* p, const ScanClass& sc, const double* J, const T* y, T* out, T* jout, int* flag, hipStream_t s) {
  const float* ht = p->htab;
  if (sc.n_small > 0) {
    const auto f = k_scan_small<NX, MODE, BACK, T>;
    const int bytes = sc.small_waves * Lay<NX>::SIZE * (int)sizeof(double);
    lds_limit(f, small_waves<NX>() * Lay<NX>::SIZE * (int)sizeof(double));
    hipLaunchKernelGGL(f, dim3(sc.n_small), dim3(64 * sc.small_waves), bytes, s, J, ht, y, sc.dev, sc.small, out, jout,
                       flag);
  }
  if constexpr (MODE == kConst && four_nx(NX)) {
    if (sc.four.n_tile > 0) {
      const ScanTiles& f = sc.four;
      const dim3 g(f.n_tile), b(64);
      hipLaunchKernelGGL((k_four_reduce<NX, BACK, T>), g, b, 0, s, J, y, f.dev, f.tiles, p->scan);
      hipLaunchKernelGGL(k_scan_tiles<NX>, dim3(f.n_group), b, 0, s, p->scan, f.dev, f.groups);
      hipLaunchKernelGGL((k_four_apply<NX, BACK, T>), g, b, 0, s, J, y, f.dev, f.tiles, (const double*)p->scan, out, jout,
                         flag);
      return;
    }
  }
  if (sc.n_tile > 0) {
    const dim3 g(sc.n_tile), b(64);
    if constexpr (NX <= kLaneNx)
      hipLaunchKernelGGL((k_lane_reduce<NX, MODE, BACK, T>), g, b, 0, s, J, ht, y, sc.dev, sc.tiles, p->scan);
    else
      hipLaunchKernelGGL((k_scan_reduce<NX, MODE, BACK, T>), g, b, 0, s, J, ht, y, sc.dev, sc.tiles, p->scan);
    if (sc.n_group > 0)
      hipLaunchKernelGGL(k_scan_tiles<NX>, dim3(sc.n_group), b, 0, s, p->scan, sc.dev, sc.groups);
    if constexpr (NX <= kLaneNx)
      hipLaunchKernelGGL((k_lane_apply<NX, MODE, BACK, T>), g, b, 0, s, J, ht, y, sc.dev, sc.tiles,
                         (const double*)p->scan, out, jout, flag);
    else
      hipLaunchKernelGGL((k_scan_apply<NX, MODE, BACK, T>), g, b, 0, s, J, ht, y, sc.dev, sc.tiles,
                         (const double*)p->scan, out, jout, flag);
  }
}

#define SCAN_NX_SWITCH(nx, CALL)                    \
  switch (nx) {                                     \
    case 1: { constexpr int NXC = 1; CALL; } break; \
    case 2: { constexpr int NXC = 2; CALL; } break; \
    case 3: { constexpr int NXC = 3; CALL; } break; \
    case 4: { constexpr int NXC = 4; CALL; } break; \
    case 5: { constexpr int NXC = 5; CALL; } break; \
    case 6: { constexpr int NXC = 6; CALL; } break; \
    case 7: { constexpr int NXC = 7; CALL; } break; \
    case 8: { constexpr int NXC = 8; CALL; } break; \
    default: return hipErrorInvalidValue;           \
  }

// Rounds per tile: all tiles run at once.  A CU holds 8 waves of the kernels at n_x = 5 and
// 4, 5, 7 at n_x = 8, 7, 6 (LDS records).  With fewer slots assumed than there are, tiles get
// longer for nothing (n_x = 6, N = 2^20: 4 a CU 244 us, 7 a CU 227); with more, a second set
// runs for a few tiles.  Below n_x = 5 what counts is the number of groups of 64 tiles that
// the last tiles' start state walks (n_x = 3, 4 at N = 3e5: 12 a CU 33.6 and 44.6 us, 8 a CU
// 34.1 and 54; n_x = 1: 16 a CU 13.8, 24 a CU 15.5).
int scan_rounds(int64_t Nn, int nx) {
  static constexpr int waves[kScanNx + 1] = {0, 16, 16, 12, 12, 8, 7, 5, 4};
  const int64_t per_round = (int64_t)64 * kCus * waves[nx];
  return (int)((Nn + per_round - 1) / per_round);
}

// Four nodes a lane: rounds per tile (8 waves a CU), and the nodes of a class, its one-launch
// instances aside, from which on it is taken.
int four_rounds(int64_t Nn) {
  const int64_t per_round = (int64_t)kFourRound * kCus * 8;
  return (int)((Nn + per_round - 1) / per_round);
}
constexpr int64_t kFourNodes = 100000;

}  // namespace

int64_t scan_scratch(int64_t Nn, int nx) {
  if (nx > kWideNx) return 0;   // no preconditioner
  if (nx > kScanNx) {
    const int64_t R = wide_rounds(Nn), nt = (Nn + kWideNodes * R - 1) / (kWideNodes * R);
    return ((int64_t)nx * nx + nx) * (nt + (nt + kWideGroup - 1) / kWideGroup);
  }
  const int64_t F = (int64_t)nx * nx + nx, R = scan_rounds(Nn, nx), nt = (Nn + 64 * R - 1) / (64 * R);
  const int64_t need = F * (nt * (kC * R + 1) + (nt + 63) / 64);
  if (!four_nx(nx)) return need;
  const int64_t R4 = four_rounds(Nn), nt4 = (Nn + kFourRound * R4 - 1) / (kFourRound * R4);
  return std::max(need, F * (nt4 * (64 * R4 + 1) + (nt4 + 63) / 64));
}

int64_t scan_htab(int64_t Nn, int nx, birk_precision prec) {
  return nx <= kScanNx && prec == BIRK_F32_REFINE_F64 ? Nn * nx * nx : 0;
}

hipError_t plan_scan(birk_plan* p) {
  hipError_t e = hipSuccess;
  p->sclass.clear();
  for (int nx = 1; nx <= kWideNx; ++nx) {
    const bool wide = nx > kScanNx;
    const int per = wide ? kWideNodes : 64, group = wide ? kWideGroup : 64;
    ScanClass sc;
    sc.nx = nx;
    std::vector<ScanDesc> h, h4;
    std::vector<int2> tt, tg, tn, t4, g4;
    std::vector<int> ts;
    int64_t nodes = 0;   // of the instances worked in tiles
    int most = 0;
    if (!wide) SCAN_NX_SWITCH(nx, most = small_waves<NXC>())
    for (const Instance& in : p->inst) {
      if (in.nx != nx) continue;
      const int k = (int)h.size();
      ScanDesc d;
      d.Nn = in.Nn;
      d.off = in.off;
      d.joff = in.joff;
      d.jcoff = in.jcoff;
      d.hoff = in.htab_off;
      d.w = in.w;
      d.rounds = wide ? wide_rounds(in.Nn) : scan_rounds(in.Nn, nx);
      d.ntile = (int)((in.Nn + per * d.rounds - 1) / (per * d.rounds));
      const int64_t F = (int64_t)nx * nx + nx;
      d.cmap = in.scan_off;
      d.tmap = d.cmap + (wide ? 0 : F * kC * d.rounds * d.ntile);
      d.gmap = d.tmap + F * d.ntile;
      h.push_back(d);
      // four nodes a lane
      ScanDesc f = d;
      f.rounds = four_rounds(in.Nn);
      f.ntile = (int)((in.Nn + kFourRound * f.rounds - 1) / (kFourRound * f.rounds));
      f.tmap = d.cmap + 64 * F * f.rounds * f.ntile;
      f.gmap = f.tmap + F * f.ntile;
      h4.push_back(f);
      for (int64_t b = 0; b * 256 < in.Nn; ++b) tn.push_back(make_int2(k, (int)b));
      if (d.ntile <= most) {
        ts.push_back(k);
        sc.small_waves = std::max(sc.small_waves, d.ntile);
        continue;
      }
      for (int b = 0; b < d.ntile; ++b) tt.push_back(make_int2(k, b));
      if (d.ntile > 1)
        for (int b = 0; b * group + 1 < d.ntile; ++b) tg.push_back(make_int2(k, b));
      nodes += in.Nn;
      for (int b = 0; b < f.ntile; ++b) t4.push_back(make_int2(k, b));
      for (int b = 0; b * 64 + 1 < f.ntile; ++b) g4.push_back(make_int2(k, b));
    }
    if (h.empty()) continue;
    sc.n_tile = (int)tt.size();
    sc.n_group = (int)tg.size();
    sc.n_small = (int)ts.size();
    sc.n_nodes = (int)tn.size();
    void* x = nullptr;
    auto up = [&](const void* src, size_t bytes) -> void* {
      if (e == hipSuccess) e = upload_raw(p, src, bytes, &x);
      return e == hipSuccess ? x : nullptr;
    };
    sc.dev = (ScanDesc*)up(h.data(), h.size() * sizeof(ScanDesc));
    sc.tiles = (int2*)up(tt.data(), tt.size() * sizeof(int2));
    sc.groups = (int2*)up(tg.data(), tg.size() * sizeof(int2));
    sc.nodes = (int2*)up(tn.data(), tn.size() * sizeof(int2));
    sc.small = (int*)up(ts.data(), ts.size() * sizeof(int));
    if (four_nx(nx) && nodes >= kFourNodes && !g4.empty()) {
      sc.four.dev = (ScanDesc*)up(h4.data(), h4.size() * sizeof(ScanDesc));
      sc.four.tiles = (int2*)up(t4.data(), t4.size() * sizeof(int2));
      sc.four.groups = (int2*)up(g4.data(), g4.size() * sizeof(int2));
      sc.four.n_tile = (int)t4.size();
      sc.four.n_group = (int)g4.size();
    }
    if (e != hipSuccess) return e;
    p->sclass.push_back(sc);
  }
  return e;
}

hipError_t scan_prepare(birk_plan* p, const double* J, hipStream_t s) {
  for (const ScanClass& sc : p->sclass) {
    if (sc.nx > kScanNx) continue;
    SCAN_NX_SWITCH(sc.nx, hipLaunchKernelGGL(k_make_h<NXC>, dim3(sc.n_nodes), dim3(256), 0, s, J, p->htab, sc.dev,
                                             sc.nodes, p->flag))
  }
  return hipGetLastError();
}

template <typename T>
hipError_t scan_inverse(birk_plan* p, int jac_kind, const double* J, const T* y, T* out, T* jout, int cached,
                        hipStream_t s, int* flag) {
  const bool pn = jac_kind == BIRK_J_PER_NODE;
  for (const ScanClass& sc : p->sclass) {
    if (sc.nx > kScanNx) {
      const hipError_t e = wide_inverse<T>(p, sc, pn, J, y, out, jout, flag, s);
      if (e != hipSuccess) return e;
    } else if (pn && cached && std::is_same<T, float>::value) {
      if constexpr (std::is_same<T, float>::value) {
        SCAN_NX_SWITCH(sc.nx, (launch<NXC, kCachedH, false, T>(p, sc, J, y, out, jout, flag, s)))
      }
    } else if (pn) {
      SCAN_NX_SWITCH(sc.nx, (launch<NXC, kPerNode, false, T>(p, sc, J, y, out, jout, flag, s)))
    } else {
      SCAN_NX_SWITCH(sc.nx, (launch<NXC, kConst, false, T>(p, sc, J, y, out, jout, flag, s)))
    }
  }
  return hipGetLastError();
}

hipError_t scan_inverse_t(birk_plan* p, int jac_kind, const double* J, const double* y, double* out, hipStream_t s) {
  for (const ScanClass& sc : p->sclass) {
    if (sc.nx > kScanNx) {
      const hipError_t e = wide_inverse_t(p, sc, jac_kind == BIRK_J_PER_NODE, J, y, out, s);
      if (e != hipSuccess) return e;
    } else if (jac_kind == BIRK_J_PER_NODE) {
      SCAN_NX_SWITCH(sc.nx, (launch<NXC, kPerNode, true, double>(p, sc, J, y, out, nullptr, nullptr, s)))
    } else {
      SCAN_NX_SWITCH(sc.nx, (launch<NXC, kConst, true, double>(p, sc, J, y, out, nullptr, nullptr, s)))
    }
  }
  return hipGetLastError();
}

#undef SCAN_NX_SWITCH

template hipError_t scan_inverse<double>(birk_plan*, int, const double*, const double*, double*, double*, int,
                                         hipStream_t, int*);
template hipError_t scan_inverse<float>(birk_plan*, int, const double*, const float*, float*, float*, int, hipStream_t,
                                         int*);

}  // namespace birk
