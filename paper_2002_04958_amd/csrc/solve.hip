// Solve-phase structures and kernels: union construction, CF-l1-Jacobi
// half-sweeps, residual, restriction, prolongation, dense coarsest solve,
// and the V(n_pre, n_post) cycle driver.
#include <algorithm>
#include <array>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <fstream>
#include <mutex>
#include <sstream>

#include "kernels.hpp"
#include "rowdot.hpp"
#include "solve.hpp"

namespace mgd {

// ===========================================================================
// union construction
// ===========================================================================
// The rows of a union level are numbered member after member ("natural", see
// RowRanges); ext maps a natural row to its place in extended stored order and
// perm back.  All levels are mapped and measured first, with one readback of
// their sizes, then every level's matrices are gathered row by row straight
// into stored order with their columns mapped on the way.  One set of launches
// serves all members, and the windows of the length order are sorted here: a
// wait per member and step and a sort on the host cost 60 of the 280 ms of a
// step with new coefficients at 3D 64^3, G = 20, and 11.5 of the 21.8 ms of a
// scalar hierarchy of 2D 1024^2.

// one member at one level, as the kernels see it
struct UMember {
  const int* rp;      // its rows of the level matrix, columns ci - cbase local
  const int* ci;
  const double* v;
  const int8_t* cf;   // C/F marker; null where the member has no coarser level
  const int* prp;     // its rows of the interpolation, columns pci - pbase local
  const int* pci;
  const double* pv;
  const int* colour;  // multicolour Gauss-Seidel only
  int cbase, pbase;
  int off, n;         // natural rows [off, off + n)
  int coff;           // its first row at the next level (natural)
  int nc;
  int kind;           // 0 coarsening, 1 relaxed last level, 2 dense last level
  int dense_before;   // rows of kind 2 in the members before it
};

UMember SetupHierarchy::member(size_t l) const {
  UMember u{};
  if (l >= n_levels()) return u;
  const SetupLevel& L = b->levels[l];
  const int r0 = L.off[m];
  u.rp = L.A.rp.get() + r0;
  u.ci = L.A.ci.get();
  u.v = L.A.v.get();
  u.cbase = r0;
  u.n = n(l);
  u.colour = L.colour.p ? L.colour.get() + r0 : nullptr;
  if (!last(l)) {
    u.cf = L.cf.get() + r0;
    u.prp = L.P.rp.get() + r0;
    u.pci = L.P.ci.get();
    u.pv = L.P.v.get();
    u.pbase = L.coff[m];
    u.nc = L.coff[m + 1] - L.coff[m];
  } else {
    u.kind = coarse_kind() == 1 ? 1 : 2;
  }
  return u;
}

// isc[i] = 1 for C rows.  Members without a coarser level are all F.
__global__ void k_u_flags(int n, RowRanges R, const UMember* __restrict__ tab,
                          int* __restrict__ isc) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const UMember m = tab[member_of(R, i)];
  isc[i] = m.cf ? (m.cf[i - m.off] == kC ? 1 : 0) : 0;
}

// extended stored position of every row: C rows in order, then F rows (and rows
// of relaxed last levels), then dense rows.  The candidates are combined by
// arithmetic rather than by a select between kernel arguments under a divergent
// branch.
__global__ void k_u_map(int n, int nC, int nS, RowRanges R, const UMember* __restrict__ tab,
                        const int* __restrict__ isc, const int* __restrict__ cidx,
                        int* __restrict__ ext, int* __restrict__ perm, int* __restrict__ err) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const UMember m = tab[member_of(R, i)];
  const int c = isc[i], d = m.kind == 2 ? 1 : 0;
  const int sc = cidx[i], sf = nC + i - cidx[i] - m.dense_before;
  const int sd = nS + m.dense_before + (i - m.off);
  int s = sf + c * (sc - sf);
  s = s + d * (sd - s);
  ext[i] = s;
  if (s < 0 || s >= n) {
    atomicOr(err, 1);
    return;
  }
  perm[s] = i;
}
// n rows on n places, each place taken (perm starts as -1): a permutation
__global__ void k_u_check(int n, const int* __restrict__ ext, const int* __restrict__ perm,
                          int* __restrict__ err) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const int i = perm[k];
  if (i < 0 || i >= n || ext[i] != k) atomicOr(err, 2);
}

constexpr int kSortWindow = 128;  // two 64-row slices: less padding, gathers stay local

// Windows of the length order: segment q holds rows [row[q], row[q + 1]) and
// windows [win[q], win[q + 1]), the last one cut at the segment's end.
struct SortWindows {
  int nseg = 0;
  int win[2 * kMaxMembers + 1] = {}, row[2 * kMaxMembers + 1] = {};
  void add(int rows) {
    if (rows <= 0) return;
    win[nseg + 1] = win[nseg] + cdiv(rows, kSortWindow);
    row[nseg + 1] = row[nseg] + rows;
    ++nseg;
  }
};

// Rows of each segment in order of decreasing length (stable) within windows of
// kSortWindow rows, one workgroup per window: a row's rank is the number of
// longer rows, and of equally long ones before it.
__global__ void __launch_bounds__(kSortWindow) k_u_window_sort(SortWindows W, RowRanges R,
                                                               const UMember* __restrict__ tab,
                                                               int* __restrict__ ext,
                                                               int* __restrict__ perm,
                                                               const int* __restrict__ err) {
  __shared__ int lens[kSortWindow];
  if (*err) return;
  const int b = blockIdx.x, t = threadIdx.x;
  int q = 0;
  while (q + 1 < W.nseg && W.win[q + 1] <= b) ++q;
  const int w0 = W.row[q] + (b - W.win[q]) * kSortWindow;
  const int w1 = min(W.row[q + 1], w0 + kSortWindow);
  int i = 0, len = -1;
  if (w0 + t < w1) {
    i = perm[w0 + t];
    const UMember m = tab[member_of(R, i)];
    len = m.rp[i - m.off + 1] - m.rp[i - m.off];
  }
  lens[t] = len;
  __syncthreads();
  if (w0 + t >= w1) return;
  int rank = 0;
  for (int u = 0; u < kSortWindow; ++u) rank += (lens[u] > len || (lens[u] == len && u < t)) ? 1 : 0;
  perm[w0 + rank] = i;
  ext[i] = w0 + rank;
}

// the colour of every stored row (multicolour Gauss-Seidel)
__global__ void k_u_colours(int nS, RowRanges R, const UMember* __restrict__ tab,
                            const int* __restrict__ perm, int* __restrict__ col) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= nS) return;
  const int i = perm[k];
  const UMember m = tab[member_of(R, i)];
  col[k] = m.colour[i - m.off];
}

// row lengths in stored order: the level matrix, and W (F rows)
__global__ void k_u_len(int nC, int nS, RowRanges R, const UMember* __restrict__ tab,
                        const int* __restrict__ perm, int* __restrict__ alen,
                        int* __restrict__ wlen, const int* __restrict__ err) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= nS) return;
  if (*err) {  // a malformed map: empty rows, reported with the sizes
    alen[k] = 0;
    if (k >= nC) wlen[k - nC] = 0;
    return;
  }
  const int i = perm[k];
  const UMember m = tab[member_of(R, i)];
  const int r = i - m.off;
  alen[k] = m.rp[r + 1] - m.rp[r];
  if (k >= nC) wlen[k - nC] = m.kind == 0 ? m.prp[r + 1] - m.prp[r] : 0;
}

// 64 x the longest row of every 64-row slice, and the longest row of all: one
// wave per slice.  What bounds it are the additions to the one maximum, about
// 12 ns each one after the other: one per workgroup, of at most kStatBlocks, and
// none that would not raise it.  One per wave of 1024 workgroups took 48 us at
// 2^20 rows, this 5.6 us.
constexpr int kStatBlocks = 512;
__global__ void __launch_bounds__(256) k_row_stats(int rows, const int* __restrict__ rp,
                                                   int* __restrict__ w64, int* longest) {
  __shared__ int s_most[4];
  int most = 0;
  const int ns = (rows + 63) / 64;
  for (int s = blockIdx.x * 4 + (threadIdx.x >> 6); s < ns; s += gridDim.x * 4) {
    const int k = 64 * s + (threadIdx.x & 63);
    int m = k < rows ? rp[k + 1] - rp[k] : 0;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) m = max(m, __shfl_xor(m, off, 64));
    if ((threadIdx.x & 63) == 0) w64[s] = (int)min(64LL * m, (long long)INT_MAX);
    most = max(most, m);
  }
  if ((threadIdx.x & 63) == 0) s_most[threadIdx.x >> 6] = most;
  __syncthreads();
  if (threadIdx.x == 0) {
    most = max(max(s_most[0], s_most[1]), max(s_most[2], s_most[3]));
    // a value read late only costs an addition
    if (most > __hip_atomic_load(longest, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      atomicMax(longest, most);
  }
}

// sizes of one level for the readback (slots may be absent)
__global__ void k_u_sizes(const int* __restrict__ arp, int nS, int nC, const int* __restrict__ wrp,
                          int nF, const int* __restrict__ err, int* __restrict__ out) {
  out[0] = nS > 0 ? arp[nS] : 0;
  out[1] = nS > 0 ? arp[nC] : 0;
  out[2] = nF > 0 ? wrp[nF] : 0;
  out[3] = *err;
}

// GL lanes copy one stored row: entries in source order, columns through the map
template <int GL>
__global__ void __launch_bounds__(256) k_u_rows(int nS, int n, RowRanges R,
                                                const UMember* __restrict__ tab,
                                                const int* __restrict__ perm,
                                                const int* __restrict__ ext,
                                                const int* __restrict__ arp, int* __restrict__ ci,
                                                double* __restrict__ v, int* __restrict__ err) {
  const int k = blockIdx.x * (256 / GL) + threadIdx.x / GL, lane = threadIdx.x % GL;
  if (k >= nS) return;
  const int i = perm[k];
  const UMember m = tab[member_of(R, i)];
  const int e0 = m.rp[i - m.off], len = m.rp[i - m.off + 1] - e0, p = arp[k];
  if (len != arp[k + 1] - p) {  // another length than the row was given
    if (lane == 0) atomicOr(err, 4);
    return;
  }
  for (int e = lane; e < len; e += GL) {
    const int j = m.ci[e0 + e] - m.cbase;
    if (j < 0 || j >= m.n) {
      atomicOr(err, 16);
      ci[p + e] = 0;
      continue;
    }
    ci[p + e] = ext[m.off + j];
    v[p + e] = m.v[e0 + e];
  }
}
// W: the interpolation's F rows, columns in the next level's extended order
template <int GL>
__global__ void __launch_bounds__(256) k_u_wrows(int nC, int nF, RowRanges R,
                                                 const UMember* __restrict__ tab,
                                                 const int* __restrict__ perm,
                                                 const int* __restrict__ ext_next,
                                                 const int* __restrict__ wrp,
                                                 int* __restrict__ ci, double* __restrict__ v,
                                                 int* __restrict__ err) {
  const int f = blockIdx.x * (256 / GL) + threadIdx.x / GL, lane = threadIdx.x % GL;
  if (f >= nF) return;
  const int i = perm[nC + f];
  const UMember m = tab[member_of(R, i)];
  if (m.kind != 0) return;
  const int e0 = m.prp[i - m.off], len = m.prp[i - m.off + 1] - e0, p = wrp[f];
  if (len != wrp[f + 1] - p) {
    if (lane == 0) atomicOr(err, 4);
    return;
  }
  for (int e = lane; e < len; e += GL) {
    const int j = m.pci[e0 + e] - m.pbase;
    if (j < 0 || j >= m.nc) {
      atomicOr(err, 16);
      ci[p + e] = 0;
      continue;
    }
    ci[p + e] = ext_next[m.coff + j];
    v[p + e] = m.pv[e0 + e];
  }
}
// C position <-> the next level's extended index (a C row's interpolation is
// its one coarse point)
__global__ void k_u_cmap(int nC, int n_next, RowRanges R, const UMember* __restrict__ tab,
                         const int* __restrict__ perm, const int* __restrict__ ext_next,
                         int* __restrict__ cmap, int* __restrict__ cpos, int* __restrict__ err) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= nC) return;
  const int i = perm[k];
  const UMember m = tab[member_of(R, i)];
  const int j = m.pci[m.prp[i - m.off]] - m.pbase;
  if (j < 0 || j >= m.nc || m.coff + j >= n_next) {
    atomicOr(err, 64);
    cmap[k] = 0;
    return;
  }
  const int x = ext_next[m.coff + j];
  cmap[k] = x;
  cpos[x] = k;
}
// every C position is the one its coarse point names
__global__ void k_u_cmap_check(int nC, const int* __restrict__ cmap, const int* __restrict__ cpos,
                               int* __restrict__ err) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < nC && cpos[cmap[k]] != k) atomicOr(err, 8);
}
// 1 / l1 diagonal of the stored rows (a_kk, then |a_kj| in entry order), and
// 1 / a_kk where wanted
// GL lanes per row read its entries side by side; the sum adds them in order (a
// lane per row took 1.42 ms for the unions at 3D 64^3, G = 20, this 0.70 ms).
template <int GL, typename T>
__global__ void __launch_bounds__(256) k_u_dinv(int nS, const int* __restrict__ rp,
                                                const int* __restrict__ ci,
                                                const double* __restrict__ v,
                                                T* __restrict__ dinv, T* __restrict__ dgs) {
  const int k = blockIdx.x * (256 / GL) + threadIdx.x / GL, lane = threadIdx.x % GL;
  if (k >= nS) return;
  const int e0 = rp[k], e1 = rp[k + 1];
  double dg = 0.0;
  bool has = false;
  for (int e = e0 + lane; e < e1; e += GL)
    if (ci[e] == k) {
      dg = v[e];
      has = true;
    }
#pragma unroll
  for (int o = GL / 2; o > 0; o >>= 1) {
    const double od = __shfl_xor(dg, o, GL);
    if (__shfl_xor((int)has, o, GL) && !has) {
      dg = od;
      has = true;
    }
  }
  double acc = dg;
  for (int b = e0; b < e1; b += GL) {
    const int e = b + lane;
    const bool off = e < e1 && ci[e] != k;
    const double a = off ? fabs(v[e]) : 0.0;  // adding 0 to the sum changes nothing
    const int cnt = min(GL, e1 - b);
    for (int q = 0; q < cnt; ++q) acc = acc + __shfl(a, q, GL);
  }
  if (lane == 0) {
    dinv[k] = (T)(1.0 / acc);
    if (dgs) dgs[k] = (T)(1.0 / dg);
  }
}
template <typename T>
__global__ void k_dinv_nat(int n, int nC, const int* __restrict__ iperm,
                           const T* __restrict__ dinv, T* __restrict__ dn) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= n) return;
  const int k = iperm[p];
  dn[p] = k < nC ? dinv[k] : (T)0;
}

static void row_stats(Ctx* c, int rows, const int* rp, DBuf<int>& w64, DBuf<int>& soff,
                      int* longest);

// Level products between the mapping pass and the layouts.
template <typename T>
struct BuildLevel {
  int n = 0, nS = 0, nC = 0, nF = 0, n_coarse = 0;
  RowRanges R;
  size_t tab = 0;            // its members in the device table
  bool bottom = false;       // runs one member per workgroup (or may, see build_bottom)
  long long want_a = 0, want_w = 0;  // entries the stored matrix and W must end with
  DBuf<int> ext, perm;       // natural -> extended stored order, and back
  DBuf<int> arp, wrp;
  DBuf<int> aw64, asoff, ww64, wsoff, tw64, tsoff;  // SELL widths and offsets (A, W, W^T)
  Csr<double> A, W, Wt;      // stored order
};
template <typename T>
static void layout_levels(Ctx* c, std::vector<BuildLevel<T>>& bl, const int* stats, Union<T>& U,
                          int autotune);
template <typename T>
static void build_bottom(Ctx* c, std::vector<BuildLevel<T>>& bl, const std::vector<UMember>& tab,
                         int cand, const int* widths_dev, const std::vector<int>& widths,
                         Union<T>& U);
template <typename T>
static std::vector<int> bot_widths(Ctx* c, const std::vector<BuildLevel<T>>& bl,
                                   const std::vector<UMember>& tab, int cand, DBuf<int>& out);
static long long sell_min_rows();
static long long tune_min_rows();
constexpr int kBotRows = 2048;
// rows of a member in the F-block (F points, or a relaxed last level)
static int f_rows(const UMember& m) { return m.kind == 0 ? m.n - m.nc : (m.kind == 1 ? m.n : 0); }

static long long env_ll(const char* name, long long dflt) {
  const char* e = std::getenv(name);
  return e && *e ? std::atoll(e) : dflt;
}

// Host-side verification of a union level (MGD_DEBUG_UNION=1): the map is a
// permutation and every stored row equals its source row.  Throws with the
// first mismatch; used to diagnose, never needed for correct operation.
static bool debug_union() {
  static const bool on = [] {
    const char* e = std::getenv("MGD_DEBUG_UNION");
    return e && e[0] == '1';
  }();
  return on;
}
template <typename T>
static void verify_union_level(Ctx* c, const std::vector<UMember>& tab, const BuildLevel<T>& b) {
  std::vector<int> ext(b.n), arp((size_t)b.nS + 1), aci((size_t)std::max(b.A.nnz, 1)), seen(b.n, 0);
  std::vector<double> av((size_t)std::max(b.A.nnz, 1));
  copy_d2h(c, ext.data(), b.ext.get(), (size_t)b.n);
  if (b.nS > 0) copy_d2h(c, arp.data(), b.A.rp.get(), (size_t)b.nS + 1);
  copy_d2h(c, aci.data(), b.A.ci.get(), (size_t)b.A.nnz);
  copy_d2h(c, av.data(), b.A.v.get(), (size_t)b.A.nnz);
  for (int q = 0; q < b.R.nm; ++q) {
    const UMember& m = tab[b.tab + q];
    if (m.n == 0) continue;
    std::vector<int> rp((size_t)m.n + 1);
    copy_d2h(c, rp.data(), m.rp, (size_t)m.n + 1);
    const int e0 = rp[0], ne = rp[m.n] - e0;
    std::vector<int> ci((size_t)std::max(ne, 1));
    std::vector<double> v((size_t)std::max(ne, 1));
    copy_d2h(c, ci.data(), m.ci + e0, (size_t)ne);
    copy_d2h(c, v.data(), m.v + e0, (size_t)ne);
    for (int i = 0; i < m.n; ++i) {
      const int s = ext[m.off + i];
      const std::string at = "member " + std::to_string(q) + " row " + std::to_string(i) +
                             " -> stored " + std::to_string(s);
      if (s < 0 || s >= b.n) fail(MGD_EHIP, "union debug: " + at + " out of range");
      if (seen[s]++) fail(MGD_EHIP, "union debug: " + at + " taken twice");
      if ((m.kind == 2) != (s >= b.nS)) fail(MGD_EHIP, "union debug: " + at + " in the wrong region");
      if (m.kind == 2) continue;
      const int len = rp[i + 1] - rp[i];
      if (arp[s + 1] - arp[s] != len)
        fail(MGD_EHIP, "union debug: " + at + " length " + std::to_string(arp[s + 1] - arp[s]) +
                           ", source " + std::to_string(len));
      for (int k = 0; k < len; ++k)
        if (aci[(size_t)arp[s] + k] != ext[m.off + ci[(size_t)rp[i] - e0 + k] - m.cbase] ||
            av[(size_t)arp[s] + k] != v[(size_t)rp[i] - e0 + k])
          fail(MGD_EHIP, "union debug: " + at + " entry " + std::to_string(k) + " differs");
    }
  }
}

// multicolour Gauss-Seidel: stored rows of each block in order of their colour
template <typename T>
static void colour_order(Ctx* c, BuildLevel<T>& b, const UMember* tab,
                         std::vector<std::array<int, 4>>& cranges) {
  const int nS = b.nS, nC = b.nC;
  DBuf<int> cold(c, (size_t)nS);
  hipLaunchKernelGGL(k_u_colours, dim3(cdiv(nS, 256)), dim3(256), 0, c->stream, nS, b.R, tab,
                     (const int*)b.perm.get(), cold.get());
  MGD_CHECK_LAUNCH();
  std::vector<int> col(nS), pm(nS), order(nS), ext(b.n);
  copy_d2h(c, col.data(), cold.get(), (size_t)nS);
  copy_d2h(c, pm.data(), b.perm.get(), (size_t)nS);
  copy_d2h(c, ext.data(), b.ext.get(), (size_t)b.n);
  for (int k = 0; k < nS; ++k) order[k] = k;
  auto by_col = [&](int x, int y) { return col[x] < col[y]; };
  std::stable_sort(order.begin(), order.begin() + nC, by_col);
  std::stable_sort(order.begin() + nC, order.end(), by_col);
  int ncol = 0;
  for (int k = 0; k < nS; ++k) ncol = std::max(ncol, col[k] + 1);
  cranges.assign(ncol, {nC, nC, nS, nS});
  for (int k = nS - 1; k >= 0; --k) cranges[col[order[k]]][k < nC ? 0 : 2] = k;
  for (int k = 0; k < nS; ++k) cranges[col[order[k]]][k < nC ? 1 : 3] = k + 1;
  for (auto& r : cranges) {  // colours absent from a block: empty range
    if (r[1] <= r[0]) r[0] = r[1] = 0;
    if (r[3] <= r[2]) r[2] = r[3] = 0;
  }
  std::vector<int> pm2(nS);
  for (int k = 0; k < nS; ++k) {
    pm2[k] = pm[order[k]];
    MGD_REQUIRE(pm2[k] >= 0 && pm2[k] < b.n, "internal: malformed stored-row map");
    ext[pm2[k]] = k;
  }
  copy_h2d(c, b.perm.get(), pm2.data(), (size_t)nS);
  copy_h2d(c, b.ext.get(), ext.data(), (size_t)b.n);
}

template <typename T>
std::unique_ptr<Union<T>> build_union(Ctx* c, const std::vector<const SetupHierarchy*>& members,
                                      int n_pre, int n_post, int autotune, int smoother) {
  DeferFrees frees(c);
  auto U = std::make_unique<Union<T>>();
  U->n_pre = n_pre;
  U->n_post = n_post;
  U->gs = smoother == 1;
  U->members = (int)members.size();
  MGD_REQUIRE(members.size() <= (size_t)kMaxMembers, "internal: too many members in a union");
  size_t maxL = 0;
  for (auto* H : members) maxL = std::max(maxL, H->n_levels());
  // host side: the levels' sizes and the members' places in them
  std::vector<BuildLevel<T>> bl;
  std::vector<UMember> tab;
  for (size_t l = 0; l < maxL; ++l) {
    BuildLevel<T> b;
    b.tab = tab.size();
    b.R.nm = (int)members.size();
    int dense = 0;
    for (size_t q = 0; q < members.size(); ++q) {
      const SetupHierarchy* H = members[q];
      UMember m = H->member(l);
      m.off = b.n;
      m.coff = b.n_coarse;
      m.dense_before = dense;
      b.R.off[q] = b.n;
      if (m.n > 0) {
        if (m.kind == 2)
          dense += m.n;
        else
          b.want_a += H->nnz(l);
        if (m.kind == 0) b.want_w += H->nnz_P(l) - m.nc;
      }
      b.n += m.n;
      b.nC += m.nc;
      b.n_coarse += m.nc;
      tab.push_back(m);
    }
    b.R.off[b.R.nm] = b.n;
    b.nS = b.n - dense;
    b.nF = b.nS - b.nC;
    MGD_REQUIRE(b.want_a < INT32_MAX && b.want_w < INT32_MAX, "union too large for int32 indices");
    bl.push_back(std::move(b));
    if (bl.back().n_coarse == 0) break;
  }
  const int nl = (int)bl.size();
  DBuf<UMember> dtab(c, std::max<size_t>(tab.size(), 1));
  copy_h2d(c, dtab.get(), tab.data(), tab.size());
  // first level from which every member is small enough for one workgroup
  int cand = nl;
  if (smoother != 1)
    while (cand > 0) {
      const BuildLevel<T>& b = bl[cand - 1];
      // (levels whose layouts may be tuned or sliced are not, tuned now or before)
      bool ok = b.nS < std::min(sell_min_rows(), tune_min_rows());
      for (int q = 0; q < b.R.nm; ++q) ok = ok && tab[b.tab + q].n <= kBotRows;
      if (!ok) break;
      --cand;
    }
  U->L.resize(nl);
  int* err = c->err_flag();
  // maps and row lengths of every level
  DBuf<int> sizes(c, (size_t)nl * 4), stats(c, (size_t)nl * 6);
  fill<int>(c, stats.get(), 0, (size_t)nl * 6);
  for (int l = 0; l < nl; ++l) {
    StepScope st("solve-phase build: order of level " + std::to_string(l) + " of " +
                 std::to_string(members.size()) + " hierarchies");
    BuildLevel<T>& b = bl[l];
    const UMember* dt = dtab.get() + b.tab;
    const int n = b.n, g = cdiv(std::max(n, 1), 256);
    b.ext.alloc(c, (size_t)std::max(n, 1));
    b.perm.alloc(c, (size_t)std::max(n, 1));
    fill<int>(c, b.perm.get(), -1, (size_t)n);
    if (n > 0) {
      DBuf<int> isc(c, (size_t)n), cidx(c, (size_t)n + 1);
      hipLaunchKernelGGL(k_u_flags, dim3(g), dim3(256), 0, c->stream, n, b.R, dt, isc.get());
      MGD_CHECK_LAUNCH();
      exclusive_scan(c, isc.get(), cidx.get(), n);
      hipLaunchKernelGGL(k_u_map, dim3(g), dim3(256), 0, c->stream, n, b.nC, b.nS, b.R, dt,
                         (const int*)isc.get(), (const int*)cidx.get(), b.ext.get(), b.perm.get(),
                         err);
      hipLaunchKernelGGL(k_u_check, dim3(g), dim3(256), 0, c->stream, n, (const int*)b.ext.get(),
                         (const int*)b.perm.get(), err);
      MGD_CHECK_LAUNCH();
    }
    // Below the finest level, rows of the C-block and of the F-block are ordered
    // by decreasing length (stable) within windows of kSortWindow rows, so that
    // 64-row slices hold rows of similar length while neighbouring rows stay
    // close.  With multicolour Gauss-Seidel the blocks are ordered by colour
    // instead, so each colour is one range of the C-block and one of the F-block.
    if (b.nS > 0 && smoother == 1) {
      c->check_device_errors("stored-row map of a solve-phase level");
      colour_order(c, b, dt, U->L[l].cranges);
    } else if (b.nS > 0 && l > 0) {
      // levels that may run one member per workgroup keep a member's rows together
      SortWindows win;
      if (l >= cand) {
        for (int q = 0; q < b.R.nm; ++q) win.add(tab[b.tab + q].nc);
        for (int q = 0; q < b.R.nm; ++q) win.add(f_rows(tab[b.tab + q]));
      } else {
        win.add(b.nC);
        win.add(b.nF);
      }
      hipLaunchKernelGGL(k_u_window_sort, dim3(win.win[win.nseg]), dim3(kSortWindow), 0, c->stream,
                         win, b.R, dt, b.ext.get(), b.perm.get(), (const int*)err);
      MGD_CHECK_LAUNCH();
    }
    DBuf<int> alen(c, (size_t)std::max(b.nS, 1)), wlen(c, (size_t)std::max(b.nF, 1));
    b.arp.alloc(c, (size_t)b.nS + 1);
    b.wrp.alloc(c, (size_t)b.nF + 1);
    if (b.nS > 0) {
      hipLaunchKernelGGL(k_u_len, dim3(cdiv(b.nS, 256)), dim3(256), 0, c->stream, b.nC, b.nS, b.R,
                         dt, (const int*)b.perm.get(), alen.get(), wlen.get(), (const int*)err);
      MGD_CHECK_LAUNCH();
    }
    exclusive_scan(c, alen.get(), b.arp.get(), b.nS);
    exclusive_scan(c, wlen.get(), b.wrp.get(), b.nF);
    row_stats(c, b.nS, b.arp.get(), b.aw64, b.asoff, stats.get() + 6 * l);
    row_stats(c, b.nF, b.wrp.get(), b.ww64, b.wsoff, stats.get() + 6 * l + 2);
    hipLaunchKernelGGL(k_u_sizes, dim3(1), dim3(1), 0, c->stream, (const int*)b.arp.get(), b.nS,
                       b.nC, (const int*)b.wrp.get(), b.nF, (const int*)err, sizes.get() + 4 * l);
    MGD_CHECK_LAUNCH();
  }
  const std::vector<int> sz = read_vec(c, sizes.get(), (size_t)nl * 4);
  c->throw_device_errors(nl ? sz[4 * nl - 1] : 0, "stored order of the solve-phase levels");
  // matrices in stored order
  for (int l = 0; l < nl; ++l) {
    StepScope st("solve-phase build: matrices of level " + std::to_string(l));
    BuildLevel<T>& b = bl[l];
    const UMember* dt = dtab.get() + b.tab;
    ULevel<T>& lv = U->L[l];
    if (sz[4 * l] != b.want_a || sz[4 * l + 2] != b.want_w)
      fail(MGD_EHIP, "internal check failed: stored level matrix has " + std::to_string(sz[4 * l]) +
                         " entries and W " + std::to_string(sz[4 * l + 2]) + ", their members " +
                         std::to_string(b.want_a) + " and " + std::to_string(b.want_w) +
                         step_suffix());
    const bool coarsens = l + 1 < nl && b.n_coarse > 0;
    lv.n = lv.nX = b.n;
    lv.nS = b.nS;
    lv.nC = b.nC;
    lv.nnz_C = sz[4 * l + 1];
    lv.nnz_F = b.want_a - lv.nnz_C;
    lv.dinv.alloc(c, (size_t)std::max(b.nS, 1));
    if (smoother == 1) lv.dgs.alloc(c, (size_t)std::max(b.nS, 1));
    b.A.n_rows = b.nS;
    b.A.n_cols = b.nS;
    b.A.nnz = (int)b.want_a;
    b.A.rp = std::move(b.arp);
    b.A.ci.alloc(c, (size_t)std::max(b.A.nnz, 1));
    b.A.v.alloc(c, (size_t)std::max(b.A.nnz, 1));
    // lanes per copied row: about the mean row length
#define MGD_ROWS_GL(K, N_, GL, ...)                                                                \
  hipLaunchKernelGGL(K<GL>, dim3(cdiv(N_, 256 / GL)), dim3(256), 0, c->stream, __VA_ARGS__)
#define MGD_ROWS(K, N_, AVG, ...)                                                                  \
  switch (fit_lanes(N_, (AVG) <= 10.0 ? 8 : (AVG) <= 24.0 ? 16 : 64)) {                            \
    case 1: MGD_ROWS_GL(K, N_, 1, __VA_ARGS__); break;                                             \
    case 8: MGD_ROWS_GL(K, N_, 8, __VA_ARGS__); break;                                             \
    case 16: MGD_ROWS_GL(K, N_, 16, __VA_ARGS__); break;                                           \
    default: MGD_ROWS_GL(K, N_, 64, __VA_ARGS__);                                                  \
  }                                                                                                \
  MGD_CHECK_LAUNCH()
    if (b.nS > 0) {
      const double avg = (double)b.A.nnz / b.nS;
      MGD_ROWS(k_u_rows, b.nS, avg, b.nS, b.n, b.R, dt, (const int*)b.perm.get(),
               (const int*)b.ext.get(), (const int*)b.A.rp.get(), b.A.ci.get(), b.A.v.get(), err);
      auto dinv = [&](auto kernel, int lanes) {
        hipLaunchKernelGGL(kernel, dim3(cdiv(b.nS, 256 / lanes)), dim3(256), 0, c->stream, b.nS,
                           (const int*)b.A.rp.get(), (const int*)b.A.ci.get(),
                           (const double*)b.A.v.get(), lv.dinv.get(), lv.dgs.get());
        MGD_CHECK_LAUNCH();
      };
      switch (fit_lanes(b.nS, avg <= 10.0 ? 8 : 16)) {
        case 1: dinv(k_u_dinv<1, T>, 1); break;
        case 8: dinv(k_u_dinv<8, T>, 8); break;
        default: dinv(k_u_dinv<16, T>, 16);
      }
    }
    check_structure_async(c, b.nS, b.nS, b.A.nnz, b.A.rp.get(), b.A.ci.get(), false, true);
    // dense members: offsets in the extended order
    for (int q = 0; q < b.R.nm; ++q) {
      const UMember& m = tab[b.tab + q];
      if (m.n == 0 || m.kind != 2) continue;
      lv.dense.push_back({b.nS + m.dense_before, m.n, members[q]->inverse()});
      lv.dense_max_n = std::max(lv.dense_max_n, m.n);
      lv.dense_entries += (long long)m.n * m.n;
    }
    if (!lv.dense.empty()) {
      lv.dense_dev.alloc(c, lv.dense.size());
      copy_h2d(c, lv.dense_dev.get(), lv.dense.data(), lv.dense.size());
    }
    if (coarsens) {
      BuildLevel<T>& nb = bl[l + 1];
      MGD_REQUIRE(nb.n == b.n_coarse && b.nC == b.n_coarse,
                  "internal: coarse level size differs from the C-block");
      lv.nX_next = nb.n;
      lv.nC_next = nb.nC;
      lv.nS_next = nb.nS;
      b.W.n_rows = b.nF;
      b.W.n_cols = nb.n;
      b.W.nnz = (int)b.want_w;
      b.W.rp = std::move(b.wrp);
      b.W.ci.alloc(c, (size_t)std::max(b.W.nnz, 1));
      b.W.v.alloc(c, (size_t)std::max(b.W.nnz, 1));
      if (b.nF > 0) {
        const double avg = (double)b.W.nnz / b.nF;
        MGD_ROWS(k_u_wrows, b.nF, avg, b.nC, b.nF, b.R, dt, (const int*)b.perm.get(),
                 (const int*)nb.ext.get(), (const int*)b.W.rp.get(), b.W.ci.get(), b.W.v.get(),
                 err);
      }
#undef MGD_ROWS
#undef MGD_ROWS_GL
      // C-block position -> level l+1 index; level l+1 index -> C-block position
      lv.cmap.alloc(c, (size_t)std::max(b.nC, 1));
      lv.cpos.alloc(c, (size_t)std::max(nb.n, 1));
      fill<int>(c, lv.cpos.get(), 0, (size_t)nb.n);
      hipLaunchKernelGGL(k_u_cmap, dim3(cdiv(b.nC, 256)), dim3(256), 0, c->stream, b.nC, nb.n, b.R,
                         dt, (const int*)b.perm.get(), (const int*)nb.ext.get(), lv.cmap.get(),
                         lv.cpos.get(), err);
      hipLaunchKernelGGL(k_u_cmap_check, dim3(cdiv(b.nC, 256)), dim3(256), 0, c->stream, b.nC,
                         (const int*)lv.cmap.get(), (const int*)lv.cpos.get(), err);
      MGD_CHECK_LAUNCH();
      check_structure_async(c, b.nF, nb.n, b.W.nnz, b.W.rp.get(), b.W.ci.get(), false, true);
      // W^T: rows in level l+1 extended order, columns F indices ascending
      transpose(c, b.W, b.Wt);
      row_stats(c, b.Wt.n_rows, b.Wt.rp.get(), b.tw64, b.tsoff, stats.get() + 6 * l + 4);
    }
    if (debug_union()) verify_union_level(c, tab, b);
  }
  DBuf<int> widths;  // slice widths of each member's rows at the candidate bottom levels
  const std::vector<int> hw = bot_widths(c, bl, tab, cand, widths);
  const std::vector<int> hs = read_vec(c, stats.get(), (size_t)nl * 6);
  c->check_device_errors("stored-order matrices of the solve-phase levels");
  build_bottom<T>(c, bl, tab, cand, widths.get(), hw, *U);
  layout_levels<T>(c, bl, hs.data(), *U, autotune);
  if (nl > 0) {
    // level 0 seen from the natural side, for entry kernels that read their
    // inputs in natural order: the inverse permutation and d^-1 of C rows
    ULevel<T>& l0 = U->L[0];
    const int nX = l0.nX, g = cdiv(std::max(nX, 1), 256);
    l0.iperm = std::move(bl[0].ext);
    l0.dinv_nat.alloc(c, (size_t)std::max(nX, 1));
    if (nX > 0) {
      hipLaunchKernelGGL(k_dinv_nat<T>, dim3(g), dim3(256), 0, c->stream, nX, l0.nC,
                         (const int*)l0.iperm.get(), (const T*)l0.dinv.get(), l0.dinv_nat.get());
      MGD_CHECK_LAUNCH();
    }
  }
  U->build_tail(c);
  c->check_device_errors("solve-phase build");
  return U;
}

// ===========================================================================
// solve kernels (stored order)
// ===========================================================================
// Iterate gathers.  A level's iterate has a C region [0, nC) and an F region
// [nC, nS) that alternate independently between two buffers, and a dense
// region [nS, nX) kept in the first buffer.  The region is chosen by index
// arithmetic on a buffer distance (a select of values, never a branch).
template <typename T>
struct GatherCF {
  const T* base;        // buffer holding the C region
  ptrdiff_t f_minus_c;  // (buffer holding the F region) - base, in elements
  int nC;
  __device__ __forceinline__ T operator()(int j) const {
    return base[j + (j < nC ? 0 : f_minus_c)];
  }
};
template <typename T>
struct GatherCFD {
  const T* base;  // C region buffer
  ptrdiff_t f_minus_c, d_minus_c;
  int nC, nS;
  __device__ __forceinline__ T operator()(int j) const {
    const ptrdiff_t o = j < nC ? 0 : (j < nS ? f_minus_c : d_minus_c);
    return base[j + o];
  }
};
template <typename T>
struct Gather1 {
  const T* x;
  __device__ __forceinline__ T operator()(int j) const { return x[j]; }
};
template <typename T>
struct GatherPerm {  // natural vector seen in stored order
  const T* x;
  const int* perm;
  __device__ __forceinline__ T operator()(int j) const { return x[perm[j]]; }
};
template <typename T>
struct GatherCOnly {  // first F half-sweep: F values are still zero
  const T* xc;
  int nC;
};

// position of row `row` in its slice: o its first value, oc its first column
// code, w the slice width; for SELL16 the slice's two column bases (fb < 0:
// the slice keeps 32-bit columns, oc then counts 32-bit words)
template <int FMT>
__device__ __forceinline__ void sell_slice(const int* __restrict__ rp, int row, int& o, int& oc,
                                           int& w, int& cb, int& fb) {
  if (FMT == kFmtSELL16) {
    const int s4 = 4 * (row >> 6);
    o = rp[s4] + (row & 63);
    w = (rp[s4 + 4] - rp[s4]) >> 6;
    cb = rp[s4 + 2];
    fb = rp[s4 + 3];
    oc = (fb < 0 ? rp[s4 + 1] >> 1 : rp[s4 + 1]) + (row & 63);
  } else {
    o = rp[row >> 6] + (row & 63);
    oc = o;
    w = (rp[(row >> 6) + 1] - rp[row >> 6]) >> 6;
    cb = fb = 0;
  }
}
__device__ __forceinline__ int sell16_decode(unsigned u, int cb, int fb) {
  return (u & 0x8000u) ? fb + (int)(u & 0x7fffu) : cb + (int)u;
}
// column of code idx of a sliced layout: a 16-bit code (NARROW) or a 32-bit column
template <bool NARROW>
__device__ __forceinline__ int sell_col(const int* __restrict__ ci, int idx, int cb, int fb) {
  if (NARROW) return sell16_decode(reinterpret_cast<const uint16_t*>(ci)[idx], cb, fb);
  return ci[idx];
}
// sum of a_rj g(j) over one sliced row (values from o, column codes from oc)
template <bool NARROW, typename T, typename G>
__device__ __forceinline__ T sell_row(const int* __restrict__ ci, const T* __restrict__ v,
                                      const G& g, int o, int oc, int w, int cb, int fb) {
  T s = 0;
  int e = 0;
  for (; e + 4 <= w; e += 4) {  // four entries' loads in flight (sum order unchanged)
    int j[4];
    T a[4], x[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) j[q] = sell_col<NARROW>(ci, oc + 64 * (e + q), cb, fb);
#pragma unroll
    for (int q = 0; q < 4; ++q) a[q] = v[o + 64 * (e + q)];
#pragma unroll
    for (int q = 0; q < 4; ++q) x[q] = g(j[q]);
#pragma unroll
    for (int q = 0; q < 4; ++q) s += a[q] * x[q];
  }
  for (; e < w; ++e) s += v[o + 64 * e] * g(sell_col<NARROW>(ci, oc + 64 * e, cb, fb));
  return s;
}
// the same over the C columns only (j < nC), F columns weighted zero
template <bool NARROW, typename T>
__device__ __forceinline__ T sell_row_c(const int* __restrict__ ci, const T* __restrict__ v,
                                        const T* __restrict__ xc, int nC, int o, int oc, int w,
                                        int cb, int fb) {
  T s = 0;
  int e = 0;
  for (; e + 4 <= w; e += 4) {
    int j[4];
    T a[4], x[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) j[q] = sell_col<NARROW>(ci, oc + 64 * (e + q), cb, fb);
#pragma unroll
    for (int q = 0; q < 4; ++q) a[q] = j[q] < nC ? v[o + 64 * (e + q)] : (T)0;
#pragma unroll
    for (int q = 0; q < 4; ++q) x[q] = xc[j[q] < nC ? j[q] : 0];
#pragma unroll
    for (int q = 0; q < 4; ++q) s += a[q] * x[q];
  }
  for (; e < w; ++e) {
    const int j = sell_col<NARROW>(ci, oc + 64 * e, cb, fb);
    if (j < nC) s += v[o + 64 * e] * xc[j];
  }
  return s;
}

// The same sums for a wave whose 64 lanes are the 64 rows of one slice (the
// launch is aligned to slices): the slice header is read once into scalar
// registers, and the entries go in groups of eight with every column code and
// value of a group in flight together, then every gather of the group.  The
// entries past the row width in the last group load the last entry again and
// are not added, so the sum, its order and its rounding are those above.
template <bool NARROW, typename T, typename G>
__device__ __forceinline__ T sell_row8(const int* __restrict__ ci, const T* __restrict__ v,
                                       const G& g, int o, int oc, int w, int cb, int fb) {
  T s = 0;
  for (int e = 0; e < w; e += 8) {
    int j[8];
    T a[8], x[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int eq = min(e + q, w - 1);
      j[q] = sell_col<NARROW>(ci, oc + 64 * eq, cb, fb);
      a[q] = v[o + 64 * eq];
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) x[q] = g(j[q]);
#pragma unroll
    for (int q = 0; q < 8; ++q)
      if (e + q < w) s += a[q] * x[q];
  }
  return s;
}
// C columns only: an F column's product is zero (adding a zero product leaves
// the sum as it is: a sum that starts at +0 is never -0)
template <bool NARROW, typename T>
__device__ __forceinline__ T sell_row8_c(const int* __restrict__ ci, const T* __restrict__ v,
                                         const T* __restrict__ xc, int nC, int o, int oc, int w,
                                         int cb, int fb) {
  T s = 0;
  for (int e = 0; e < w; e += 8) {
    int j[8];
    T a[8], x[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int eq = min(e + q, w - 1);
      j[q] = sell_col<NARROW>(ci, oc + 64 * eq, cb, fb);
      a[q] = v[o + 64 * eq];
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) x[q] = xc[j[q] < nC ? j[q] : 0];
#pragma unroll
    for (int q = 0; q < 8; ++q)
      if (e + q < w && j[q] < nC) s += a[q] * x[q];
  }
  return s;
}
// slice header of the wave's slice (uniform), then the lane's row in it
template <int FMT>
__device__ __forceinline__ void sell_slice_wave(const int* __restrict__ rp, int row, int& o,
                                                int& oc, int& w, int& cb, int& fb) {
  const int r64 = __builtin_amdgcn_readfirstlane(row & ~63);
  sell_slice<FMT>(rp, r64, o, oc, w, cb, fb);
  o += row & 63;
  oc += row & 63;
}

// sum over row `row` of a_rj g(j), entries in stored order; SELL uses one
// lane per row, CSR `TPR` lanes of a wavefront per row (butterfly combine).
// WAVE: sliced rows of a launch aligned to slices (every lane of a wave in the
// same slice)
template <int FMT, int TPR, bool WAVE = false, typename T, typename G>
__device__ __forceinline__ T mrow(const int* __restrict__ rp, const int* __restrict__ ci,
                                  const T* __restrict__ v, const G& g, int row, int lane) {
  T s = 0;
  if ((FMT == kFmtSELL || FMT == kFmtSELL16) && WAVE) {
    int o, oc, w, cb, fb;
    sell_slice_wave<FMT>(rp, row, o, oc, w, cb, fb);
    if (FMT == kFmtSELL16 && fb >= 0)
      s = sell_row8<true>(ci, v, g, o, oc, w, cb, fb);
    else
      s = sell_row8<false>(ci, v, g, o, oc, w, cb, fb);
  } else if (FMT == kFmtSELL || FMT == kFmtSELL16) {
    int o, oc, w, cb, fb;
    sell_slice<FMT>(rp, row, o, oc, w, cb, fb);
    // a slice is 16-bit or 32-bit as a whole: lanes diverge only in the waves
    // that straddle two slices
    if (FMT == kFmtSELL16 && fb >= 0)
      s = sell_row<true>(ci, v, g, o, oc, w, cb, fb);
    else
      s = sell_row<false>(ci, v, g, o, oc, w, cb, fb);
  } else {
    // eight of the lane's entries at a time, every column, value and gather
    // of the batch in flight together (loads past the row's end masked off),
    // the lane's sum in entry order
    const int e1 = rp[row + 1];
    for (int e = rp[row] + lane; e < e1; e += 8 * TPR) {
      int j[8];
      T a[8], x[8];
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (e + q * TPR < e1) {
          j[q] = ci[e + q * TPR];
          a[q] = v[e + q * TPR];
        }
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (e + q * TPR < e1) x[q] = g(j[q]);
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (e + q * TPR < e1) s += a[q] * x[q];
    }
    if (TPR > 1) {
#pragma unroll
      for (int off = TPR / 2; off > 0; off >>= 1) s += __shfl_xor(s, off, TPR);
    }
  }
  return s;
}
// the same, with only C columns (the F part of the iterate is zero): F columns
// read the first C value with weight zero, so every lane issues the same loads
template <int FMT, int TPR, bool WAVE = false, typename T>
__device__ __forceinline__ T mrow_c(const int* __restrict__ rp, const int* __restrict__ ci,
                                    const T* __restrict__ v, const T* __restrict__ xc, int nC,
                                    int row, int lane) {
  T s = 0;
  if (nC == 0) return s;
  if ((FMT == kFmtSELL || FMT == kFmtSELL16) && WAVE) {
    int o, oc, w, cb, fb;
    sell_slice_wave<FMT>(rp, row, o, oc, w, cb, fb);
    if (FMT == kFmtSELL16 && fb >= 0)
      s = sell_row8_c<true>(ci, v, xc, nC, o, oc, w, cb, fb);
    else
      s = sell_row8_c<false>(ci, v, xc, nC, o, oc, w, cb, fb);
  } else if (FMT == kFmtSELL || FMT == kFmtSELL16) {
    int o, oc, w, cb, fb;
    sell_slice<FMT>(rp, row, o, oc, w, cb, fb);
    if (FMT == kFmtSELL16 && fb >= 0)
      s = sell_row_c<true>(ci, v, xc, nC, o, oc, w, cb, fb);
    else
      s = sell_row_c<false>(ci, v, xc, nC, o, oc, w, cb, fb);
  } else {
    const int e1 = rp[row + 1];
    for (int e = rp[row] + lane; e < e1; e += 8 * TPR) {  // batches as in mrow
      int j[8];
      T a[8], x[8];
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (e + q * TPR < e1) {
          j[q] = ci[e + q * TPR];
          a[q] = v[e + q * TPR];
        }
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (e + q * TPR < e1 && j[q] < nC) x[q] = xc[j[q]];
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (e + q * TPR < e1 && j[q] < nC) s += a[q] * x[q];
    }
    if (TPR > 1) {
#pragma unroll
      for (int off = TPR / 2; off > 0; off >>= 1) s += __shfl_xor(s, off, TPR);
    }
  }
  return s;
}

// Row ranges per workgroup.  Workgroups are dispatched to the device's
// chiplets (XCDs, each with its own L2) in turn; with c_xcd_rows set,
// workgroup b takes the rows of workgroup xcd_block(b), so that each chiplet
// works on one contiguous share of the rows and finds the iterate values its
// rows gather (mostly near its own rows) in its own L2.
__constant__ int c_xcd_rows = 0;
template <int FMT>
constexpr bool kSliced = FMT == kFmtSELL || FMT == kFmtSELL16;
template <int FMT>
__host__ __device__ __forceinline__ int launch_start(int r0) {
  return kSliced<FMT> ? (r0 & ~63) : r0;
}
constexpr int kXcds = 8;
__device__ __forceinline__ long xcd_block(long b, long nb) {
  const long q = nb / kXcds, r = nb % kXcds, x = b % kXcds;
  return x * q + (x < r ? x : r) + b / kXcds;
}
void set_xcd_rows(int on) {
  MGD_HIP(hipMemcpyToSymbol(HIP_SYMBOL(c_xcd_rows), &on, sizeof(int)));
}
// Sliced layouts (one lane per row) start at r0 rounded down to a 64-row
// slice, so that every wave works on one slice (kSliced, launch_start).
#define MGD_ROWS_TPR                                                              \
  const long b_ = c_xcd_rows ? xcd_block(blockIdx.x, gridDim.x) : (long)blockIdx.x; \
  const long t_ = b_ * blockDim.x + threadIdx.x;                                  \
  const int lane = (int)(t_ % TPR);                                               \
  const int k = launch_start<FMT>(r0) + (int)(t_ / TPR);                          \
  if (k >= r1 || k < r0) return;

// level-0 entry: B[k] = b[perm[k]]; C values of the first sweep X_C = B_C / d_C
template <typename T, bool PRE>
__global__ void k_entry(int nX, int nC, const int* __restrict__ perm, const T* __restrict__ dinv,
                        const T* __restrict__ b, T* __restrict__ B, T* __restrict__ XC) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= nX) return;
  const T bb = b[perm[k]];
  B[k] = bb;
  if (k < nC) XC[k] = PRE ? bb * dinv[k] : (T)0;
}
// level-0 entry with the members' right-hand sides formed here from a block
// vector, read in natural order (member m = blockIdx.y, row i, coalesced):
// (T)(r[seg_m N + i] - coef_m[i] w[i]) written at its stored position iperm[.]
template <typename T, bool PRE>
__global__ void k_entry_nat(int N, int nC, const int* __restrict__ iperm,
                            const T* __restrict__ dinv_nat, const SegIn* __restrict__ tab,
                            const double* __restrict__ r, const T* __restrict__ w,
                            T* __restrict__ B, T* __restrict__ XC) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N) return;
  const SegIn d = tab[blockIdx.y];
  const size_t p = (size_t)blockIdx.y * N + i;
  double v = r[(size_t)d.seg * N + i];
  if (d.coef) v = v - d.coef[i] * (double)w[i];
  const T bb = (T)v;
  const int k = iperm[p];
  B[k] = bb;
  if (k < nC) XC[k] = PRE ? bb * dinv_nat[p] : (T)0;
}
// later cycles: B = (b - A z) in stored order (dense rows: 0), X_C as above
template <typename T, int FMT, int TPR, bool PRE>
__global__ void __launch_bounds__(256) k_entry_resid(int r0, int r1, int nS, int nC,
                                                     const int* __restrict__ rp,
                                                     const int* __restrict__ ci,
                                                     const T* __restrict__ v,
                                                     const int* __restrict__ perm,
                                                     const T* __restrict__ dinv,
                                                     const T* __restrict__ b,
                                                     const T* __restrict__ z, T* __restrict__ B,
                                                     T* __restrict__ XC) {
  MGD_ROWS_TPR
  if (k >= nS) {
    if (lane == 0) B[k] = (T)0;
    return;
  }
  const T bk = b[perm[k]];
  const T s = mrow<FMT, TPR, true>(rp, ci, v, GatherPerm<T>{z, perm}, k, lane);
  if (lane == 0) {
    const T bb = bk - s;
    B[k] = bb;
    if (k < nC) XC[k] = PRE ? bb * dinv[k] : (T)0;
  }
}

// first F half-sweep of a cycle (F iterate zero): X_F = (B_F - A_FC X_C) / d_F
template <typename T, int FMT, int TPR>
__global__ void __launch_bounds__(256) k_fhalf0(int r0, int r1, int nC, const int* __restrict__ rp,
                                                const int* __restrict__ ci,
                                                const T* __restrict__ v,
                                                const T* __restrict__ dinv,
                                                const T* __restrict__ B, const T* __restrict__ XC,
                                                T* __restrict__ Xout) {
  MGD_ROWS_TPR
  const T bk = B[k], dk = dinv[k];
  const T s = mrow_c<FMT, TPR, true>(rp, ci, v, XC, nC, k, lane);
  if (lane == 0) Xout[k] = (T)0 + (bk - s) * dk;
}

// half-sweep on rows [r0, r1): Xout = Xold + (B - A X) / d
template <typename T, int FMT, int TPR>
__global__ void __launch_bounds__(256) k_half(int r0, int r1, const int* __restrict__ rp,
                                              const int* __restrict__ ci, const T* __restrict__ v,
                                              const T* __restrict__ dinv, const T* __restrict__ B,
                                              GatherCF<T> X, const T* __restrict__ Xold,
                                              T* __restrict__ Xout) {
  MGD_ROWS_TPR
  const T xk = Xold[k], bk = B[k], dk = dinv[k];
  const T s = mrow<FMT, TPR, true>(rp, ci, v, X, k, lane);
  if (lane == 0) Xout[k] = xk + (bk - s) * dk;
}

// level-0 final C half-sweep fused with the output: z[perm[k]] = new X_C on
// C rows, the current F and dense values on the other rows
template <typename T, int FMT, int TPR>
__global__ void __launch_bounds__(256) k_half_out(int r0, int r1, int nC, int nS,
                                                  const int* __restrict__ rp,
                                                  const int* __restrict__ ci,
                                                  const T* __restrict__ v,
                                                  const T* __restrict__ dinv,
                                                  const T* __restrict__ B, GatherCF<T> X,
                                                  const T* __restrict__ XD,
                                                  const int* __restrict__ perm, T* __restrict__ z) {
  MGD_ROWS_TPR
  if (k < nC) {
    const T xk = X.base[k], bk = B[k], dk = dinv[k];
    const int pk = perm[k];
    const T s = mrow<FMT, TPR, true>(rp, ci, v, X, k, lane);
    if (lane == 0) z[pk] = xk + (bk - s) * dk;
  } else if (lane == 0) {
    if (k < nS)
      z[perm[k]] = X.base[k + X.f_minus_c];
    else
      z[perm[k]] = XD[k];
  }
}
// multicolour Gauss-Seidel on the rows of one colour, [r0, r0+n1) u [r2, r2+n2),
// in place: no two rows of a colour are coupled
template <typename T, int FMT, int TPR>
__global__ void __launch_bounds__(256) k_gs(int r0, int n1, int r2, int n2,
                                            const int* __restrict__ rp,
                                            const int* __restrict__ ci, const T* __restrict__ v,
                                            const T* __restrict__ dg, const T* __restrict__ B,
                                            T* __restrict__ X) {
  const long t = blockIdx.x * (long)blockDim.x + threadIdx.x;
  const int lane = (int)(t % TPR);
  const int q = (int)(t / TPR);
  if (q >= n1 + n2) return;
  const int k = q < n1 ? r0 + q : r2 + (q - n1);
  const T s = mrow<FMT, TPR>(rp, ci, v, Gather1<T>{X}, k, lane);
  if (lane == 0) X[k] = X[k] + (B[k] - s) * dg[k];
}

// level-0 output without post-smoothing
template <typename T>
__global__ void k_out(int nX, GatherCFD<T> X, const int* __restrict__ perm, T* __restrict__ z) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < nX) z[perm[k]] = X(k);
}

template <typename T, int FMT, int TPR>
__global__ void __launch_bounds__(256) k_resid(int r0, int r1, const int* __restrict__ rp,
                                               const int* __restrict__ ci,
                                               const T* __restrict__ v, const T* __restrict__ B,
                                               GatherCF<T> X, T* __restrict__ R) {
  MGD_ROWS_TPR
  const T bk = B[k];
  const T s = mrow<FMT, TPR, true>(rp, ci, v, X, k, lane);
  if (lane == 0) R[k] = bk - s;
}

// restriction into level l+1 (rows in its extended order):
// Bn[k] = R[cpos[k]] + sum_f Wt[k, f] R[nC + f], and its first-sweep C values
template <typename T, int FMT, int TPR, bool PRE>
__global__ void __launch_bounds__(256) k_restrict(int r0, int r1, int nC, int nCn,
                                                  const int* __restrict__ rp,
                                                  const int* __restrict__ ci,
                                                  const T* __restrict__ v,
                                                  const int* __restrict__ cpos,
                                                  const T* __restrict__ R,
                                                  const T* __restrict__ dinv_n,
                                                  T* __restrict__ Bn, T* __restrict__ XCn) {
  MGD_ROWS_TPR
  const T rc = R[cpos[k]];
  const T s = mrow<FMT, TPR, true>(rp, ci, v, Gather1<T>{R + nC}, k, lane);
  if (lane == 0) {
    const T bb = rc + s;
    Bn[k] = bb;
    if (k < nCn) XCn[k] = PRE ? bb * dinv_n[k] : (T)0;
  }
}

// prolongation: X_C[k] += E(cmap[k]) (k < nC); X_F[k] += W[k - nC, :] E
template <typename T, int FMT, int TPR>
__global__ void __launch_bounds__(256) k_prolong(int r0, int r1, int nC,
                                                 const int* __restrict__ rp,
                                                 const int* __restrict__ ci,
                                                 const T* __restrict__ v,
                                                 const int* __restrict__ cmap, GatherCFD<T> E,
                                                 T* __restrict__ XC, T* __restrict__ XF) {
  MGD_ROWS_TPR
  if (k < nC) {
    if (lane == 0) XC[k] += E(cmap[k]);
  } else {
    const T xk = XF[k];
    const T s = mrow<FMT, TPR>(rp, ci, v, E, k - nC, lane);
    if (lane == 0) XF[k] = xk + s;
  }
}

// x = A^{-1} b for every dense-solved member (FP64 arithmetic).  A workgroup
// of four waves takes 64 rows of one member; wave q sums the columns of its
// quarter in ascending order, eight column loads in flight per step, and the
// four partial sums are added in wave order.
template <typename T>
__global__ void __launch_bounds__(256) k_dense(const DenseDev* __restrict__ tab,
                                               const T* __restrict__ b, T* __restrict__ X) {
  __shared__ double part[4][64];
  const DenseDev d = tab[blockIdx.y];
  const int lane = threadIdx.x & 63;
  const int q = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // the wave: a scalar
  const int i = blockIdx.x * 64 + lane;
  const int quarter = (d.n + 3) / 4;
  const int j0 = min(d.n, q * quarter), j1 = min(d.n, j0 + quarter);
  double s = 0.0;
  if (i < d.n) {
    const double* __restrict__ col = d.inv + i;
    const T* __restrict__ bb = b + d.off;
    // eight columns at a time, the last batch cut at j1 (a scalar, like j0:
    // the branches are uniform); the sum in column order
    for (int j = j0; j < j1; j += 8) {
      double a[8], x[8];
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (j + k < j1) {
          a[k] = col[(size_t)(j + k) * d.n];
          x[k] = (double)bb[j + k];
        }
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (j + k < j1) s += a[k] * x[k];
    }
  }
  part[q][lane] = s;
  __syncthreads();
  if (q == 0 && i < d.n)
    X[d.off + i] = (T)(((part[0][lane] + part[1][lane]) + part[2][lane]) + part[3][lane]);
}

template <typename T>
__global__ void k_axpy_t(int n, const T* __restrict__ x, T* __restrict__ y) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) y[i] += x[i];
}

// ---------------------------------------------------------------------------
// the bottom of a cycle: one workgroup per member
// ---------------------------------------------------------------------------
// A cycle's small levels are a chain of dependent launches of 2 to 5 us each
// (six per level), whose work is a few hundred nanoseconds.  One workgroup runs
// the whole chain for its member between barriers of its own, with the same
// arithmetic as per-level launches with one lane per row.  What bounds it is one
// compute unit's instruction issue (a wave's instruction takes four cycles), so
// the layout is chosen for few instructions per entry: 64-row slices stored
// column by column (C rows and F rows in slices of their own), every address a
// constant step from the last, rows padded to the slice's even width with zero
// values; iterates in one buffer, so a column is its position.  A row's entries
// are added by one lane in sequence, in T, where up to 64 lanes shared a long row
// before: with FP32 hierarchies the bound of a row's rounding error grows with its
// length instead of its length over the lanes.  The error of an FP32 cycle against
// the FP64 one is that of the values' own rounding and did not move: over 12 inputs
// each, monolithic matrices of 2D 40^2 and 64^2, G = 20, 3D 16^3, G = 2 and 2D
// 64^2, G = 5 gave 6.33, 6.28, 6.70 and 6.42e-8 (relative, 2-norm) with shared rows
// and 6.35, 6.27, 6.70 and 6.38e-8 so.  The three lower
// levels of a 64^2 hierarchy (FP64) take 40 us as 13 launches, 33 us here with
// rows in CSR order (25 instructions per entry) and 20 us as slices.  A Schur1
// apply at 2D 101^2, G = 5 went from 777 to 507 us by it, a PCTL apply at 2D
// 256^2, G = 20 from 644 to 561 us.
extern __shared__ __align__(16) unsigned char bot_sm[];

// an array of a level, in the LDS copy or in memory
template <bool IN, typename U>
__device__ __forceinline__ const U* bot_at(const unsigned char* __restrict__ g, unsigned o) {
  if (IN) return reinterpret_cast<const U*>(bot_sm + o);
  return reinterpret_cast<const U*>(g + o);
}

// K entries of the lane's row, their loads together, added in order
template <int K, typename T>
__device__ __forceinline__ T bot_part(const uint16_t* ci, const T* v, const T* x, T s) {
  int j[K];
  T a[K], xv[K];
#pragma unroll
  for (int q = 0; q < K; ++q) {
    j[q] = ci[64 * q];
    a[q] = v[64 * q];
  }
#pragma unroll
  for (int q = 0; q < K; ++q) xv[q] = x[j[q]];
#pragma unroll
  for (int q = 0; q < K; ++q) s += a[q] * xv[q];
  return s;
}
// the lane's row of slice `sl`
template <bool IN, typename T>
__device__ __forceinline__ T bot_row(const unsigned char* __restrict__ g, const BotOp& op,
                                     const T* x, int sl, int lane) {
  const uint16_t* so = bot_at<true, uint16_t>(g, op.so);
  const int o = __builtin_amdgcn_readfirstlane(so[sl]);
  int w = __builtin_amdgcn_readfirstlane(so[sl + 1]) - o;
  const uint16_t* ci = bot_at<IN, uint16_t>(g, op.co) + 64 * o + lane;
  const T* v = bot_at<IN, T>(g, op.vo) + 64 * o + lane;
  T s = 0;
  if (!IN) {
    // from memory: sixteen columns' loads in flight, cut at the (scalar) width
    for (; w > 0; w -= 16, ci += 1024, v += 1024) {
      int j[16];
      T a[16], xv[16];
#pragma unroll
      for (int q = 0; q < 16; q += 2)
        if (q < w) {
          j[q] = ci[64 * q];
          j[q + 1] = ci[64 * q + 64];
          a[q] = v[64 * q];
          a[q + 1] = v[64 * q + 64];
        }
#pragma unroll
      for (int q = 0; q < 16; q += 2)
        if (q < w) {
          xv[q] = x[j[q]];
          xv[q + 1] = x[j[q + 1]];
        }
#pragma unroll
      for (int q = 0; q < 16; q += 2)
        if (q < w) {
          s += a[q] * xv[q];
          s += a[q + 1] * xv[q + 1];
        }
    }
    return s;
  }
  for (; w >= 8; w -= 8, ci += 512, v += 512) s = bot_part<8>(ci, v, x, s);
  if (w >= 4) {
    s = bot_part<4>(ci, v, x, s);
    w -= 4;
    ci += 256;
    v += 256;
  }
  if (w >= 2) s = bot_part<2>(ci, v, x, s);
  return s;
}

// one operation: a wave per slice
template <int NT, bool IN, typename T>
__device__ __forceinline__ void bot_rows(const unsigned char* __restrict__ g, const BotOp& op,
                                         T* vec) {
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint16_t* map = bot_at<true, uint16_t>(g, op.map);
  const T* dv = bot_at<true, T>(g, op.dv);
  const T* x = vec + op.x;
  // a half-sweep's new values wait for every row to have read the old ones: in a
  // register while a wave has one slice, else at op.out
  const bool one = op.s1 - op.s0 <= NT / 64;
  T keep = 0;
  int kept = -1;
  for (int sl = op.s0 + w; sl < op.s1; sl += NT / 64) {
    // slices [0, sC) hold rows [0, rC), the others the rows from rC on
    const bool first = sl < op.sC;
    const int r = first ? 64 * sl + lane : op.rC + 64 * (sl - op.sC) + lane;
    const int rs = min(r, (first ? op.rC : op.rows) - 1);  // a row of the slice
    if (op.kind == kBotHalf || op.kind == kBotFHalf0) {
      const T old = op.kind == kBotHalf ? vec[op.x + rs] : (T)0;
      const T bk = vec[op.b + rs], dk = dv[rs];
      const T s = bot_row<IN>(g, op, x, sl, lane);
      keep = old + (bk - s) * dk;
      kept = r == rs ? r : -1;
      if (!one && r == rs) vec[op.out + r] = keep;
    } else if (op.kind == kBotResid) {
      const T bk = vec[op.b + rs];
      const T s = bot_row<IN>(g, op, x, sl, lane);
      if (r == rs) vec[op.out + r] = bk - s;
    } else if (op.kind == kBotRestrict) {
      const T rc = vec[op.b + map[rs]], dk = dv[min(rs, op.nd)];
      const T s = bot_row<IN>(g, op, x, sl, lane);
      const T bb = rc + s;
      if (r == rs) {
        vec[op.out + r] = bb;
        vec[op.out2 + r] = r < op.nC ? bb * dk : (T)0;
      }
    } else {  // kBotProlong: F rows, in place
      const T xk = vec[op.out + rs];
      const T s = bot_row<IN>(g, op, x, sl, lane);
      if (r == rs) vec[op.out + r] = xk + s;
    }
  }
  if (op.kind == kBotProlong)  // C rows: their coarse points' values
    for (int k = threadIdx.x; k < op.nC; k += NT) vec[op.out2 + k] += x[map[k]];
  if (op.kind == kBotHalf || op.kind == kBotFHalf0) {
    __syncthreads();
    if (one) {
      if (kept >= 0) vec[op.x + kept] = keep;
      return;
    }
    for (int sl = op.s0 + w; sl < op.s1; sl += NT / 64) {
      const bool first = sl < op.sC;
      const int r = first ? 64 * sl + lane : op.rC + 64 * (sl - op.sC) + lane;
      if (r < (first ? op.rC : op.rows)) vec[op.x + r] = vec[op.out + r];
    }
  }
}

// x = A^{-1} b of a dense last level: k_dense's sums (four quarters of the
// columns, added in order), NT / 256 64-row chunks at a time
template <int NT, bool IN, typename T>
__device__ __forceinline__ void bot_dense(const unsigned char* __restrict__ g, const BotOp& op,
                                          T* vec, double (*part)[4][64]) {
  const double* inv = bot_at<IN, double>(g, op.vo);
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), q = w & 3, h = w >> 2;
  const int n = op.rows, quarter = (n + 3) / 4;
  const int j0 = min(n, q * quarter), j1 = min(n, j0 + quarter);
  for (int c0 = 0; c0 < n; c0 += 64 * (NT / 256)) {
    const int i = c0 + 64 * h + lane;
    double s = 0.0;
    if (i < n) {
      int j = j0;
      for (; j + 16 <= j1; j += 16) {
        double a[16], x[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
          a[k] = inv[(j + k) * n + i];
          x[k] = (double)vec[op.b + j + k];
        }
#pragma unroll
        for (int k = 0; k < 16; ++k) s += a[k] * x[k];
      }
      if (j < j1) {  // the rest: loads past it repeat the last column and are not added
        double a[16], x[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
          const int jk = min(j + k, j1 - 1);
          a[k] = inv[jk * n + i];
          x[k] = (double)vec[op.b + jk];
        }
#pragma unroll
        for (int k = 0; k < 16; ++k)
          if (j + k < j1) s += a[k] * x[k];
      }
    }
    part[h][q][lane] = s;
    __syncthreads();
    if (q == 0 && i < n)
      vec[op.out + i] =
          (T)(((part[h][0][lane] + part[h][1][lane]) + part[h][2][lane]) + part[h][3][lane]);
    __syncthreads();
  }
}

template <typename T, int NT>
__global__ void __launch_bounds__(NT) k_bottom(const BotMember* __restrict__ mem,
                                               const unsigned char* __restrict__ buf,
                                               const T* __restrict__ B, T* __restrict__ X) {
  __shared__ double part[NT / 256][4][64];
  const BotMember m = mem[blockIdx.x];
  const unsigned char* __restrict__ g = buf + m.buf;
  T* vec = reinterpret_cast<T*>(bot_sm + m.vec_at);
  const int t = threadIdx.x;
  auto place = [&](int i) { return i < m.nC ? m.cb + i : m.fb + (i - m.nC); };
  // the right-hand side, its diagonals and the member's data, all in flight
  constexpr int kPer = kBotRows / NT;
  T bb[kPer], dd[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int i = t + k * NT;
    bb[k] = i < m.n ? B[place(i)] : (T)0;
    dd[k] = i < m.nC ? bot_at<false, T>(g, m.dv)[i] : (T)0;
  }
  for (unsigned i0 = 16 * t; i0 < m.lds; i0 += 5 * 16 * NT) {
    uint4 c[5];
#pragma unroll
    for (int k = 0; k < 5; ++k)
      c[k] = *reinterpret_cast<const uint4*>(g + min(i0 + k * 16 * NT, m.lds - 16));
#pragma unroll
    for (int k = 0; k < 5; ++k)
      if (i0 + k * 16 * NT < m.lds) *reinterpret_cast<uint4*>(bot_sm + i0 + k * 16 * NT) = c[k];
  }
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int i = t + k * NT;
    if (i < m.n) {
      vec[i] = bb[k];
      vec[m.n + i] = i < m.nC ? bb[k] * dd[k] : (T)0;
    }
  }
  __syncthreads();
  for (int p = 0; p < m.nops; ++p) {
    // the operation, from LDS into scalars
    BotOp op;
    {
      constexpr int kWords = sizeof(BotOp) / 4;
      const int* src = reinterpret_cast<const int*>(bot_sm + m.ops) + p * kWords;
      int w[kWords];
#pragma unroll
      for (int k = 0; k < kWords; ++k) w[k] = __builtin_amdgcn_readfirstlane(src[k]);
      __builtin_memcpy(&op, w, sizeof(op));
    }
    if (op.kind == kBotDense) {
      if (op.in)
        bot_dense<NT, true, T>(g, op, vec, part);
      else
        bot_dense<NT, false, T>(g, op, vec, part);
    } else {
      if (op.in)
        bot_rows<NT, true, T>(g, op, vec);
      else
        bot_rows<NT, false, T>(g, op, vec);
      __syncthreads();
    }
  }
  for (int i = t; i < m.n; i += NT) X[place(i)] = vec[m.n + i];
}

// Even widths of the 64-row slices of member blockIdx.x's rows at one level: of
// A (C rows, then F rows), of W (F rows) and of W^T (the next level's rows), at
// out[blockIdx.x][matrix][slice]; the slices of a matrix are counted by its rows.
constexpr int kBotSlices = 2 * (kBotRows / 64) / 2 + 4;
struct BotRows {       // a member's place in a level's extended stored order
  int cb, fb, db, nC, nF, kind;
};
__global__ void __launch_bounds__(256) k_bot_widths(const BotRows* __restrict__ at,
                                                    const BotRows* __restrict__ next, int nC_u,
                                                    const int* __restrict__ arp,
                                                    const int* __restrict__ wrp,
                                                    const int* __restrict__ trp,
                                                    int* __restrict__ out) {
  const BotRows m = at[blockIdx.x];
  int* o = out + (size_t)blockIdx.x * 3 * kBotSlices;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int sC = (m.nC + 63) / 64, sF = (m.nF + 63) / 64;
  auto emit = [&](int mat, int sl, int len) {
#pragma unroll
    for (int f = 32; f > 0; f >>= 1) len = max(len, __shfl_xor(len, f, 64));
    if (lane == 0) o[mat * kBotSlices + sl] = (len + 1) & ~1;
  };
  if (m.kind == 2) return;
  for (int sl = wave; sl < sC + sF; sl += 4) {
    const int r = sl < sC ? 64 * sl + lane : 64 * (sl - sC) + lane;
    const int k = sl < sC ? m.cb + r : m.fb + r;
    const bool in = r < (sl < sC ? m.nC : m.nF);
    emit(0, sl, in ? arp[k + 1] - arp[k] : 0);
  }
  if (m.kind != 0) return;
  for (int sl = wave; sl < sF; sl += 4) {
    const int r = 64 * sl + lane, k = m.fb - nC_u + r;
    emit(1, sl, r < m.nF ? wrp[k + 1] - wrp[k] : 0);
  }
  const BotRows x = next[blockIdx.x];
  for (int sl = wave; sl < sC; sl += 4) {  // the next level's rows: as many as C rows here
    const int r = 64 * sl + lane;
    const int k = x.kind == 2 ? x.db + r : (r < x.nC ? x.cb + r : x.fb + (r - x.nC));
    emit(2, sl, r < m.nC ? trp[k + 1] - trp[k] : 0);
  }
}

// Packs member blockIdx.y's rows of one bottom level: local rows and columns,
// values in T.
struct BotPack {
  unsigned char* buf;  // the member's part
  BotLevel L;
  BotRows at, next;
  const double* inv;
  int q;               // the member's row of the slice widths
};
// local row of extended stored index k
__device__ __forceinline__ int bot_local(int k, int nC_u, int nS_u, const BotRows& m) {
  return k < nC_u ? k - m.cb : (k < nS_u ? m.nC + k - m.fb : k - m.db);
}
template <typename T>
__global__ void k_bot_pack(const BotPack* __restrict__ tab, int nC, int nS, int nCn, int nSn,
                           const int* __restrict__ widths, const int* __restrict__ arp,
                           const int* __restrict__ aci, const double* __restrict__ av,
                           const int* __restrict__ wrp, const int* __restrict__ wci,
                           const double* __restrict__ wv, const int* __restrict__ trp,
                           const int* __restrict__ tci, const double* __restrict__ tv,
                           const T* __restrict__ dinv, const int* __restrict__ cmap,
                           const int* __restrict__ cpos, int* __restrict__ err) {
  const BotPack p = tab[blockIdx.y];
  const BotLevel L = p.L;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  unsigned char* g = p.buf;
  if (L.kind == 2) {
    double* inv = reinterpret_cast<double*>(g + L.vA);
    for (int e = i; e < L.n * L.n; e += gridDim.x * blockDim.x) inv[e] = p.inv[e];
    return;
  }
  const int* wd = widths + (size_t)p.q * 3 * kBotSlices;
  bool bad = false;
  // one row of matrix `mat` into slice sl, lane ln: entry(e, column, value)
  auto put = [&](int mat, int sl, int ln, int len, int pad, unsigned co, unsigned vo, auto entry) {
    int o = 0;
    for (int k = 0; k < sl; ++k) o += wd[mat * kBotSlices + k];
    const int w = wd[mat * kBotSlices + sl];
    bad = bad || len > w;
    uint16_t* ci = reinterpret_cast<uint16_t*>(g + co) + 64 * o + ln;
    T* v = reinterpret_cast<T*>(g + vo) + 64 * o + ln;
    for (int e = 0; e < w; ++e) {
      int j = pad;
      double a = 0.0;
      if (e < len) entry(e, j, a);
      ci[64 * e] = (uint16_t)j;
      v[64 * e] = (T)a;
    }
  };
  auto offsets = [&](int mat, int ns, unsigned so) {  // one thread per slice offset
    if (i > ns) return;
    int o = 0;
    for (int k = 0; k < i; ++k) o += wd[mat * kBotSlices + k];
    reinterpret_cast<uint16_t*>(g + so)[i] = (uint16_t)o;
  };
  const int nF = L.n - L.nC, sC = (L.nC + 63) / 64, sF = (nF + 63) / 64;
  offsets(0, sC + sF, L.sA);
  // the slice's 64 lanes, those past its last row with rows of padding
  if (i < 64 * (sC + sF)) {
    const int sl = i >> 6, ln = i & 63;
    const bool c = sl < sC;
    const int r = c ? i : i - 64 * sC;  // row of its block
    const bool in = r < (c ? L.nC : nF);
    const int k = (c ? p.at.cb : p.at.fb) + (in ? r : 0), row = c ? r : L.nC + r;
    put(0, sl, ln, in ? arp[k + 1] - arp[k] : 0, in ? row : 0, L.cA, L.vA,
        [&](int e, int& j, double& a) {
          j = bot_local(aci[arp[k] + e], nC, nS, p.at);
          a = av[arp[k] + e];
          bad = bad || j < 0 || j >= L.n;
        });
    if (in) reinterpret_cast<T*>(g + L.dv)[row] = dinv[k];
  }
  if (L.kind == 0) {
    const int f0 = p.at.fb - nC;
    offsets(1, sF, L.sW);
    offsets(2, sC, L.sT);
    if (i < 64 * sF) {
      const bool in = i < nF;
      const int k = f0 + (in ? i : 0);
      put(1, i >> 6, i & 63, in ? wrp[k + 1] - wrp[k] : 0, 0, L.cW, L.vW,
          [&](int e, int& j, double& a) {
            j = bot_local(wci[wrp[k] + e], nCn, nSn, p.next);
            a = wv[wrp[k] + e];
            bad = bad || j < 0 || j >= L.nn;
          });
    }
    if (i < 64 * sC) {
      const bool in = i < L.nn;
      const int r = in ? i : 0;
      const BotRows& x = p.next;
      const int k = x.kind == 2 ? x.db + r : (r < x.nC ? x.cb + r : x.fb + (r - x.nC));
      put(2, i >> 6, i & 63, in ? trp[k + 1] - trp[k] : 0, 0, L.cT, L.vT,
          [&](int e, int& j, double& a) {
            const int f = tci[trp[k] + e] - f0;  // local F row, read from the residual
            j = L.nC + f;
            a = tv[trp[k] + e];
            bad = bad || f < 0 || f >= nF;
          });
      if (in) {
        const int cl = cpos[k] - p.at.cb;
        bad = bad || cl < 0 || cl >= L.nC;
        reinterpret_cast<uint16_t*>(g + L.cp)[i] = (uint16_t)cl;
      }
    }
    if (i < L.nC) {
      const int j = bot_local(cmap[p.at.cb + i], nCn, nSn, p.next);
      bad = bad || j < 0 || j >= L.nn;
      reinterpret_cast<uint16_t*>(g + L.cm)[i] = (uint16_t)j;
    }
  }
  if (bad) atomicOr(err, 32);
}

// ---------------------------------------------------------------------------
// persistent tail: every level from a threshold down (and back up) in one
// launch.  Each phase does what the per-level kernel of the same name does,
// with the same arithmetic, over a grid-stride loop; phases are separated by
// a grid-wide barrier.  The grid is sized so that all its workgroups are
// resident at once; a barrier wait that exceeds its spin bound reports
// through the error flag and lets the workgroup go on, so the kernel always
// ends.  The last workgroup to finish resets the counters for the next launch.
// Pointers to vectors that earlier phases write are read without __restrict__,
// so every such load goes through the memory system after the barrier's fence.
// ---------------------------------------------------------------------------
constexpr int kTailThreads = 256;
constexpr unsigned kTailSpinLimit = 1u << 17;  // about 0.1 s of polling
constexpr int kTailSyncStride = 32;  // counters 128 bytes apart
constexpr int kErrTailBarrier = 64;

__device__ __forceinline__ void tail_barrier(unsigned* arrive, unsigned target, int* err) {
  __syncthreads();
  if (threadIdx.x == 0) {
    __hip_atomic_fetch_add(arrive, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    unsigned spins = 0;
    while (__hip_atomic_load(arrive, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
      // once any wait has timed out, later waits of the launch end at once
      if (++spins > kTailSpinLimit ||
          (__hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kErrTailBarrier)) {
        atomicOr(err, kErrTailBarrier);
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  }
  __syncthreads();
}

template <int FMT, int TPR, typename T>
__device__ __forceinline__ void tail_rows(const TailOp<T>& op) {
  const long long n = (long long)(op.r1 - op.r0) * TPR;
  const long long stride = (long long)gridDim.x * kTailThreads;
  for (long long t = blockIdx.x * (long long)kTailThreads + threadIdx.x; t < n; t += stride) {
    // a group of TPR lanes shares a row: the whole group is in or out of range
    const int lane = (int)(t % TPR);
    const int k = op.r0 + (int)(t / TPR);
    if (op.kind == kTopFHalf0) {
      const T s = mrow_c<FMT, TPR>(op.rp, op.ci, op.v, op.xc, op.nC, k, lane);
      if (lane == 0) op.out[k] = (T)0 + (op.B[k] - s) * op.dinv[k];
    } else if (op.kind == kTopHalf) {
      const T s = mrow<FMT, TPR>(op.rp, op.ci, op.v, GatherCF<T>{op.xc, op.f_minus_c, op.nC}, k,
                                 lane);
      if (lane == 0) op.out[k] = op.xold[k] + (op.B[k] - s) * op.dinv[k];
    } else if (op.kind == kTopResid) {
      const T s = mrow<FMT, TPR>(op.rp, op.ci, op.v, GatherCF<T>{op.xc, op.f_minus_c, op.nC}, k,
                                 lane);
      if (lane == 0) op.out[k] = op.B[k] - s;
    } else if (op.kind == kTopRestrict) {
      const T s = mrow<FMT, TPR>(op.rp, op.ci, op.v, Gather1<T>{op.B + op.nC}, k, lane);
      if (lane == 0) {
        const T bb = op.B[op.map[k]] + s;
        op.out[k] = bb;
        if (k < op.nCn) op.out2[k] = op.pre ? bb * op.dinv[k] : (T)0;
      }
    } else {  // kTopProlong
      const GatherCFD<T> E{op.xc, (ptrdiff_t)op.f_minus_c, (ptrdiff_t)op.d_minus_c, op.nC, op.nS};
      if (k < op.nCn) {
        if (lane == 0) op.out2[k] += E(op.map[k]);
      } else {
        const T s = mrow<FMT, TPR>(op.rp, op.ci, op.v, E, k - op.nCn, lane);
        if (lane == 0) op.out[k] += s;
      }
    }
  }
}

// k_dense over virtual workgroups (member, 64-row chunk)
template <typename T>
__device__ __forceinline__ void tail_dense(const TailOp<T>& op) {
  __shared__ double part[4][64];
  const int nvb = op.ndense * op.dchunks;
  const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
  for (int vb = blockIdx.x; vb < nvb; vb += gridDim.x) {
    const DenseDev d = op.dense[vb / op.dchunks];
    const int i = (vb % op.dchunks) * 64 + lane;
    const int quarter = (d.n + 3) / 4;
    const int j0 = min(d.n, q * quarter), j1 = min(d.n, j0 + quarter);
    double sum = 0.0;
    if (i < d.n) {
      const double* __restrict__ col = d.inv + i;
      const T* bb = op.B + d.off;
      int j = j0;
      for (; j + 8 <= j1; j += 8) {
        double a[8], x[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          a[k] = col[(size_t)(j + k) * d.n];
          x[k] = (double)bb[j + k];
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) sum += a[k] * x[k];
      }
      for (; j < j1; ++j) sum += col[(size_t)j * d.n] * (double)bb[j];
    }
    part[q][lane] = sum;
    __syncthreads();
    if (q == 0 && i < d.n)
      op.out[d.off + i] = (T)(((part[0][lane] + part[1][lane]) + part[2][lane]) + part[3][lane]);
    __syncthreads();
  }
}

template <typename T>
__device__ __forceinline__ void tail_phase(const TailOp<T>& op) {
  if (op.kind == kTopDense) {
    tail_dense(op);
    return;
  }
  if (op.fmt == kFmtSELL) return tail_rows<kFmtSELL, 1>(op);
  if (op.fmt == kFmtSELL16) return tail_rows<kFmtSELL16, 1>(op);
  switch (op.tpr) {
    case 1: tail_rows<kFmtCSR, 1>(op); break;
    case 2: tail_rows<kFmtCSR, 2>(op); break;
    case 4: tail_rows<kFmtCSR, 4>(op); break;
    case 8: tail_rows<kFmtCSR, 8>(op); break;
    case 16: tail_rows<kFmtCSR, 16>(op); break;
    case 32: tail_rows<kFmtCSR, 32>(op); break;
    default: tail_rows<kFmtCSR, 64>(op); break;
  }
}

template <typename T>
__global__ void __launch_bounds__(kTailThreads) k_tail(const TailOp<T>* __restrict__ ops, int nops,
                                                       unsigned* sync, int* err) {
  for (int p = 0; p < nops; ++p) {
    if (p > 0) tail_barrier(sync, (unsigned)p * gridDim.x, err);
    const TailOp<T> op = ops[p];
    tail_phase(op);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    // every workgroup has passed every barrier once it counts itself out here;
    // only the counters are touched (atomically), so no data fence is needed
    const unsigned k =
        __hip_atomic_fetch_add(sync + kTailSyncStride, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (k == gridDim.x - 1) {
      __hip_atomic_store(sync, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(sync + kTailSyncStride, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// ---------------------------------------------------------------------------
// launchers: one row per lane (SELL) or TPR lanes per row (CSR)
// ---------------------------------------------------------------------------
template <typename T>
struct MatArgs {
  const LMat<T>* m;
};
static inline dim3 rows_grid(int rows, int tpr, int bs) { return dim3(cdiv((long long)rows * tpr, bs)); }

// Calls F.template go<FMT, TPR>() for the matrix's layout.
template <typename F>
static void with_layout(int fmt, int tpr, F&& f) {
  if (fmt == kFmtSELL) {
    f.template go<kFmtSELL, 1>();
    return;
  }
  if (fmt == kFmtSELL16) {
    f.template go<kFmtSELL16, 1>();
    return;
  }
  switch (tpr) {
    case 1: f.template go<kFmtCSR, 1>(); break;
    case 2: f.template go<kFmtCSR, 2>(); break;
    case 4: f.template go<kFmtCSR, 4>(); break;
    case 8: f.template go<kFmtCSR, 8>(); break;
    case 16: f.template go<kFmtCSR, 16>(); break;
    case 32: f.template go<kFmtCSR, 32>(); break;
    default: f.template go<kFmtCSR, 64>(); break;
  }
}
// Level and union size of the launches being profiled, appended to the kernel
// symbol as "@L<level>/<members>" (the symbol itself comes before the '@').
static thread_local int t_prof_level = -1, t_prof_members = 0;
static std::string level_tag() {
  return t_prof_level < 0 ? std::string()
                          : "@L" + std::to_string(t_prof_level) + "/" + std::to_string(t_prof_members);
}
template <typename T>
static std::string kname(const Ctx* c, const char* base, const LMat<T>& m,
                         std::initializer_list<std::string> extra = {}) {
  if (!c->profiling) return std::string();
  std::vector<std::string> a{type_name<T>(), std::to_string(m.fmt),
                             std::to_string(m.fmt != kFmtCSR ? 1 : tpr_of(m.tpr))};
  for (const auto& e : extra) a.push_back(e);
  std::string s(base);
  const char* sep = "<";
  for (const auto& x : a) {
    s += sep;
    s += x;
    sep = ", ";
  }
  return s + ">" + level_tag();
}

template <typename T>
struct HalfL {
  Ctx* c;
  const LMat<T>& A;
  int r0, r1;
  const T *dinv, *B;
  GatherCF<T> X;
  const T* Xold;
  T* Xout;
  template <int FMT, int TPR>
  void go() const {
    if (r1 <= r0) return;
    hipLaunchKernelGGL((k_half<T, FMT, TPR>), rows_grid(r1 - launch_start<FMT>(r0), TPR, A.bs),
                       dim3(A.bs), 0, c->stream,
                       r0, r1, A.rp.get(), A.ci.get(), A.v.get(), dinv, B, X, Xold, Xout);
    MGD_CHECK_LAUNCH();
  }
};
template <typename T>
struct FHalf0L {
  Ctx* c;
  const LMat<T>& A;
  int r0, r1, nC;
  const T *dinv, *B, *XC;
  T* Xout;
  template <int FMT, int TPR>
  void go() const {
    if (r1 <= r0) return;
    hipLaunchKernelGGL((k_fhalf0<T, FMT, TPR>), rows_grid(r1 - launch_start<FMT>(r0), TPR, A.bs),
                       dim3(A.bs), 0, c->stream,
                       r0, r1, nC, A.rp.get(), A.ci.get(), A.v.get(), dinv, B, XC, Xout);
    MGD_CHECK_LAUNCH();
  }
};
template <typename T>
struct HalfOutL {
  Ctx* c;
  const LMat<T>& A;
  int nX, nC, nS;
  const T *dinv, *B;
  GatherCF<T> X;
  const T* XD;
  const int* perm;
  T* z;
  template <int FMT, int TPR>
  void go() const {
    if (nX <= 0) return;
    hipLaunchKernelGGL((k_half_out<T, FMT, TPR>), rows_grid(nX, TPR, A.bs), dim3(A.bs), 0, c->stream, 0,
                       nX, nC, nS, A.rp.get(), A.ci.get(), A.v.get(), dinv, B, X, XD, perm, z);
    MGD_CHECK_LAUNCH();
  }
};
template <typename T>
struct GsL {
  Ctx* c;
  const LMat<T>& A;
  int r0, n1, r2, n2;
  const T *dg, *B;
  T* X;
  template <int FMT, int TPR>
  void go() const {
    if (n1 + n2 <= 0) return;
    hipLaunchKernelGGL((k_gs<T, FMT, TPR>), rows_grid(n1 + n2, TPR, A.bs), dim3(A.bs), 0, c->stream, r0,
                       n1, r2, n2, A.rp.get(), A.ci.get(), A.v.get(), dg, B, X);
    MGD_CHECK_LAUNCH();
  }
};
template <typename T>
struct ResidL {
  Ctx* c;
  const LMat<T>& A;
  int nS;
  const T* B;
  GatherCF<T> X;
  T* R;
  template <int FMT, int TPR>
  void go() const {
    if (nS <= 0) return;
    hipLaunchKernelGGL((k_resid<T, FMT, TPR>), rows_grid(nS, TPR, A.bs), dim3(A.bs), 0, c->stream, 0, nS,
                       A.rp.get(), A.ci.get(), A.v.get(), B, X, R);
    MGD_CHECK_LAUNCH();
  }
};
template <typename T>
struct EntryResidL {
  Ctx* c;
  const LMat<T>& A;
  int nX, nS, nC;
  const int* perm;
  const T *dinv, *b, *z;
  T *B, *XC;
  bool pre;
  template <int FMT, int TPR>
  void go() const {
    if (nX <= 0) return;
    if (pre)
      hipLaunchKernelGGL((k_entry_resid<T, FMT, TPR, true>), rows_grid(nX, TPR, A.bs), dim3(A.bs), 0,
                         c->stream, 0, nX, nS, nC, A.rp.get(), A.ci.get(), A.v.get(), perm, dinv,
                         b, z, B, XC);
    else
      hipLaunchKernelGGL((k_entry_resid<T, FMT, TPR, false>), rows_grid(nX, TPR, A.bs), dim3(A.bs), 0,
                         c->stream, 0, nX, nS, nC, A.rp.get(), A.ci.get(), A.v.get(), perm, dinv,
                         b, z, B, XC);
    MGD_CHECK_LAUNCH();
  }
};
template <typename T>
struct RestrictL {
  Ctx* c;
  const LMat<T>& Wt;
  int nXn, nC, nCn;
  const int* cpos;
  const T *R, *dinv_n;
  T *Bn, *XCn;
  bool pre;
  template <int FMT, int TPR>
  void go() const {
    if (nXn <= 0) return;
    if (pre)
      hipLaunchKernelGGL((k_restrict<T, FMT, TPR, true>), rows_grid(nXn, TPR, Wt.bs), dim3(Wt.bs), 0,
                         c->stream, 0, nXn, nC, nCn, Wt.rp.get(), Wt.ci.get(), Wt.v.get(), cpos, R,
                         dinv_n, Bn, XCn);
    else
      hipLaunchKernelGGL((k_restrict<T, FMT, TPR, false>), rows_grid(nXn, TPR, Wt.bs), dim3(Wt.bs), 0,
                         c->stream, 0, nXn, nC, nCn, Wt.rp.get(), Wt.ci.get(), Wt.v.get(), cpos, R,
                         dinv_n, Bn, XCn);
    MGD_CHECK_LAUNCH();
  }
};
template <typename T>
struct ProlongL {
  Ctx* c;
  const LMat<T>& W;
  int nS, nC;
  const int* cmap;
  GatherCFD<T> E;
  T *XC, *XF;
  template <int FMT, int TPR>
  void go() const {
    if (nS <= 0) return;
    hipLaunchKernelGGL((k_prolong<T, FMT, TPR>), rows_grid(nS, TPR, W.bs), dim3(W.bs), 0, c->stream, 0,
                       nS, nC, W.rp.get(), W.ci.get(), W.v.get(), cmap, E, XC, XF);
    MGD_CHECK_LAUNCH();
  }
};

// algorithmic bytes per launch: every matrix entry (value + column), every
// per-row vector element read or written, and the gathered iterate once
template <typename T>
static double mat_bytes(const LMat<T>& m, long long nnz) {
  return (double)nnz * (sizeof(T) + (m.fmt == kFmtSELL16 ? 2 : 4));
}
// profiling scope of a launch that reads `nnz` entries of m over `rows` rows
// plus vec_bytes of vectors: stored-layout bytes, and the same launch priced
// as plain CSR (value and 4-byte column per entry, 4-byte row pointer per row)
template <typename T>
static ProfScope prof_level(Ctx* c, int cls, const LMat<T>& m, long long nnz, long long rows,
                            double vec_bytes, std::string name) {
  return ProfScope(c, cls, mat_bytes(m, nnz) + vec_bytes, std::move(name),
                   (double)nnz * (sizeof(T) + 4) + 4.0 * (double)rows + vec_bytes);
}
static inline int cls_of(int l, int cls0) { return l == 0 ? cls0 : KC_VCYCLE_COARSE; }

template <typename T>
static GatherCF<T> gather_cf(const T* xc, const T* xf, int nC) {
  return GatherCF<T>{xc, (ptrdiff_t)(xf - xc), nC};
}
template <typename T>
static GatherCFD<T> gather_cfd(const T* xc, const T* xf, const T* xd, int nC, int nS) {
  return GatherCFD<T>{xc, (ptrdiff_t)(xf - xc), (ptrdiff_t)(xd - xc), nC, nS};
}

template <typename T>
void Union<T>::vcycle(Ctx* c, T* z) {
  const int nl = (int)L.size();
  const size_t ts = sizeof(T);
  // current buffer (0: X0, 1: X1) of the C and the F region, per level
  std::vector<int> cc(nl, 0), cf(nl, 0);
  auto Xb = [&](int l, int which) -> T* { return which ? X1[l].get() : X0[l].get(); };
  t_prof_members = members;
  const int lt = bot_from >= 0 ? bot_from : (tail_from >= 0 ? tail_from : nl);
  for (int l = 0; l < lt; ++l) {
    t_prof_level = l;
    ULevel<T>& lv = L[l];
    const int nF = lv.nS - lv.nC;
    // the C values of the first sweep were written with B (entry / restriction)
    if (lv.nS > 0) {
      for (int s = 0; s < n_pre; ++s) {
        if (s > 0) {  // C half of a later sweep
          ProfScope ps = prof_level(c, cls_of(l, KC_SMOOTH_L0), lv.A, lv.nnz_C, lv.nC,
                                    (double)lv.nC * 4 * ts + lv.nS * ts, kname(c, "k_half", lv.A));
          with_layout(lv.A.fmt, lv.A.tpr,
                      HalfL<T>{c, lv.A, 0, lv.nC, lv.dinv.get(), B[l].get(),
                               gather_cf<T>(Xb(l, cc[l]), Xb(l, cf[l]), lv.nC), Xb(l, cc[l]),
                               Xb(l, 1 - cc[l])});
          cc[l] = 1 - cc[l];
        }
        if (nF > 0) {
          if (s == 0) {
            ProfScope ps = prof_level(c, cls_of(l, KC_SMOOTH_L0), lv.A, lv.nnz_F, nF,
                                      (double)nF * 3 * ts + lv.nC * ts, kname(c, "k_fhalf0", lv.A));
            with_layout(lv.A.fmt, lv.A.tpr,
                        FHalf0L<T>{c, lv.A, lv.nC, lv.nS, lv.nC, lv.dinv.get(), B[l].get(),
                                   Xb(l, cc[l]), Xb(l, 1 - cf[l])});
          } else {
            ProfScope ps = prof_level(c, cls_of(l, KC_SMOOTH_L0), lv.A, lv.nnz_F, nF,
                                      (double)nF * 4 * ts + lv.nS * ts, kname(c, "k_half", lv.A));
            with_layout(lv.A.fmt, lv.A.tpr,
                        HalfL<T>{c, lv.A, lv.nC, lv.nS, lv.dinv.get(), B[l].get(),
                                 gather_cf<T>(Xb(l, cc[l]), Xb(l, cf[l]), lv.nC), Xb(l, cf[l]),
                                 Xb(l, 1 - cf[l])});
          }
          cf[l] = 1 - cf[l];
        }
      }
      if (n_pre == 0 && nF > 0) fill<T>(c, Xb(l, cf[l]) + lv.nC, (T)0, (size_t)nF);
      if (lv.nX_next > 0) {
        {
          ProfScope ps = prof_level(c, cls_of(l, KC_RESID_L0), lv.A, lv.A.nnz, lv.nS,
                                    (double)lv.nS * 3 * ts, kname(c, "k_resid", lv.A));
          with_layout(lv.A.fmt, lv.A.tpr,
                      ResidL<T>{c, lv.A, lv.nS, B[l].get(),
                                gather_cf<T>(Xb(l, cc[l]), Xb(l, cf[l]), lv.nC), R[l].get()});
        }
        const ULevel<T>& nx = L[l + 1];
        ProfScope ps = prof_level(c, cls_of(l, KC_TRANSFER_L0), lv.Wt, lv.Wt.nnz, lv.Wt.rows,
                                  (double)lv.nX_next * (4 + ts) + (double)nx.nC * 2 * ts +
                                      lv.nS * ts,
                                  kname(c, "k_restrict", lv.Wt, {n_pre > 0 ? "true" : "false"}));
        with_layout(lv.Wt.fmt, lv.Wt.tpr,
                    RestrictL<T>{c, lv.Wt, lv.nX_next, lv.nC, nx.nC, lv.cpos.get(), R[l].get(),
                                 nx.dinv.get(), B[l + 1].get(), Xb(l + 1, 0), n_pre > 0});
      }
    }
    if (!lv.dense.empty()) {
      ProfScope ps(c, KC_COARSE_SOLVE, 8.0 * lv.dense_entries + 2.0 * ts * (lv.nX - lv.nS),
                   ksym(c, "k_dense", {type_name<T>()}));
      dim3 grid(cdiv(lv.dense_max_n, 64), (unsigned)lv.dense.size());
      hipLaunchKernelGGL(k_dense<T>, grid, dim3(256), 0, c->stream,
                         (const DenseDev*)lv.dense_dev.get(), (const T*)B[l].get(), X0[l].get());
      MGD_CHECK_LAUNCH();
    }
  }
  if (bot_from >= 0) {  // levels lt .. nl-1, down and up, one workgroup per member
    t_prof_level = lt;
    ProfScope ps(c, cls_of(lt, KC_SMOOTH_L0), bot_bytes,
                 ksym(c, "k_bottom", {type_name<T>(), std::to_string(bot_threads)}) + level_tag());
    auto bottom = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3(bot_members), dim3(bot_threads), bot_lds, c->stream,
                         (const BotMember*)bot_mem.get(), (const unsigned char*)bot_buf.get(),
                         (const T*)B[lt].get(), X0[lt].get());
    };
    if (bot_threads == 1024)
      bottom(k_bottom<T, 1024>);
    else
      bottom(k_bottom<T, 512>);
    MGD_CHECK_LAUNCH();
  } else if (lt < nl) {  // levels lt .. nl-1, down and up, in one launch
    t_prof_level = lt;
    ProfScope ps(c, KC_VCYCLE_COARSE, tail_bytes, ksym(c, "k_tail", {type_name<T>()}) + level_tag(),
                 tail_bytes_csr);
    hipLaunchKernelGGL(k_tail<T>, dim3(tail_blocks), dim3(kTailThreads), 0, c->stream,
                       (const TailOp<T>*)tail_ops.get(), tail_nops, tail_sync.get(), c->err_flag());
    MGD_CHECK_LAUNCH();
    cc[lt] = tail_cc;
    cf[lt] = tail_cf;
  }
  for (int l = lt - 1; l >= 0; --l) {
    t_prof_level = l;
    ULevel<T>& lv = L[l];
    const int nF = lv.nS - lv.nC;
    if (lv.nS > 0 && lv.nX_next > 0) {
      const ULevel<T>& nx = L[l + 1];
      ProfScope ps = prof_level(c, cls_of(l, KC_TRANSFER_L0), lv.W, lv.W.nnz, lv.W.rows,
                                (double)lv.nC * 4 + lv.nS * 2.0 * ts + (double)lv.nX_next * ts,
                                kname(c, "k_prolong", lv.W));
      with_layout(lv.W.fmt, lv.W.tpr,
                  ProlongL<T>{c, lv.W, lv.nS, lv.nC, lv.cmap.get(),
                              gather_cfd<T>(Xb(l + 1, cc[l + 1]), Xb(l + 1, cf[l + 1]),
                                            X0[l + 1].get(), nx.nC, nx.nS),
                              Xb(l, cc[l]), Xb(l, cf[l])});
    }
    const bool last_out = (l == 0);
    if (lv.nS > 0) {
      for (int s = 0; s < n_post; ++s) {
        if (nF > 0) {
          ProfScope ps = prof_level(c, cls_of(l, KC_SMOOTH_L0), lv.A, lv.nnz_F, nF,
                                    (double)nF * 4 * ts + lv.nS * ts, kname(c, "k_half", lv.A));
          with_layout(lv.A.fmt, lv.A.tpr,
                      HalfL<T>{c, lv.A, lv.nC, lv.nS, lv.dinv.get(), B[l].get(),
                               gather_cf<T>(Xb(l, cc[l]), Xb(l, cf[l]), lv.nC), Xb(l, cf[l]),
                               Xb(l, 1 - cf[l])});
          cf[l] = 1 - cf[l];
        }
        if (last_out && z && s == n_post - 1) {  // final C half writes the natural result
          ProfScope ps = prof_level(c, KC_SMOOTH_L0, lv.A, lv.nnz_C, lv.nC,
                                    (double)lv.nC * 3 * ts + lv.nS * ts + (double)lv.nX * (4 + ts),
                                    kname(c, "k_half_out", lv.A));
          with_layout(lv.A.fmt, lv.A.tpr,
                      HalfOutL<T>{c, lv.A, lv.nX, lv.nC, lv.nS, lv.dinv.get(), B[l].get(),
                                  gather_cf<T>(Xb(l, cc[l]), Xb(l, cf[l]), lv.nC), X0[l].get(),
                                  lv.perm.get(), z});
          return;
        }
        ProfScope ps = prof_level(c, cls_of(l, KC_SMOOTH_L0), lv.A, lv.nnz_C, lv.nC,
                                  (double)lv.nC * 4 * ts + lv.nS * ts, kname(c, "k_half", lv.A));
        with_layout(lv.A.fmt, lv.A.tpr,
                    HalfL<T>{c, lv.A, 0, lv.nC, lv.dinv.get(), B[l].get(),
                             gather_cf<T>(Xb(l, cc[l]), Xb(l, cf[l]), lv.nC), Xb(l, cc[l]),
                             Xb(l, 1 - cc[l])});
        cc[l] = 1 - cc[l];
      }
    }
    if (last_out && !z) {  // the result stays in stored order
      out_cc = cc[0];
      out_cf = cf[0];
      return;
    }
    if (last_out) {  // no post-smoothing (or no stored rows): copy out
      hipLaunchKernelGGL(k_out<T>, dim3(cdiv(lv.nX, 256)), dim3(256), 0, c->stream, lv.nX,
                         gather_cfd<T>(Xb(0, cc[0]), Xb(0, cf[0]), X0[0].get(), lv.nC, lv.nS),
                         (const int*)lv.perm.get(), z);
      MGD_CHECK_LAUNCH();
    }
  }
  if (lt == 0 && bot_from == 0) {  // the whole cycle was the bottom: its result is in X0
    out_cc = out_cf = 0;
    if (!z) return;
    ULevel<T>& lv = L[0];
    hipLaunchKernelGGL(k_out<T>, dim3(cdiv(lv.nX, 256)), dim3(256), 0, c->stream, lv.nX,
                       gather_cfd<T>(X0[0].get(), X0[0].get(), X0[0].get(), lv.nC, lv.nS),
                       (const int*)lv.perm.get(), z);
    MGD_CHECK_LAUNCH();
  }
}

// Levels from which the persistent tail takes over: the first level from
// which every level has at most MGD_TAIL_ROWS extended rows (default
// kTailRows = 0: off, the per-level launches measure faster on gfx950, where
// the barrier's device-scope release and acquire write back and invalidate
// the L2 of the workgroup's chiplet at every phase).  Workgroups:
// MGD_TAIL_BLOCKS (default kTailBlocks), capped by what the device holds
// resident at once.
constexpr int kTailRows = 0;
constexpr int kTailBlocks = 256;

// The phase table of vcycle() for levels >= tail_from, recorded with the same
// buffer choices (the two iterate buffers of every level start at X0 in each
// cycle, so the table is the same for every cycle).
template <typename T>
void Union<T>::build_tail(Ctx* c) {
  tail_from = -1;
  const int nl = (int)L.size();
  const long long rows = env_ll("MGD_TAIL_ROWS", kTailRows);
  if (gs || n_pre < 1 || rows <= 0 || nl < 2 || bot_from >= 0) return;
  int lt = nl;
  while (lt > 1 && L[lt - 1].nX <= rows) --lt;
  if (lt >= nl) return;
  std::vector<int> cc(nl, 0), cf(nl, 0);
  auto Xb = [&](int l, int which) -> T* { return which ? X1[l].get() : X0[l].get(); };
  std::vector<TailOp<T>> ops;
  double bytes = 0, bytes_csr = 0;
  const size_t ts = sizeof(T);
  auto mat_op = [&](int kind, const LMat<T>& m, int r0, int r1, long long nnz, double vec) {
    TailOp<T> o{};
    o.kind = kind;
    o.fmt = m.fmt;
    o.tpr = m.fmt == kFmtCSR ? tpr_of(m.tpr) : 1;
    o.r0 = r0;
    o.r1 = r1;
    o.rp = m.rp.get();
    o.ci = m.ci.get();
    o.v = m.v.get();
    bytes += mat_bytes(m, nnz) + vec;
    bytes_csr += (double)nnz * (ts + 4) + 4.0 * (r1 - r0) + vec;
    return o;
  };
  auto gather = [&](TailOp<T>& o, int l) {
    o.xc = Xb(l, cc[l]);
    o.f_minus_c = Xb(l, cf[l]) - Xb(l, cc[l]);
    o.nC = L[l].nC;
  };
  for (int l = lt; l < nl; ++l) {  // down: the same steps as vcycle()
    ULevel<T>& lv = L[l];
    const int nF = lv.nS - lv.nC;
    if (lv.nS > 0) {
      for (int s = 0; s < n_pre; ++s) {
        if (s > 0) {
          if (lv.nC > 0) {
            TailOp<T> o = mat_op(kTopHalf, lv.A, 0, lv.nC, lv.nnz_C, (double)lv.nC * 4 * ts + lv.nS * ts);
            gather(o, l);
            o.dinv = lv.dinv.get();
            o.B = B[l].get();
            o.xold = Xb(l, cc[l]);
            o.out = Xb(l, 1 - cc[l]);
            ops.push_back(o);
          }
          cc[l] = 1 - cc[l];
        }
        if (nF > 0) {
          TailOp<T> o = mat_op(s == 0 ? kTopFHalf0 : kTopHalf, lv.A, lv.nC, lv.nS, lv.nnz_F,
                               (double)nF * (s == 0 ? 3 : 4) * ts + (s == 0 ? lv.nC : lv.nS) * ts);
          gather(o, l);
          o.dinv = lv.dinv.get();
          o.B = B[l].get();
          o.xold = Xb(l, cf[l]);
          o.out = Xb(l, 1 - cf[l]);
          ops.push_back(o);
          cf[l] = 1 - cf[l];
        }
      }
      if (lv.nX_next > 0) {
        TailOp<T> o = mat_op(kTopResid, lv.A, 0, lv.nS, lv.A.nnz, (double)lv.nS * 3 * ts);
        gather(o, l);
        o.B = B[l].get();
        o.out = R[l].get();
        ops.push_back(o);
        const ULevel<T>& nx = L[l + 1];
        TailOp<T> q = mat_op(kTopRestrict, lv.Wt, 0, lv.nX_next, lv.Wt.nnz,
                             (double)lv.nX_next * (4 + ts) + (double)nx.nC * 2 * ts + lv.nS * ts);
        q.nC = lv.nC;
        q.nCn = nx.nC;
        q.pre = 1;
        q.map = lv.cpos.get();
        q.B = R[l].get();
        q.dinv = nx.dinv.get();
        q.out = B[l + 1].get();
        q.out2 = X0[l + 1].get();
        ops.push_back(q);
      }
    }
    if (!lv.dense.empty()) {
      TailOp<T> o{};
      o.kind = kTopDense;
      o.dense = (const DenseDev*)lv.dense_dev.get();
      o.ndense = (int)lv.dense.size();
      o.dchunks = cdiv(lv.dense_max_n, 64);
      o.B = B[l].get();
      o.out = X0[l].get();
      bytes += 8.0 * lv.dense_entries + 2.0 * ts * (lv.nX - lv.nS);
      bytes_csr += 8.0 * lv.dense_entries + 2.0 * ts * (lv.nX - lv.nS);
      ops.push_back(o);
    }
  }
  for (int l = nl - 1; l >= lt; --l) {  // up
    ULevel<T>& lv = L[l];
    const int nF = lv.nS - lv.nC;
    if (lv.nS > 0 && lv.nX_next > 0) {
      const ULevel<T>& nx = L[l + 1];
      TailOp<T> o = mat_op(kTopProlong, lv.W, 0, lv.nS, lv.W.nnz,
                           (double)lv.nC * 4 + lv.nS * 2.0 * ts + (double)lv.nX_next * ts);
      o.xc = Xb(l + 1, cc[l + 1]);
      o.f_minus_c = Xb(l + 1, cf[l + 1]) - Xb(l + 1, cc[l + 1]);
      o.d_minus_c = X0[l + 1].get() - Xb(l + 1, cc[l + 1]);
      o.nC = nx.nC;
      o.nS = nx.nS;
      o.nCn = lv.nC;
      o.map = lv.cmap.get();
      o.out2 = Xb(l, cc[l]);
      o.out = Xb(l, cf[l]);
      ops.push_back(o);
    }
    if (lv.nS > 0) {
      for (int s = 0; s < n_post; ++s) {
        if (nF > 0) {
          TailOp<T> o = mat_op(kTopHalf, lv.A, lv.nC, lv.nS, lv.nnz_F, (double)nF * 4 * ts + lv.nS * ts);
          gather(o, l);
          o.dinv = lv.dinv.get();
          o.B = B[l].get();
          o.xold = Xb(l, cf[l]);
          o.out = Xb(l, 1 - cf[l]);
          ops.push_back(o);
          cf[l] = 1 - cf[l];
        }
        if (lv.nC > 0) {
          TailOp<T> o = mat_op(kTopHalf, lv.A, 0, lv.nC, lv.nnz_C, (double)lv.nC * 4 * ts + lv.nS * ts);
          gather(o, l);
          o.dinv = lv.dinv.get();
          o.B = B[l].get();
          o.xold = Xb(l, cc[l]);
          o.out = Xb(l, 1 - cc[l]);
          ops.push_back(o);
        }
        cc[l] = 1 - cc[l];
      }
    }
  }
  if (ops.empty()) return;
  // workgroups resident at once on the whole device
  int dev = 0, cus = 0, per_cu = 0;
  MGD_HIP(hipGetDevice(&dev));
  MGD_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
  MGD_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_tail<T>, kTailThreads, 0));
  const long long want = env_ll("MGD_TAIL_BLOCKS", kTailBlocks);
  tail_blocks = (int)std::max(1LL, std::min(want, (long long)cus * std::max(per_cu, 1)));
  tail_ops.alloc(c, ops.size());
  copy_h2d(c, tail_ops.get(), ops.data(), ops.size());
  tail_sync.alloc(c, 2 * kTailSyncStride);
  fill<unsigned>(c, tail_sync.get(), 0u, 2 * kTailSyncStride);
  tail_nops = (int)ops.size();
  tail_cc = cc[lt];
  tail_cf = cf[lt];
  tail_bytes = bytes;
  tail_bytes_csr = bytes_csr;
  tail_from = lt;
}

template <typename T>
void Union<T>::gs_sweep(Ctx* c, int l, bool descending) {
  ULevel<T>& lv = L[l];
  const int nc = (int)lv.cranges.size();
  for (int q = 0; q < nc; ++q) {
    const auto& r = lv.cranges[descending ? nc - 1 - q : q];
    const int n1 = r[1] - r[0], n2 = r[3] - r[2];
    if (n1 + n2 == 0) continue;
    ProfScope ps(c, cls_of(l, KC_SMOOTH_L0), 0.0, kname(c, "k_gs", lv.A));
    with_layout(lv.A.fmt, lv.A.tpr,
                GsL<T>{c, lv.A, r[0], n1, r[2], n2, lv.dgs.get(), B[l].get(), X0[l].get()});
  }
}

// V-cycle with multicolour Gauss-Seidel: one iterate buffer per level, updated
// in place colour by colour (ascending going down, descending going up)
template <typename T>
void Union<T>::vcycle_gs(Ctx* c, T* z) {
  const int nl = (int)L.size();
  for (int l = 0; l < nl; ++l) {
    ULevel<T>& lv = L[l];
    const int nF = lv.nS - lv.nC;
    if (lv.nS > 0) {
      if (nF > 0) fill<T>(c, X0[l].get() + lv.nC, (T)0, (size_t)nF);  // C part zeroed with B
      for (int s = 0; s < n_pre; ++s) gs_sweep(c, l, false);
      if (lv.nX_next > 0) {
        {
          ProfScope ps(c, cls_of(l, KC_RESID_L0), 0.0, kname(c, "k_resid", lv.A));
          with_layout(lv.A.fmt, lv.A.tpr,
                      ResidL<T>{c, lv.A, lv.nS, B[l].get(),
                                gather_cf<T>(X0[l].get(), X0[l].get(), lv.nC), R[l].get()});
        }
        const ULevel<T>& nx = L[l + 1];
        ProfScope ps(c, cls_of(l, KC_TRANSFER_L0), 0.0, kname(c, "k_restrict", lv.Wt, {"false"}));
        with_layout(lv.Wt.fmt, lv.Wt.tpr,
                    RestrictL<T>{c, lv.Wt, lv.nX_next, lv.nC, nx.nC, lv.cpos.get(), R[l].get(),
                                 nx.dinv.get(), B[l + 1].get(), X0[l + 1].get(), false});
      }
    }
    if (!lv.dense.empty()) {
      ProfScope ps(c, KC_COARSE_SOLVE, 8.0 * lv.dense_entries, ksym(c, "k_dense", {type_name<T>()}));
      dim3 grid(cdiv(lv.dense_max_n, 64), (unsigned)lv.dense.size());
      hipLaunchKernelGGL(k_dense<T>, grid, dim3(256), 0, c->stream,
                         (const DenseDev*)lv.dense_dev.get(), (const T*)B[l].get(), X0[l].get());
      MGD_CHECK_LAUNCH();
    }
  }
  for (int l = nl - 1; l >= 0; --l) {
    ULevel<T>& lv = L[l];
    if (lv.nS > 0 && lv.nX_next > 0) {
      const ULevel<T>& nx = L[l + 1];
      ProfScope ps(c, cls_of(l, KC_TRANSFER_L0), 0.0, kname(c, "k_prolong", lv.W));
      with_layout(lv.W.fmt, lv.W.tpr,
                  ProlongL<T>{c, lv.W, lv.nS, lv.nC, lv.cmap.get(),
                              gather_cfd<T>(X0[l + 1].get(), X0[l + 1].get(), X0[l + 1].get(),
                                            nx.nC, nx.nS),
                              X0[l].get(), X0[l].get()});
    }
    if (lv.nS > 0)
      for (int s = 0; s < n_post; ++s) gs_sweep(c, l, true);
  }
  ULevel<T>& l0 = L[0];
  hipLaunchKernelGGL(k_out<T>, dim3(cdiv(l0.nX, 256)), dim3(256), 0, c->stream, l0.nX,
                     gather_cfd<T>(X0[0].get(), X0[0].get(), X0[0].get(), l0.nC, l0.nS),
                     (const int*)l0.perm.get(), z);
  MGD_CHECK_LAUNCH();
}

template <typename T>
void Union<T>::apply_seg(Ctx* c, int N, const SegIn* tab, const double* r, const T* w, T* z) {
  ULevel<T>& l0 = L[0];
  MGD_REQUIRE(N > 0 && (long long)N * members == l0.nX, "apply_seg: rows do not match the union");
  MGD_REQUIRE(z || (!gs && tail_from != 0), "apply_seg: stored-order result needs level-0 launches");
  const bool pre = n_pre > 0 && !gs;
  {
    // iperm, r and the coefficients (FP64), w, d^-1 on C rows, B and X_C written
    ProfScope ps(c, KC_TRANSFER_L0,
                 (double)l0.nX * (4 + 16 + 2.0 * sizeof(T)) + l0.nC * 2.0 * sizeof(T),
                 ksym(c, "k_entry_nat", {type_name<T>(), pre ? "true" : "false"}));
    const dim3 grid(cdiv(N, 256), members);
    if (pre)
      hipLaunchKernelGGL((k_entry_nat<T, true>), grid, dim3(256), 0, c->stream, N, l0.nC,
                         (const int*)l0.iperm.get(), (const T*)l0.dinv_nat.get(), tab, r, w,
                         B[0].get(), X0[0].get());
    else
      hipLaunchKernelGGL((k_entry_nat<T, false>), grid, dim3(256), 0, c->stream, N, l0.nC,
                         (const int*)l0.iperm.get(), (const T*)l0.dinv_nat.get(), tab, r, w,
                         B[0].get(), X0[0].get());
    MGD_CHECK_LAUNCH();
  }
  if (gs)
    vcycle_gs(c, z);
  else
    vcycle(c, z);
  t_prof_level = -1;
}

template <typename T>
StoredOut<T> Union<T>::stored_out() const {
  const ULevel<T>& l0 = L[0];
  return {l0.iperm.get(), (out_cc ? X1[0] : X0[0]).get(), (out_cf ? X1[0] : X0[0]).get(),
          X0[0].get(), l0.nC, l0.nS};
}

template <typename T>
void Union<T>::apply(Ctx* c, const T* bvec, T* z, int cycles) {
  ULevel<T>& l0 = L[0];
  const bool pre = n_pre > 0 && !gs;  // first-sweep C values (CF-l1-Jacobi only)
  {
    ProfScope ps(c, KC_TRANSFER_L0, (double)l0.nX * (4 + 2.0 * sizeof(T)) + l0.nC * 2.0 * sizeof(T),
                 ksym(c, "k_entry", {type_name<T>(), pre ? "true" : "false"}));
    if (pre)
      hipLaunchKernelGGL((k_entry<T, true>), dim3(cdiv(l0.nX, 256)), dim3(256), 0, c->stream,
                         l0.nX, l0.nC, (const int*)l0.perm.get(), (const T*)l0.dinv.get(), bvec,
                         B[0].get(), X0[0].get());
    else
      hipLaunchKernelGGL((k_entry<T, false>), dim3(cdiv(l0.nX, 256)), dim3(256), 0, c->stream,
                         l0.nX, l0.nC, (const int*)l0.perm.get(), (const T*)l0.dinv.get(), bvec,
                         B[0].get(), X0[0].get());
    MGD_CHECK_LAUNCH();
  }
  if (gs)
    vcycle_gs(c, z);
  else
    vcycle(c, z);
  for (int k = 1; k < cycles; ++k) {
    {
      ProfScope ps = prof_level(c, KC_RESID_L0, l0.A, l0.A.nnz, l0.nS,
                                (double)l0.nX * (8 + 3.0 * sizeof(T)),
                                kname(c, "k_entry_resid", l0.A, {pre ? "true" : "false"}));
      with_layout(l0.A.fmt, l0.A.tpr,
                  EntryResidL<T>{c, l0.A, l0.nX, l0.nS, l0.nC, l0.perm.get(), l0.dinv.get(), bvec,
                                 z, B[0].get(), X0[0].get(), pre});
    }
    if (gs)
      vcycle_gs(c, t1.get());
    else
      vcycle(c, t1.get());
    hipLaunchKernelGGL(k_axpy_t<T>, dim3(cdiv(n0, 256)), dim3(256), 0, c->stream, n0,
                       (const T*)t1.get(), z);
    MGD_CHECK_LAUNCH();
  }
  t_prof_level = -1;
}

template <typename T>
double Union<T>::bytes_per_vcycle() const {
  const double ts = sizeof(T);
  double s = 0;
  for (size_t l = 0; l < L.size(); ++l) {
    const auto& lv = L[l];
    const double nF = lv.nS - lv.nC;
    if (lv.nS > 0) {
      s += mat_bytes(lv.A, lv.nnz_F) * (n_pre + n_post) + mat_bytes(lv.A, lv.nnz_C) * (n_pre + n_post - 1);
      s += (nF * 4 * ts + lv.nS * ts) * (n_pre + n_post) +
           (lv.nC * 4 * ts + lv.nS * ts) * (n_pre + n_post - 1);
      if (lv.nX_next > 0) {
        s += mat_bytes(lv.A, lv.A.nnz) + lv.nS * 3 * ts;
        s += mat_bytes(lv.Wt, lv.Wt.nnz) + lv.nX_next * (4 + ts) + lv.nS * ts;
        s += mat_bytes(lv.W, lv.W.nnz) + lv.nC * 4.0 + lv.nS * 2.0 * ts + lv.nX_next * ts;
      }
    }
    s += 8.0 * lv.dense_entries;
  }
  return s;
}

static std::mutex g_tune_mu;
static std::map<std::string, int> g_tune;
static bool g_tune_loaded = false;

static std::string tune_key(long long rows, long long nnz, int maxrow, bool fp32,
                            const char* kind) {
  std::ostringstream o;
  o << (fp32 ? "f32:" : "f64:") << kind << rows << ":" << nnz << ":" << maxrow;
  return o.str();
}
static void tune_load_locked() {
  if (g_tune_loaded) return;
  g_tune_loaded = true;
  const char* path = std::getenv("MGD_AUTOTUNE_CACHE");
  if (!path) return;
  std::ifstream f(path);
  std::string tok;
  // format: {"key": value, ...}
  std::string all((std::istreambuf_iterator<char>(f)), std::istreambuf_iterator<char>());
  size_t p = 0;
  while ((p = all.find('"', p)) != std::string::npos) {
    size_t q = all.find('"', p + 1);
    if (q == std::string::npos) break;
    std::string key = all.substr(p + 1, q - p - 1);
    size_t colon = all.find(':', q);
    if (colon == std::string::npos) break;
    g_tune[key] = std::atoi(all.c_str() + colon + 1);
    p = colon + 1;
  }
}
static void tune_save_locked() {
  const char* path = std::getenv("MGD_AUTOTUNE_CACHE");
  if (!path) return;
  std::ofstream f(path);
  f << "{";
  bool first = true;
  for (auto& kv : g_tune) {
    f << (first ? "" : ",") << "\n  \"" << kv.first << "\": " << kv.second;
    first = false;
  }
  f << "\n}\n";
}
int autotune_lookup(long long rows, long long nnz, int maxrow, bool fp32, const char* kind) {
  std::lock_guard<std::mutex> g(g_tune_mu);
  tune_load_locked();
  auto it = g_tune.find(tune_key(rows, nnz, maxrow, fp32, kind));
  return it == g_tune.end() ? 0 : it->second;
}
void autotune_store(long long rows, long long nnz, int maxrow, bool fp32, int tpr,
                    const char* kind) {
  std::lock_guard<std::mutex> g(g_tune_mu);
  tune_load_locked();
  g_tune[tune_key(rows, nnz, maxrow, fp32, kind)] = tpr;
  tune_save_locked();
}

// ---------------------------------------------------------------------------
// level layouts
// ---------------------------------------------------------------------------
template <typename T>
__global__ void k_sell_fill(int rows, const int* __restrict__ rp, const int* __restrict__ ci,
                            const double* __restrict__ v, const int* __restrict__ off,
                            int self_pad, int* __restrict__ sci, T* __restrict__ sv) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= rows) return;
  const int o = off[r >> 6] + (r & 63), w = (off[(r >> 6) + 1] - off[r >> 6]) >> 6;
  const int e0 = rp[r], len = rp[r + 1] - e0;
  const int pad = self_pad ? r : 0;  // padding reads a defined element with weight zero
  for (int e = 0; e < w; ++e) {
    const bool in = e < len;
    sci[o + 64 * e] = in ? ci[e0 + e] : pad;
    sv[o + 64 * e] = in ? (T)v[e0 + e] : (T)0;
  }
}

// Test override: MGD_SELL16_SPAN lowers the column span a slice side may have
// in the 16-bit layout (so that small systems get 32-bit slices too).
static int sell16_span() {
  const char* e = std::getenv("MGD_SELL16_SPAN");
  const int d = 0x7fff;
  return e && *e ? std::min(d, std::max(0, std::atoi(e))) : d;
}

// SELL16 bases of slice s from the real entries of its rows (CSR M): the
// smallest column below `split` and the smallest at or above it (0 without
// one); a side spanning more than `span` (<= 2^15 - 1) columns makes the
// slice keep 32-bit columns (F base -1).  units[s]: the slice's code size in
// 16-bit units.
// One wave per slice, one lane per row.
__global__ void __launch_bounds__(256) k_sell16_bases(int rows, const int* __restrict__ rp,
                                                      const int* __restrict__ ci, int split,
                                                      int span, const int* __restrict__ off,
                                                      int* __restrict__ rp4,
                                                      int* __restrict__ units) {
  const int r = blockIdx.x * 256 + threadIdx.x, s = r >> 6;
  const int ns = (rows + 63) / 64;
  int cmin = INT_MAX, cmax = -1, fmin = INT_MAX, fmax = -1;
  if (r < rows)
    for (int e = rp[r]; e < rp[r + 1]; ++e) {
      const int j = ci[e];
      if (j < split) {
        cmin = min(cmin, j);
        cmax = max(cmax, j);
      } else {
        fmin = min(fmin, j);
        fmax = max(fmax, j);
      }
    }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    cmin = min(cmin, __shfl_xor(cmin, o, 64));
    cmax = max(cmax, __shfl_xor(cmax, o, 64));
    fmin = min(fmin, __shfl_xor(fmin, o, 64));
    fmax = max(fmax, __shfl_xor(fmax, o, 64));
  }
  if ((threadIdx.x & 63) != 0 || s >= ns) return;
  const bool wide = (cmax >= 0 && cmax - cmin > span) || (fmax >= 0 && fmax - fmin > span);
  rp4[4 * s] = off[s];
  rp4[4 * s + 2] = cmax >= 0 ? cmin : 0;
  rp4[4 * s + 3] = wide ? -1 : (fmax >= 0 ? fmin : 0);
  units[s] = (off[s + 1] - off[s]) * (wide ? 2 : 1);
  if (s == ns - 1) rp4[4 * ns] = off[ns];
}
__global__ void k_sell16_coff(int ns, const int* __restrict__ coff, int* __restrict__ rp4) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s <= ns) rp4[4 * s + 1] = coff[s];
}
// codes of row r: column - C base below the split, (column - F base) | 2^15
// at or above it, or the column itself in a 32-bit slice; padding elements
// get code 0 (the C base, or column 0, with weight zero)
__global__ void k_sell16_encode(int rows, const int* __restrict__ rp, const int* __restrict__ ci,
                                int split, const int* __restrict__ rp4, uint16_t* __restrict__ c16) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= rows) return;
  const int s4 = 4 * (r >> 6);
  const int w = (rp4[s4 + 4] - rp4[s4]) >> 6;
  const int cb = rp4[s4 + 2], fb = rp4[s4 + 3];
  const int e0 = rp[r], len = rp[r + 1] - e0;
  if (fb < 0) {
    int* c32 = reinterpret_cast<int*>(c16) + (rp4[s4 + 1] >> 1) + (r & 63);
    for (int q = 0; q < w; ++q) c32[64 * q] = q < len ? ci[e0 + q] : 0;
    return;
  }
  const int oc = rp4[s4 + 1] + (r & 63);
  for (int q = 0; q < w; ++q) {
    unsigned code = 0;
    if (q < len) {
      const int j = ci[e0 + q];
      code = j < split ? (unsigned)(j - cb) : (0x8000u | (unsigned)(j - fb));
    }
    c16[oc + 64 * q] = (uint16_t)code;
  }
}
// every real element decodes to its CSR column, every padding element to a
// column inside [0, ncols)
__global__ void k_sell16_check(int rows, int ncols, const int* __restrict__ rp,
                               const int* __restrict__ ci, const int* __restrict__ rp4,
                               const int* __restrict__ codes, int* __restrict__ err) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= rows) return;
  int o, oc, w, cb, fb;
  sell_slice<kFmtSELL16>(rp4, r, o, oc, w, cb, fb);
  const int e0 = rp[r], len = rp[r + 1] - e0;
  for (int q = 0; q < w; ++q) {
    const int j = fb >= 0 ? sell_col<true>(codes, oc + 64 * q, cb, fb)
                          : sell_col<false>(codes, oc + 64 * q, cb, fb);
    if (q < len ? j != ci[e0 + q] : (j < 0 || j >= ncols)) atomicOr(err, 4);
  }
}

// Longest row (longest[0]) and SELL layout of a CSR structure: slice widths in
// w64, slice offsets in soff, the stored entries with padding in longest[1]
// (kScanTooLarge where int32 cannot hold them: soff is of no use then).
static void row_stats(Ctx* c, int rows, const int* rp, DBuf<int>& w64, DBuf<int>& soff,
                      int* longest) {
  if (rows <= 0) return;
  const int ns = cdiv(rows, 64);
  w64.alloc(c, (size_t)ns);
  soff.alloc(c, (size_t)ns + 1);
  hipLaunchKernelGGL(k_row_stats, dim3(std::min(cdiv(rows, 256), kStatBlocks)), dim3(256), 0, c->stream, rows, rp,
                     w64.get(), longest);
  MGD_CHECK_LAUNCH();
  exclusive_scan(c, w64.get(), soff.get(), ns);
  copy_d2d(c, longest + 1, soff.get() + ns, 1);
}

// CSR (FP64 values) -> layout `fmt` with values in T; `self_pad` pads SELL rows
// with their own index as column (square stored-order matrices), else column 0.
// A SELL result (slice offsets soff, `stored` entries) becomes SELL16 when
// split16 >= 0.
template <typename T>
static void to_layout(Ctx* c, const Csr<double>& M, int fmt, int tpr, bool self_pad,
                      LMat<T>& out, const DBuf<int>& soff, long long stored, int split16 = -1) {
  out.rows = M.n_rows;
  out.nnz = M.nnz;
  out.fmt = fmt;
  out.tpr = tpr;
  if (fmt == kFmtCSR || M.n_rows == 0) {
    out.fmt = kFmtCSR;
    out.stored = M.nnz;
    out.rp.alloc(c, (size_t)M.n_rows + 1);
    copy_d2d(c, out.rp.get(), M.rp.get(), (size_t)M.n_rows + 1);
    out.ci.alloc(c, (size_t)std::max(M.nnz, 1));
    copy_d2d(c, out.ci.get(), M.ci.get(), (size_t)M.nnz);
    out.v.alloc(c, (size_t)std::max(M.nnz, 1));
    cast_copy<T, double>(c, out.v.get(), M.v.get(), (size_t)M.nnz, KC_VEC);
    return;
  }
  const int ns = cdiv(M.n_rows, 64);
  out.rp.alloc(c, (size_t)ns + 1);
  copy_d2d(c, out.rp.get(), soff.get(), (size_t)ns + 1);
  out.stored = stored;
  out.ci.alloc(c, (size_t)std::max(out.stored, 1LL));
  out.v.alloc(c, (size_t)std::max(out.stored, 1LL));
  hipLaunchKernelGGL(k_sell_fill<T>, dim3(cdiv(M.n_rows, 256)), dim3(256), 0, c->stream,
                     M.n_rows, (const int*)M.rp.get(), (const int*)M.ci.get(),
                     (const double*)M.v.get(), (const int*)out.rp.get(), self_pad ? 1 : 0,
                     out.ci.get(), out.v.get());
  MGD_CHECK_LAUNCH();
  if (split16 < 0 || M.nnz == 0) return;
  DBuf<int> rp4(c, 4 * (size_t)ns + 2), units(c, (size_t)ns), coff(c, (size_t)ns + 1);
  hipLaunchKernelGGL(k_sell16_bases, dim3(cdiv(M.n_rows, 256)), dim3(256), 0, c->stream, M.n_rows,
                     (const int*)M.rp.get(), (const int*)M.ci.get(), split16, sell16_span(),
                     (const int*)out.rp.get(), rp4.get(), units.get());
  MGD_CHECK_LAUNCH();
  exclusive_scan(c, units.get(), coff.get(), ns);
  const long long total = read1(c, coff.get() + ns);
  if (total < 0) return;  // codes past int32: the 32-bit columns stay
  hipLaunchKernelGGL(k_sell16_coff, dim3(cdiv(ns + 1, 256)), dim3(256), 0, c->stream, ns,
                     (const int*)coff.get(), rp4.get());
  MGD_CHECK_LAUNCH();
  DBuf<int> codes(c, (size_t)std::max(1LL, (total + 1) / 2));
  hipLaunchKernelGGL(k_sell16_encode, dim3(cdiv(M.n_rows, 256)), dim3(256), 0, c->stream,
                     M.n_rows, (const int*)M.rp.get(), (const int*)M.ci.get(), split16,
                     (const int*)rp4.get(), reinterpret_cast<uint16_t*>(codes.get()));
  MGD_CHECK_LAUNCH();
  hipLaunchKernelGGL(k_sell16_check, dim3(cdiv(M.n_rows, 256)), dim3(256), 0, c->stream,
                     M.n_rows, M.n_cols, (const int*)M.rp.get(), (const int*)M.ci.get(),
                     (const int*)rp4.get(), (const int*)codes.get(), c->err_flag());
  MGD_CHECK_LAUNCH();
  out.rp = std::move(rp4);
  out.ci = std::move(codes);
  out.fmt = kFmtSELL16;
}
template <typename T>
static void tune_layout(Ctx* c, ULevel<T>& lv, const BuildLevel<T>& b, const int* st, int autotune,
                        bool fp32);
template <typename T>
static void tune_restrict(Ctx* c, const ULevel<T>& lv, const BuildLevel<T>& b, const int* st,
                          LMat<T>& out, int autotune, bool fp32);

constexpr long long kFillLanes = 1 << 17;  // lanes that keep all compute units busy
constexpr int kSellMinRows = 1 << 17;
// Test overrides: MGD_SELL_MIN_ROWS lowers the row count from which sliced
// layouts are considered (so that small systems exercise them), MGD_SELL16=0
// keeps sliced layouts at 32-bit columns.
static long long sell_min_rows() {
  const char* e = std::getenv("MGD_SELL_MIN_ROWS");
  return e && *e ? std::max(1LL, std::atoll(e)) : (long long)kSellMinRows;
}
// Matrices with fewer rows keep the default layout rule: their launches are
// latency bound, and timing them back to back with their data in cache does
// not rank the layouts as their launches inside a cycle do.  MGD_TUNE_MIN_ROWS
// (tests) lowers the bound.
constexpr int kTuneMinRows = 1 << 17;
static long long tune_min_rows() {
  const char* e = std::getenv("MGD_TUNE_MIN_ROWS");
  return e && *e ? std::max(1LL, std::atoll(e)) : (long long)kTuneMinRows;
}
static bool sell16_enabled() {
  const char* e = std::getenv("MGD_SELL16");
  return !(e && e[0] == '0');
}
// lanes per row so that a small matrix still spreads over the device
static int small_level_tpr(long long rows, double avg) {
  int t = 1;
  while (t < 64 && rows * t < kFillLanes && t < avg) t *= 2;
  return t;
}
// Padding up to which a large matrix is stored as SELL without timing it.  Its
// 2-byte columns and unit-stride loads pay for padding that CSR does not read:
// with 1.3, 1.4, 1.5, 1.6 and 2.0 a solve at 3D 64^3, G = 20 (lower levels pad
// by 1.34 and 1.46) took 52.0, 48.8, 48.2, 48.2 and 48.2 ms with FP32
// hierarchies and 66.9, 62.2, 61.9, 61.9, 61.8 ms with FP64, at 3D 80^3, G = 2
// 32.6, 31.8, 31.8, 31.8, 31.8 ms; 2D 256^2 and 512^2 were the same throughout.
constexpr double kSellPad = 1.5;
// entries of a SELL layout; one that int32 cannot index is more than any limit
constexpr long long kSellTooLarge = 1LL << 62;
static long long sell_entries_of(int stat) { return stat < 0 ? kSellTooLarge : stat; }
// interpolation / restriction layout: SELL for large matrices with little
// padding (sell_entries: the SELL layout's stored entries), otherwise CSR with
// enough lanes per row; the result is kTuneSell (1000) or the lanes per row
static int transfer_default(const Csr<double>& M, long long sell_entries) {
  const double avg = M.n_rows ? (double)M.nnz / M.n_rows : 1.0;
  if (M.nnz > 0 && M.n_rows >= sell_min_rows() && sell_entries <= (long long)(kSellPad * M.nnz))
    return 1000;
  return std::max(small_level_tpr(M.n_rows, avg), default_tpr(avg));
}
template <typename T>
static void layout_transfer(Ctx* c, const Csr<double>& M, LMat<T>& out, const DBuf<int>& soff,
                            long long stored, int split16) {
  const int d = transfer_default(M, stored);
  if (d == 1000)
    to_layout<T>(c, M, kFmtSELL, 1, false, out, soff, stored, sell16_enabled() ? split16 : -1);
  else
    to_layout<T>(c, M, kFmtCSR, d, false, out, soff, stored);
}

// The operations of a member's cycle over its levels lev[0 .. n), the same as
// Union::vcycle's launches; tmp: values shared by the levels (the residual, and
// the new values of a half-sweep).
static void bot_program(const BotLevel* lev, int n, int n_pre, int n_post, int tmp,
                        std::vector<BotOp>& ops) {
  auto on_A = [&](int l, int kind) {
    const BotLevel& L = lev[l];
    BotOp o{};
    o.kind = kind;
    o.in = L.in_lds;
    o.sC = cdiv(L.nC, 64);
    o.rC = L.nC;
    o.rows = L.n;
    o.s1 = o.sC + cdiv(L.n - L.nC, 64);
    o.so = L.sA;
    o.co = L.cA;
    o.vo = L.vA;
    o.x = L.vec + L.n;
    o.b = L.vec;
    o.out = tmp;
    o.dv = o.map = L.dv;
    o.nd = L.n - 1;
    return o;
  };
  auto half = [&](int l, bool F, int kind) {
    BotOp o = on_A(l, kind);
    if (F)
      o.s0 = o.sC;
    else
      o.s1 = o.sC;
    if (o.s1 > o.s0) ops.push_back(o);
  };
  for (int l = 0; l < n; ++l) {
    const BotLevel& L = lev[l];
    if (L.kind == 2) {
      BotOp o{};
      o.kind = kBotDense;
      o.in = L.in_lds;
      o.rows = L.n;
      o.vo = L.vA;
      o.b = L.vec;
      o.out = L.vec + L.n;
      ops.push_back(o);
      break;
    }
    half(l, true, kBotFHalf0);
    for (int s = 1; s < n_pre; ++s) {
      half(l, false, kBotHalf);
      half(l, true, kBotHalf);
    }
    if (L.kind != 0) continue;
    ops.push_back(on_A(l, kBotResid));
    const BotLevel& N = lev[l + 1];
    BotOp r{};
    r.kind = kBotRestrict;
    r.in = L.in_lds;
    r.sC = r.s1 = cdiv(L.nn, 64);
    r.rC = r.rows = L.nn;
    r.so = L.sT;
    r.co = L.cT;
    r.vo = L.vT;
    r.x = r.b = tmp;
    r.map = L.cp;
    r.out = N.vec;
    r.out2 = N.vec + N.n;
    r.nC = N.nC;
    r.dv = N.nC > 0 ? N.dv : L.dv;
    r.nd = N.nC > 0 ? N.n - 1 : 0;
    ops.push_back(r);
  }
  for (int l = n - 1; l >= 0; --l) {
    const BotLevel& L = lev[l];
    if (L.kind == 2) continue;
    if (L.kind == 0) {
      const BotLevel& N = lev[l + 1];
      BotOp o{};
      o.kind = kBotProlong;
      o.in = L.in_lds;
      o.sC = o.s1 = cdiv(L.n - L.nC, 64);
      o.rC = o.rows = L.n - L.nC;
      o.so = L.sW;
      o.co = L.cW;
      o.vo = L.vW;
      o.x = N.vec + N.n;
      o.b = L.vec;
      o.dv = L.dv;
      o.map = L.cm;
      o.nC = L.nC;
      o.out = L.vec + L.n + L.nC;
      o.out2 = L.vec + L.n;
      ops.push_back(o);
    }
    for (int s = 0; s < n_post; ++s) {
      half(l, true, kBotHalf);
      half(l, false, kBotHalf);
    }
  }
}

// The bottom of the cycle (BotLevel, k_bottom): the levels from which on every
// member has at most kBotRows rows, none of them too long, if any of them coarsens (a lone dense level
// stays with k_dense).  MGD_BOTTOM=0 (or MGD_TAIL_ROWS, whose launch takes these
// levels instead) keeps per-level launches, with one lane per row there: the
// same bits.  With members of at most 0 (no bottom), 300, 600, 1200 and 2048 rows
// an apply took, in us: 2D 101^2 G = 5 Schur1 777, 728, 605, 509, 507; 2D 64^2
// Schur2 303, 197, 203, 170, 169; 3D 20^3 G = 3 Schur2 447, 486, 335, 329, 347
// (its 300-row bottom has one short level); batched 2D 256^2 G = 20 PCTL 644, 589,
// 588, 561, 561.  Above 2048 rows a matrix outgrows LDS and 16 rows a lane would
// be in sequence.  A matrix is limited to what LDS could hold (values and 16-bit
// columns): past it one compute unit reads it from L2 four times a cycle.  With
// limits of 2^14 (FP64's, nearly), 2^15 and 2^16 entries FP64 applies of one hierarchy with long rows took 176, 174 and 187
// us (2D 101^2 G = 20), 360, 379 and 379 us (3D 46^3 G = 6; 355 with launches), on
// the first of the cases above 504, 500 and 500, an FP32 solve at 2D 256^2 G = 20
// 18.7, 18.6 and 18.6 ms.
// While the finest level leaves compute units free beside a concurrent block
// matvec (one workgroup per 512 rows), a member takes a whole unit; above that,
// 512 threads and 110 KB, which fit beside a workgroup of the matvec.
constexpr long long kBotWholeRows = 512 * 192;
constexpr unsigned kBotLdsWhole = 150 * 1024, kBotLdsShared = 110 * 1024;
constexpr long long kBotMatrix = 160 * 1024;  // bytes of a matrix and member
// Longest row: one lane adds it entry after entry, a launch of the level shares it
// among up to 64.  With limits of 96, 128, 192 entries and none, FP64 applies of a
// grid of 30^2 rows with one row of 128 couplings took 45.3, 45.1, 51.3 and 51.3 us
// (46.0 with launches alone), of 14^2 with 96 couplings 26.2, 17.5, 17.7 and 17.6
// (26.4); FP32 applies of 44^2 with 96, 128 and 190 couplings took 58.7, 79.4 and
// 79.4 us with 128, 68.6, 62.3 and 67.1 with 192, 68.5, 77.0 and 90.7 with none
// (80.0, 78.2 and 75.9).
template <typename T>
constexpr int kBotWidth = sizeof(T) == 8 ? 128 : 192;
constexpr int kBotDenseRows = 256;  // larger dense levels are spread over workgroups

// places of the members in a level's extended stored order
template <typename T>
static std::vector<BotRows> bot_rows_of(const BuildLevel<T>& b, const std::vector<UMember>& tab) {
  std::vector<BotRows> v;
  int cb = 0, fb = b.nC;
  for (int q = 0; q < b.R.nm; ++q) {
    const UMember& m = tab[b.tab + q];
    v.push_back({cb, fb, b.nS + m.dense_before, m.nc, f_rows(m), m.kind});
    cb += m.nc;
    fb += f_rows(m);
  }
  return v;
}

template <typename T>
static std::vector<int> bot_widths(Ctx* c, const std::vector<BuildLevel<T>>& bl,
                                   const std::vector<UMember>& tab, int cand, DBuf<int>& out) {
  const int nl = (int)bl.size(), nm = nl ? bl[0].R.nm : 0;
  if (cand >= nl) return {};
  const size_t per = (size_t)nm * 3 * kBotSlices;
  out.alloc(c, per * (nl - cand));
  fill<int>(c, out.get(), 0, per * (nl - cand));
  std::vector<BotRows> at;
  for (int l = cand; l <= nl; ++l) {
    std::vector<BotRows> r(nm);
    if (l < nl) r = bot_rows_of(bl[l], tab);
    at.insert(at.end(), r.begin(), r.end());
  }
  DBuf<BotRows> dev(c, at.size());
  copy_h2d(c, dev.get(), at.data(), at.size());
  for (int l = cand; l < nl; ++l) {
    if (bl[l].nS == 0) continue;
    const BotRows* d = dev.get() + (size_t)(l - cand) * nm;
    hipLaunchKernelGGL(k_bot_widths, dim3(nm), dim3(256), 0, c->stream, d, d + nm, bl[l].nC,
                       (const int*)bl[l].A.rp.get(), (const int*)bl[l].W.rp.get(),
                       (const int*)bl[l].Wt.rp.get(), out.get() + per * (l - cand));
    MGD_CHECK_LAUNCH();
  }
  return read_vec(c, out.get(), per * (nl - cand));
}

template <typename T>
static void build_bottom(Ctx* c, std::vector<BuildLevel<T>>& bl, const std::vector<UMember>& tab,
                         int cand, const int* widths_dev, const std::vector<int>& widths,
                         Union<T>& U) {
  const int nl = (int)bl.size(), nm = nl ? bl[0].R.nm : 0;
  if (U.gs || U.n_pre < 1 || cand >= nl) return;
  int rows0 = 0;
  for (int q = 0; q < nm; ++q) rows0 = std::max(rows0, tab[bl[0].tab + q].n);
  const bool whole = rows0 <= kBotWholeRows;
  const unsigned budget = whole ? kBotLdsWhole : kBotLdsShared;
  auto wid = [&](int l, int q, int mat) {
    return widths.data() + (((size_t)(l - cand) * nm + q) * 3 + mat) * kBotSlices;
  };
  auto sum = [](const int* w, int n) {
    int s = 0;
    for (int k = 0; k < n; ++k) s += w[k];
    return s;
  };
  // slice columns (64 stored entries each) of the member's A, W and W^T
  auto stored = [&](int l, int q, int mat) {
    const UMember& m = tab[bl[l].tab + q];
    const int sC = cdiv(m.nc, 64), sF = cdiv(f_rows(m), 64);
    if (m.n == 0 || m.kind == 2) return 0;
    if (mat > 0 && m.kind != 0) return 0;
    return sum(wid(l, q, mat), mat == 0 ? sC + sF : (mat == 1 ? sF : sC));
  };
  auto widest = [&](int l, int q, int mat) {  // its longest row there, rounded up to even
    const UMember& m = tab[bl[l].tab + q];
    const int sC = cdiv(m.nc, 64), sF = cdiv(f_rows(m), 64);
    if (m.n == 0 || m.kind == 2 || (mat > 0 && m.kind != 0)) return 0;
    const int* w = wid(l, q, mat);
    return *std::max_element(w, w + std::max(1, mat == 0 ? sC + sF : (mat == 1 ? sF : sC)));
  };
  int lt = nl;
  while (lt > cand) {
    bool ok = true;
    for (int q = 0; q < nm; ++q) {
      const UMember& m = tab[bl[lt - 1].tab + q];
      for (int mat = 0; mat < 3; ++mat)
        ok = ok && 64LL * stored(lt - 1, q, mat) * (long long)(sizeof(T) + 2) <= kBotMatrix &&
             widest(lt - 1, q, mat) <= kBotWidth<T>;
      ok = ok && (m.kind != 2 || m.n <= kBotDenseRows);
    }
    if (!ok) break;
    --lt;
  }
  // vectors and index arrays of every member in LDS
  for (; lt < nl; ++lt) {
    bool fits = true;
    for (int q = 0; q < nm; ++q) {
      size_t v = 0, top = 0, small = 0;
      for (int l = lt; l < nl; ++l) {
        const size_t n = tab[bl[l].tab + q].n;
        v += 2 * n;
        top = std::max(top, n);
        small += n * (sizeof(T) + 4) + 6 * kBotSlices + 128;
        small += (2 * (U.n_pre + U.n_post) + 3) * sizeof(BotOp);
      }
      fits = fits && (v + top) * sizeof(T) + small <= budget;
    }
    if (fits) break;
  }
  bool coarsens = false;
  for (int l = lt; l < nl; ++l) coarsens = coarsens || bl[l].n_coarse > 0;
  if (!coarsens) return;
  for (int l = lt; l < nl; ++l) bl[l].bottom = bl[l].nS > 0;
  const char* off = std::getenv("MGD_BOTTOM");
  if ((off && off[0] == '0') || env_ll("MGD_TAIL_ROWS", 0) > 0) return;
  std::vector<BotMember> mem;
  std::vector<std::vector<BotOp>> progs;
  std::vector<BotPack> pack;            // level by level
  std::vector<size_t> first(nl + 1, 0);
  std::vector<std::vector<BotLevel>> levs;
  std::vector<int> who;
  size_t total = 0;
  for (int q = 0; q < nm; ++q) {
    if (tab[bl[lt].tab + q].n == 0) continue;
    BotMember M{};
    M.buf = total;
    int last = lt;
    while (last + 1 < nl && tab[bl[last + 1].tab + q].n > 0 && tab[bl[last].tab + q].kind == 0) ++last;
    std::vector<BotLevel> lev(last - lt + 1);
    int vec = 0, top = 0;
    for (int l = lt; l <= last; ++l) {
      const UMember& m = tab[bl[l].tab + q];
      BotLevel& L = lev[l - lt];
      L.n = m.n;
      L.kind = m.kind;
      L.nC = L.nn = m.kind == 0 ? m.nc : 0;
      L.vec = vec;
      vec += 2 * m.n;
      top = std::max(top, m.n);
    }
    const int tmp = vec;
    const unsigned vbytes = (unsigned)(((size_t)(vec + top) * sizeof(T) + 15) / 16 * 16);
    unsigned at = 0;
    auto take = [&](size_t bytes) {
      const unsigned o = at;
      at += (unsigned)((bytes + 7) / 8 * 8);
      return o;
    };
    // in LDS in any case: the index arrays and diagonals
    for (int l = last; l >= lt; --l) {
      BotLevel& L = lev[l - lt];
      if (L.kind == 2) continue;
      const int sC = cdiv(L.nC, 64), sF = cdiv(L.n - L.nC, 64);
      L.dv = take(L.n * sizeof(T));
      L.sA = take(2 * (size_t)(sC + sF + 1));
      L.sW = take(2 * (size_t)(sF + 1));
      L.sT = take(2 * (size_t)(sC + 1));
      L.cm = take(2 * (size_t)L.nC);
      L.cp = take(2 * (size_t)L.nn);
    }
    at = (at + 15) / 16 * 16;
    M.ops = at;
    {
      std::vector<BotOp> count;  // as many as the program will have
      bot_program(lev.data(), (int)lev.size(), U.n_pre, U.n_post, tmp, count);
      M.nops = (int)count.size();
    }
    at += (unsigned)((M.nops * sizeof(BotOp) + 15) / 16 * 16);
    M.lds = at;
    // then, while there is room, the matrices (read four times a cycle), the
    // coarsest first, and the dense inverse (read once)
    bool room = true;
    auto place = [&](BotLevel& L) {
      at = (at + 15) / 16 * 16;
      room = room && at + vbytes <= budget;
      L.in_lds = room ? 1 : 0;
      if (room) M.lds = at;
    };
    for (int l = last; l >= lt; --l) {
      BotLevel& L = lev[l - lt];
      if (L.kind == 2) continue;
      const size_t nA = 64 * (size_t)stored(l, q, 0), nW = 64 * (size_t)stored(l, q, 1),
                   nT = 64 * (size_t)stored(l, q, 2);
      L.vA = take(nA * sizeof(T));
      L.vW = take(nW * sizeof(T));
      L.vT = take(nT * sizeof(T));
      L.cA = take(2 * nA);
      L.cW = take(2 * nW);
      L.cT = take(2 * nT);
      place(L);
    }
    if (lev.back().kind == 2) {
      lev.back().vA = take(sizeof(double) * (size_t)lev.back().n * lev.back().n);
      place(lev.back());
    }
    M.vec_at = M.lds;
    U.bot_lds = std::max(U.bot_lds, M.lds + vbytes);
    U.bot_bytes += at + 2.0 * lev[0].n * sizeof(T);
    total += (at + 255) / 256 * 256;
    M.n = lev[0].n;
    M.nC = lev[0].nC;
    M.dv = lev[0].dv;
    progs.emplace_back();
    bot_program(lev.data(), (int)lev.size(), U.n_pre, U.n_post, tmp, progs.back());
    mem.push_back(M);
    levs.push_back(std::move(lev));
    who.push_back(q);
  }
  U.bot_buf.alloc(c, std::max<size_t>(total, 16));
  for (int l = lt; l < nl; ++l) {
    first[l] = pack.size();
    const std::vector<BotRows> at = bot_rows_of(bl[l], tab);
    std::vector<BotRows> next(nm);
    if (l + 1 < nl) next = bot_rows_of(bl[l + 1], tab);
    for (size_t k = 0; k < mem.size(); ++k) {
      const int q = who[k];
      if (l - lt >= (int)levs[k].size()) continue;
      if (l == lt) {
        mem[k].cb = at[q].cb;
        mem[k].fb = at[q].kind == 2 ? at[q].db : at[q].fb;
      }
      BotPack P{};
      P.buf = U.bot_buf.get() + mem[k].buf;
      P.L = levs[k][l - lt];
      P.at = at[q];
      P.next = next[q];
      P.q = (l - cand) * nm + q;
      if (P.L.kind == 2) {
        for (const DenseDev& d : U.L[l].dense)
          if (d.off == at[q].db) P.inv = d.inv;
        MGD_REQUIRE(P.inv, "internal: dense member without an inverse");
      }
      pack.push_back(P);
    }
  }
  first[nl] = pack.size();
  U.bot_mem.alloc(c, mem.size());
  copy_h2d(c, U.bot_mem.get(), mem.data(), mem.size());
  for (size_t k = 0; k < mem.size(); ++k)
    MGD_HIP(hipMemcpyAsync(U.bot_buf.get() + mem[k].buf + mem[k].ops, progs[k].data(),
                           progs[k].size() * sizeof(BotOp), hipMemcpyHostToDevice, c->stream));
  DBuf<BotPack> dp(c, pack.size());
  copy_h2d(c, dp.get(), pack.data(), pack.size());
  for (int l = lt; l < nl; ++l) {
    const unsigned cnt = (unsigned)(first[l + 1] - first[l]);
    if (!cnt) continue;
    const BuildLevel<T>& b = bl[l];
    const BuildLevel<T>* nb = l + 1 < nl ? &bl[l + 1] : nullptr;
    int rows = 1;
    for (size_t k = first[l]; k < first[l + 1]; ++k)
      rows = std::max(rows, 64 * (cdiv(pack[k].L.nC, 64) + cdiv(pack[k].L.n - pack[k].L.nC, 64) + 1));
    hipLaunchKernelGGL(k_bot_pack<T>, dim3(cdiv(rows, 256), cnt), dim3(256), 0, c->stream,
                       (const BotPack*)(dp.get() + first[l]), b.nC, b.nS, nb ? nb->nC : 0,
                       nb ? nb->nS : 0, widths_dev, (const int*)b.A.rp.get(),
                       (const int*)b.A.ci.get(), (const double*)b.A.v.get(),
                       (const int*)b.W.rp.get(), (const int*)b.W.ci.get(),
                       (const double*)b.W.v.get(), (const int*)b.Wt.rp.get(),
                       (const int*)b.Wt.ci.get(), (const double*)b.Wt.v.get(),
                       (const T*)U.L[l].dinv.get(), (const int*)U.L[l].cmap.get(),
                       (const int*)U.L[l].cpos.get(), c->err_flag());
    MGD_CHECK_LAUNCH();
  }
  c->check_device_errors("packed bottom levels");
  const void* kernel = whole ? reinterpret_cast<const void*>(&k_bottom<T, 1024>)
                             : reinterpret_cast<const void*>(&k_bottom<T, 512>);
  MGD_HIP(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)budget));
  U.bot_threads = whole ? 1024 : 512;
  U.bot_members = (int)mem.size();
  U.bot_from = lt;
}

// stats: per level the longest row and the SELL entries of A, W and W^T
template <typename T>
static void layout_levels(Ctx* c, std::vector<BuildLevel<T>>& bl, const int* stats, Union<T>& U,
                          int autotune) {
  const int nl = (int)bl.size();
  for (int l = 0; l < nl; ++l) {
    StepScope st("solve-phase build: layouts of level " + std::to_string(l));
    BuildLevel<T>& b = bl[l];
    ULevel<T>& lv = U.L[l];
    const int* s6 = stats + 6 * l;
    const bool packed = U.bot_from >= 0 && l >= U.bot_from;  // in bot_buf instead
    if (b.bottom && (!packed || l == 0)) {
      // one lane per row, so that per-level launches add a row's entries in the
      // bottom's order (and, at level 0, the residual between cycles, which is
      // always a launch of its own)
      to_layout<T>(c, b.A, kFmtCSR, 1, true, lv.A, b.asoff, 0);
      if (lv.nX_next > 0 && !packed) {
        to_layout<T>(c, b.W, kFmtCSR, 1, false, lv.W, b.wsoff, 0);
        to_layout<T>(c, b.Wt, kFmtCSR, 1, false, lv.Wt, b.tsoff, 0);
      }
      lv.perm = std::move(b.perm);
      continue;
    }
    if (packed) {
      lv.perm = std::move(b.perm);
      continue;
    }
    if (lv.nX_next > 0) {
      // W gathers from three regions of the next level: 32-bit columns;
      // W^T's columns are F indices, one region
      layout_transfer<T>(c, b.W, lv.W, b.wsoff, sell_entries_of(s6[3]), -1);
      tune_restrict<T>(c, lv, b, s6 + 4, lv.Wt, autotune, sizeof(T) == 4);
    }
    tune_layout<T>(c, lv, b, s6, autotune, sizeof(T) == 4);
    lv.perm = std::move(b.perm);
  }
  // workspace
  U.B.resize(nl);
  U.X0.resize(nl);
  U.X1.resize(nl);
  U.R.resize(nl);
  U.n0 = nl ? U.L[0].nX : 0;
  for (int l = 0; l < nl; ++l) {
    auto& lv = U.L[l];
    if (U.bot_from >= 0 && l > U.bot_from) break;  // in LDS
    U.B[l].alloc(c, (size_t)std::max(lv.nX, 1));
    U.X0[l].alloc(c, (size_t)std::max(lv.nX, 1));
    U.X1[l].alloc(c, (size_t)std::max(lv.nX, 1));
    U.R[l].alloc(c, (size_t)std::max(lv.nS, 1));
  }
  U.t1.alloc(c, (size_t)std::max(U.n0, 1));
}

// Layout of a level matrix: the tuned choice cached per (rows, nnz, longest
// row) key as code + (threads per workgroup / 64) * kTuneBsUnit, code 1000 =
// SELL, t = CSR with t lanes per row (a value below kTuneBsUnit keeps 256
// threads); without a cached choice and with autotuning off, SELL when
// padding stays within kSellPad, else CSR with a lane count from the mean row
// length, on 256-thread workgroups.  Autotuning times the residual kernel for
// every layout with 64, 128 and 256 threads per workgroup (rows per workgroup
// = threads / lanes per row; 64-row slices for SELL): the best of three runs
// of back-to-back launches (enough launches for about 0.2 ms per run), and
// keeps the fastest unless the default layout is within kTuneMargin of it, so
// that timing noise does not pick the layout.  A restriction W^T is tuned the
// same way with the restriction kernel (its own cache entries).  Only matrices
// of at least tune_min_rows() rows are timed.
constexpr int kTuneSell = 1000;
constexpr int kTuneBsUnit = 100000;
constexpr double kTuneMargin = 1.03;

// candidate layouts: SELL while its padding stays within 2x, CSR with 1 lane
// and with up to twice the mean row length in lanes, and the default
static std::vector<int> tune_layouts(long long sell_entries, long long nnz, double avg, int dflt) {
  std::vector<int> layouts;
  if (sell_entries <= 2 * nnz) layouts.push_back(kTuneSell);
  for (int t : {1, 2, 4, 8, 16, 32})
    if (t == 1 || t <= 2 * std::max(avg, 1.0)) layouts.push_back(t);
  if (std::find(layouts.begin(), layouts.end(), dflt) == layouts.end()) layouts.push_back(dflt);
  return layouts;
}
// the timed choice among layouts x {64, 128, 256} threads: apply(value) sets a
// layout up, run() launches the kernel once on it; reps launches per run
template <typename Apply, typename Run>
static int tune_pick(Ctx* c, const std::vector<int>& layouts, int dflt, int reps,
                     const Apply& apply, const Run& run) {
  hipEvent_t e0, e1;
  MGD_HIP(hipEventCreate(&e0));
  MGD_HIP(hipEventCreate(&e1));
  const int dflt_value = dflt + 4 * kTuneBsUnit;  // the default layout, 256 threads
  float best = 1e30f, t_dflt = 1e30f;
  int bt = dflt_value;
  const bool prof = c->profiling;
  c->profiling = false;
  for (int code : layouts)
    for (int bs : {64, 128, 256}) {
      const int cand = code + (bs / 64) * kTuneBsUnit;
      apply(cand);
      run();
      float ms = 1e30f;
      for (int trial = 0; trial < 3; ++trial) {
        MGD_HIP(hipEventRecord(e0, c->stream));
        for (int rep = 0; rep < reps; ++rep) run();
        MGD_HIP(hipEventRecord(e1, c->stream));
        MGD_HIP(hipEventSynchronize(e1));
        float t = 0;
        MGD_HIP(hipEventElapsedTime(&t, e0, e1));
        ms = std::min(ms, t);
      }
      c->sync();  // the candidate's predecessors go back to the allocator
      if (cand == dflt_value) t_dflt = ms;
      if (ms < best) {
        best = ms;
        bt = cand;
      }
    }
  if (t_dflt <= best * kTuneMargin) bt = dflt_value;
  c->profiling = prof;
  MGD_HIP(hipEventDestroy(e0));
  MGD_HIP(hipEventDestroy(e1));
  return bt;
}
// launches per timed run: about 0.2 ms of work at 5 TB/s, 4 to 64 launches
static int tune_reps(double bytes) {
  return (int)std::min(64.0, std::max(4.0, 1e9 / std::max(bytes, 1.0)));
}

template <typename T>
static void tune_layout(Ctx* c, ULevel<T>& lv, const BuildLevel<T>& b, const int* stat,
                        int autotune, bool fp32) {
  const Csr<double>& A = b.A;
  if (lv.nS == 0) {
    to_layout<T>(c, A, kFmtCSR, 1, true, lv.A, b.asoff, 0);
    return;
  }
  const int maxrow = stat[0];
  const double avg = (double)A.nnz / lv.nS;
  const long long st = sell_entries_of(stat[1]);
  auto apply = [&](int value) {
    const int code = value % kTuneBsUnit, units = value / kTuneBsUnit;
    if (code == kTuneSell)
      to_layout<T>(c, A, kFmtSELL, 1, true, lv.A, b.asoff, st, sell16_enabled() ? lv.nC : -1);
    else
      to_layout<T>(c, A, kFmtCSR, code, true, lv.A, b.asoff, st);
    lv.A.bs = units ? 64 * units : 256;
  };
  const int cached = autotune_lookup(lv.nS, A.nnz, maxrow, fp32);
  if (cached > 0 && !(st == kSellTooLarge && cached % kTuneBsUnit == kTuneSell)) {
    apply(cached);
    return;
  }
  // enough lanes to occupy the device on small levels (a lane per row serialises
  // long rows), SELL when the level is large and its padding within kSellPad
  const int dflt = (lv.nS >= sell_min_rows() && st <= (long long)(kSellPad * A.nnz))
                       ? kTuneSell
                       : std::max(small_level_tpr(lv.nS, avg), default_tpr(avg));
  if (!autotune || lv.nS < tune_min_rows()) {
    apply(dflt);
    return;
  }
  DBuf<T> x(c, (size_t)std::max(lv.nX, 1)), bb(c, (size_t)lv.nS), r(c, (size_t)lv.nS);
  fill<T>(c, x.get(), (T)1, (size_t)std::max(lv.nX, 1));
  fill<T>(c, bb.get(), (T)1, (size_t)lv.nS);
  const auto g = gather_cf<T>(x.get(), x.get(), lv.nC);
  auto run = [&]() {
    ResidL<T> launch{c, lv.A, lv.nS, bb.get(), g, r.get()};
    with_layout(lv.A.fmt, lv.A.tpr, launch);
  };
  const int reps = tune_reps((double)A.nnz * (sizeof(T) + 4) + 4.0 * sizeof(T) * lv.nS);
  const int bt = tune_pick(c, tune_layouts(st, A.nnz, avg, dflt), dflt, reps, apply, run);
  apply(bt);
  autotune_store(lv.nS, A.nnz, maxrow, fp32, bt);
}

// Layout of the restriction W^T of level l (rows: level l+1 in its extended
// order, columns: level l's F-block), chosen like a level matrix's with the
// restriction kernel timed into scratch vectors of the two levels' sizes
// (cpos, the C-block position of each coarse row, is the level's own).
template <typename T>
static void tune_restrict(Ctx* c, const ULevel<T>& lv, const BuildLevel<T>& b, const int* stat,
                          LMat<T>& out, int autotune, bool fp32) {
  const Csr<double>& Wt = b.Wt;
  const int nS = b.nS, nC = b.nC, nCn = lv.nC_next;
  const int maxrow = stat[0];
  const long long st = sell_entries_of(stat[1]);
  if (Wt.n_rows == 0 || Wt.nnz == 0) {
    layout_transfer<T>(c, Wt, out, b.tsoff, st, 0);
    return;
  }
  auto apply = [&](int value) {
    const int code = value % kTuneBsUnit, units = value / kTuneBsUnit;
    if (code == kTuneSell)
      to_layout<T>(c, Wt, kFmtSELL, 1, false, out, b.tsoff, st, sell16_enabled() ? 0 : -1);
    else
      to_layout<T>(c, Wt, kFmtCSR, code, false, out, b.tsoff, st);
    out.bs = units ? 64 * units : 256;
  };
  const int cached = autotune_lookup(Wt.n_rows, Wt.nnz, maxrow, fp32, "wt:");
  if (cached > 0 && !(st == kSellTooLarge && cached % kTuneBsUnit == kTuneSell)) {
    apply(cached);
    return;
  }
  if (!autotune || Wt.n_rows < tune_min_rows()) {
    layout_transfer<T>(c, Wt, out, b.tsoff, st, 0);
    return;
  }
  const double avg = (double)Wt.nnz / Wt.n_rows;
  const int dflt = transfer_default(Wt, st);
  const int nXn = Wt.n_rows;
  DBuf<T> R(c, (size_t)std::max(nS, 1)), dn(c, (size_t)std::max(nCn, 1));
  DBuf<T> Bn(c, (size_t)nXn), XCn(c, (size_t)std::max(nCn, 1));
  fill<T>(c, R.get(), (T)1, (size_t)std::max(nS, 1));
  fill<T>(c, dn.get(), (T)1, (size_t)std::max(nCn, 1));
  auto run = [&]() {
    RestrictL<T> launch{c, out, nXn, nC, nCn, lv.cpos.get(), R.get(), dn.get(), Bn.get(),
                        XCn.get(), true};
    with_layout(out.fmt, out.tpr, launch);
  };
  const int reps = tune_reps((double)Wt.nnz * (sizeof(T) + 4) + 3.0 * sizeof(T) * nXn);
  const int bt = tune_pick(c, tune_layouts(st, Wt.nnz, avg, dflt), dflt, reps, apply, run);
  apply(bt);
  autotune_store(Wt.n_rows, Wt.nnz, maxrow, fp32, bt, "wt:");
}

template struct Union<double>;
template struct Union<float>;
template std::unique_ptr<Union<double>> build_union<double>(
    Ctx*, const std::vector<const SetupHierarchy*>&, int, int, int, int);
template std::unique_ptr<Union<float>> build_union<float>(
    Ctx*, const std::vector<const SetupHierarchy*>&, int, int, int, int);

}  // namespace mgd
