// AMG setup kernels: strength of connection, PMIS, classical modified
// interpolation, sorted transpose, canonical-order SpGEMM, l1 diagonal and
// the dense coarsest-level inverse.
//
// Every floating-point sum here is evaluated left to right in a fixed order
// with separately rounded products and additions (no contraction into fused
// multiply-adds), so the results are reproducible bit for bit by any other
// implementation that follows the same order.
#pragma clang fp contract(off)

#include <algorithm>
#include <climits>
#include <type_traits>

#include "kernels.hpp"
#include "setup.hpp"

namespace mgd {

// ---------------------------------------------------------------------------
// copies
// ---------------------------------------------------------------------------
void csr_copy_from(Ctx* c, const mgd_csr* A, Csr<double>& out) {
  out.alloc(c, A->n_rows, A->n_cols, (int)A->nnz);
  copy_d2d(c, out.rp.get(), A->row_ptr, (size_t)A->n_rows + 1);
  copy_d2d(c, out.ci.get(), A->col_idx, (size_t)A->nnz);
  copy_d2d(c, out.v.get(), A->val, (size_t)A->nnz);
}

// ---------------------------------------------------------------------------
// strength of connection
// ---------------------------------------------------------------------------
// GL lanes per row read its entries side by side, the row sum adds them in
// order (it decides dominance).  One lane per row, 64 rows apart in every load,
// took 2.3 ms for the five levels of a setup at 3D 64^3, G = 20 (1.3 ms for the
// 1.6M rows of 17 entries at the second); this takes 0.76 ms.
template <int GL>
__global__ void __launch_bounds__(256) k_strength(int n, const int* __restrict__ rp,
                                                  const int* __restrict__ ci,
                                                  const double* __restrict__ v, double theta,
                                                  double dom, uint8_t* __restrict__ S,
                                                  int* __restrict__ stc,
                                                  double* __restrict__ diag,
                                                  const int* __restrict__ err) {
  const int i = blockIdx.x * (256 / GL) + threadIdx.x / GL, lane = threadIdx.x % GL;
  if (i >= n || *err) return;
  const int e0 = rp[i], e1 = rp[i + 1];
  double m = -INFINITY, rs = 0.0, dg = 0.0;
  bool has = false;
  for (int b = e0; b < e1; b += GL) {
    const int e = b + lane;
    double a = 0.0;
    if (e < e1) {
      a = v[e];
      if (ci[e] == i) {
        dg = a;
        has = true;
      } else if (-a > m) {
        m = -a;
      }
    }
    const int cnt = min(GL, e1 - b);
    for (int q = 0; q < cnt; ++q) rs = rs + __shfl(a, q, GL);
  }
#pragma unroll
  for (int o = GL / 2; o > 0; o >>= 1) {
    const double om = __shfl_xor(m, o, GL), od = __shfl_xor(dg, o, GL);
    const int oh = __shfl_xor((int)has, o, GL);
    if (om > m) m = om;
    if (!has && oh) {
      dg = od;
      has = true;
    }
  }
  if (lane == 0) diag[i] = dg;
  bool empty = !(m > 0.0);
  if (dom > 0.0 && rs >= dom * dg) empty = true;
  const double thr = theta * m;
  for (int e = e0 + lane; e < e1; e += GL) {
    const int j = ci[e];
    const bool s = !empty && j != i && (-v[e] >= thr);
    S[e] = s ? 1 : 0;
    if (s) atomicAdd(&stc[j], 1);
  }
}

// S: one flag per entry; stc: how many rows depend on each; diag: a_ii
static void strength(Ctx* c, const Csr<double>& A, double theta, double dom, DBuf<uint8_t>& S,
                     DBuf<int>& stc, DBuf<double>& diag) {
  S.alloc(c, (size_t)A.nnz);
  stc.alloc(c, (size_t)A.n_rows);
  diag.alloc(c, (size_t)A.n_rows);
  fill<int>(c, stc.get(), 0, (size_t)A.n_rows);
  if (A.n_rows == 0) return;
  auto launch = [&](auto kernel, int lanes) {
    hipLaunchKernelGGL(kernel, dim3(cdiv(A.n_rows, 256 / lanes)), dim3(256), 0, c->stream,
                       A.n_rows, A.rp.get(), A.ci.get(), A.v.get(), theta, dom, S.get(), stc.get(),
                       diag.get(), (const int*)c->err_flag());
    MGD_CHECK_LAUNCH();
  };
  switch (fit_lanes(A.n_rows, A.nnz <= 10LL * A.n_rows ? 8 : 16)) {
    case 1: launch(k_strength<1>, 1); break;
    case 8: launch(k_strength<8>, 8); break;
    default: launch(k_strength<16>, 16);
  }
}

// ---------------------------------------------------------------------------
// PMIS
// ---------------------------------------------------------------------------
// First output of SplitMix64 for the given state (Steele, Lea, Flood 2014).
__device__ __forceinline__ uint64_t splitmix64_first(uint64_t z) {
  z += 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// members that coarsen at this level
struct MemberFlags {
  uint8_t on[kMaxMembers] = {};
};

// keys and first states; rows of members that do not coarsen are F
__global__ void k_pmis_init(int n, RowRanges R, MemberFlags M, const int* __restrict__ stc,
                            uint64_t seed, int level, uint64_t* __restrict__ key,
                            int* __restrict__ loser, int8_t* __restrict__ state) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int m = member_of(R, i);
  const uint64_t own = (uint64_t)(i - R.off[m]);
  const uint64_t h = splitmix64_first(seed ^ ((uint64_t)level << 56) ^ own) >> 32;
  key[i] = ((uint64_t)stc[i] << 32) | h;
  loser[i] = 0;
  state[i] = (!M.on[m] || stc[i] == 0) ? kF : kU;
}

__global__ void k_st_fill(int n, const int* __restrict__ rp, const int* __restrict__ ci,
                          const uint8_t* __restrict__ S, int* __restrict__ fillpos,
                          int* __restrict__ st_ci, int cap, int* __restrict__ err) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  for (int e = rp[i]; e < rp[i + 1]; ++e)
    if (S[e]) {
      const int p = atomicAdd(&fillpos[ci[e]], 1);
      if (p >= 0 && p < cap)
        st_ci[p] = i;
      else
        atomicOr(err, 1);
    }
}

__device__ __forceinline__ bool beats(uint64_t kj, int j, uint64_t ki, int i) {
  return kj > ki || (kj == ki && j > i);
}

// A round: an undecided row none of whose undecided neighbours, in either
// direction of the strength graph, beats it becomes C, and rows that depend
// strongly on a new C point become F.  The first kernel walks each edge from the
// row that stores it and marks the loser with the round's number, so no
// transposed graph is formed; the second settles the rows.  Its reads of
// neighbours' states may see them settled or not: a new C point is a row not
// marked this round and not F either way (an undecided row has no older C point
// among its dependencies).
//
// A round walks the list of rows the last one left undecided, kPmisLanes lanes
// per row (a workgroup past the list's end exits), and the second kernel writes
// the next list, in any order.  With a lane per row and every row visited, and
// two counters per undecided row in LDS, the rounds of a setup at 3D 64^3, G = 20
// took 3.7 ms and those of a hierarchy at 2D 1024^2 1.06 ms; now 2.6 and 0.78 ms.
constexpr int kPmisLanes = 8;
__global__ void __launch_bounds__(256) k_pmis_lose(
    const int* __restrict__ list, const int* __restrict__ left, const int* __restrict__ rp,
    const int* __restrict__ ci, const uint8_t* __restrict__ S, const uint64_t* __restrict__ key,
    const int8_t* __restrict__ state, int round, int* __restrict__ loser,
    const int* __restrict__ err) {
  constexpr int kRows = 256 / kPmisLanes, kBatch = 4;
  const int nl = *left, lane = threadIdx.x % kPmisLanes;
  if (*err) return;
  // a group's rows in a pass, whose loads wait for each other together
  const int per = nl > (int)gridDim.x * kRows ? kBatch : 1;
  for (int p0 = blockIdx.x * kRows * per; p0 < nl; p0 += gridDim.x * kRows * per) {
    int i[kBatch], f0[kBatch], f1[kBatch];
    uint64_t ki[kBatch];
    bool lose[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int p = p0 + kRows * u + threadIdx.x / kPmisLanes;
      i[u] = u < per && p < nl ? list[p] : -1;
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      f0[u] = f1[u] = 0;
      ki[u] = 0;
      lose[u] = false;
      if (i[u] < 0) continue;
      f0[u] = rp[i[u]] + lane;
      f1[u] = rp[i[u] + 1];
      ki[u] = key[i[u]];
    }
    for (bool more = true; __any(more);) {
      more = false;
      int j[kBatch];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) j[u] = f0[u] < f1[u] && S[f0[u]] ? ci[f0[u]] : -1;
#pragma unroll
      for (int u = 0; u < kBatch; ++u)
        if (j[u] >= 0 && state[j[u]] != kU) j[u] = -1;
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        if (j[u] >= 0) {
          if (beats(key[j[u]], j[u], ki[u], i[u]))
            lose[u] = true;
          else
            loser[j[u]] = round;
        }
        f0[u] += kPmisLanes;
        more = more || f0[u] < f1[u];
      }
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u)
      if (lose[u]) loser[i[u]] = round;
  }
}

// The undecided rows: list[0 .. cnt[nm]), and a flag per member that has any
// (cnt[m]).  SETTLE: of the rows in `from`, after the second half of a round;
// otherwise of all n.  A workgroup takes 256 * CHUNKS rows at a time and adds to
// the list once for all of them: few workgroups meet in the counter.
template <bool SETTLE, int CHUNKS>
__global__ void __launch_bounds__(256) k_pmis_settle(int n, RowRanges R,
                                                     const int* __restrict__ from,
                                                     const int* __restrict__ left,
                                                     const int* __restrict__ rp,
                                                     const int* __restrict__ ci,
                                                     const uint8_t* __restrict__ S, int round,
                                                     const int* __restrict__ loser, int8_t* state,
                                                     int* __restrict__ list, int* __restrict__ cnt,
                                                     const int* __restrict__ err) {
  __shared__ int s_any[kMaxMembers], s_n, s_base;
  constexpr int kRows = 256 / kPmisLanes;
  const int nl = SETTLE ? *left : n;
  // rows of a workgroup at a time; one per lane group where the list is short
  const bool thin = SETTLE && nl <= (int)gridDim.x * kRows;
  const int per = thin ? kRows : 256 * CHUNKS;
  if (*err || (int)blockIdx.x * per >= nl) return;
  const int grp = threadIdx.x / kPmisLanes, lane = threadIdx.x % kPmisLanes;
  const int sh = (threadIdx.x & 63) / kPmisLanes * kPmisLanes;
  constexpr uint64_t kGroup = (1ull << kPmisLanes) - 1;
  if (threadIdx.x < R.nm) s_any[threadIdx.x] = 0;
  for (int p0 = blockIdx.x * per; p0 < nl; p0 += gridDim.x * per) {
    if (threadIdx.x == 0) s_n = 0;
    __syncthreads();
    int row[CHUNKS], pos[CHUNKS];  // undecided rows, -1: none
#pragma unroll
    for (int t = 0; t < CHUNKS; ++t) {
      row[t] = -1;
      if (!SETTLE) {
        const int i = p0 + 256 * t + threadIdx.x;
        if (i < n && state[i] == kU) row[t] = i;
      } else {
        // kPmisLanes rows of the group together: their loads wait for each other
        // four deep once, not once per row
        int i[kPmisLanes], f0[kPmisLanes], f1[kPmisLanes];  // f1 = -1: a winner
        bool hit[kPmisLanes];
#pragma unroll
        for (int u = 0; u < kPmisLanes; ++u) {
          const int p = p0 + 256 * t + kRows * u + grp;
          i[u] = p < nl && (!thin || t + u == 0) ? from[p] : -1;
        }
#pragma unroll
        for (int u = 0; u < kPmisLanes; ++u) {
          f0[u] = f1[u] = 0;
          if (i[u] < 0) continue;
          f0[u] = rp[i[u]] + lane;
          f1[u] = loser[i[u]] == round ? rp[i[u] + 1] : -1;
        }
#pragma unroll
        for (int u = 0; u < kPmisLanes; ++u) hit[u] = false;
        for (bool more = true; __any(more);) {
          more = false;
          int j[kPmisLanes];
#pragma unroll
          for (int u = 0; u < kPmisLanes; ++u)
            j[u] = f0[u] < f1[u] && S[f0[u]] ? ci[f0[u]] : -1;
#pragma unroll
          for (int u = 0; u < kPmisLanes; ++u) {
            if (j[u] >= 0 && loser[j[u]] != round && state[j[u]] != kF) hit[u] = true;
            f0[u] += kPmisLanes;
            more = more || (f0[u] < f1[u] && !hit[u]);
          }
        }
#pragma unroll
        for (int u = 0; u < kPmisLanes; ++u) {
          const bool f = ((__ballot(hit[u]) >> sh) & kGroup) != 0;
          if (i[u] < 0) continue;
          if (f1[u] < 0 || f) {
            if (lane == 0) state[i[u]] = f ? kF : kC;
          } else if (lane == u) {
            row[t] = i[u];
          }
        }
      }
      const uint64_t w = __ballot(row[t] >= 0);
      int base = 0;
      if ((threadIdx.x & 63) == 0 && w) base = atomicAdd(&s_n, (int)__popcll(w));
      pos[t] = __shfl(base, 0, 64) + (int)__popcll(w & ((1ull << (threadIdx.x & 63)) - 1));
      if (row[t] >= 0) s_any[member_of(R, row[t])] = 1;
    }
    __syncthreads();
    if (threadIdx.x == 0) s_base = s_n ? atomicAdd(&cnt[R.nm], s_n) : 0;
    __syncthreads();
#pragma unroll
    for (int t = 0; t < CHUNKS; ++t)
      if (row[t] >= 0) list[s_base + pos[t]] = row[t];
  }
  __syncthreads();
  if (threadIdx.x < R.nm && s_any[threadIdx.x]) cnt[threadIdx.x] = 1;
}

// rows of members that turn out not to coarsen become F
__global__ void k_mask_f(int n, RowRanges R, MemberFlags M, int8_t* __restrict__ state) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n && !M.on[member_of(R, i)]) state[i] = kF;
}

// out[m] = scan[off[m]] for every member and one past the last, then the error flag
__global__ void k_bounds(RowRanges R, const int* __restrict__ scan, const int* __restrict__ err,
                         int* __restrict__ out) {
  for (int m = threadIdx.x; m <= R.nm; m += blockDim.x) out[m] = scan[R.off[m]];
  if (threadIdx.x == 0) out[R.nm + 1] = *err;
}

__global__ void k_is_c(int n, const int8_t* __restrict__ st, int* __restrict__ out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = st[i] == kC ? 1 : 0;
}

static RowRanges row_ranges(const std::vector<int>& off) {
  RowRanges R;
  R.nm = (int)off.size() - 1;
  MGD_REQUIRE(R.nm >= 1 && R.nm <= kMaxMembers, "internal: too many hierarchies in a batch");
  std::copy(off.begin(), off.end(), R.off);
  return R;
}

// scan values at the members' bounds; throws if a device check has failed
static std::vector<int> read_bounds(Ctx* c, const RowRanges& R, const int* scan, const char* where) {
  DBuf<int> d(c, (size_t)R.nm + 2);
  hipLaunchKernelGGL(k_bounds, dim3(1), dim3(64), 0, c->stream, R, scan, (const int*)c->err_flag(),
                     d.get());
  MGD_CHECK_LAUNCH();
  std::vector<int> h = read_vec(c, d.get(), (size_t)R.nm + 2);
  c->throw_device_errors(h[R.nm + 1], where);
  h.pop_back();
  return h;
}

// ---------------------------------------------------------------------------
// HMIS: Ruge-Stueben first pass inside tiles of consecutive rows (one
// workgroup per tile, state in LDS), then PMIS for the points it leaves open
// ---------------------------------------------------------------------------
constexpr int kMaxHmisTile = 1024;

__device__ __forceinline__ uint64_t block_max_u64(uint64_t v, uint64_t* red) {
  for (int off = 32; off > 0; off >>= 1) {
    const uint64_t o = __shfl_xor(v, off, 64);
    v = o > v ? o : v;
  }
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  uint64_t m = red[0];
  for (int w = 1; w < (int)(blockDim.x >> 6); ++w) m = red[w] > m ? red[w] : m;
  __syncthreads();
  return m;
}

// One workgroup (256 threads) per tile [t0, t1).  The measure of a point is
// the number of undecided tile points depending strongly on it; the point of
// largest (measure, hash, index) with a positive measure becomes C, the
// undecided tile points depending on it become F, the measures of those new F
// points' undecided tile dependencies rise by one, then the measures of the new
// C point's undecided tile dependencies drop by one.  c0[i] = 1 for the C points.
__global__ void __launch_bounds__(256) k_rs_tiles(int n, int tile, uint64_t seed, int level,
                                                  const int* __restrict__ rp,
                                                  const int* __restrict__ ci,
                                                  const uint8_t* __restrict__ S,
                                                  const int* __restrict__ st_rp,
                                                  const int* __restrict__ st_ci,
                                                  int8_t* __restrict__ c0) {
  __shared__ int lam[kMaxHmisTile];
  __shared__ int8_t st[kMaxHmisTile];
  __shared__ uint8_t newf[kMaxHmisTile];
  __shared__ uint32_t hk[kMaxHmisTile];
  __shared__ uint64_t red[4];
  const int t0 = blockIdx.x * tile, t1 = min(n, t0 + tile), nt = t1 - t0;
  for (int i = threadIdx.x; i < nt; i += 256) {
    st[i] = 0;
    newf[i] = 0;
    hk[i] = (uint32_t)(splitmix64_first(seed ^ ((uint64_t)level << 56) ^ (uint64_t)(t0 + i)) >> 32);
    int m = 0;
    for (int e = st_rp[t0 + i]; e < st_rp[t0 + i + 1]; ++e) {
      const int j = st_ci[e];
      m += (j >= t0 && j < t1) ? 1 : 0;
    }
    lam[i] = m;
  }
  __syncthreads();
  for (int step = 0; step < nt; ++step) {
    uint64_t best = 0;
    for (int i = threadIdx.x; i < nt; i += 256) {
      if (st[i] == 0 && lam[i] > 0) {
        const uint64_t k = ((uint64_t)lam[i] << 48) | ((uint64_t)hk[i] << 16) | (uint64_t)i;
        best = k > best ? k : best;
      }
    }
    best = block_max_u64(best, red);
    if (best == 0) break;  // the same value in every thread
    const int pl = (int)(best & 0xffff), pg = t0 + pl;
    if (threadIdx.x == 0) st[pl] = 1;
    __syncthreads();
    // undecided tile points depending on the new C point become F
    for (int e = st_rp[pg] + threadIdx.x; e < st_rp[pg + 1]; e += 256) {
      const int j = st_ci[e] - t0;
      if (j >= 0 && j < nt && st[j] == 0) {
        st[j] = -1;
        newf[j] = 1;
      }
    }
    __syncthreads();
    // their undecided tile dependencies gain one
    for (int e = st_rp[pg] + threadIdx.x; e < st_rp[pg + 1]; e += 256) {
      const int j = st_ci[e] - t0;
      if (j >= 0 && j < nt && newf[j]) {
        newf[j] = 0;
        for (int f = rp[t0 + j]; f < rp[t0 + j + 1]; ++f) {
          const int k = ci[f] - t0;
          if (S[f] && k >= 0 && k < nt && st[k] == 0) atomicAdd(&lam[k], 1);
        }
      }
    }
    __syncthreads();
    // the new C point's undecided tile dependencies lose one
    for (int f = rp[pg] + threadIdx.x; f < rp[pg + 1]; f += 256) {
      const int k = ci[f] - t0;
      if (S[f] && k >= 0 && k < nt && st[k] == 0) atomicAdd(&lam[k], -1);
    }
    __syncthreads();
  }
  for (int i = threadIdx.x; i < nt; i += 256) c0[t0 + i] = st[i] == 1 ? 1 : 0;
}

// HMIS initial state: first-pass C points; F for points nobody depends on or
// that depend strongly on a first-pass C point; undecided otherwise
__global__ void k_hmis_init(int n, const int* __restrict__ rp, const int* __restrict__ ci,
                            const uint8_t* __restrict__ S, const int* __restrict__ stc,
                            const int8_t* __restrict__ c0, int8_t* __restrict__ state) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  if (c0[i]) {
    state[i] = kC;
    return;
  }
  bool dep = stc[i] == 0;
  for (int e = rp[i]; e < rp[i + 1] && !dep; ++e)
    if (S[e] && c0[ci[e]]) dep = true;
  state[i] = dep ? kF : kU;
}

// C/F splitting of the members flagged in M (PMIS, or HMIS with tiles of
// hmis_tile rows), the coarse numbers cidx (n + 1) of its C points, each member's
// first coarse number (returned) and its rounds.  Rounds are enqueued several at
// a time, with the numbering behind them; a round with nothing left to decide
// does nothing, and the counters read back say which rounds a member took.
constexpr int kPmisAhead = 6;
// A row per lane group while kPmisThinGrid workgroups hold the list: rows of 30
// entries eight to a group took 34 us a round however few were left.
constexpr int kPmisGrid = 16384, kPmisThinGrid = 2048, kPmisManyFrom = 1 << 20;
static std::vector<int> pmis(Ctx* c, const Csr<double>& A, const DBuf<uint8_t>& S,
                             const DBuf<int>& stc, const RowRanges& R, const MemberFlags& M,
                             uint64_t seed, int level, int hmis_tile, DBuf<int8_t>& state,
                             DBuf<int>& cidx, std::vector<int>& rounds) {
  const int n = A.n_rows, nm = R.nm, stride = nm + 1;
  rounds.assign(nm, 0);
  state.alloc(c, (size_t)std::max(n, 1));
  cidx.alloc(c, (size_t)n + 1);
  const int g = cdiv(std::max(n, 1), 256);
  const int* err = c->err_flag();
  DBuf<uint64_t> key(c, (size_t)std::max(n, 1));
  DBuf<int> loser(c, (size_t)std::max(n, 1)), isc(c, (size_t)std::max(n, 1));
  // counters per round (row 0: before the first), then the members' bounds and the flag
  const size_t at = (size_t)(kPmisAhead + 1) * stride;
  DBuf<int> cnt(c, at + nm + 2), lists(c, (size_t)2 * std::max(n, 1));
  if (n > 0) {
    hipLaunchKernelGGL(k_pmis_init, dim3(g), dim3(256), 0, c->stream, n, R, M, stc.get(), seed,
                       level, key.get(), loser.get(), state.get());
    MGD_CHECK_LAUNCH();
  }
  if (hmis_tile > 0 && n > 0) {
    DBuf<int> st_rp(c, (size_t)n + 1), fillpos(c, (size_t)n);
    const int nst = exclusive_scan_total(c, stc.get(), st_rp.get(), n);
    DBuf<int> st_ci(c, (size_t)std::max(nst, 1));
    copy_d2d(c, fillpos.get(), st_rp.get(), (size_t)n);
    hipLaunchKernelGGL(k_st_fill, dim3(g), dim3(256), 0, c->stream, n, A.rp.get(), A.ci.get(),
                       S.get(), fillpos.get(), st_ci.get(), nst, c->err_flag());
    MGD_CHECK_LAUNCH();
    c->check_device_errors("transposed strength graph");
    check_index_structure(c, n, n, nst, st_rp.get(), st_ci.get(), "transposed strength graph");
    DBuf<int8_t> c0(c, (size_t)n);
    hipLaunchKernelGGL(k_rs_tiles, dim3(cdiv(n, hmis_tile)), dim3(256), 0, c->stream, n, hmis_tile,
                       seed, level, A.rp.get(), A.ci.get(), S.get(), (const int*)st_rp.get(),
                       (const int*)st_ci.get(), c0.get());
    MGD_CHECK_LAUNCH();
    hipLaunchKernelGGL(k_hmis_init, dim3(g), dim3(256), 0, c->stream, n, A.rp.get(), A.ci.get(),
                       S.get(), stc.get(), (const int8_t*)c0.get(), state.get());
    MGD_CHECK_LAUNCH();
    c->sync();
  }
  // settles round r (or lists the rows there are) and counts into the row of
  // counters behind `before`'s
  auto settle = [&](auto settles, int r, const int* from, int* list, int* before) {
    constexpr bool kSettle = decltype(settles)::value;
    auto launch = [&](auto kernel, int chunks) {
      const int g = std::max(cdiv(n, 256 * chunks),  // short lists with a row per lane group
                             std::min(cdiv(n, 256 / kPmisLanes), kPmisThinGrid));
      hipLaunchKernelGGL(kernel, dim3(std::clamp(g, 1, kPmisGrid)), dim3(256), 0,
                         c->stream, n, R, from, (const int*)before, A.rp.get(), A.ci.get(),
                         S.get(), r, (const int*)loser.get(), state.get(), list,
                         kSettle ? before + 1 : before, err);
      MGD_CHECK_LAUNCH();
    };
    if (n < kPmisManyFrom)
      launch(k_pmis_settle<kSettle, 1>, 1);
    else
      launch(k_pmis_settle<kSettle, 4>, 4);
  };
  for (int base = 0;; base += kPmisAhead) {
    fill<int>(c, cnt.get(), 0, at);
    // row 0 is counted again rather than carried over
    settle(std::false_type{}, 0, nullptr, lists.get(), cnt.get());
    for (int r = 1; r <= kPmisAhead; ++r) {
      const int* from = lists.get() + (size_t)((r - 1) & 1) * n;
      int* before = cnt.get() + (size_t)(r - 1) * stride + nm;
      hipLaunchKernelGGL(k_pmis_lose, dim3(std::clamp(cdiv(n, 256 / kPmisLanes), 1, kPmisGrid)),
                         dim3(256), 0, c->stream, from, (const int*)before, A.rp.get(), A.ci.get(),
                         S.get(), (const uint64_t*)key.get(), (const int8_t*)state.get(), base + r,
                         loser.get(), err);
      MGD_CHECK_LAUNCH();
      settle(std::true_type{}, base + r, from, lists.get() + (size_t)(r & 1) * n, before);
    }
    if (n > 0) {
      hipLaunchKernelGGL(k_is_c, dim3(g), dim3(256), 0, c->stream, n, (const int8_t*)state.get(),
                         isc.get());
      MGD_CHECK_LAUNCH();
    }
    exclusive_scan(c, isc.get(), cidx.get(), n);
    hipLaunchKernelGGL(k_bounds, dim3(1), dim3(64), 0, c->stream, R, (const int*)cidx.get(), err,
                       cnt.get() + at);
    MGD_CHECK_LAUNCH();
    const std::vector<int> h = read_vec(c, cnt.get(), at + nm + 2);
    c->throw_device_errors(h[at + nm + 1], "PMIS");
    for (int m = 0; m < nm; ++m)
      for (int r = 1; r <= kPmisAhead; ++r)
        if (h[(size_t)(r - 1) * stride + m] > 0) rounds[m] = base + r;
    if (h[(size_t)kPmisAhead * stride + nm] == 0)
      return std::vector<int>(h.begin() + at, h.begin() + at + nm + 1);
    // each round decides at least the undecided row of largest (key, index)
    if (base > n) fail(MGD_EHIP, "PMIS did not terminate");
  }
}

// one matrix, every row
static int pmis_one(Ctx* c, const Csr<double>& A, const DBuf<uint8_t>& S, const DBuf<int>& stc,
                    uint64_t seed, int level, DBuf<int8_t>& state, int hmis_tile) {
  MemberFlags M;
  M.on[0] = 1;
  DBuf<int> cidx;
  std::vector<int> rounds;
  pmis(c, A, S, stc, row_ranges({0, A.n_rows}), M, seed, level, hmis_tile, state, cidx, rounds);
  return rounds[0];
}

// ---------------------------------------------------------------------------
// classical modified interpolation
// ---------------------------------------------------------------------------
__device__ __forceinline__ int sgn(double x) { return (x > 0.0) - (x < 0.0); }

// Between LDS accesses of one wave to places other lanes wrote: the hardware
// does them in program order, this keeps the compiler to it.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// position of column j in the sorted row [e0, e1), or -1
__device__ __forceinline__ int find_col(const int* __restrict__ ci, int e0, int e1, int j) {
  int lo = e0, hi = e1;
  while (lo < hi) {
    int mid = (lo + hi) >> 1;
    if (ci[mid] < j)
      lo = mid + 1;
    else
      hi = mid;
  }
  return (lo < e1 && ci[lo] == j) ? lo : -1;
}

__global__ void k_interp_count(int n, const int* __restrict__ rp, const int* __restrict__ ci,
                               const uint8_t* __restrict__ S, const int8_t* __restrict__ st,
                               int* __restrict__ cnt) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  if (st[i] == kC) {
    cnt[i] = 1;
    return;
  }
  int k = 0;
  for (int e = rp[i]; e < rp[i + 1]; ++e)
    if (S[e] && st[ci[e]] == kC) ++k;
  cnt[i] = k;
}

// One F row by one lane: sigma (scratch per matrix entry) first, then the
// modified diagonal, then the weights.  Rows with more strong C neighbours than
// the lane-group kernel keeps in LDS.
__device__ __forceinline__ void interp_row_serial(
    int i, const int* __restrict__ rp, const int* __restrict__ ci, const double* __restrict__ v,
    const double* __restrict__ diag, const uint8_t* __restrict__ S, const int8_t* __restrict__ st,
    const int* __restrict__ cidx, int p, int pend, int* __restrict__ pci, double* __restrict__ pv,
    double* __restrict__ sigma, int* __restrict__ err) {
  const int e0 = rp[i], e1 = rp[i + 1];
  // 1. sigma_ik = sum over j in C_i (ascending j) of ahat_kj, for strong F k
  for (int e = e0; e < e1; ++e) {
    const int k = ci[e];
    if (!S[e] || st[k] != kF) continue;
    const int f0 = rp[k], f1 = rp[k + 1];
    const int skk = sgn(diag[k]);
    double s = 0.0;
    int q = e0;
    for (int f = f0; f < f1; ++f) {
      const int j = ci[f];
      while (q < e1 && ci[q] < j) ++q;
      if (q < e1 && ci[q] == j && S[q] && st[j] == kC) {
        const double a = v[f];
        s = s + (sgn(a) != skk ? a : 0.0);
      }
    }
    sigma[e] = s;
  }
  // 2. modified diagonal: a_ii + weak neighbours + strong F without common C
  double at = diag[i];
  for (int e = e0; e < e1; ++e) {
    const int j = ci[e];
    if (j == i) continue;
    if (!S[e])
      at = at + v[e];
    else if (st[j] == kF && sigma[e] == 0.0)
      at = at + v[e];
  }
  // 3. weights for each strong C point, distribution over ascending k
  for (int e = e0; e < e1; ++e) {
    const int j = ci[e];
    if (!S[e] || st[j] != kC) continue;
    double num = v[e];
    for (int e2 = e0; e2 < e1; ++e2) {
      const int k = ci[e2];
      if (!S[e2] || st[k] != kF) continue;
      const double sg = sigma[e2];
      if (sg == 0.0) continue;
      const int f = find_col(ci, rp[k], rp[k + 1], j);
      if (f < 0) continue;
      const double a = v[f];
      const double ah = sgn(a) != sgn(diag[k]) ? a : 0.0;
      num = num + (v[e2] * ah) / sg;
    }
    if (p >= pend) {  // more entries than the count pass gave this row
      atomicOr(err, 1);
      return;
    }
    pci[p] = cidx[j];
    pv[p] = -num / at;
    ++p;
  }
  if (p != pend) atomicOr(err, 2);
}

// GL lanes per row.  A row is a chain of dependent reads (the row, its strong F
// neighbours' row pointers, their rows, the common C points); with one lane per
// row that chain was about a thread's whole life (k, j and a bisection nested),
// so the lanes share it: they read the row's entries and every neighbour's row
// pointers at once, keep the row's strong C columns in LDS (sorted, as the row
// is), read one neighbour row k at a time side by side and look each column up
// in that list.  The sums stay the serial ones: sigma_ik adds the common C
// points in list order, which is ascending j; a weight's numerator is owned by
// its list position and gets its terms in ascending k; the modified diagonal is
// added in entry order.  The 22 hierarchies of the 3D 64^3, G = 20 system spend
// 3.9 ms here; one lane per row took 106 ms.
template <int GL>
__global__ void __launch_bounds__(256) k_interp_fill(
    int n, const int* __restrict__ rp, const int* __restrict__ ci, const double* __restrict__ v,
    const double* __restrict__ diag, const uint8_t* __restrict__ S, const int8_t* __restrict__ st,
    const int* __restrict__ cidx, const int* __restrict__ prp, int* __restrict__ pci,
    double* __restrict__ pv, double* __restrict__ sigma, int* __restrict__ err) {
  constexpr int kCap = 4 * GL;        // strong C neighbours kept in LDS
  constexpr int kGroups = 256 / GL;
  __shared__ int s_col[kGroups][kCap];
  __shared__ int s_hit[kGroups][kCap];
  __shared__ double s_num[kGroups][kCap];
  __shared__ double s_ah[kGroups][kCap];
  const int grp = threadIdx.x / GL, lane = threadIdx.x % GL;
  const int i = blockIdx.x * kGroups + grp;
  if (i >= n) return;
  // the lanes of a group exchange data through these without a barrier: they are
  // in one wave, with a wave_lds_fence between
  int* col = s_col[grp];
  int* hit = s_hit[grp];
  double* num = s_num[grp];
  double* ahs = s_ah[grp];
  const int p = prp[i], pend = prp[i + 1], m = pend - p;
  if (st[i] == kC) {
    if (lane) return;
    if (m != 1) {  // the count pass gives C rows exactly one entry
      atomicOr(err, 2);
      return;
    }
    pci[p] = cidx[i];
    pv[p] = 1.0;
    return;
  }
  if (m == 0) return;
  if (m > kCap || m < 0) {
    if (lane == 0) {
      if (m < 0)
        atomicOr(err, 2);
      else
        interp_row_serial(i, rp, ci, v, diag, S, st, cidx, p, pend, pci, pv, sigma, err);
    }
    return;
  }
  const int e0 = rp[i], e1 = rp[i + 1];
  const int sh = (threadIdx.x & 63) / GL * GL;
  const uint64_t gm = (GL == 64 ? ~0ull : ((1ull << (GL & 63)) - 1)) << sh;
  // the row's strong C columns and the numerators' first terms
  int nc = 0;
  for (int b = e0; b < e1; b += GL) {
    const int e = b + lane;
    bool c = false;
    int j = 0;
    double a = 0.0;
    if (e < e1) {
      j = ci[e];
      a = v[e];
      c = S[e] && st[j] == kC;
    }
    const uint64_t w = (__ballot(c) & gm) >> sh;
    const int at = nc + __popcll(w & ((1ull << lane) - 1));
    if (c && at < m) {
      col[at] = j;
      num[at] = a;
    }
    nc += __popcll(w);
  }
  if (nc != m) {  // another number of entries than the count pass found
    if (lane == 0) atomicOr(err, 2);
    return;
  }
  wave_lds_fence();
  double at = diag[i];
  for (int b = e0; b < e1; b += GL) {
    const int e = b + lane;
    // kind of the lane's entry: 0 none (diagonal or strong C), 1 weak, 2 strong F
    int j = 0, f0 = 0, f1 = 0, kind = 0, sk = 0;
    double a = 0.0;
    if (e < e1) {
      j = ci[e];
      a = v[e];
      if (j != i) kind = !S[e] ? 1 : (st[j] == kF ? 2 : 0);
      if (kind == 2) {
        f0 = rp[j];
        f1 = rp[j + 1];
        sk = sgn(diag[j]);
      }
    }
    const int cnt = min(GL, e1 - b);
    for (int q = 0; q < cnt; ++q) {
      const int kq = __shfl(kind, q, GL);
      if (kq == 0) continue;
      const double aq = __shfl(a, q, GL);
      if (kq == 1) {
        at = at + aq;
        continue;
      }
      const int k0 = __shfl(f0, q, GL), k1 = __shfl(f1, q, GL), skk = __shfl(sk, q, GL);
      wave_lds_fence();  // every lane has read the hits of the neighbour before
      for (int s = lane; s < m; s += GL) hit[s] = 0;
      wave_lds_fence();
      for (int f = k0 + lane; f < k1; f += GL) {
        const int jj = ci[f];
        const double af = v[f];
        int lo = 0, hi = m;
        while (lo < hi) {
          const int mid = (lo + hi) >> 1;
          if (col[mid] < jj)
            lo = mid + 1;
          else
            hi = mid;
        }
        if (lo < m && col[lo] == jj) {
          ahs[lo] = sgn(af) != skk ? af : 0.0;
          hit[lo] = 1;
        }
      }
      wave_lds_fence();
      double sg = 0.0;
      for (int s = 0; s < m; ++s)
        if (hit[s]) sg = sg + ahs[s];
      if (sg == 0.0) {
        at = at + aq;
        continue;
      }
      for (int s = lane; s < m; s += GL)
        if (hit[s]) num[s] = num[s] + (aq * ahs[s]) / sg;
    }
  }
  for (int s = lane; s < m; s += GL) {
    pci[p + s] = cidx[col[s]];
    pv[p + s] = -num[s] / at;
  }
}

// nc coarse points in all; poff: every member's first entry of P
static void interpolation(Ctx* c, const Csr<double>& A, const DBuf<double>& diag,
                          const DBuf<uint8_t>& S, const DBuf<int8_t>& state, const DBuf<int>& cidx,
                          const RowRanges& R, int nc, Csr<double>& P, std::vector<int>& poff) {
  const int n = A.n_rows;
  DBuf<int> cnt(c, (size_t)n);
  DBuf<double> sigma(c, (size_t)std::max(A.nnz, 1));
  const int g = cdiv(n, 256);
  hipLaunchKernelGGL(k_interp_count, dim3(g), dim3(256), 0, c->stream, n, A.rp.get(), A.ci.get(),
                     S.get(), state.get(), cnt.get());
  MGD_CHECK_LAUNCH();
  P.n_rows = n;
  P.n_cols = nc;
  P.rp.alloc(c, (size_t)n + 1);
  exclusive_scan(c, cnt.get(), P.rp.get(), n);
  poff = read_bounds(c, R, P.rp.get(), "interpolation");
  P.nnz = poff.back();
  P.ci.alloc(c, (size_t)std::max(P.nnz, 1));
  P.v.alloc(c, (size_t)std::max(P.nnz, 1));
  // as many lanes as a row has entries on average, up to half a wave: the
  // lanes read one neighbour's row side by side
#define MGD_INTERP(GL)                                                                           \
  hipLaunchKernelGGL(k_interp_fill<GL>, dim3(cdiv(n, 256 / GL)), dim3(256), 0, c->stream, n,     \
                     A.rp.get(), A.ci.get(), A.v.get(), diag.get(), S.get(), state.get(),        \
                     cidx.get(), P.rp.get(), P.ci.get(), P.v.get(), sigma.get(), c->err_flag())
  const double avg = (double)A.nnz / std::max(n, 1);
  switch (fit_lanes(n, avg <= 10.0 ? 8 : avg <= 24.0 ? 16 : 32)) {
    case 1: MGD_INTERP(1); break;
    case 8: MGD_INTERP(8); break;
    case 16: MGD_INTERP(16); break;
    default: MGD_INTERP(32);
  }
#undef MGD_INTERP
  MGD_CHECK_LAUNCH();
}

// ---------------------------------------------------------------------------
// sorted transpose
// ---------------------------------------------------------------------------
__global__ void k_count_cols(int nnz, const int* __restrict__ ci, int* __restrict__ cnt,
                             const int* __restrict__ err) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e < nnz && !*err) atomicAdd(&cnt[ci[e]], 1);
}
__global__ void k_transpose_fill(int n, const int* __restrict__ rp, const int* __restrict__ ci,
                                 const double* __restrict__ v, int* __restrict__ fillpos,
                                 int* __restrict__ tci, double* __restrict__ tv, int cap,
                                 int* __restrict__ err) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n || *err) return;
  for (int e = rp[i]; e < rp[i + 1]; ++e) {
    const int p = atomicAdd(&fillpos[ci[e]], 1);
    if (p < 0 || p >= cap) {
      atomicOr(err, 1);
      continue;
    }
    tci[p] = i;
    tv[p] = v[e];
  }
}
// rows sorted by column out of place, GL lanes per row: an entry's place is the
// number of smaller columns in its row (columns of a transpose are distinct)
template <int GL>
__global__ void __launch_bounds__(256) k_sort_rows(int n, const int* __restrict__ rp,
                                                   const int* __restrict__ ci,
                                                   const double* __restrict__ v,
                                                   int* __restrict__ oci, double* __restrict__ ov,
                                                   const int* __restrict__ err) {
  const int i = blockIdx.x * (256 / GL) + threadIdx.x / GL, lane = threadIdx.x % GL;
  if (i >= n || *err) return;
  const int e0 = rp[i], m = rp[i + 1] - e0;
  for (int t = lane; t < m; t += GL) {
    const int k = ci[e0 + t];
    int rank = 0;
    for (int u = 0; u < m; ++u) rank += ci[e0 + u] < k ? 1 : 0;
    oci[e0 + rank] = k;
    ov[e0 + rank] = v[e0 + t];
  }
}

// Enqueued without waiting inside a DeferFrees scope (a malformed result then
// shows in the error flag), otherwise complete and checked on return.
void transpose(Ctx* c, const Csr<double>& A, Csr<double>& T) {
  T.n_rows = A.n_cols;
  T.n_cols = A.n_rows;
  T.nnz = A.nnz;
  DBuf<int> cnt(c, (size_t)std::max(A.n_cols, 1)), fillpos(c, (size_t)std::max(A.n_cols, 1));
  DBuf<int> uci(c, (size_t)std::max(A.nnz, 1));  // rows in arrival order
  DBuf<double> uv(c, (size_t)std::max(A.nnz, 1));
  fill<int>(c, cnt.get(), 0, (size_t)A.n_cols);
  if (A.nnz)
    hipLaunchKernelGGL(k_count_cols, dim3(cdiv(A.nnz, 256)), dim3(256), 0, c->stream, A.nnz,
                       A.ci.get(), cnt.get(), (const int*)c->err_flag());
  MGD_CHECK_LAUNCH();
  T.rp.alloc(c, (size_t)A.n_cols + 1);
  exclusive_scan(c, cnt.get(), T.rp.get(), A.n_cols);
  T.ci.alloc(c, (size_t)std::max(A.nnz, 1));
  T.v.alloc(c, (size_t)std::max(A.nnz, 1));
  copy_d2d(c, fillpos.get(), T.rp.get(), (size_t)A.n_cols);
  if (A.n_rows)
    hipLaunchKernelGGL(k_transpose_fill, dim3(cdiv(A.n_rows, 256)), dim3(256), 0, c->stream,
                       A.n_rows, A.rp.get(), A.ci.get(), A.v.get(), fillpos.get(), uci.get(),
                       uv.get(), A.nnz, c->err_flag());
  MGD_CHECK_LAUNCH();
  if (T.n_rows && T.nnz) {
    auto sort = [&](auto kernel, int lanes) {
      hipLaunchKernelGGL(kernel, dim3(cdiv(T.n_rows, 256 / lanes)), dim3(256), 0, c->stream,
                         T.n_rows, T.rp.get(), (const int*)uci.get(), (const double*)uv.get(),
                         T.ci.get(), T.v.get(), (const int*)c->err_flag());
    };
    switch (fit_lanes(T.n_rows, (double)T.nnz <= 16.0 * T.n_rows ? 8 : 64)) {
      case 1: sort(k_sort_rows<1>, 1); break;
      case 64: sort(k_sort_rows<64>, 64); break;
      default: sort(k_sort_rows<8>, 8);
    }
    MGD_CHECK_LAUNCH();
  }
  if (c->defer) {
    check_structure_async(c, T.n_rows, T.n_cols, T.nnz, T.rp.get(), T.ci.get(), false, false);
    return;
  }
  c->check_device_errors("transpose");
  check_structure(c, T, "transpose", false);
}

// ---------------------------------------------------------------------------
// SpGEMM.  Row i of C = A B holds every column some b_k of the row's entries
// reaches, ascending, with the value 0 + a_ik1 b_k1j + a_ik2 b_k2j + ... over
// the row's entries in ascending k.
//
// A row is collected in a hash table in LDS by a group of GL lanes.  The lanes
// take the products of GL entries k of the row side by side (a search among the
// entries' running totals gives each lane its entry), find their slots together,
// and add one entry's products after the other's: the columns of one row of B
// are distinct, so no two lanes meet in a slot, and a slot gets its terms in
// ascending k, the sum above term by term.  With the lanes over one row of B at a
// time, one to four of eight worked at the finest level.
//
// Rows are sorted into classes by the table they need (load at most 3/4): from
// the sum of their B rows' lengths before the columns are counted, from the
// count itself before the values are formed, and from the number of columns that
// exist at all in both.  What bounds a row is instructions and the LDS its table
// takes from other waves, hence the small first table (24 columns hold nearly
// every row of A P and the Galerkin rows of the first levels) and 16-byte
// accesses where a table is cleared, read out and ranked.  The kernels of a class
// walk its list with a grid of at most kSpGrid workgroups and read the list's
// length on the device, so classes without rows cost an empty launch and no
// readback.  Rows too long for the largest table are formed one range of columns
// after another.
//
// At 3D 64^3, G = 20 (22 hierarchies), products of a setup: one lane per row
// merging the B rows' heads through memory 200 ms; tables from 64 slots, lanes
// over one row of B 9.9 ms; tables from 32 slots 8.4; products side by side 6.0;
// 16-byte accesses 5.2.
// ---------------------------------------------------------------------------
constexpr int kSpClasses = 5;             // four table sizes, then ranges of columns
constexpr int kSpGrid = 4096;
// Rows per thread of the sorting kernel: few where the rows' walks over A bound
// it (at 276K rows 8 took 145 us; one up to 2^19, for a workgroup per compute
// unit), many where the workgroups meet in the counters,
// one addition after the other.  For the same reason a workgroup has 1024 threads:
// with 256 sorting the rows of A P took 34.6 and 27.2 us at 2^20 rows (before and
// after the count), with 1024 16.9 and 10.2.
constexpr int kSpBinFew = 2, kSpBinMany = 8, kSpBinWg = 1024;
constexpr int kSpBinFewFrom = 1 << 19, kSpBinManyFrom = 1 << 21;

__host__ __device__ constexpr int sp_class(int cols) {
  return cols <= 24 ? 0 : cols <= 96 ? 1 : cols <= 384 ? 2 : cols <= 3072 ? 3 : 4;
}

// lists[c * n ...] = the rows of class c, count[c] their number.  COUNTED: the
// class from crp's row lengths, else from the B rows' total length; rows
// without entries are in no list (cnt[i] = 0 for them before the count).
template <bool COUNTED, int ROWS>
__global__ void __launch_bounds__(kSpBinWg) k_spgemm_bin(int n, int max_cols,
                                                    const int* __restrict__ arp,
                                                    const int* __restrict__ aci,
                                                    const int* __restrict__ brp,
                                                    const int* __restrict__ crp,
                                                    int* __restrict__ cnt,
                                                    int* __restrict__ lists,
                                                    int* __restrict__ count,
                                                    const int* __restrict__ err) {
  __shared__ int s_n[kSpClasses], s_base[kSpClasses];
  if (*err) return;  // an operand is malformed: empty lists, reported with the sizes
  if (threadIdx.x < kSpClasses) s_n[threadIdx.x] = 0;
  __syncthreads();
  const int r0 = blockIdx.x * kSpBinWg * ROWS;
  int cls[ROWS], pos[ROWS];
#pragma unroll
  for (int t = 0; t < ROWS; ++t) {
    const int i = r0 + t * kSpBinWg + threadIdx.x;
    cls[t] = -1;
    pos[t] = 0;
    if (i < n) {
      long long len = 0;
      if (COUNTED) {
        len = crp[i + 1] - crp[i];
      } else {
        for (int e = arp[i]; e < arp[i + 1]; ++e) {
          const int k = aci[e];
          len += brp[k + 1] - brp[k];
        }
        if (len == 0) cnt[i] = 0;
      }
      if (len > 0) cls[t] = sp_class((int)min(len, (long long)max_cols));
    }
#pragma unroll
    for (int c = 0; c < kSpClasses; ++c) {
      const uint64_t w = __ballot(cls[t] == c);
      if (w == 0) continue;
      int base = 0;
      if ((threadIdx.x & 63) == 0) base = atomicAdd(&s_n[c], (int)__popcll(w));
      base = __shfl(base, 0, 64);
      if (cls[t] == c) pos[t] = base + (int)__popcll(w & ((1ull << (threadIdx.x & 63)) - 1));
    }
  }
  __syncthreads();
  if (threadIdx.x < kSpClasses)
    s_base[threadIdx.x] = s_n[threadIdx.x] ? atomicAdd(&count[threadIdx.x], s_n[threadIdx.x]) : 0;
  __syncthreads();
#pragma unroll
  for (int t = 0; t < ROWS; ++t)
    if (cls[t] >= 0)
      lists[(size_t)cls[t] * n + s_base[cls[t]] + pos[t]] = r0 + t * kSpBinWg + threadIdx.x;
}

template <int H, int GL, int WG, bool FILL>
__global__ void __launch_bounds__(WG) k_spgemm_hash(
    const int* __restrict__ list, const int* __restrict__ count, const int* __restrict__ arp,
    const int* __restrict__ aci, const double* __restrict__ av, const int* __restrict__ brp,
    const int* __restrict__ bci, const double* __restrict__ bv, const int* __restrict__ crp,
    int* __restrict__ cnt_or_cci, double* __restrict__ cv, int* __restrict__ err) {
  constexpr int kGroups = WG / GL, kMost = 3 * H / 4;
  constexpr int kShift = 32 - (H == 32 ? 5 : H == 128 ? 7 : H == 512 ? 9 : 12);
  constexpr int kQuads = H / (4 * GL);  // int4s of a table per lane
  __shared__ int4 s_key4[kGroups][H / 4];
  __shared__ double2 s_val2[FILL ? kGroups : 1][FILL ? H / 2 : 1];
  __shared__ int4 s_col4[FILL ? kGroups : 1][FILL ? kMost / 4 : 1];
  __shared__ uint16_t s_slot[FILL ? kGroups : 1][FILL ? kMost : 1];
  const int grp = threadIdx.x / GL, lane = threadIdx.x % GL;
  const int sh = (threadIdx.x & 63) / GL * GL;
  const uint64_t gm = (GL == 64 ? ~0ull : ((1ull << (GL & 63)) - 1)) << sh;
  // a group's lanes are in one wave: a wave_lds_fence between their accesses, no
  // barrier (volatile: a key may be taken by another lane between two looks)
  int* keys = reinterpret_cast<int*>(s_key4[grp]);
  volatile int* key = keys;
  double* val = reinterpret_cast<double*>(s_val2[FILL ? grp : 0]);
  int* col = reinterpret_cast<int*>(s_col4[FILL ? grp : 0]);
  uint16_t* slot = s_slot[FILL ? grp : 0];
  const int nr = *count;
  for (int r = blockIdx.x * kGroups + grp; r < nr; r += gridDim.x * kGroups) {
    const int i = list[r];
    const int e0 = arp[i], e1 = arp[i + 1];
    wave_lds_fence();  // every lane is done with the row before
#pragma unroll
    for (int s = 0; s < kQuads; ++s) {
      s_key4[grp][s * GL + lane] = make_int4(-1, -1, -1, -1);
      if (FILL) {
        s_val2[grp][2 * s * GL + lane] = make_double2(0.0, 0.0);
        s_val2[grp][(2 * s + 1) * GL + lane] = make_double2(0.0, 0.0);
      }
    }
    wave_lds_fence();
    int fresh = 0;
    bool lost = false;
    for (int b = e0; b < e1; b += GL) {
      // GL entries of the row, then the products of all of them side by side
      const int e = b + lane;
      int f0 = 0, len = 0;
      double a = 0.0;
      if (e < e1) {
        const int k = aci[e];
        f0 = brp[k];
        len = brp[k + 1] - f0;
        if (FILL) a = av[e];
      }
      int upto = len;  // products of the entries up to the lane's
#pragma unroll
      for (int o = 1; o < GL; o <<= 1) {
        const int t = __shfl_up(upto, o, GL);
        if (lane >= o) upto += t;
      }
      const int total = __shfl(upto, GL - 1, GL), from = f0 - (upto - len);
      for (int p0 = 0; p0 < total; p0 += GL) {
        const int p = p0 + lane;
        int q = 0;  // the entry product p belongs to
#pragma unroll
        for (int o = GL / 2; o > 0; o >>= 1)
          if (__shfl(upto, q + o - 1, GL) <= p) q += o;
        const int f = __shfl(from, q, GL) + p;
        const double aq = FILL ? __shfl(a, q, GL) : 0.0;
        int h = -1;
        double x = 0.0;
        if (p < total) {
          const int j = bci[f];
          if (FILL) x = aq * bv[f];
          h = (int)(((unsigned)j * 2654435769u) >> kShift);
          int tries = 0;
          for (; tries < H; ++tries) {  // a table is at most 3/4 full
            int at = key[h];
            if (at == -1) {
              at = atomicCAS(&keys[h], -1, j);
              if (at == -1) {
                ++fresh;
                break;
              }
            }
            if (at == j) break;
            h = (h + 1) & (H - 1);
          }
          if (tries == H) {
            lost = true;
            h = -1;
          }
        }
        if (FILL) {  // one entry's products after the other's
          const int last = __shfl(q, min(GL, total - p0) - 1, GL);
          for (int t = __shfl(q, 0, GL); t <= last; ++t) {
            if (q == t && h >= 0) val[h] = val[h] + x;
            wave_lds_fence();
          }
        }
      }
    }
    if (lost) atomicOr(err, 1);
    if (!FILL) {
#pragma unroll
      for (int o = GL / 2; o > 0; o >>= 1) fresh += __shfl_xor(fresh, o, GL);
      if (lane == 0) cnt_or_cci[i] = fresh;
      continue;
    }
    // the columns present, in slot order, then each at its rank
    wave_lds_fence();
    int m = 0;
#pragma unroll
    for (int s = 0; s < kQuads; ++s) {
      const int4 k4 = s_key4[grp][s * GL + lane];
      const int k[4] = {k4.x, k4.y, k4.z, k4.w};
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const uint64_t w = (__ballot(k[t] >= 0) & gm) >> sh;
        const int at = m + (int)__popcll(w & ((1ull << lane) - 1));
        if (k[t] >= 0 && at < kMost) {
          col[at] = k[t];
          slot[at] = (uint16_t)(4 * (s * GL + lane) + t);
        }
        m += (int)__popcll(w);
      }
    }
    const int o = crp[i];
    if (m != crp[i + 1] - o || m > kMost) {  // another number of columns than were counted
      if (lane == 0) atomicOr(err, 2);
      continue;
    }
    if (lane < (-m & 3)) col[m + lane] = INT_MAX;  // m <= kMost, a multiple of 4
    wave_lds_fence();
    for (int t = lane; t < m; t += GL) {
      const int k = col[t];
      int rank = 0;
      for (int u = 0; u < (m + 3) / 4; ++u) {
        const int4 c4 = s_col4[grp][u];
        rank += (c4.x < k) + (c4.y < k) + (c4.z < k) + (c4.w < k);
      }
      cnt_or_cci[o + rank] = k;
      cv[o + rank] = val[slot[t]];
    }
  }
}

// Rows of the last class, one wave per row: the columns kSpRange at a time, each
// range in an array indexed by column (the row's products are read again for
// every range), so the columns come out in order without a search or a sort.  Only
// ranges between the row's first and last column are walked: in a matrix of
// several members a row reaches its own member's columns (22 members of 67,600 rows
// with 20 rows of 2,500 to 20,000 couplings each are set up in 314 ms; with all
// ranges walked 1870 ms).
constexpr int kSpRange = 4096;
template <bool FILL>
__global__ void __launch_bounds__(64) k_spgemm_range(
    const int* __restrict__ list, const int* __restrict__ count,
    const int* __restrict__ arp, const int* __restrict__ aci, const double* __restrict__ av,
    const int* __restrict__ brp, const int* __restrict__ bci, const double* __restrict__ bv,
    const int* __restrict__ crp, int* __restrict__ cnt_or_cci, double* __restrict__ cv,
    int* __restrict__ err) {
  __shared__ double val[FILL ? kSpRange : 1];
  __shared__ unsigned bits[kSpRange / 32];
  const int lane = threadIdx.x;
  const int nr = *count;
  for (int r = blockIdx.x; r < nr; r += gridDim.x) {
    const int i = list[r];
    const int e0 = arp[i], e1 = arp[i + 1];
    int out = FILL ? crp[i] : 0;
    const int oend = FILL ? crp[i + 1] : INT_MAX;
    int first = INT_MAX, last = -1;  // B's rows are sorted
    for (int e = e0 + lane; e < e1; e += 64) {
      const int k = aci[e], f0 = brp[k], f1 = brp[k + 1];
      if (f0 < f1) {
        first = min(first, bci[f0]);
        last = max(last, bci[f1 - 1]);
      }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      first = min(first, __shfl_xor(first, o, 64));
      last = max(last, __shfl_xor(last, o, 64));
    }
    for (long long lo = first; lo <= last; lo += kSpRange) {
      wave_lds_fence();  // every lane has read the range before
      for (int s = lane; s < kSpRange / 32; s += 64) bits[s] = 0;
      if (FILL)
        for (int s = lane; s < kSpRange; s += 64) val[s] = 0.0;
      wave_lds_fence();
      for (int b = e0; b < e1; b += 64) {
        const int e = b + lane;
        int f0 = 0, f1 = 0;
        double a = 0.0;
        if (e < e1) {
          const int k = aci[e];
          f0 = brp[k];
          f1 = brp[k + 1];
          if (FILL) a = av[e];
        }
        const int cnt = min(64, e1 - b);
        for (int q = 0; q < cnt; ++q) {
          const int k0 = __shfl(f0, q, 64), k1 = __shfl(f1, q, 64);
          const double aq = FILL ? __shfl(a, q, 64) : 0.0;
          for (int f = k0 + lane; f < k1; f += 64) {
            const long long s = (long long)bci[f] - lo;
            if (s < 0 || s >= kSpRange) continue;
            atomicOr(&bits[s >> 5], 1u << (s & 31));
            if (FILL) val[s] = val[s] + aq * bv[f];
          }
          wave_lds_fence();  // the next B row may reach a column through another lane
        }
      }
      for (int s0 = 0; s0 < kSpRange; s0 += 64) {
        const uint64_t w = (uint64_t)bits[s0 >> 5] | ((uint64_t)bits[(s0 >> 5) + 1] << 32);
        const int at = out + (int)__popcll(w & ((1ull << lane) - 1));
        if (FILL && ((w >> lane) & 1) && at < oend) {
          cnt_or_cci[at] = (int)lo + s0 + lane;
          cv[at] = val[s0 + lane];
        }
        out += (int)__popcll(w);
      }
    }
    if (!FILL && lane == 0) cnt_or_cci[i] = out;
    if (FILL && out != oend && lane == 0) atomicOr(err, 2);  // not the columns counted
  }
}

template <bool FILL>
static void spgemm_pass(Ctx* c, const Csr<double>& A, const Csr<double>& B, int max_cols,
                        DBuf<int>& lists, DBuf<int>& count, const int* crp, int* cnt_or_cci, double* cv) {
  const int n = A.n_rows;
  fill<int>(c, count.get(), 0, kSpClasses);
  auto bin = [&](auto kernel, int rows) {
    hipLaunchKernelGGL(kernel, dim3(cdiv(n, kSpBinWg * rows)), dim3(kSpBinWg), 0, c->stream, n, max_cols,
                       A.rp.get(), A.ci.get(), B.rp.get(), crp, FILL ? (int*)nullptr : cnt_or_cci,
                       lists.get(), count.get(), (const int*)c->err_flag());
    MGD_CHECK_LAUNCH();
  };
  if (n < kSpBinFewFrom)
    bin(k_spgemm_bin<FILL, 1>, 1);
  else if (n < kSpBinManyFrom)
    bin(k_spgemm_bin<FILL, kSpBinFew>, kSpBinFew);
  else
    bin(k_spgemm_bin<FILL, kSpBinMany>, kSpBinMany);
  const int top = sp_class(max_cols);  // no row needs more than all columns
#define MGD_SPGEMM(CLS, H, GL, WG)                                                                \
  if (CLS <= top) {                                                                               \
    hipLaunchKernelGGL((k_spgemm_hash<H, GL, WG, FILL>), dim3(std::min(cdiv(n, WG / GL), kSpGrid)), \
                       dim3(WG), 0, c->stream, (const int*)lists.get() + (size_t)CLS * n,         \
                       (const int*)count.get() + CLS, A.rp.get(), A.ci.get(), A.v.get(),          \
                       B.rp.get(), B.ci.get(), B.v.get(), crp, cnt_or_cci, cv, c->err_flag());    \
    MGD_CHECK_LAUNCH();                                                                           \
  }
  MGD_SPGEMM(0, 32, 8, 256)
  MGD_SPGEMM(1, 128, 16, 256)
  MGD_SPGEMM(2, 512, 64, 256)
  MGD_SPGEMM(3, 4096, 64, 64)
#undef MGD_SPGEMM
  if (top == 4) {
    hipLaunchKernelGGL(k_spgemm_range<FILL>, dim3(std::min(n, kSpGrid)), dim3(64), 0, c->stream,
                       (const int*)lists.get() + (size_t)4 * n, (const int*)count.get() + 4,
                       A.rp.get(), A.ci.get(), A.v.get(), B.rp.get(), B.ci.get(),
                       B.v.get(), crp, cnt_or_cci, cv, c->err_flag());
    MGD_CHECK_LAUNCH();
  }
}

void spgemm(Ctx* c, const Csr<double>& A, const Csr<double>& B, int max_cols, Csr<double>& C) {
  MGD_REQUIRE(A.n_cols == B.n_rows, "spgemm: inner dimensions differ");
  const int n = A.n_rows;
  DBuf<int> cnt(c, (size_t)std::max(n, 1)), lists(c, (size_t)kSpClasses * std::max(n, 1));
  DBuf<int> count(c, kSpClasses);
  C.n_rows = n;
  C.n_cols = B.n_cols;
  C.rp.alloc(c, (size_t)n + 1);
  if (n) spgemm_pass<false>(c, A, B, max_cols, lists, count, nullptr, cnt.get(), nullptr);
  exclusive_scan(c, cnt.get(), C.rp.get(), n);
  C.nnz = read_bounds(c, row_ranges({0, n}), C.rp.get(), "SpGEMM count").back();
  MGD_REQUIRE(C.nnz >= 0, "sparse product too large for int32 indices");
  C.ci.alloc(c, (size_t)std::max(C.nnz, 1));
  C.v.alloc(c, (size_t)std::max(C.nnz, 1));
  if (n) spgemm_pass<true>(c, A, B, max_cols, lists, count, C.rp.get(), C.ci.get(), C.v.get());
}

// ---------------------------------------------------------------------------
// aggressive coarsening: a second pass of the same coarsening over the first
// pass's C points, on their strength graph of distance two (j depends on i
// when j is in S_i or in S_k for some k in S_i), numbered by ascending fine
// index; hash keys of level + kAggressiveSalt.  The graph is the pattern of
// X Y minus its diagonal, X = the strong entries of the C rows and
// Y = I + S restricted to C columns.
// ---------------------------------------------------------------------------
constexpr int kAggressiveSalt = 64;

__global__ void k_d2x_count(int n, const int* __restrict__ rp, const uint8_t* __restrict__ S,
                            const int8_t* __restrict__ st, const int* __restrict__ cidx,
                            int* __restrict__ cnt) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n || st[i] != kC) return;
  int k = 0;
  for (int e = rp[i]; e < rp[i + 1]; ++e) k += S[e] ? 1 : 0;
  cnt[cidx[i]] = k;
}
__global__ void k_d2x_fill(int n, const int* __restrict__ rp, const int* __restrict__ ci,
                           const uint8_t* __restrict__ S, const int8_t* __restrict__ st,
                           const int* __restrict__ cidx, const int* __restrict__ xrp,
                           int* __restrict__ xci, double* __restrict__ xv) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n || st[i] != kC) return;
  int p = xrp[cidx[i]];
  for (int e = rp[i]; e < rp[i + 1]; ++e)
    if (S[e]) {
      xci[p] = ci[e];
      xv[p] = 1.0;
      ++p;
    }
}
__global__ void k_d2y_count(int n, const int* __restrict__ rp, const int* __restrict__ ci,
                            const uint8_t* __restrict__ S, const int8_t* __restrict__ st,
                            int* __restrict__ cnt) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int k = st[i] == kC ? 1 : 0;
  for (int e = rp[i]; e < rp[i + 1]; ++e) k += (S[e] && st[ci[e]] == kC) ? 1 : 0;
  cnt[i] = k;
}
// row i of Y: i itself when it is C, and its strong C dependencies, in
// ascending coarse index (strength never flags the diagonal)
__global__ void k_d2y_fill(int n, const int* __restrict__ rp, const int* __restrict__ ci,
                           const uint8_t* __restrict__ S, const int8_t* __restrict__ st,
                           const int* __restrict__ cidx, const int* __restrict__ yrp,
                           int* __restrict__ yci, double* __restrict__ yv) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int p = yrp[i];
  bool self = st[i] == kC;
  for (int e = rp[i]; e < rp[i + 1]; ++e) {
    const int j = ci[e];
    if (self && j > i) {
      yci[p] = cidx[i];
      yv[p] = 1.0;
      ++p;
      self = false;
    }
    if (S[e] && st[j] == kC) {
      yci[p] = cidx[j];
      yv[p] = 1.0;
      ++p;
    }
  }
  if (self) {
    yci[p] = cidx[i];
    yv[p] = 1.0;
  }
}
__global__ void k_offdiag_count(int n, const int* __restrict__ rp, const int* __restrict__ ci,
                                int* __restrict__ cnt) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int k = 0;
  for (int e = rp[i]; e < rp[i + 1]; ++e) k += ci[e] != i ? 1 : 0;
  cnt[i] = k;
}
__global__ void k_offdiag_fill(int n, const int* __restrict__ rp, const int* __restrict__ ci,
                               const int* __restrict__ orp, int* __restrict__ oci,
                               double* __restrict__ ov) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int p = orp[i];
  for (int e = rp[i]; e < rp[i + 1]; ++e)
    if (ci[e] != i) {
      oci[p] = ci[e];
      ov[p] = 1.0;
      ++p;
    }
}
__global__ void k_d2_combine(int n, const int8_t* __restrict__ st1, const int* __restrict__ cidx1,
                             const int8_t* __restrict__ st2, int8_t* __restrict__ st) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  st[i] = (st1[i] == kC && st2[cidx1[i]] == kC) ? kC : kF;
}

// state: first-pass C/F splitting in, final splitting out; returns the rounds
// of the second pass
static int aggressive_split(Ctx* c, const Csr<double>& A, const DBuf<uint8_t>& S,
                            const DBuf<int>& cidx1, int n1, uint64_t seed, int level,
                            int hmis_tile, DBuf<int8_t>& state) {
  const int n = A.n_rows;
  const int g = cdiv(n, 256);
  Csr<double> X, Y, Z, G2;
  {
    DBuf<int> cnt(c, (size_t)std::max(n1, 1));
    hipLaunchKernelGGL(k_d2x_count, dim3(g), dim3(256), 0, c->stream, n, A.rp.get(), S.get(),
                       state.get(), cidx1.get(), cnt.get());
    MGD_CHECK_LAUNCH();
    X.n_rows = n1;
    X.n_cols = n;
    X.rp.alloc(c, (size_t)n1 + 1);
    X.nnz = exclusive_scan_total(c, cnt.get(), X.rp.get(), n1);
    X.ci.alloc(c, (size_t)std::max(X.nnz, 1));
    X.v.alloc(c, (size_t)std::max(X.nnz, 1));
    hipLaunchKernelGGL(k_d2x_fill, dim3(g), dim3(256), 0, c->stream, n, A.rp.get(), A.ci.get(),
                       S.get(), state.get(), cidx1.get(), (const int*)X.rp.get(), X.ci.get(),
                       X.v.get());
    MGD_CHECK_LAUNCH();
  }
  {
    DBuf<int> cnt(c, (size_t)n);
    hipLaunchKernelGGL(k_d2y_count, dim3(g), dim3(256), 0, c->stream, n, A.rp.get(), A.ci.get(),
                       S.get(), state.get(), cnt.get());
    MGD_CHECK_LAUNCH();
    Y.n_rows = n;
    Y.n_cols = n1;
    Y.rp.alloc(c, (size_t)n + 1);
    Y.nnz = exclusive_scan_total(c, cnt.get(), Y.rp.get(), n);
    Y.ci.alloc(c, (size_t)std::max(Y.nnz, 1));
    Y.v.alloc(c, (size_t)std::max(Y.nnz, 1));
    hipLaunchKernelGGL(k_d2y_fill, dim3(g), dim3(256), 0, c->stream, n, A.rp.get(), A.ci.get(),
                       S.get(), state.get(), cidx1.get(), (const int*)Y.rp.get(), Y.ci.get(),
                       Y.v.get());
    MGD_CHECK_LAUNCH();
  }
  check_structure(c, X, "distance-two graph: X", false);
  check_structure(c, Y, "distance-two graph: Y", false);
  spgemm(c, X, Y, n1, Z);
  check_structure(c, Z, "distance-two graph", false);
  {
    const int g1 = cdiv(n1, 256);
    DBuf<int> cnt(c, (size_t)std::max(n1, 1));
    hipLaunchKernelGGL(k_offdiag_count, dim3(g1), dim3(256), 0, c->stream, n1, Z.rp.get(),
                       Z.ci.get(), cnt.get());
    MGD_CHECK_LAUNCH();
    G2.n_rows = G2.n_cols = n1;
    G2.rp.alloc(c, (size_t)n1 + 1);
    G2.nnz = exclusive_scan_total(c, cnt.get(), G2.rp.get(), n1);
    G2.ci.alloc(c, (size_t)std::max(G2.nnz, 1));
    G2.v.alloc(c, (size_t)std::max(G2.nnz, 1));
    hipLaunchKernelGGL(k_offdiag_fill, dim3(g1), dim3(256), 0, c->stream, n1, Z.rp.get(),
                       Z.ci.get(), (const int*)G2.rp.get(), G2.ci.get(), G2.v.get());
    MGD_CHECK_LAUNCH();
  }
  DBuf<uint8_t> S2(c, (size_t)std::max(G2.nnz, 1));
  fill<uint8_t>(c, S2.get(), (uint8_t)1, (size_t)G2.nnz);
  DBuf<int> stc2(c, (size_t)std::max(n1, 1));
  fill<int>(c, stc2.get(), 0, (size_t)n1);
  if (G2.nnz)
    hipLaunchKernelGGL(k_count_cols, dim3(cdiv(G2.nnz, 256)), dim3(256), 0, c->stream, G2.nnz,
                       G2.ci.get(), stc2.get(), (const int*)c->err_flag());
  MGD_CHECK_LAUNCH();
  DBuf<int8_t> st2;
  const int rounds = pmis_one(c, G2, S2, stc2, seed, level + kAggressiveSalt, st2, hmis_tile);
  DBuf<int8_t> out(c, (size_t)n);
  hipLaunchKernelGGL(k_d2_combine, dim3(g), dim3(256), 0, c->stream, n, state.get(), cidx1.get(),
                     (const int8_t*)st2.get(), out.get());
  MGD_CHECK_LAUNCH();
  c->sync();
  state = std::move(out);
  return rounds;
}

// ---------------------------------------------------------------------------
// multipass interpolation (Stueben 2001): C rows are the identity; a point of
// pass m (its nearest C point is m strong dependencies away) interpolates
// through its strong dependencies P_i of pass m - 1:
//   alpha = (sum of negative off-diagonal a_ij) / (sum_{j in P_i} a_ij),
//   d = a_ii + (sum of the other off-diagonal a_ij),
//   w_ik = -(alpha * (0 + sum_{j in P_i, ascending} a_ij w_jk)) / d.
// Rows are built pass by pass into a buffer per pass; off[i], len[i] locate
// row i in its pass's buffer.  Points no chain reaches get empty rows.
// ---------------------------------------------------------------------------
__global__ void k_mp_init(int n, const int8_t* __restrict__ st, const int* __restrict__ cidx,
                          int* __restrict__ pass, int* __restrict__ off, int* __restrict__ len) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const bool isc = st[i] == kC;
  pass[i] = isc ? 0 : -1;
  off[i] = isc ? cidx[i] : 0;
  len[i] = isc ? 1 : 0;
}
__global__ void k_iota(int n, int* __restrict__ out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = i;
}
// pass m for every unreached point with a strong dependency of pass m - 1
// (a point set in this launch reads as m or -1, never as m - 1)
__global__ void k_mp_assign(int n, int m, const int* __restrict__ rp, const int* __restrict__ ci,
                            const uint8_t* __restrict__ S, int* __restrict__ pass,
                            int* __restrict__ added) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  bool hit = false;
  if (i < n && pass[i] < 0)
    for (int e = rp[i]; e < rp[i + 1]; ++e)
      if (S[e] && pass[ci[e]] == m - 1) {
        hit = true;
        break;
      }
  if (hit) pass[i] = m;
  const uint64_t b = __ballot(hit);
  if ((threadIdx.x & 63) == 0 && b) atomicAdd(added, (int)__popcll(b));
}
template <bool FILL>
__global__ void k_mp_rows(int n, int m, const int* __restrict__ rp, const int* __restrict__ ci,
                          const double* __restrict__ v, const uint8_t* __restrict__ S,
                          const int* __restrict__ pass, const int* __restrict__ bci,
                          const double* __restrict__ bv, int* __restrict__ off,
                          int* __restrict__ len, int* __restrict__ head, int* __restrict__ hend,
                          const int* __restrict__ orp, int* __restrict__ cnt_or_oci,
                          double* __restrict__ ov, int* __restrict__ err) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  if (pass[i] != m) {
    if (!FILL) cnt_or_oci[i] = 0;
    return;
  }
  const int e0 = rp[i], e1 = rp[i + 1];
  double dg = 0.0, sn = 0.0, sp = 0.0, sP = 0.0;
  for (int e = e0; e < e1; ++e) {
    const int j = ci[e];
    const double a = v[e];
    if (j == i)
      dg = a;
    else if (a < 0.0)
      sn = sn + a;
    else
      sp = sp + a;
    if (S[e] && pass[j] == m - 1) {
      sP = sP + a;
      head[e] = off[j];
      hend[e] = off[j] + len[j];
    } else {
      head[e] = 0;
      hend[e] = 0;
    }
  }
  const double alpha = sn / sP, d = dg + sp;
  int out = FILL ? orp[i] : 0;
  const int oend = FILL ? orp[i + 1] : INT_MAX;
  for (;;) {
    int kmin = INT_MAX;
    for (int e = e0; e < e1; ++e)
      if (head[e] < hend[e]) kmin = min(kmin, bci[head[e]]);
    if (kmin == INT_MAX) break;
    double acc = 0.0;
    for (int e = e0; e < e1; ++e) {
      const int h = head[e];
      if (h < hend[e] && bci[h] == kmin) {
        if (FILL) acc = acc + v[e] * bv[h];
        head[e] = h + 1;
      }
    }
    if (FILL) {
      if (out >= oend) {  // more columns than the count pass gave this row
        atomicOr(err, 1);
        return;
      }
      cnt_or_oci[out] = kmin;
      ov[out] = -(alpha * acc) / d;
    }
    ++out;
  }
  if (!FILL) {
    cnt_or_oci[i] = out;
  } else {
    if (out != oend) atomicOr(err, 2);
    off[i] = orp[i];
    len[i] = out - orp[i];
  }
}
__global__ void k_mp_copy(int n, int m, const int* __restrict__ pass, const int* __restrict__ off,
                          const int* __restrict__ len, const int* __restrict__ bci,
                          const double* __restrict__ bv, const int* __restrict__ prp,
                          int* __restrict__ pci, double* __restrict__ pv) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n || pass[i] != m) return;
  const int o = off[i], p = prp[i];
  for (int q = 0; q < len[i]; ++q) {
    pci[p + q] = bci[o + q];
    pv[p + q] = bv[o + q];
  }
}

static void multipass_interpolation(Ctx* c, const Csr<double>& A, const DBuf<uint8_t>& S,
                                    const DBuf<int8_t>& state, const DBuf<int>& cidx, int nc,
                                    Csr<double>& P) {
  const int n = A.n_rows;
  const int g = cdiv(n, 256);
  DBuf<int> pass(c, (size_t)n), off(c, (size_t)n), len(c, (size_t)n), added(c, 1);
  hipLaunchKernelGGL(k_mp_init, dim3(g), dim3(256), 0, c->stream, n, state.get(), cidx.get(),
                     pass.get(), off.get(), len.get());
  MGD_CHECK_LAUNCH();
  std::vector<DBuf<int>> bci;
  std::vector<DBuf<double>> bv;
  bci.emplace_back(c, (size_t)std::max(nc, 1));
  bv.emplace_back(c, (size_t)std::max(nc, 1));
  hipLaunchKernelGGL(k_iota, dim3(cdiv(std::max(nc, 1), 256)), dim3(256), 0, c->stream, nc,
                     bci[0].get());
  MGD_CHECK_LAUNCH();
  fill<double>(c, bv[0].get(), 1.0, (size_t)nc);
  DBuf<int> head(c, (size_t)std::max(A.nnz, 1)), hend(c, (size_t)std::max(A.nnz, 1));
  DBuf<int> cnt(c, (size_t)n), orp(c, (size_t)n + 1);
  for (int m = 1;; ++m) {
    if (m > n) fail(MGD_EHIP, "multipass interpolation did not terminate");
    fill<int>(c, added.get(), 0, 1);
    hipLaunchKernelGGL(k_mp_assign, dim3(g), dim3(256), 0, c->stream, n, m, A.rp.get(),
                       A.ci.get(), S.get(), pass.get(), added.get());
    MGD_CHECK_LAUNCH();
    if (read1(c, added.get()) == 0) break;
    hipLaunchKernelGGL(k_mp_rows<false>, dim3(g), dim3(256), 0, c->stream, n, m, A.rp.get(),
                       A.ci.get(), A.v.get(), S.get(), (const int*)pass.get(),
                       (const int*)bci[m - 1].get(), (const double*)bv[m - 1].get(), off.get(),
                       len.get(), head.get(), hend.get(), (const int*)nullptr, cnt.get(),
                       (double*)nullptr, c->err_flag());
    MGD_CHECK_LAUNCH();
    const int tot = exclusive_scan_total(c, cnt.get(), orp.get(), n);
    bci.emplace_back(c, (size_t)std::max(tot, 1));
    bv.emplace_back(c, (size_t)std::max(tot, 1));
    hipLaunchKernelGGL(k_mp_rows<true>, dim3(g), dim3(256), 0, c->stream, n, m, A.rp.get(),
                       A.ci.get(), A.v.get(), S.get(), (const int*)pass.get(),
                       (const int*)bci[m - 1].get(), (const double*)bv[m - 1].get(), off.get(),
                       len.get(), head.get(), hend.get(), (const int*)orp.get(), bci[m].get(),
                       bv[m].get(), c->err_flag());
    MGD_CHECK_LAUNCH();
    c->check_device_errors("multipass interpolation");
  }
  P.n_rows = n;
  P.n_cols = nc;
  P.rp.alloc(c, (size_t)n + 1);
  P.nnz = exclusive_scan_total(c, len.get(), P.rp.get(), n);
  P.ci.alloc(c, (size_t)std::max(P.nnz, 1));
  P.v.alloc(c, (size_t)std::max(P.nnz, 1));
  for (int m = 0; m < (int)bci.size(); ++m)
    hipLaunchKernelGGL(k_mp_copy, dim3(g), dim3(256), 0, c->stream, n, m, (const int*)pass.get(),
                       (const int*)off.get(), (const int*)len.get(), (const int*)bci[m].get(),
                       (const double*)bv[m].get(), (const int*)P.rp.get(), P.ci.get(), P.v.get());
  MGD_CHECK_LAUNCH();
  c->sync();
}

// ---------------------------------------------------------------------------
// Jones-Plassmann colouring (multicolour Gauss-Seidel): every stored
// off-diagonal entry of A is an edge in both directions; in round c every
// uncoloured row whose (hash32(seed, level, i), i) beats all uncoloured
// neighbours gets colour c
// ---------------------------------------------------------------------------
__global__ void k_jp_select(int n, int round, uint64_t seed, int level,
                            const int* __restrict__ rp, const int* __restrict__ ci,
                            const int* __restrict__ trp, const int* __restrict__ tci,
                            const int* __restrict__ colour, uint8_t* __restrict__ win) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  if (colour[i] >= 0) {
    win[i] = 0;
    return;
  }
  const uint64_t salt = seed ^ ((uint64_t)level << 56);
  const uint32_t ki = (uint32_t)(splitmix64_first(salt ^ (uint64_t)i) >> 32);
  bool best = true;
  for (int e = rp[i]; e < rp[i + 1] && best; ++e) {
    const int j = ci[e];
    if (j == i || colour[j] >= 0) continue;
    const uint32_t kj = (uint32_t)(splitmix64_first(salt ^ (uint64_t)j) >> 32);
    if (kj > ki || (kj == ki && j > i)) best = false;
  }
  for (int e = trp[i]; e < trp[i + 1] && best; ++e) {
    const int j = tci[e];
    if (j == i || colour[j] >= 0) continue;
    const uint32_t kj = (uint32_t)(splitmix64_first(salt ^ (uint64_t)j) >> 32);
    if (kj > ki || (kj == ki && j > i)) best = false;
  }
  win[i] = best ? 1 : 0;
}
__global__ void k_jp_assign(int n, int round, const uint8_t* __restrict__ win,
                            int* __restrict__ colour, int* __restrict__ remaining) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  bool left = false;
  if (i < n) {
    if (win[i]) colour[i] = round;
    left = colour[i] < 0;
  }
  const uint64_t m = __ballot(left);
  if ((threadIdx.x & 63) == 0 && m) atomicAdd(remaining, (int)__popcll(m));
}

int jp_colouring(Ctx* c, const Csr<double>& A, uint64_t seed, int level, DBuf<int>& colour) {
  const int n = A.n_rows;
  colour.alloc(c, (size_t)std::max(n, 1));
  if (n == 0) return 0;
  fill<int>(c, colour.get(), -1, (size_t)n);
  Csr<double> T;
  transpose(c, A, T);
  DBuf<uint8_t> win(c, (size_t)n);
  DBuf<int> remaining(c, 1);
  const int g = cdiv(n, 256);
  int round = 0;
  for (;;) {
    fill<int>(c, remaining.get(), 0, 1);
    hipLaunchKernelGGL(k_jp_select, dim3(g), dim3(256), 0, c->stream, n, round, seed, level,
                       A.rp.get(), A.ci.get(), (const int*)T.rp.get(), (const int*)T.ci.get(),
                       (const int*)colour.get(), win.get());
    MGD_CHECK_LAUNCH();
    hipLaunchKernelGGL(k_jp_assign, dim3(g), dim3(256), 0, c->stream, n, round,
                       (const uint8_t*)win.get(), colour.get(), remaining.get());
    MGD_CHECK_LAUNCH();
    ++round;
    if (read1(c, remaining.get()) == 0) break;
    // every round colours at least the uncoloured row of largest (key, index)
    if (round > n) fail(MGD_EHIP, "colouring did not terminate");
  }
  return round;
}

// ---------------------------------------------------------------------------
// dense inverses of the members' coarsest matrices (FP64): LU with partial
// pivoting (first row of maximum magnitude), then one triangular solve pair per
// column of the identity.  One workgroup per member; n <= dense_max.
// ---------------------------------------------------------------------------
struct DenseJob {
  const int* rp;  // the member's rows, columns ci - cbase
  const int* ci;
  const double* v;
  int n, cbase;
  double* M;      // n x n work, row-major (members larger than kLdsDense only)
  int* piv;
  double* inv;    // n x n, column-major
};

// Up to kLdsDense rows (the default coarsest size): matrix and inverse in LDS.
// Every entry goes through the operations of the factorisation below in the
// same order: the forward solves apply row k to all later rows at once
// (ascending k for each), the backward solves, whose sums start at the row just
// finished, run one column per thread.
constexpr int kLdsDense = 100;
__global__ void __launch_bounds__(1024) k_dense_inverse(const DenseJob* __restrict__ jobs,
                                                        int* __restrict__ singular) {
  __shared__ double M[kLdsDense * kLdsDense], X[kLdsDense * kLdsDense];
  __shared__ int piv[kLdsDense];
  const DenseJob J = jobs[blockIdx.x];
  const int n = J.n, t = threadIdx.x, lane = t & 63;
  if (n > kLdsDense) return;
  for (int q = t; q < n * n; q += 1024) {
    M[q] = 0.0;
    X[q] = 0.0;
  }
  __syncthreads();
  for (int i = t; i < n; i += 1024)
    for (int e = J.rp[i]; e < J.rp[i + 1]; ++e) {
      const int j = J.ci[e] - J.cbase;
      if (j >= 0 && j < n) M[i * n + j] = J.v[e];
    }
  __syncthreads();
  for (int col = 0; col < n; ++col) {
    // pivot: largest |M[r][col]|, smallest r on ties; every wave finds it
    double best = -1.0;
    int bi = INT_MAX;
    for (int r = col + lane; r < n; r += 64) {
      const double a = fabs(M[r * n + col]);
      if (a > best) {
        best = a;
        bi = r;
      }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const double ov = __shfl_xor(best, o, 64);
      const int oi = __shfl_xor(bi, o, 64);
      if (ov > best || (ov == best && oi < bi)) {
        best = ov;
        bi = oi;
      }
    }
    if (!(best > 0.0)) {  // the same in every thread
      if (t == 0) singular[0] = 1;
      return;
    }
    __syncthreads();
    if (t == 0) piv[col] = bi;
    if (bi != col)
      for (int j = t; j < n; j += 1024) {
        const double tmp = M[col * n + j];
        M[col * n + j] = M[bi * n + j];
        M[bi * n + j] = tmp;
      }
    __syncthreads();
    const double d = M[col * n + col];
    for (int r = col + 1 + t; r < n; r += 1024) M[r * n + col] = M[r * n + col] / d;
    __syncthreads();
    const int m = n - col - 1;
    for (int q = t; q < m * m; q += 1024) {
      const int r = col + 1 + q / m, j = col + 1 + q % m;
      M[r * n + j] = M[r * n + j] - M[r * n + col] * M[col * n + j];
    }
    __syncthreads();
  }
  if (t < n) {  // column t of the permuted identity
    int at = t;
    for (int i = 0; i < n; ++i) {
      const int p = piv[i];
      at = at == i ? p : (at == p ? i : at);
    }
    X[at * n + t] = 1.0;
  }
  __syncthreads();
  for (int k = 0; k + 1 < n; ++k) {  // unit lower
    const int m = n - k - 1;
    for (int q = t; q < m * n; q += 1024) {
      const int i = k + 1 + q / n, j = q % n;
      X[i * n + j] = X[i * n + j] - M[i * n + k] * X[k * n + j];
    }
    __syncthreads();
  }
  if (t < n) {  // upper
    for (int i = n - 1; i >= 0; --i) {
      double s = X[i * n + t];
      for (int k = i + 1; k < n; ++k) s = s - M[i * n + k] * X[k * n + t];
      X[i * n + t] = s / M[i * n + i];
    }
  }
  __syncthreads();
  for (int q = t; q < n * n; q += 1024) J.inv[(size_t)(q % n) * n + q / n] = X[q];
}

// Larger coarsest matrices (coarsening stalled above the default size): in memory.
__global__ void k_csr_to_dense(const DenseJob* __restrict__ jobs) {
  const DenseJob J = jobs[blockIdx.y];
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (J.n <= kLdsDense || i >= J.n) return;
  for (int e = J.rp[i]; e < J.rp[i + 1]; ++e) {
    const int j = J.ci[e] - J.cbase;
    if (j >= 0 && j < J.n) J.M[(size_t)i * J.n + j] = J.v[e];
  }
}

__global__ void __launch_bounds__(1024) k_lu(const DenseJob* __restrict__ jobs,
                                             int* __restrict__ singular) {
  __shared__ double sval[1024];
  __shared__ int sidx[1024];
  const DenseJob J = jobs[blockIdx.x];
  const int n = J.n;
  if (n <= kLdsDense) return;
  double* __restrict__ M = J.M;
  const int t = threadIdx.x;
  for (int col = 0; col < n; ++col) {
    // pivot search: max |M[r][col]|, smallest r on ties
    double best = -1.0;
    int bi = INT_MAX;
    for (int r = col + t; r < n; r += 1024) {
      const double a = fabs(M[(size_t)r * n + col]);
      if (a > best) {
        best = a;
        bi = r;
      }
    }
    sval[t] = best;
    sidx[t] = bi;
    __syncthreads();
    for (int s = 512; s > 0; s >>= 1) {
      if (t < s) {
        const double ov = sval[t + s];
        const int oi = sidx[t + s];
        if (ov > sval[t] || (ov == sval[t] && oi < sidx[t])) {
          sval[t] = ov;
          sidx[t] = oi;
        }
      }
      __syncthreads();
    }
    const int p = sidx[0];
    const double pv = sval[0];
    __syncthreads();
    if (!(pv > 0.0)) {
      if (t == 0) singular[0] = 1;
      return;
    }
    if (t == 0) J.piv[col] = p;
    if (p != col)
      for (int j = t; j < n; j += 1024) {
        const double tmp = M[(size_t)col * n + j];
        M[(size_t)col * n + j] = M[(size_t)p * n + j];
        M[(size_t)p * n + j] = tmp;
      }
    __syncthreads();
    const double d = M[(size_t)col * n + col];
    for (int r = col + 1 + t; r < n; r += 1024) M[(size_t)r * n + col] = M[(size_t)r * n + col] / d;
    __syncthreads();
    const int m = n - col - 1;
    for (long q = t; q < (long)m * m; q += 1024) {
      const int r = col + 1 + (int)(q / m);
      const int j = col + 1 + (int)(q % m);
      M[(size_t)r * n + j] = M[(size_t)r * n + j] - M[(size_t)r * n + col] * M[(size_t)col * n + j];
    }
    __syncthreads();
  }
}

// inverse column j: solve L U x = P e_j; written column-major inv[j*n + i]
__global__ void k_lu_inverse(const DenseJob* __restrict__ jobs, const int* __restrict__ singular) {
  const DenseJob J = jobs[blockIdx.y];
  const int n = J.n, j = blockIdx.x * blockDim.x + threadIdx.x;
  if (n <= kLdsDense || j >= n || *singular) return;
  const double* __restrict__ M = J.M;
  double* x = J.inv + (size_t)j * n;
  for (int i = 0; i < n; ++i) x[i] = (i == j) ? 1.0 : 0.0;
  for (int i = 0; i < n; ++i) {  // apply the row interchanges in order
    const int p = J.piv[i];
    if (p != i) {
      const double t = x[i];
      x[i] = x[p];
      x[p] = t;
    }
  }
  for (int i = 0; i < n; ++i) {  // unit lower
    double s = x[i];
    for (int k = 0; k < i; ++k) s = s - M[(size_t)i * n + k] * x[k];
    x[i] = s;
  }
  for (int i = n - 1; i >= 0; --i) {  // upper
    double s = x[i];
    for (int k = i + 1; k < n; ++k) s = s - M[(size_t)i * n + k] * x[k];
    x[i] = s / M[(size_t)i * n + i];
  }
}

// coarse_kind and inverses of every member
static void coarsest_inverses(Ctx* c, const amg_params& p, SetupBatch& H) {
  const int nm = (int)H.n_levels.size();
  H.coarse_kind.assign(nm, 0);
  H.inv_at.assign(nm, 0);
  size_t total = 0, work = 0, pivs = 0;
  int top = 0;
  std::vector<DenseJob> jobs;
  std::vector<size_t> m_at, p_at;
  std::vector<int> who;
  for (int m = 0; m < nm; ++m) {
    const SetupLevel& L = H.levels[H.n_levels[m] - 1];
    const int n = L.off[m + 1] - L.off[m];
    if (n > p.dense_max) {
      H.coarse_kind[m] = 1;
      continue;
    }
    H.inv_at[m] = total;
    total += (size_t)n * n;
    if (n == 0) continue;
    jobs.push_back({L.A.rp.get() + L.off[m], L.A.ci.get(), L.A.v.get(), n, L.off[m], nullptr,
                    nullptr, nullptr});
    m_at.push_back(work);
    p_at.push_back(pivs);
    who.push_back(m);
    if (n > kLdsDense) {
      work += (size_t)n * n;
      pivs += n;
      top = std::max(top, n);
    }
  }
  if (jobs.empty()) return;
  H.inv.alloc(c, std::max<size_t>(total, 1));
  DBuf<double> M(c, std::max<size_t>(work, 1));
  DBuf<int> piv(c, std::max<size_t>(pivs, 1)), sing(c, 1);
  for (size_t q = 0; q < jobs.size(); ++q) {
    jobs[q].M = M.get() + m_at[q];
    jobs[q].piv = piv.get() + p_at[q];
    jobs[q].inv = H.inv.get() + H.inv_at[who[q]];
  }
  DBuf<DenseJob> dj(c, jobs.size());
  copy_h2d(c, dj.get(), jobs.data(), jobs.size());
  fill<int>(c, sing.get(), 0, 1);
  const unsigned nj = (unsigned)jobs.size();
  hipLaunchKernelGGL(k_dense_inverse, dim3(nj), dim3(1024), 0, c->stream,
                     (const DenseJob*)dj.get(), sing.get());
  MGD_CHECK_LAUNCH();
  if (top > 0) {
    fill<double>(c, M.get(), 0.0, work);
    hipLaunchKernelGGL(k_csr_to_dense, dim3(cdiv(top, 256), nj), dim3(256), 0, c->stream,
                       (const DenseJob*)dj.get());
    hipLaunchKernelGGL(k_lu, dim3(nj), dim3(1024), 0, c->stream, (const DenseJob*)dj.get(),
                       sing.get());
    hipLaunchKernelGGL(k_lu_inverse, dim3(cdiv(top, 64), nj), dim3(64), 0, c->stream,
                       (const DenseJob*)dj.get(), (const int*)sing.get());
    MGD_CHECK_LAUNCH();
  }
  if (read1(c, sing.get())) fail(MGD_ESINGULAR, "zero pivot in the coarsest-level LU");
}

// ---------------------------------------------------------------------------
// hierarchy driver
// ---------------------------------------------------------------------------
void amg_build(Ctx* c, Csr<double>&& A0, const std::vector<int>& off0,
               const std::vector<int>& eoff0, const amg_params& p, SetupBatch& H) {
  DeferFrees frees(c);
  const int nm = (int)off0.size() - 1;
  MGD_REQUIRE(nm == 1 || setup_batches(p), "internal: these parameters set up one matrix at a time");
  H.levels.clear();
  H.n_levels.assign(nm, 0);
  const int tile = p.coarsening == 1 ? p.hmis_tile : 0;
  Csr<double> A = std::move(A0);
  std::vector<int> off = off0, eoff = eoff0;
  for (int lvl = 0;; ++lvl) {
    const int n = A.n_rows;
    SetupLevel L;
    L.off = off;
    L.eoff = eoff;
    const RowRanges R = row_ranges(off);
    MemberFlags M;
    bool any = false;
    for (int m = 0; m < nm; ++m) {
      const int rows = off[m + 1] - off[m];
      const bool on =
          rows > p.coarse_max && lvl != p.max_levels - 1 && lvl != MGD_MAX_LEVELS - 1;
      M.on[m] = on ? 1 : 0;
      any = any || on;
      if (rows > 0 || lvl == 0) H.n_levels[m] = lvl + 1;  // the last level, so far
    }
    if (!any) {
      L.A = std::move(A);
      H.levels.push_back(std::move(L));
      break;
    }
    const std::string at = " (level " + std::to_string(lvl) + ", " + std::to_string(n) + " rows)";
    DBuf<uint8_t> S;
    DBuf<int> stc, cidx;
    DBuf<double> diag;
    DBuf<int8_t> state;
    StepScope st_strength("amg setup: strength" + at);
    strength(c, A, p.strength_theta, p.dominance_theta, S, stc, diag);
    StepScope st_pmis("amg setup: pmis" + at);
    std::vector<int> coff =
        pmis(c, A, S, stc, R, M, p.seed, lvl, tile, state, cidx, L.rounds);
    StepScope st_cnum("amg setup: coarse numbering" + at);
    auto number = [&]() {
      DBuf<int> isc(c, (size_t)n);
      hipLaunchKernelGGL(k_is_c, dim3(cdiv(n, 256)), dim3(256), 0, c->stream, n,
                         (const int8_t*)state.get(), isc.get());
      MGD_CHECK_LAUNCH();
      exclusive_scan(c, isc.get(), cidx.get(), n);
      coff = read_bounds(c, R, cidx.get(), "coarse numbering");
    };
    const bool aggressive = lvl < p.aggressive_levels;
    if (aggressive && coff.back() > 0) {  // one matrix
      StepScope st_agg("amg setup: aggressive second pass" + at);
      L.rounds[0] += aggressive_split(c, A, S, cidx, coff.back(), p.seed, lvl, tile, state);
      number();
    }
    // members whose coarsening stalled end here
    bool stalled = false;
    any = false;
    for (int m = 0; m < nm; ++m) {
      const int rows = off[m + 1] - off[m], nc = coff[m + 1] - coff[m];
      if (M.on[m] && (nc == 0 || 10LL * nc > 9LL * rows)) {
        M.on[m] = 0;
        stalled = true;
      }
      any = any || M.on[m];
    }
    if (!any) {
      L.A = std::move(A);
      H.levels.push_back(std::move(L));
      break;
    }
    if (stalled) {
      hipLaunchKernelGGL(k_mask_f, dim3(cdiv(n, 256)), dim3(256), 0, c->stream, n, R, M,
                         state.get());
      MGD_CHECK_LAUNCH();
      number();
    }
    const int nc = coff.back();
    int max_cols = 0;  // no product row leaves its member
    for (int m = 0; m < nm; ++m) max_cols = std::max(max_cols, coff[m + 1] - coff[m]);
    Csr<double> P, Rt, AP, Ac;
    {
      StepScope st("amg setup: interpolation" + at);
      if (aggressive) {
        multipass_interpolation(c, A, S, state, cidx, nc, P);
        L.poff = {0, P.nnz};
      } else {
        interpolation(c, A, diag, S, state, cidx, R, nc, P, L.poff);
      }
      check_structure_async(c, P.n_rows, P.n_cols, P.nnz, P.rp.get(), P.ci.get(), false, false);
    }
    {
      StepScope st("amg setup: transpose of P" + at);
      transpose(c, P, Rt);
    }
    {
      StepScope st("amg setup: A P" + at);
      spgemm(c, A, P, max_cols, AP);
      check_structure_async(c, AP.n_rows, AP.n_cols, AP.nnz, AP.rp.get(), AP.ci.get(), false, false);
    }
    {
      StepScope st("amg setup: R (A P)" + at);
      spgemm(c, Rt, AP, max_cols, Ac);
      check_structure_async(c, Ac.n_rows, Ac.n_cols, Ac.nnz, Ac.rp.get(), Ac.ci.get(), true, false);
      eoff = read_bounds(c, row_ranges(coff), Ac.rp.get(), "coarse operator");
    }
    L.A = std::move(A);
    L.cf = std::move(state);
    L.P = std::move(P);
    L.coff = coff;
    off = coff;
    H.levels.push_back(std::move(L));
    A = std::move(Ac);
  }
  if (p.smoother == 1) {
    for (size_t l = 0; l < H.levels.size(); ++l) {
      StepScope st("amg setup: colouring (level " + std::to_string(l) + ")");
      auto& L = H.levels[l];
      L.ncolours = jp_colouring(c, L.A, p.seed, (int)l, L.colour);
    }
  }
  StepScope st("amg setup: coarsest LU");
  coarsest_inverses(c, p, H);
}

}  // namespace mgd
