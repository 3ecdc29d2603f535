// AMG setup on the device (natural ordering).
#pragma once
#include <memory>
#include <vector>

#include "common.hpp"

namespace mgd {

constexpr int8_t kC = 1, kF = -1, kU = 0;

// Rows of a level member after member: member q has [off[q], off[q + 1]), none
// where the two are equal.  Passed by value as a kernel argument.
constexpr int kMaxMembers = 66;
struct RowRanges {
  int nm = 0;
  int off[kMaxMembers + 1] = {};
};
__device__ __forceinline__ int member_of(const RowRanges& R, int i) {
  int lo = 0, hi = R.nm;  // off[lo] <= i < off[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (R.off[mid] <= i)
      lo = mid;
    else
      hi = mid;
  }
  return lo;
}

struct UMember;  // a member's arrays at one level, for the union builder

// Hierarchies built together: level l holds the level matrices of all members
// that have one as the diagonal blocks of one matrix (columns numbered through),
// so one set of launches and one wait serve them all.  A member keeps the values
// it would have alone: its rows only see its own columns, and whatever depends
// on a row's number (hash keys, tie breaks) uses the number within the member.
// The 22 hierarchies of the 3D 64^3, G = 20 system take 29 ms together; one
// after another they took 145 ms, most of it launches and waits on small levels.
struct SetupLevel {
  Csr<double> A;
  DBuf<int8_t> cf;            // empty on the last level; all F for members that end here
  Csr<double> P;              // A.n_rows x next level's rows; empty rows for members that end here
  std::vector<int> off, eoff;    // per member its first row and entry (members + 1)
  std::vector<int> coff, poff;   // its first coarse row and entry of P (members + 1)
  std::vector<int> rounds;       // PMIS rounds per member
  DBuf<int> colour;  // Jones-Plassmann colours (multicolour Gauss-Seidel only)
  int ncolours = 0;
};

struct SetupBatch {
  std::vector<SetupLevel> levels;
  std::vector<int> n_levels;     // per member
  std::vector<int> coarse_kind;  // per member: 0 dense LU (explicit inverse), 1 l1-Jacobi sweeps
  DBuf<double> inv;              // the inverses, n_L x n_L, column-major
  std::vector<size_t> inv_at;    // per member its first value in inv
};

// A member's level-0 matrix inside its batch: row i at rp[i], columns ci - base.
struct MemberCsr {
  int n = 0, nnz = 0, base = 0;
  const int* rp = nullptr;
  const int* ci = nullptr;
  const double* v = nullptr;
};

struct SetupHierarchy {
  std::shared_ptr<SetupBatch> b;
  int m = 0;
  size_t n_levels() const { return b->n_levels[m]; }
  bool last(size_t l) const { return l + 1 == n_levels(); }
  int n(size_t l) const { return b->levels[l].off[m + 1] - b->levels[l].off[m]; }
  int nnz(size_t l) const { return b->levels[l].eoff[m + 1] - b->levels[l].eoff[m]; }
  int nnz_P(size_t l) const { return last(l) ? 0 : b->levels[l].poff[m + 1] - b->levels[l].poff[m]; }
  int rounds(size_t l) const { return last(l) ? 0 : b->levels[l].rounds[m]; }
  int coarse_kind() const { return b->coarse_kind[m]; }
  const double* inverse() const { return b->inv.get() + b->inv_at[m]; }
  MemberCsr level0() const {
    const SetupLevel& L = b->levels[0];
    return {n(0), nnz(0), L.off[m], L.A.rp.get() + L.off[m], L.A.ci.get(), L.A.v.get()};
  }
  UMember member(size_t l) const;
};

// Copy a caller matrix into an owned one.
void csr_copy_from(Ctx* c, const mgd_csr* A, Csr<double>& out);
// Build the hierarchies of the diagonal blocks of A0 (member q: rows and columns
// [off[q], off[q + 1]), entries [eoff[q], eoff[q + 1])), already validated.  More
// than one member needs setup_batches(p).
void amg_build(Ctx* c, Csr<double>&& A0, const std::vector<int>& off,
               const std::vector<int>& eoff, const amg_params& p, SetupBatch& H);
// Whether hierarchies with these parameters can be built together (HMIS tiles,
// the distance-two pass and colourings are formed for one matrix at a time).
inline bool setup_batches(const amg_params& p) {
  return p.coarsening == 0 && p.aggressive_levels == 0 && p.smoother == 0;
}

// Sorted transpose (values copied).
void transpose(Ctx* c, const Csr<double>& A, Csr<double>& T);
// C = A B, structural pattern, entries summed over ascending k from 0.  No row of
// C has more than max_cols columns.
void spgemm(Ctx* c, const Csr<double>& A, const Csr<double>& B, int max_cols, Csr<double>& C);
// Jones-Plassmann colouring of the structural graph of A; returns the number of colours
int jp_colouring(Ctx* c, const Csr<double>& A, uint64_t seed, int level, DBuf<int>& colour);
}  // namespace mgd
