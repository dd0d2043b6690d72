// LDS layouts of the dense step and adjoint kernels (one environment per 64-lane workgroup): plain C++ with no HIP
// dependency, shared by the host runtime, the kernels and the host-side replay of the tests (dense_lds_check.cpp), which knows
// the phases in which each array is alive.
#pragma once

#include "../../include/ags.h"

namespace ags {

constexpr int kDenseMaxV = 31;      // columns: one lane each below 32, and one more lane for the right-hand side
constexpr int kDenseMaxLinks = 32;  // links: one lane and one mask bit each
constexpr int kDenseRows = 64;      // rows solved one per lane; more go through global scratch
constexpr int kDenseZWords = 32 * kDenseRows;  // tiles of Z^T of up to 64 rows in scratch
constexpr int kDenseChunk = 32;     // rows whose Jacobian columns are formed at a time
constexpr int kDenseLdsRows = 32;   // rows whose Delassus matrix is kept in LDS (small batches: kDenseRows)
constexpr int kDenseXStride = 17;   // words per link of the subtree sums (10 inertia, 6 force; odd: no bank conflicts)
constexpr int kDensePose = 7;       // words per link pose: quaternion xyzw, origin

// Size class of a model: NC - 1 columns and NC links at most, NC a multiple of four (the contraction step of a matrix
// tile).  The kernels are compiled per class, so that these offsets are constants and loops over columns and links have
// no bounds tests; columns and links past the model's are zeros.  28 is the humanoid's class (27 columns).
constexpr int dense_class(int n_v, int n_links) {
  return n_v <= 15 && n_links <= 16 ? 16 : n_v <= 27 && n_links <= 28 ? 28 : 32;
}

constexpr int kDenseContacts = 21;  // contacts of an environment whose rows fit its lanes

// Offsets in 8-byte words, except the integer arrays (t_*, lrow, rm, clk), which are in ints.  The overlays keep a
// workgroup at 10-15 KB, so that the registers and not the LDS bound how many fit a CU.
template <int NC, int LR = kDenseLdsRows>
struct DenseLds {
  static constexpr int max2(int a, int b) { return a > b ? a : b; }
  // model masks: ancestors of a link, columns moving a link, columns of a row of M
  static constexpr int t_la = 0, t_lcm = NC, t_ccm = 2 * NC;
  // live through a substep: positions, rates, v* (before it, the right-hand side), limit rows, reference point
  static constexpr int qj = 3 * NC / 2, qd = qj + NC, vs = qd + NC, lrow = 2 * (vs + NC), org = vs + NC + 32;
  // Dynamics region.  S: column axes.  pose: link poses.  V: link velocities, the columns' momenta, the factor's
  // broadcast window, link velocities under v*.  X: per-link sums, the packed mass matrix and behind it a 1 among 63
  // zeros; later the rows' column masks (rm), the coefficients of the factor's columns (co), the contacts (normal,
  // point, distance, links) and the limit rows' biases.  The rows' forces of one chunk overlay pose and V.
  static constexpr int S = org + 4, pose = S + 6 * NC, V = pose + kDensePose * NC, X = V + 6 * NC, strip = X + NC * (NC + 1) / 2,
                       rm = 2 * X, co = X + 64, cn = X + 128, cx = cn + 66, cphi = cx + 66, clk = 2 * (cphi + 22),
                       lbias = cphi + 34,
                       x_words = max2(max2(kDenseXStride * NC, NC * (NC + 1) / 2 + 64), 128 + 66 + 66 + 34 + 64);
  // The Delassus matrix of at most LR rows (row stride odd: its transposed tile is written without bank conflicts) overlays the region from its start, after the sweeps the impulses
  // and the velocity change in the factor's columns.  G: pairs of columns of the factor's inverse transpose, column pair
  // m as (2 m + 2) x 2 words, behind the Delassus matrix (over the tail of X, written when the mass matrix has been read).
  static constexpr int A = S, lam = A, u = A + kDenseRows, A_stride = LR + 1, G = A + LR * A_stride,
                       g_words = NC / 2 * (NC / 2 + 1) * 2;
  // (the sweeps read up to three rows behind the matrix) then the model's root states
  static constexpr int fixed = max2(max2(X + x_words, G + g_words), A + (LR + 3) * A_stride);
  static_assert(S % 2 == 0 && V % 2 == 0 && co % 2 == 0 && u % 2 == 0 && G % 2 == 0, "16-byte aligned pairs");
  static_assert(kDensePose * NC + 6 * NC >= 6 * kDenseChunk && 6 * NC >= 64, "overlaid arrays fit");
  static_assert(lbias + 64 <= G, "the factor's columns leave what is read after them alone");
};

struct DenseDyn {
  int root;   // 13 words per actor
  int total;  // words
};
inline DenseDyn make_dense_layout(const ags_model_info& info, int fixed_words) {
  return {fixed_words, (fixed_words + 13 * info.n_actors + 1) & ~1};
}
template <int LR>
inline int dense_fixed_words(int nc) {
  return nc == 16 ? DenseLds<16, LR>::fixed : nc == 28 ? DenseLds<28, LR>::fixed : DenseLds<32, LR>::fixed;
}
inline int dense_fixed_words(int nc, int lds_rows) {
  return lds_rows == kDenseRows ? dense_fixed_words<kDenseRows>(nc) : dense_fixed_words<kDenseLdsRows>(nc);
}
inline int dense_x_words(int nc) {
  return nc == 16 ? DenseLds<16>::x_words : nc == 28 ? DenseLds<28>::x_words : DenseLds<32>::x_words;
}

// LDS of the dense adjoint (RT tiles of 16 rows), offsets in 8-byte words except t_*, rm, lrow, clk, cel (ints).  What the
// reverse could recompute (velocities, accelerations, inertias, momenta) is not kept through the sweeps: five instead of
// four workgroups of the humanoid's class would fit a CU with it, six fit without.
template <int NC, int RT>
struct DenseAdjLds {
  static constexpr int max2(int a, int b) { return a > b ? a : b; }
  static constexpr int rows = 16 * RT, contacts = rows / 3;
  static constexpr int A_stride = rows + 1, Z_stride = 33;  // odd: columns are read without bank conflicts
  static constexpr int t_la = 0, t_lcm = NC, t_ccm = 2 * NC;
  // per column: velocity change of the impulses, z = M^-1 nubar, free acceleration, w = M^-1 h v*bar (these four one after
  // the other: a lane group steps from one to the next); v*, rates, positions, nubar (then v*bar), rate adjoints, G^T nubar
  static constexpr int dv = 3 * NC / 2, z = dv + NC, qdd = z + NC, w = qdd + NC, vs = w + NC, nu = vs + NC, qj = nu + NC,
                       nub = qj + NC, nui = nub + NC, nh = nui + NC, u = nh + NC, org = u + 64;
  // column axes, link poses, factor
  static constexpr int S = org + 4, pose = S + 6 * NC, G = pose + kDensePose * NC, g_words = NC / 2 * (NC / 2 + 1) * 2,
                       co = G + g_words;
  // rows: forces (before them the factor's window, after them the contacts' wrenches), masks, impulses and their adjoints
  static constexpr int rowf = co + 2 * NC, rm = 2 * (rowf + 6 * rows), lamy = rowf + 7 * rows, cx = lamy + 2 * rows,
                       cel = 2 * (cx + 3 * contacts), work = (cx + 4 * contacts + 3) & ~1;
  // work, before the rows: X (17 words per link, then the packed mass matrix and a 1 among zeros), velocities,
  // accelerations, momenta; then velocities under v*, limits and contacts; then the Delassus matrix and behind it the tape;
  // then rows x columns products (X of the reverse), P; then again X, velocities, accelerations, momenta
  static constexpr int X = work, V = X + max2(kDenseXStride * NC, NC * (NC + 1) / 2 + 64), Acc = V + 6 * NC, Fm = Acc + 6 * NC,
                       Vs = work, lbias = Vs + 6 * NC, lrow = 2 * (lbias + 64), cn = lbias + 96, cphi = cn + 3 * contacts,
                       clk = 2 * (cphi + contacts), A = work, tape = A + rows * A_stride,
                       sb = max2(Fm + 6 * NC, work + max2(rows, 32) * Z_stride),  // axis adjoint of every column
                       fixed = sb + 6 * NC;
  static_assert(S % 2 == 0 && G % 2 == 0 && co % 2 == 0 && rowf % 2 == 0 && u % 2 == 0 && work % 2 == 0, "16-byte aligned pairs");
  static_assert(6 * (2 * contacts + 4) <= 6 * rows && cphi + 2 * contacts <= fixed, "overlaid arrays fit");
};

struct DenseAdjDyn {
  int iters4;               // sweeps, rounded up to the contraction step of a tile.  Tape: per sweep and row the change of
                            // the impulse, then (reverse) the row adjoint after the sweep
  int mask;                 // per sweep: bits of the rows updated freely, of those at the upper bound
  int st, rbar, dbar;       // state at every substep's start; adjoints of roots and of DOFs
  int state_words, rows_cap, total;
};
inline DenseAdjDyn make_dense_adj_layout(const ags_model_info& info, int substeps, int iters, int row_cap, int fixed, int tape,
                                         int rows) {
  DenseAdjDyn d{};
  d.iters4 = (iters + 3) & ~3;
  d.mask = tape + 2 * d.iters4 * rows;
  int off = d.mask + 2 * d.iters4;
  off = ((off > fixed ? off : fixed) + 1) & ~1;
  auto take = [&](int n) {
    const int o = off;
    off += n;
    return o;
  };
  d.state_words = 13 * info.n_actors + 2 * info.n_dof;
  d.st = take(substeps * d.state_words);
  d.rbar = take(13 * info.n_actors);
  d.dbar = take(2 * info.n_dof);
  const int rc = info.max_rows > 1 ? info.max_rows : 1;
  d.rows_cap = rc < row_cap ? rc : row_cap;
  d.total = off;
  return d;
}
template <int NC, int RT>
inline DenseAdjDyn make_dense_adj_layout(const ags_model_info& info, int substeps, int iters, int row_cap) {
  using L = DenseAdjLds<NC, RT>;
  return make_dense_adj_layout(info, substeps, iters, row_cap, L::fixed, L::tape, L::rows);
}
inline DenseAdjDyn make_dense_adj_layout(int nc, int big, const ags_model_info& info, int substeps, int iters, int row_cap) {
  if (nc == 16)
    return big ? make_dense_adj_layout<16, 4>(info, substeps, iters, row_cap) : make_dense_adj_layout<16, 2>(info, substeps, iters, row_cap);
  if (nc == 28)
    return big ? make_dense_adj_layout<28, 4>(info, substeps, iters, row_cap) : make_dense_adj_layout<28, 2>(info, substeps, iters, row_cap);
  return big ? make_dense_adj_layout<32, 4>(info, substeps, iters, row_cap) : make_dense_adj_layout<32, 2>(info, substeps, iters, row_cap);
}

}  // namespace ags
