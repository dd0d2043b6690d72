// Host-side replay of the dense kernels' LDS layouts (built with -fsanitize=address,undefined by the test).  Every array of
// DenseLds and DenseAdjLds is listed with the words that the kernels index (from the loops' extreme indices) and the phases of a
// substep in which its contents are alive; every word is touched in a heap buffer of exactly the launch's size, arrays alive in
// a common phase must not share a word, and what lanes read past an array's end (results that are not used) must stay
// inside the workgroup's LDS.  Prints one JSON line and exits nonzero on a violation.
//   dense_lds_check step n_links n_v n_dof n_actors n_tendon_joints
//   dense_lds_check adjoint n_links n_v n_dof n_actors max_rows substeps sweeps row_cap
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "ags_dense_layout.h"

using namespace ags;

namespace {
int g_fail = 0;

struct Arr {
  std::string name;
  long word, words;  // 8-byte words
  int from, to;      // first and last phase
};
Arr ints(const char* name, long at, long n, int from, int to) { return {name, at / 2, (at % 2 + n + 1) / 2, from, to}; }

void check(const char* what, const std::vector<Arr>& arrays, const std::vector<Arr>& past, long total) {
  std::vector<double> lds((size_t)total, 0.0);
  auto fail = [&](const std::string& why) {
    std::fprintf(stderr, "%s: %s\n", what, why.c_str());
    g_fail = 1;
  };
  for (const Arr& a : arrays) {
    if (a.word < 0 || a.words < 0 || a.word + a.words > total) {
      fail(a.name + " [" + std::to_string(a.word) + ", " + std::to_string(a.word + a.words) + ") of " + std::to_string(total));
      continue;
    }
    for (long k = a.word; k < a.word + a.words; ++k) lds[k] += 1.0;  // through the buffer that the sanitizer watches
  }
  for (const Arr& a : past)
    if (a.word < 0 || a.word + a.words > total) fail(a.name + " is read past the workgroup's LDS");
  for (size_t i = 0; i < arrays.size(); ++i)
    for (size_t j = 0; j < i; ++j) {
      const Arr &a = arrays[i], &b = arrays[j];
      if (a.from <= b.to && b.from <= a.to && a.word < b.word + b.words && b.word < a.word + a.words)
        fail(a.name + " and " + b.name + " share words while both are alive");
    }
}

// phases of a substep of the step
enum { CONTROLS, POSES, VELOCITIES, TERMS, ACCELERATIONS, FORCES, SUBTREE, MOMENTA, MASS, LOAD, FACTOR, COEFFICIENTS, VSTAR,
       NARROW, ROWS, CHUNK, DELASSUS, SWEEPS, CHANGE, OUTPUTS };

template <int NC, int LR>
long step(int n_links, int n_v, int n_dof, const ags_model_info& info, int n_tj) {
  using L = DenseLds<NC, LR>;
  const DenseDyn dyn = make_dense_layout(info, dense_fixed_words(NC, LR));
  const int CT = NC > 16 ? 2 : 1, tri = NC * (NC + 1) / 2, last = 16 * CT - 1;
  const std::vector<Arr> arrays = {
      ints("la", L::t_la, NC, 0, OUTPUTS), ints("lcm", L::t_lcm, NC, 0, OUTPUTS), ints("ccm", L::t_ccm, NC, 0, OUTPUTS),
      {"qj", L::qj, n_dof, 0, OUTPUTS}, {"qd", L::qd, NC, 0, OUTPUTS}, {"vs", L::vs, NC, 0, OUTPUTS},
      ints("lrow", L::lrow, 2l * n_dof, NARROW, OUTPUTS), {"org", L::org, 3, 0, OUTPUTS},
      {"root", dyn.root, 13l * info.n_actors, 0, OUTPUTS},
      {"tendon lengths and rates", L::X, 2l * n_tj, CONTROLS, CONTROLS},
      {"S", L::S, 6l * NC, POSES, CHUNK}, {"pose", L::pose, (long)kDensePose * n_links, POSES, ROWS},
      {"V", L::V, 6l * NC, VELOCITIES, FORCES}, {"F", L::V, 6l * NC, MOMENTA, MASS},
      // 16-byte pairs at lane - k - 2 < 30; the last pair read is W - 3 <= NC - 3
      {"window", L::V, 2l * std::max(30, NC - 2), FACTOR, FACTOR}, {"v* of the links", L::V, 6l * NC, VSTAR, ROWS},
      {"column terms", L::X, 6l * NC, TERMS, ACCELERATIONS}, {"accelerations", L::X + 6 * NC, 6l * NC, ACCELERATIONS, FORCES},
      // (lanes read their 16 words before the wavefront writes: the two may share words in FORCES only through registers)
      {"inertias and forces", L::X, (long)kDenseXStride * (NC - 1) + 16, SUBTREE, MOMENTA},
      {"M", L::X, tri, MASS, LOAD}, {"strip", L::strip, 64, LOAD, LOAD}, {"G", L::G, L::g_words, FACTOR, CHANGE},
      {"co", L::co, 2l * 32, COEFFICIENTS, CHUNK}, ints("rm", L::rm, 2l * kDenseChunk, CHUNK, CHUNK),
      {"cn", L::cn, 3l * kDenseContacts, NARROW, CHUNK}, {"cx", L::cx, 3l * kDenseContacts, NARROW, CHUNK},
      {"cphi", L::cphi, kDenseContacts, NARROW, CHUNK}, ints("clk", L::clk, kDenseContacts, NARROW, CHUNK),
      {"lbias", L::lbias, 2l * n_dof, NARROW, CHUNK}, {"rowf", L::pose, 6l * kDenseChunk, CHUNK, CHUNK},
      {"A", L::A, (long)(LR - 1) * L::A_stride + LR, DELASSUS, SWEEPS},
      {"lam", L::lam, kDenseRows, CHANGE, CHANGE}, {"u", L::u, 64, CHANGE, CHANGE},
  };
  const std::vector<Arr> past = {
      {"S by column tiles", L::S, 6l * last + 6, 0, 0}, {"F by column tiles", L::V, 6l * last + 6, 0, 0},
      {"ccm", 0, (L::t_ccm + NC + 1) / 2, 0, 0},
      // the sweeps' next contact: rows to LR + 2
      {"A ahead", L::A, (long)(LR + 2) * L::A_stride + LR, 0, 0},
  };
  check("step", arrays, past, dyn.total);
  if (n_v > NC - 1 || n_links > NC || 2 * n_tj > dense_x_words(NC)) g_fail = 1;
  return 8l * dyn.total;
}

// phases of a job of the adjoint
enum { A_CONTROLS, A_POSES, A_VELOCITIES, A_TERMS, A_FORCES, A_SUBTREE, A_MOMENTA, A_MASS, A_LOAD, A_FACTOR, A_VSTAR, A_NARROW,
       A_ROWS, A_DELASSUS, A_SWEEPS, A_CHANGE, A_INTEGRATION, A_REVERSE, A_SOLVE, A_PRODUCTS, A_JBAR, A_ROWS_REVERSE, A_CONTACTS,
       A_READ_P, A_AGAIN, A_MASS_TERMS, A_LINKS, A_WRENCHES, A_END };

template <int NC, int RT>
long adjoint(int n_links, int n_v, const ags_model_info& info, int substeps, int iters, int cap) {
  using L = DenseAdjLds<NC, RT>;
  const DenseAdjDyn d = make_dense_adj_layout<NC, RT>(info, substeps, iters, cap);
  const int CT = NC > 16 ? 2 : 1, tri = NC * (NC + 1) / 2, last = 16 * CT - 1, RC = L::rows, nd = info.n_dof;
  const long x16 = (long)kDenseXStride * (NC - 1) + 16, zw = (long)(RC - 1) * L::Z_stride + 16 * CT,
             pw = (long)(16 * CT - 1) * L::Z_stride + 16 * CT;
  const std::vector<Arr> arrays = {
      ints("la", L::t_la, NC, 0, A_END), ints("lcm", L::t_lcm, NC, 0, A_END), ints("ccm", L::t_ccm, NC, 0, A_END),
      {"dv", L::dv, NC, A_CHANGE, A_PRODUCTS}, {"z", L::z, NC, A_INTEGRATION, A_JBAR}, {"qdd", L::qdd, NC, A_FACTOR, A_PRODUCTS},
      {"w", L::w, NC, A_SOLVE, A_END}, {"vs", L::vs, NC, A_MOMENTA, A_JBAR}, {"nu", L::nu, NC, 0, A_LINKS},
      {"qj", L::qj, nd, 0, A_CHANGE}, {"nub", L::nub, NC, A_INTEGRATION, A_LINKS}, {"nui", L::nui, NC, A_LINKS, A_END},
      {"nh", L::nh, NC, A_INTEGRATION, A_SOLVE}, {"u", L::u, 64, A_CHANGE, A_END}, {"org", L::org, 3, 0, A_END},
      {"S", L::S, 6l * NC, A_POSES, A_END}, {"pose", L::pose, (long)kDensePose * n_links, A_POSES, A_END},
      {"G", L::G, L::g_words, A_FACTOR, A_PRODUCTS}, {"co", L::co, 2l * NC, A_FACTOR, A_PRODUCTS},
      {"window", L::rowf, 2l * std::max(30, NC - 2), A_FACTOR, A_FACTOR}, {"rowf", L::rowf, 6l * RC, A_ROWS, A_ROWS_REVERSE},
      ints("rm", L::rm, 2l * RC, A_ROWS, A_JBAR), {"lamy", L::lamy, 2l * RC, A_CHANGE, A_JBAR},
      {"cx", L::cx, 3l * L::contacts, A_NARROW, A_CONTACTS},
      // wrenches of both bodies of every contact, padded to a multiple of four
      {"ce", L::rowf, 6l * ((2 * L::contacts + 3) & ~3), A_CONTACTS, A_WRENCHES},
      ints("cel", L::cel, (2l * L::contacts + 3) & ~3l, A_CONTACTS, A_WRENCHES),
      {"column terms", L::X, 6l * NC, A_TERMS, A_TERMS}, {"V", L::V, 6l * NC, A_VELOCITIES, A_FORCES},
      {"Acc", L::Acc, 6l * NC, A_TERMS, A_FORCES}, {"inertias and forces", L::X, x16, A_FORCES, A_MOMENTA},
      {"Fm", L::Fm, 6l * NC, A_MOMENTA, A_MASS}, {"M", L::X, tri, A_MASS, A_LOAD}, {"strip", L::X + tri, 64, A_LOAD, A_LOAD},
      {"Vs", L::Vs, 6l * NC, A_VSTAR, A_ROWS}, {"lbias", L::lbias, 2l * nd, A_NARROW, A_ROWS},
      ints("lrow", L::lrow, 2l * nd, A_NARROW, A_ROWS), {"cn", L::cn, 3l * L::contacts, A_NARROW, A_ROWS},
      {"cphi", L::cphi, L::contacts, A_NARROW, A_ROWS}, ints("clk", L::clk, L::contacts, A_NARROW, A_ROWS),
      {"A", L::A, (long)(RC - 1) * L::A_stride + RC, A_DELASSUS, A_REVERSE},
      {"tape", L::tape, 2l * d.iters4 * RC, A_SWEEPS, A_PRODUCTS}, {"mask", d.mask, 2l * iters, A_SWEEPS, A_REVERSE},
      {"Z", L::X, zw, A_PRODUCTS, A_PRODUCTS}, {"T", L::X, zw, A_JBAR, A_JBAR}, {"Jbar", L::X, zw, A_ROWS_REVERSE, A_ROWS_REVERSE},
      {"sb", L::sb, 6l * NC, A_ROWS_REVERSE, A_LINKS}, {"rv", L::X, 6l * RC, A_CONTACTS, A_CONTACTS},
      {"P", L::X, pw, A_READ_P, A_READ_P}, {"V again", L::V, 6l * NC, A_AGAIN, A_LINKS}, {"Acc again", L::Acc, 6l * NC, A_AGAIN, A_LINKS},
      {"inertias again", L::X, x16, A_AGAIN, A_AGAIN}, {"Fm again", L::Fm, 6l * NC, A_AGAIN, A_AGAIN},
      {"path sums and momenta", L::X, 12l * NC, A_MASS_TERMS, A_MASS_TERMS}, {"link terms", L::X, x16, A_LINKS, A_END},
      {"st", d.st, (long)substeps * d.state_words, 0, A_END}, {"rbar", d.rbar, 13l * info.n_actors, 0, A_END},
      {"dbar", d.dbar, 2l * nd, 0, A_END},
  };
  const std::vector<Arr> past = {
      {"S by column tiles", L::S, 6l * last + 6, 0, 0}, {"Fm by column tiles", L::Fm, 6l * last + 6, 0, 0},
      {"z by column tiles", L::z, last + 1, 0, 0}, {"vs by column tiles", L::vs, last + 1, 0, 0},
      {"dv ... w by column tiles", L::dv, 3l * NC + last + 1, 0, 0}, {"nh by column tiles", L::nh, last + 1, 0, 0},
      {"A ahead", L::A, iters > 0 ? (long)(RC + 2) * L::A_stride + RC : 0, 0, 0}, {"A before its first row", L::A - 6, 6, 0, 0},
      {"P by rows", L::X, (long)(NC - 1) * L::Z_stride + 32, 0, 0},
  };
  check("adjoint", arrays, past, d.total);
  if (n_v > NC - 1 || n_links > NC || d.rows_cap > RC || d.iters4 < iters) g_fail = 1;
  return 8l * d.total;
}
}  // namespace

int main(int argc, char** argv) {
  const bool adj = argc == 10 && !std::strcmp(argv[1], "adjoint");
  if (!adj && !(argc == 7 && !std::strcmp(argv[1], "step"))) return 2;
  ags_model_info info{};
  const int nl = info.n_links = std::atoi(argv[2]), nv = info.n_v = std::atoi(argv[3]), nd = info.n_dof = std::atoi(argv[4]);
  info.n_actors = std::atoi(argv[5]);
  const int nc = dense_class(nv, nl);
  long b32 = 0, b64 = 0;
  if (!adj) {
    const int n_tj = std::atoi(argv[6]);
    auto both = [&](auto c) {
      constexpr int NC = decltype(c)::value;
      b32 = step<NC, kDenseLdsRows>(nl, nv, nd, info, n_tj);
      b64 = step<NC, kDenseRows>(nl, nv, nd, info, n_tj);
    };
    nc == 16 ? both(std::integral_constant<int, 16>{}) : nc == 28 ? both(std::integral_constant<int, 28>{}) : both(std::integral_constant<int, 32>{});
  } else {
    info.max_rows = std::atoi(argv[6]);
    const int substeps = std::atoi(argv[7]), iters = std::atoi(argv[8]), cap = std::atoi(argv[9]);
    auto both = [&](auto c) {
      constexpr int NC = decltype(c)::value;
      b32 = adjoint<NC, 2>(nl, nv, info, substeps, iters, std::min(cap, 32));
      b64 = adjoint<NC, 4>(nl, nv, info, substeps, iters, cap);
    };
    nc == 16 ? both(std::integral_constant<int, 16>{}) : nc == 28 ? both(std::integral_constant<int, 28>{}) : both(std::integral_constant<int, 32>{});
  }
  std::printf("{\"class\": %d, \"bytes_32_rows\": %ld, \"bytes_64_rows\": %ld, \"ok\": %s}\n", nc, b32, b64, g_fail ? "false" : "true");
  return g_fail;
}
