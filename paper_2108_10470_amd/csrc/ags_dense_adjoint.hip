// Dense form of the adjoint of one env-step (ags_adjoint.hip states what is differentiated) for models of at most 31
// generalized velocities and 32 links, FP64, one wavefront per environment.
//
// The recomputation is the dense step's: poses by pointer jumping, sums along the tree as products with 0/1 matrices on
// the matrix cores, M = U^T B U factored in registers, G = U^-1 B^-1/2, Z = J G, A = Z Z^T.  In reverse:
//   * solves with M are products with G: z = G (G^T nubar), lambda_bar = J z = Z (G^T nubar), w = h G (G^T nubar + Z^T ybar)
//   * Gauss-Seidel: with t = lambda_bar + A ybar per row (a lane each), the reverse of a free update of row r reads
//     g = t_r and adds -A_kr / A_rr g to every t_k (t_r becomes zero), that of a clamped one zeroes t_r and hands
//     +-mu g to its normal row.  Only the impulse changes dl and the row adjoints y per sweep are kept; the adjoint of A
//     follows from them by two products over the sweeps: for s > r, Abar_sr + Abar_rs =
//     sum_it y_s(after) dl_r + dl_s y_r(before), and 2 sum_it y_s(after) dl_s on the diagonal (which includes the adjoint
//     of 1 / A_rr)
//   * P = 1/2 W S W^T + ... = G (1/2 Z^T S Z) G^T + ...; T = S W = (S Z) G^T
//   * every adjoint of a column's axis, a link's inertia or a contact's point and direction is a sum over the columns
//     moving a link, the columns or links below a column, or the rows on it: products with the same 0/1 matrices.
//     <s, I y> terms of all columns over a link need only sum(w_s w_y^T + w_y w_s^T) and sum(v_y x w_s + v_s x w_y).
//
// What bounds it: the chain of one wavefront's dependent instructions, with 1.5 wavefronts per SIMD resident (six
// workgroups of 26 KB per CU for the humanoid-like model with room for 32 rows, 256 registers; four of 34 KB and 385
// registers were slower), and after it the few environments with more rows, in a form with room for 64 (44 of 4096
// take 0.25 ms on their own).  Cycles per environment and call, 4096 of them, three recomputations and two reversals:
// 392 k; recomputation outside Gauss-Seidel 157 k, Gauss-Seidel 65 k and its reverse 40 k, products 37 k, mass-matrix
// terms with the kinematics formed again 27 k, rows 17 k, RNEA 20 k, integration and solves 30 k.
// A lone wavefront issues an instruction about every seven cycles, so the sweeps are counted in instructions, scalar
// ones and branches included: impulses taken from the captured z after a sweep instead of selected row by row, and a
// reverse without branches, took the 52-60 row environment from 637 k to 599 k cycles.
// 4096 humanoid-like environments 0.80 ms per call (general form 4.69), relative difference 1e-13.
#include "ags_dense_ops.h"
#include "ags_adj_math.h"

namespace ags {
namespace {

// adjoint of -<Y, I X> with respect to the body's centre of mass (point) and orientation (torque)
__device__ __forceinline__ void bil_neg(const Body& b, SV Y, SV X, V3<R>& cb, V3<R>& tI) {
  const V3<R> uY = add(Y.v, cross(Y.w, b.c)), uX = add(X.v, cross(X.w, b.c));
  cb = sub(cb, mul(add(cross(uY, X.w), cross(uX, Y.w)), b.m));
  tI = sub(tI, add(cross(b.symv(X.w), Y.w), cross(b.symv(Y.w), X.w)));
}

// per-phase clock counters of the debug accounting, then the current phase and the last mark (lane 0)
__shared__ long long g_dadj_clock[kAdjPhases + 2];

template <int NC, int RT>
__device__ __forceinline__ void dense_adjoint_env(Cp<AdjArgs> P_, int ei) {
  using L = DenseAdjLds<NC, RT>;
  constexpr int CT = NC > 16 ? 2 : 1, RC = L::rows, AS = L::A_stride, ZS = L::Z_stride, KC = L::contacts;
  const Lp<R> sm = (Lp<R>)g_dense_lds;
  const Lp<int> si_ = (Lp<int>)g_dense_lds;
  const int lane_ = threadIdx.x;
  Cp<AdjArgs> P = P_;
  int lane = lane_, lc = lane & 15, lg = lane >> 4;
  const int env = __builtin_amdgcn_readfirstlane(gp(P->env_list)[ei]);
  if (P->skip_flags && __builtin_amdgcn_readfirstlane(gp(P->skip_flags)[env]) != 0) return;  // another launch runs this env
  auto phase = [&](int ph) {
    if (!P->cycles) return;
    if (lane_ == 0) {
      const long long now = (long long)clock64();
      const int cur = (int)g_dadj_clock[kAdjPhases];
      if (cur >= 0) g_dadj_clock[cur] += now - g_dadj_clock[kAdjPhases + 1];
      g_dadj_clock[kAdjPhases] = ph;
      g_dadj_clock[kAdjPhases + 1] = now;
    }
  };
#define ADJ_PHASE(ph)        \
  lane = opaque_lane(lane_); \
  lc = lane & 15;            \
  lg = lane >> 4;            \
  P = opaque_arg(P_);        \
  phase(ph)
  if (P->cycles && lane_ == 0) {
    for (int k = 0; k < kAdjPhases; ++k) g_dadj_clock[k] = 0;
    g_dadj_clock[kAdjPhases] = -1;
  }
  const int nv = P->m.n_v, ns = P->m.n_slots, na = P->m.n_actors, nd = P->m.n_dof;
  const int abase = gp(P->env_actor_base)[env], dbase = gp(P->env_dof_base)[env];
  const Lp<int> la = si_ + L::t_la, lcm = si_ + L::t_lcm, ccm = si_ + L::t_ccm;
  const Lp<R> dv = sm + L::dv, z_ = sm + L::z, qdda = sm + L::qdd, w_ = sm + L::w, vs = sm + L::vs, nu = sm + L::nu,
              qj = sm + L::qj, nub = sm + L::nub, vsb = nub, nui = sm + L::nui, u = sm + L::u, nh = sm + L::nh, org = sm + L::org;
  const Lp<R> S = sm + L::S, pose = sm + L::pose, rowf = sm + L::rowf, lamy = sm + L::lamy, cn = sm + L::cn, cx = sm + L::cx,
              cphi = sm + L::cphi, X = sm + L::X, V = sm + L::V, Acc = sm + L::Acc, Fm = sm + L::Fm, Vs = sm + L::Vs,
              lbias = sm + L::lbias, A_ = sm + L::A, tape = sm + L::tape, sb = sm + L::sb;
  const Lp<d2> co = (Lp<d2>)(sm + L::co), G2 = (Lp<d2>)(sm + L::G);
  const Lp<int> rm = si_ + L::rm, lrow = si_ + L::lrow, clk = si_ + L::clk, cel = si_ + L::cel;
  const Lp<R> st = sm + P->dd.st, rbar = sm + P->dd.rbar, dbar = sm + P->dd.dbar;
  const Lp<unsigned long long> mask = (Lp<unsigned long long>)(sm + P->dd.mask);
  const int iters4 = P->dd.iters4, sw = P->dd.state_words, subs = P->substeps;

  // ---------------------------------------------------------------- lane constants and state
  LinkLane lk{0, -1};
  ColLane cl{0};
  {
    lane_tables<NC>(&P->m, lane, lk, cl, la, lcm, ccm);
    for (int k = lane; k < 13 * na; k += 64) {
      st[k] = R(gp(P->root_state)[(long long)abase * 13 + k]);
      rbar[k] = R(gp(P->root_adj)[(long long)abase * 13 + k]);
    }
    for (int k = lane; k < 2 * nd; k += 64) {
      st[13 * na + k] = R(gp(P->dof_state)[(long long)dbase * 2 + k]);
      dbar[k] = R(gp(P->dof_adj)[(long long)dbase * 2 + k]);
    }
    if (P->mid_root)  // substep start states handed over by the forward step
      for (int s = 1; s < subs; ++s) {
        const auto mr = gp(P->mid_root) + (long long)(s - 1) * P->mid_block + (long long)abase * 13;
        const auto md = gp(P->mid_dof) + (long long)(s - 1) * P->mid_block + (long long)dbase * 2;
        for (int k = lane; k < 13 * na; k += 64) st[s * sw + k] = mr[k];
        for (int k = lane; k < 2 * nd; k += 64) st[s * sw + 13 * na + k] = md[k];
      }
    // (entries of the vectors past the model's columns stay zero)
    for (int k = lane; k < L::org - L::dv; k += 64) dv[k] = R(0);
    for (int k = lane; k < L::g_words; k += 64) sm[L::G + k] = R(0);
    wsync();
    if (lane < 3) org[lane] = st[lane];
    wsync();
  }
  // velocities of the links and their velocity-product accelerations
  auto velocities = [&]() {
    const int cm0 = lcm[lc], cm1 = 16 + lc < NC ? lcm[min(16 + lc, NC - 1)] : 0;
    path_sum<NC, true>(S, nu, V, cm0, cm1, lane);
    if (lane < NC) {
      // joint column: (V x s) qd; a free root's columns: its own term v x w on the linear part, once
      SV c{zero3(), zero3()};
      if (cl.joint()) c = mul6(crm(ld6(V + 6 * cl.link()), ld6(S + 6 * lane)), nu[lane]);
      else if (cl.root0()) c.v = cross(ld3<R>(nu + lane), ld3<R>(nu + lane + 3));
      st6(X + 6 * lane, c);
    }
    wsync();
    path_sum<NC, false>(X, X, Acc, cm0, cm1, lane);
  };
  R act_bar = R(0);  // column lane: adjoint of the joint's actuation
  bool ok = true;
  const R h = R(P->h), mu = R(P->mu);

  // the substeps before the last are recomputed for their end states (unless handed over), then every substep from the
  // last to the first is recomputed and reversed
  for (int job = P->mid_root ? subs - 1 : 0; job < 2 * subs - 1; ++job) {
    const bool reverse = job >= subs - 1;
    const int sub_i = reverse ? 2 * subs - 2 - job : job;
    const Lp<R> sin = st + sub_i * sw;
    ADJ_PHASE(0);
    // ---------------------------------------------------- controls, generalized velocity
    if (cl.joint()) {
      qj[cl.dof()] = sin[13 * na + 2 * cl.dof()];
      nu[lane] = sin[13 * na + 2 * cl.dof() + 1];
    }
    for (int k = lane; k < na; k += 64) {
      const auto ai = gp(P->m.ai) + k * AI_COLS;
      if (!ai[AI_FIXED])
        for (int q = 0; q < 6; ++q) nu[ai[AI_COL] + q] = sin[13 * k + 7 + q];
    }
    wsync();
    R tau = R(0), arm = R(0), kp = R(0), kd = R(0);
    if (cl.joint()) {
      const auto lf = gp(P->m.lf) + cl.link() * LF_COLS;
      const int d = dbase + cl.dof();
      const R pt = P->pos_tgt ? R(gp(P->pos_tgt)[d]) : R(0);
      const R vt = P->vel_tgt ? R(gp(P->vel_tgt)[d]) : R(0);
      kp = R(lf[LF_KP]);
      kd = R(lf[LF_KD]);
      tau = R(gp(P->act)[d]) + kp * (pt - qj[cl.dof()] - h * nu[lane]) + kd * (vt - nu[lane]);
      arm = finite_armature(R(lf[LF_ARM]) + h * kd + h * h * kp);
    }
    // ---------------------------------------------------- poses, axes, velocities, velocity-product accelerations
    const auto lfl = gp(P->m.lf) + (lk.is() ? lane : 0) * LF_COLS;
    {
      R Q[4];
      V3<R> o;
      poses<NC>(lfl, lk, P->m.n_jump, sin, qj, pose, S, org, nv, lane, Q, o);
      velocities();
      // every link's spatial inertia [m, m c, J] and the force it needs, about the reference point
      R w16[16];
#pragma unroll
      for (int q = 0; q < 16; ++q) w16[q] = R(0);
      if (lk.is()) {
        const Body b = link_body(lfl, Q, o);
        b.spatial(w16);
        SV acc = ld6(Acc + 6 * lane);
        acc.v = sub(acc.v, mk(R(P->gx), R(P->gy), R(P->gz)));
        const SV vel = ld6(V + 6 * lane);
        const SV f = add6(b.mul6(acc), crf(vel, b.mul6(vel)));
        w16[10] = f.w.x; w16[11] = f.w.y; w16[12] = f.w.z; w16[13] = f.v.x; w16[14] = f.v.y; w16[15] = f.v.z;
      }
      if (lane < NC) {
#pragma unroll
        for (int q = 0; q < 16; ++q) X[kDenseXStride * lane + q] = w16[q];
      }
      wsync();
    }
    ADJ_PHASE(8);
    // ---------------------------------------------------- subtree sums, mass matrix, factor
    subtree_sum<NC>(X, la, lane, X, la, 0);
    if (lane < NC) {
      const Lp<R> Y = X + kDenseXStride * cl.link();
      const SV s = ld6(S + 6 * lane);  // zero past the model's columns
      vs[lane] = tau - dot6(s, SV{mk(R(Y[10]), R(Y[11]), R(Y[12])), mk(R(Y[13]), R(Y[14]), R(Y[15]))});
      st6(Fm + 6 * lane, comp_mul(Y, s));
    }
    wsync();
    mass_matrix<NC>(Fm, S, ccm, X, lane);
    if (cl.joint()) X[lane * (lane + 1) / 2 + lane] += arm;
    R ca, cb;  // lane n: the coefficients of the stored column pair in column n of G
    {
      const Lp<R> strip = X + NC * (NC + 1) / 2;
      strip[lane] = R(lane == 31);
      wsync();
      R a[NC];
      const Lp<R> rp = lane < nv ? X + lane * (lane + 1) / 2 : lane == nv ? vs : strip + (lane < 32 ? 32 : 63 - lane);
#pragma unroll
      for (int j = 0; j < NC; ++j) a[j] = rp[j];
      wsync();
      const Lp<d2> u2 = (Lp<d2>)rowf;
      Factor f;
      f.x1 = a[0];
      f.x2 = a[1];
      f.p1 = f.p2 = R(0);
      pivot_pair(f, 0);
      int k = 0;
      if (NC == 32) {
        factor_columns<32>(a, f, k, nv, 23, u2, G2, lane);
        factor_columns<24>(a, f, k, nv, 15, u2, G2, lane);
      } else if (NC == 28) {
        factor_columns<28>(a, f, k, nv, 21, u2, G2, lane);
        factor_columns<22>(a, f, k, nv, 15, u2, G2, lane);
      }
      factor_columns<16>(a, f, k, nv, 7, u2, G2, lane);
      factor_columns<8>(a, f, k, nv, 1, u2, G2, lane);
      R qdd = -f.x1;
      if (nv & 1) {
        store_pair(f, k, u2, G2, lane);
        qdd = fma_(f.x1, lane_read(f.x1, nv) * rcp_newton(lane_read(f.x1, nv - 1)), -f.x2);
      }
      const int i = lane - 32;
      if (i >= 0 && i < nv) {
        qdda[i] = qdd;
        vs[i] = nu[i] + h * qdd;
      }
      const bool odd = lane & 1;
      const R p = dpp_move<kQuadEven>(f.p1), s1 = rsqrt_newton(p);
      const R t = f.p1 * (s1 * s1), s2 = rsqrt_newton(fma_(-f.p1, t, f.p2));
      ca = lane >= nv ? R(0) : odd ? -t * s2 : s1;
      cb = lane >= nv || !odd ? R(0) : s2;
      if (lane < NC) co[lane] = d2{ca, cb};
      wsync();
    }
    // (the right-hand side in vs past the columns is zero: their axes are)
    // y = G x, x in u[0 .. 16 CT) (y of a column lane; zero past the columns)
    auto times_G = [&]() {
      if (lane < 16 * CT) {
        const R un = u[lane], pr = ca * un, next = dpp_move<kQuadOdd>(pr);
        u[32 + lane] = lane & 1 ? cb * un : pr + next;
      }
      wsync();
      const int i = min(lane, NC - 1);
      R acc[2] = {R(0), R(0)};
      const Lp<d2> uw = (Lp<d2>)u + 16;
#pragma unroll
      for (int m = 0; m < NC / 2; ++m) {
        const d2 e = G2[m * (m + 1) + min(i, 2 * m + 1)], w = uw[m];
        const R x = fma_(R(e.y), R(w.y), R(e.x) * R(w.x));
        acc[m & 1] += i <= 2 * m + 1 ? x : R(0);
      }
      wsync();
      return lane < nv ? acc[0] + acc[1] : R(0);
    };
    ADJ_PHASE(0);
    // ---------------------------------------------------- link velocities under v*, limits, narrow phase
    path_sum<NC, true>(S, vs, Vs, lcm[lc], 16 + lc < NC ? lcm[min(16 + lc, NC - 1)] : 0, lane);
    const R beta = R(P->beta);
    int nlim, n_contacts = 0;
    {
      int alo = 0, ahi = 0;
      R glo = R(0), ghi = R(0);
      if (cl.joint()) {
        const auto lf = gp(P->m.lf) + cl.link() * LF_COLS;
        const R lo = lf[LF_LO], hi = lf[LF_HI], ml = lf[LF_ML], v = vs[lane], q = qj[cl.dof()];
        if (isfinite(lo)) {
          glo = q - lo;
          alo = min_(glo, glo + h * v) < ml;
        }
        if (isfinite(hi)) {
          ghi = hi - q;
          ahi = min_(ghi, ghi - h * v) < ml;
        }
      }
      const unsigned long long mlo = __ballot(alo), mhi = __ballot(ahi);
      nlim = __popcll(mlo) + __popcll(mhi);
      const int base = __popcll(mlo & lanes_below(lane)) + __popcll(mhi & lanes_below(lane));
      // kind (1, 2: lower, upper) | column << 8; the position error
      if (alo) {
        lrow[base] = 1 | lane << 8;
        lbias[base] = glo;
      }
      if (ahi) {
        lrow[base + alo] = 2 | lane << 8;
        lbias[base + alo] = ghi;
      }
    }
    for (int s0 = 0; s0 < ns; s0 += 64) {
      const int sl = s0 + lane;
      int act = 0, ka = 0, kb = -1;
      R phi = R(0);
      V3<R> nrm = mk(R(0), R(0), R(1)), x = nrm;
      if (sl < ns) {
        const auto si = gp(P->m.si) + sl * SI_COLS;
        const auto sf = gp(P->m.sf) + sl * SF_COLS;
        ka = si[SI_LINK_A];
        const R rad = sf[SF_R];
        const Lp<R> pa = pose + kDensePose * ka;
        const V3<R> xc = add(ld3<R>(pa + 4), qrot(pa, ld3<R>(sf + SF_P)));
        phi = org[2] + xc.z - rad;  // (a corner has no radius)
        if (si[SI_TYPE] == SLOT_SPHERE_BOX) {
          kb = si[SI_LINK_B];
          R Rb[9];
          const Lp<R> pb = pose + kDensePose * kb;
          quat_R(R(pb[0]), R(pb[1]), R(pb[2]), R(pb[3]), Rb);
          sphere_box(xc, (const R*)Rb, add(ld3<R>(pb + 4), mv(Rb, ld3<R>(sf + SF_BOXC))), ld3<R>(sf + SF_HALF), rad, phi, nrm,
                     (R*)nullptr);
        }
        x = sub(xc, mul(nrm, rad));
        const SV va = ld6(Vs + 6 * ka);
        V3<R> ua = add(va.v, cross(va.w, x));
        if (kb >= 0) {
          const SV vb = ld6(Vs + 6 * kb);
          ua = sub(ua, add(vb.v, cross(vb.w, x)));
        }
        act = (phi + h * min_(R(0), dot(nrm, ua))) < R(P->mc);
      }
      const unsigned long long m = __ballot(act);
      const int ci = n_contacts + __popcll(m & lanes_below(lane));
      if (act && ci < KC) {
        cphi[ci] = phi;
        st3(cn + 3 * ci, nrm);
        st3(cx + 3 * ci, x);
        clk[ci] = ka | (kb + 1) << 6 | sl << 12;
      }
      n_contacts += __popcll(m);
    }
    wsync();
    nlim = __builtin_amdgcn_readfirstlane(nlim);  // (the same in every lane, which the compiler does not see)
    n_contacts = __builtin_amdgcn_readfirstlane(n_contacts);
    const int Rn = nlim + 3 * n_contacts;
    if (Rn > P->dd.rows_cap) {
      ok = false;
      break;
    }
    ADJ_PHASE(9);
    // ---------------------------------------------------- rows, Z^T = G^T J^T
    int kind = 0, word = 0, col = 0;  // kind of the lane's row (1, 2: limits, 3, 4, 5: normal, t1, t2), links and slot, limit's column
    SV f{zero3(), zero3()};
    int ma = 0, mb = 0;
    R y = R(0), bias = R(0), bc = R(0);
    const bool own = lane < Rn;
    if (own) {
      R C;
      if (lane < nlim) {
        const int w = lrow[lane];
        col = w >> 8;
        kind = w & 3;
        C = lbias[lane];
        const SV s = ld6(S + 6 * col);
        const R sg = kind == 1 ? R(1) : R(-1);
        f = ccm[col] < 0 ? SV{zero3(), mul(s.v, sg)} : SV{mul(s.w, sg), zero3()};  // s . f = 1 (a unit axis)
        ma = 1 << col;
        y = sg * vs[col];
      } else {
        const int ci = (int)((unsigned)(lane - nlim) / 3u), k = lane - nlim - 3 * ci;
        kind = 3 + k;
        word = clk[ci];
        C = cphi[ci];
        const V3<R> nrm = ld3<R>(cn + 3 * ci), x = ld3<R>(cx + 3 * ci);
        V3<R> dd = nrm;
        if (k > 0) {
          V3<R> t1, t2;
          tangents(nrm, t1, t2);
          dd = k == 1 ? t1 : t2;
        }
        f = SV{cross(x, dd), dd};
        const int b = (word >> 6) & 63;
        ma = lcm[word & 63];
        y = dot6(f, ld6(Vs + 6 * (word & 63)));
        if (b) {
          mb = lcm[b - 1];
          y -= dot6(f, ld6(Vs + 6 * (b - 1)));
        }
      }
      if (kind <= 3) {
        bc = C >= R(0) ? R(1) / h : beta / h;
        bias = bc * C;
      }
    }
    if (lane < RC) {
      st6(rowf + 6 * lane, f);
      rm[2 * lane] = ma;
      rm[2 * lane + 1] = mb;
    }
    wsync();
    // columns of J^T for row tile rt
    auto jt_tile = [&](int rt, v4* jt) {
      const int r = 16 * rt + lc, w1 = min(4 + lg, 5);
      const int xa = rm[2 * r] >> lg, xb = rm[2 * r + 1] >> lg;
      const R f0 = rowf[6 * r + lg];
      R f1 = rowf[6 * r + w1];
      f1 = lg < 2 ? f1 : R(0);
#pragma unroll
      for (int t = 0; t < CT; ++t) {
        jt[t] = tile(S[6 * (16 * t + lc) + lg], f0, tile_zero());
        jt[t] = tile(S[6 * (16 * t + lc) + w1], f1, jt[t]);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int on = __builtin_amdgcn_sbfe(xa, 16 * t + 4 * v, 1), neg = __builtin_amdgcn_sbfe(xb, 16 * t + 4 * v, 1);
          const int hi = (__double2hiint(jt[t][v]) & (on | neg)) ^ (neg & (int)0x80000000);
          jt[t][v] = __hiloint2double(hi, __double2loint(jt[t][v]) & (on | neg));
        }
      }
    };
    // G[c][n] = sum of the two stored entries times the column's coefficients, zero below the diagonal's block
    auto g_entry = [&](int c, int n) {
      const int nn = min(n, NC - 1), m = nn >> 1;
      const d2 cf = co[nn], e = G2[m * (m + 1) + min(c, nn | 1)];
      const R x = fma_(R(e.y), R(cf.y), R(e.x) * R(cf.x));
      return c <= (nn | 1) && n < nv ? x : R(0);
    };
    v4 zt[RT][CT];
    {
      // G[c][n], n = 16 tn + lane % 16, c = 16 tc + 4 v + lane / 16: blocks (tn, tc) = (0, 0), (1, 0), (1, 1)
      R g[CT == 1 ? 1 : 3][4];
#pragma unroll
      for (int q = 0; q < (CT == 1 ? 1 : 3); ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          g[q][v] = (q == 2 ? 16 : 0) + 4 * v < NC ? g_entry((q == 2 ? 16 : 0) + 4 * v + lg, (q == 0 ? 0 : 16) + lc) : R(0);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
#pragma unroll
        for (int t = 0; t < CT; ++t) zt[rt][t] = tile_zero();
        if (16 * rt < Rn) {
          v4 jt[CT];
          jt_tile(rt, jt);
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            zt[rt][0] = tile(g[0][v], jt[0][v], zt[rt][0]);
            if (CT == 2) zt[rt][CT - 1] = tile(g[CT - 1][v], jt[0][v], zt[rt][CT - 1]);
          }
          if (CT == 2) {
#pragma unroll
            for (int v = 0; v < 4; ++v)
              if (16 + 4 * v < NC) zt[rt][CT - 1] = tile(g[CT == 2 ? 2 : 0][v], jt[CT - 1][v], zt[rt][CT - 1]);
          }
        }
      }
    }
    // x = Z^T l, l in LDS (one per row), into dst
    auto zt_times = [&](Lp<R> l, Lp<R> dst) {
      R lt[RT];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) lt[rt] = l[16 * rt + lc];
#pragma unroll
      for (int t = 0; t < CT; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          R x = zt[0][t][v] * lt[0];
#pragma unroll
          for (int rt = 1; rt < RT; ++rt) x = fma_(zt[rt][t][v], lt[rt], x);
          x = row16_sum(x);
          if (lc == 0) dst[16 * t + 4 * v + lg] = x;
        }
      wsync();
    };
    ADJ_PHASE(10);
    // ---------------------------------------------------- A = Z Z^T
    wsync();
#pragma unroll
    for (int r1 = 0; r1 < RT; ++r1)
      if (16 * r1 < Rn) {
#pragma unroll
        for (int r2 = 0; r2 <= r1; ++r2) {
          v4 a = tile_zero();
#pragma unroll
          for (int t = 0; t < CT; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v)
              if (16 * t + 4 * v < NC) a = tile(zt[r1][t][v], zt[r2][t][v], a);
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            A_[(16 * r1 + 4 * v + lg) * AS + 16 * r2 + lc] = a[v];
            if (r2 < r1) A_[(16 * r2 + lc) * AS + 16 * r1 + 4 * v + lg] = a[v];
          }
        }
      }
    wsync();
    ADJ_PHASE(1);
    // ---------------------------------------------------- projected Gauss-Seidel with its tape
    const int kk = min(lane, RC - 1);
    const bool fric = own && kind >= 4;
    const R akk = own ? A_[kk * AS + kk] : R(0);
    // 1 / A_rr; rows that cannot move, and friction rows of such a normal row, are dropped (every term of theirs is zero)
    R ia = akk >= R(kMinRowMass) ? R(1) / akk : R(0);
    {
      const R ian = __shfl(ia, fric ? lane - (kind - 3) : lane, 64);
      ia = ian == R(0) ? R(0) : ia;
    }
    R z = -(y + bias) * ia, rlam = R(0);
    R zn = clamp_low0(z);  // formed where z is and not where it is used
    R muv = mu;
    asm("" : "+v"(muv));
    if (lane < RC)
#pragma unroll 4
      for (int r = 0; r < Rn; ++r) {
        const int q = r * AS + lane;
        A_[q] = r == lane ? R(0) : -ia * A_[q];
      }
    wsync();
    const int iters = P->iters;
    for (int it = 0; it < iters; ++it) {
      const R lam0 = rlam;
      R zc = R(0);  // the lane's z when its own row was updated
      unsigned long long bit = 1;
      auto apply = [&](R cand, R a, int r, unsigned long long at) {
        zc = pick(zc, z, at);
        z = fma_(a, lane_read(cand - rlam, r), z);
      };
      // (columns past the last row are read within the workgroup's LDS and not used)
      Lp<R> acol = A_ + kk;
      R a0 = acol[0];
      for (int r = 0; r < nlim; ++r, bit <<= 1) {
        const R a = a0;
        acol += AS;
        a0 = acol[0];
        asm volatile("" ::: "memory");
        apply(zn, a, r, bit);
        zn = clamp_low0(z);
      }
      if (n_contacts > 0) {
        auto contact = [&](const R* c, int r) {
          const R m = muv * lane_read(zn, r);
          apply(zn, c[0], r, bit);
          apply(clamp_sym(z, m), c[1], r + 1, bit << 1);
          apply(clamp_sym(z, m), c[2], r + 2, bit << 2);
          zn = clamp_low0(z);
          bit <<= 3;
        };
        auto load = [&](R* c) {
          acol += 3 * AS;
          c[0] = acol[0];
          c[1] = acol[AS];
          c[2] = acol[2 * AS];
          asm volatile("" ::: "memory");
        };
        R ca3[3] = {a0, acol[AS], acol[2 * AS]}, cb3[3];
        for (int r = nlim;;) {
          load(cb3);
          contact(ca3, r);
          if ((r += 3) >= Rn) break;
          load(ca3);
          contact(cb3, r);
          if ((r += 3) >= Rn) break;
        }
      }
      // a row is updated once a sweep: its new impulse is its captured z within its bounds
      {
        const R n = clamp_low0(zc), m = mu * __shfl(n, fric ? lane - (kind - 3) : lane, 64);
        rlam = fric ? clamp_sym(zc, m) : n;
      }
      if (reverse) {
        const unsigned long long fr = __ballot(zc == rlam), up = __ballot(zc > rlam);
        if (lane < RC) tape[it * RC + lane] = rlam - lam0;
        if (lane == 0) {
          mask[2 * it] = fr;
          mask[2 * it + 1] = up;
        }
      }
    }
    if (!own) rlam = R(0);
    ADJ_PHASE(0);
    // ---------------------------------------------------- velocities after the impulses
    if (lane < RC) lamy[lane] = rlam;
    wsync();
    zt_times(lamy, u);
    {
      const R d = times_G();
      if (lane < NC) dv[lane] = d;
    }
    wsync();
    if (!reverse) {
      const Lp<R> sout = sin + sw;
      if (cl.joint()) {
        const R v = vs[lane] + dv[lane];
        sout[13 * na + 2 * cl.dof()] = qj[cl.dof()] + h * v;
        sout[13 * na + 2 * cl.dof() + 1] = v;
      }
      for (int a = lane; a < na; a += 64) {
        const auto ai = gp(P->m.ai) + a * AI_COLS;
        const Lp<R> rs = sin + 13 * a, ro = sout + 13 * a;
        if (ai[AI_FIXED]) {
          for (int k = 0; k < 7; ++k) ro[k] = rs[k];
          for (int k = 7; k < 13; ++k) ro[k] = R(0);
          continue;
        }
        R v[6];
        for (int k = 0; k < 6; ++k) v[k] = vs[ai[AI_COL] + k] + dv[ai[AI_COL] + k];
        for (int k = 0; k < 3; ++k) ro[k] = rs[k] + h * v[k];
        R dq[4], q1[4];
        const R q0[4] = {rs[3], rs[4], rs[5], rs[6]};
        dq_of(mul(mk(v[3], v[4], v[5]), h), dq);
        qmul(dq, q0, q1);
        const R inv = R(1) / sqrt_(q1[0] * q1[0] + q1[1] * q1[1] + q1[2] * q1[2] + q1[3] * q1[3]);
        for (int k = 0; k < 4; ++k) ro[3 + k] = q1[k] * inv;
        for (int k = 0; k < 6; ++k) ro[7 + k] = v[k];
      }
      wsync();
      continue;
    }

    // =========================================================== reverse of the substep
    ADJ_PHASE(7);
    // ---------------------------------------------------- integration
    R qbar = R(0);  // column lane: adjoint of the joint position
    if (cl.joint()) {
      const R pb = dbar[2 * cl.dof()];
      nub[lane] = dbar[2 * cl.dof() + 1] + h * pb;
      qbar = pb;
    }
    for (int a = lane; a < na; a += 64) {
      const auto ai = gp(P->m.ai) + a * AI_COLS;
      if (ai[AI_FIXED]) continue;
      const int c = ai[AI_COL];
      const Lp<R> rb = rbar + 13 * a;
      for (int k = 0; k < 3; ++k) nub[c + k] = rb[7 + k] + h * rb[k];
      const V3<R> th = mul(add(ld3<R>(vs + c + 3), ld3<R>(dv + c + 3)), h);
      R dq[4], q1[4];
      dq_of(th, dq);
      const R q0[4] = {sin[13 * a + 3], sin[13 * a + 4], sin[13 * a + 5], sin[13 * a + 6]};
      qmul(dq, q0, q1);
      const R n1 = sqrt_(q1[0] * q1[0] + q1[1] * q1[1] + q1[2] * q1[2] + q1[3] * q1[3]);
      R qo[4], qb1[4];
      R pr = R(0);
      for (int k = 0; k < 4; ++k) {
        qo[k] = rb[3 + k];
        pr += (q1[k] / n1) * qo[k];
      }
      for (int k = 0; k < 4; ++k) qb1[k] = (qo[k] - (q1[k] / n1) * pr) / n1;
      const R dqc[4] = {-dq[0], -dq[1], -dq[2], dq[3]};
      const R q0c[4] = {-q0[0], -q0[1], -q0[2], q0[3]};
      R q0b[4], dqb[4];
      qmul(dqc, qb1, q0b);
      qmul(qb1, q0c, dqb);
      for (int k = 0; k < 4; ++k) rb[3 + k] = q0b[k];  // (the position's adjoint passes through)
      const V3<R> thb = dq_adj(th, dqb);
      nub[c + 3] = rb[10] + h * thb.x;
      nub[c + 4] = rb[11] + h * thb.y;
      nub[c + 5] = rb[12] + h * thb.z;
    }
    wsync();
    // ---------------------------------------------------- G^T nubar, z = G G^T nubar, lambda_bar = Z G^T nubar
    {
      const int n = min(lane, NC - 1), m = n >> 1;
      R t1 = R(0), t2 = R(0);
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const d2 e = G2[m * (m + 1) + min(c, 2 * m + 1)];
        const R b = c <= 2 * m + 1 ? R(nub[c]) : R(0);
        t1 = fma_(R(e.x), b, t1);
        t2 = fma_(R(e.y), b, t2);
      }
      const R x = fma_(cb, t2, ca * t1);  // zero past the columns
      if (lane < NC) nh[lane] = lane < nv ? x : R(0);
      if (lane < 32) u[lane] = lane < nv ? x : R(0);
      wsync();
      const R zc = times_G();
      if (lane < NC) z_[lane] = zc;
      wsync();
    }
    R t = R(0);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      R x = R(0);
#pragma unroll
      for (int q = 0; q < CT; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v) x = fma_(zt[rt][q][v], nh[16 * q + 4 * v + lg], x);
      x += __shfl_xor(x, 16, 64);
      x += __shfl_xor(x, 32, 64);
      t = lg == rt ? x : t;
    }
    ADJ_PHASE(2);
    // ---------------------------------------------------- Gauss-Seidel reverse
    R ybar = R(0);
    {
      // The chain from row to row is a lane read and a multiply-add.  A row's own t, zero after its update, is not
      // read again in the sweep: lanes subtract what they had at their own update (gc) after it.
      const Lp<R> arow = A_ + kk * AS;
      for (int it = iters - 1; it >= 0; --it) {
        const unsigned long long fr_ = mask[2 * it], up_ = mask[2 * it + 1];
        auto scalar = [](unsigned long long x) {
          return (unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)x) |
                 (unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(x >> 32)) << 32;
        };
        unsigned long long fr = scalar(fr_), up = scalar(up_);
        const bool free_own = (fr >> lane) & 1;
        R gc = R(0);  // the lane's t when its own row was reversed
        if (n_contacts > 0) {
          fr <<= 64 - Rn;  // row r at the top bit
          up <<= 64 - Rn;
          // (entries before the first row are read within the workgroup's LDS and not used)
          const Lp<R> last = arow + Rn - 3;
          unsigned long long bit = 1ull << (Rn - 3);
          Lp<R> at = last;
          R ca3[3] = {at[0], at[1], at[2]}, cb3[3];
          auto load = [&](R* c) {
            at -= 3;
            c[0] = at[0];
            c[1] = at[1];
            c[2] = at[2];
            asm volatile("" ::: "memory");
          };
          auto contact = [&](const R* c, int r) {
            // a clamped friction row moves its normal's lane alone, by +-mu, a clamped normal none: no branches
            const R mn = pick(R(0), mu, bit);
#pragma unroll
            for (int k = 2; k >= 0; --k) {
              const R g = lane_read(t, r + k);
              gc = pick(gc, t, bit << k);
              const unsigned long long on = (unsigned long long)((long long)(fr << (2 - k)) >> 63);
              const int neg = ~(int)(up >> 32) << (2 - k) & (int)0x80000000;
              const R m = k > 0 ? __hiloint2double(__double2hiint(mn) ^ neg, __double2loint(mn)) : R(0);
              t = fma_(pick(m, c[k], on), g, t);
            }
            fr <<= 3;
            up <<= 3;
            bit >>= 3;
          };
          for (int r = Rn - 3;;) {
            load(cb3);
            contact(ca3, r);
            if ((r -= 3) < nlim) break;
            load(ca3);
            contact(cb3, r);
            if ((r -= 3) < nlim) break;
          }
        } else {
          fr <<= 63 - max(Rn - 1, 0);
        }
        if (nlim > 0) {
          unsigned long long bit = 1ull << (nlim - 1);
          R a0 = arow[nlim - 1];
          for (int r = nlim - 1; r >= 0; --r, bit >>= 1) {
            const R c0 = a0;
            a0 = arow[r - 1];
            asm volatile("" ::: "memory");
            const R g = lane_read(t, r);
            gc = pick(gc, t, bit);
            if ((int)(fr >> 32) < 0) t = fma_(c0, g, t);
            fr <<= 1;
          }
        }
        t -= gc;
        ybar = own && free_own ? fma_(-ia, gc, ybar) : ybar;
        if (lane < RC) tape[(iters4 + it) * RC + lane] = ybar;
      }
    }
    if (lane < RC) {
      lamy[RC + lane] = ybar;
      for (int it = iters; it < iters4; ++it) tape[it * RC + lane] = tape[(iters4 + it) * RC + lane] = R(0);
    }
    wsync();
    ADJ_PHASE(3);
    // ---------------------------------------------------- v*bar = nubar + J^T ybar, w = h G (G^T nubar + Z^T ybar)
    zt_times(lamy + RC, u);
    if (lane < 32) u[lane] = lane < nv ? h * (nh[lane] + u[lane]) : R(0);
    wsync();
    {
      const R wc = times_G();
      if (lane < NC) w_[lane] = wc;
    }
    wsync();
    {
      R x[CT][4];
#pragma unroll
      for (int q = 0; q < CT; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v) x[q][v] = R(0);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        if (16 * rt < Rn) {
          v4 jt[CT];
          jt_tile(rt, jt);
          const R yb = lamy[RC + 16 * rt + lc];
#pragma unroll
          for (int q = 0; q < CT; ++q)
#pragma unroll
            for (int v = 0; v < 4; ++v) x[q][v] = fma_(jt[q][v], yb, x[q][v]);
        }
      }
#pragma unroll
      for (int q = 0; q < CT; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const R s = row16_sum(x[q][v]);
          if (lc == 0) u[16 * q + 4 * v + lg] = s;
        }
      wsync();
      if (lane < nv) vsb[lane] = nub[lane] + u[lane];
      // limit rows' own axes do not enter J: they take no part below
      if (lane < nlim) rm[2 * lane] = rm[2 * lane + 1] = 0;
      wsync();
    }
    // ---------------------------------------------------- S = Abar + Abar^T, S Z, P, Jbar
    v4 tz[RT][CT];  // S Z (rows x columns)
    v4 pm[CT][CT];  // P, lower tiles (twice)
    R gt[CT == 1 ? 1 : 3][4];  // G[c][n], c = 16 tc + lane % 16, n = 16 tn + 4 v + lane / 16: (tc, tn) = (0, 0), (0, 1), (1, 1)
    {
      const Lp<R> Zl = X;
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int q = 0; q < CT; ++q)
#pragma unroll
          for (int v = 0; v < 4; ++v) Zl[(16 * rt + lc) * ZS + 16 * q + 4 * v + lg] = zt[rt][q][v];
      wsync();
      v4 zr[RT][CT];  // Z with rows 4 v + lane / 16
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int q = 0; q < CT; ++q)
#pragma unroll
          for (int v = 0; v < 4; ++v) zr[rt][q][v] = Zl[(16 * rt + 4 * v + lg) * ZS + 16 * q + lc];
#pragma unroll
      for (int rs = 0; rs < RT; ++rs)
#pragma unroll
        for (int q = 0; q < CT; ++q) tz[rs][q] = tile_zero();
      const Lp<R> dl = tape, yn = tape + iters4 * RC;
      // tile (rows of ra, columns of rb) of S, ra >= rb, and the sums that make its transpose
#pragma unroll
      for (int ra = 0; ra < RT; ++ra)
#pragma unroll
        for (int rb = 0; rb <= ra; ++rb) {
          if (16 * ra < Rn) {
            v4 c1 = tile_zero(), c2 = tile_zero(), d1 = tile_zero(), d2_ = tile_zero();
            for (int k = 0; k < iters4; k += 4) {
              const int i = k + lg;
              const R ya = yn[i * RC + 16 * ra + lc], yb = yn[i * RC + 16 * rb + lc];
              const R da = dl[i * RC + 16 * ra + lc], db = dl[i * RC + 16 * rb + lc];
              // before the sweep's reverse: after that of the next sweep
              const R na_ = i + 1 < iters4 ? R(yn[min(i + 1, iters4 - 1) * RC + 16 * ra + lc]) : R(0);
              const R nb_ = i + 1 < iters4 ? R(yn[min(i + 1, iters4 - 1) * RC + 16 * rb + lc]) : R(0);
              c1 = tile(ya, db, c1);
              c2 = tile(da, nb_, c2);
              d1 = tile(db, ya, d1);
              d2_ = tile(nb_, da, d2_);
              (void)yb;
              (void)na_;
            }
            // s row tile ra, r column tile rb: value (s, r) = c1 + c2 for s > r; the transposed tile (rows of rb,
            // columns of ra) holds d1 + d2 at (r, s)
            v4 lo, hi;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              const int i = 4 * v + lg;
              lo[v] = c1[v] + c2[v];
              hi[v] = d1[v] + d2_[v];
              if (ra == rb) lo[v] = i > lc ? lo[v] : i < lc ? hi[v] : R(2) * c1[v];
            }
#pragma unroll
            for (int q = 0; q < CT; ++q)
#pragma unroll
              for (int v = 0; v < 4; ++v) {
                if (ra == rb) {
                  tz[ra][q] = tile(lo[v], zr[ra][q][v], tz[ra][q]);
                } else {
                  tz[ra][q] = tile(hi[v], zr[rb][q][v], tz[ra][q]);
                  tz[rb][q] = tile(lo[v], zr[ra][q][v], tz[rb][q]);
                }
              }
          }
        }
#pragma unroll
      for (int tc = 0; tc < CT; ++tc)
#pragma unroll
        for (int tn = tc; tn < CT; ++tn)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            gt[tc + tn][v] = 16 * tn + 4 * v < NC ? g_entry(16 * tc + lc, 16 * tn + 4 * v + lg) : R(0);
      v4 qm[CT][CT];  // Z^T S Z
#pragma unroll
      for (int a = 0; a < CT; ++a)
#pragma unroll
        for (int b = 0; b < CT; ++b) {
          qm[a][b] = tile_zero();
#pragma unroll
          for (int rs = 0; rs < RT; ++rs)
#pragma unroll
            for (int v = 0; v < 4; ++v) qm[a][b] = tile(zr[rs][a][v], tz[rs][b][v], qm[a][b]);
        }
      v4 n1[CT][CT];  // (Z^T S Z) G^T
#pragma unroll
      for (int a = 0; a < CT; ++a)
#pragma unroll
        for (int tc = 0; tc < CT; ++tc) {
          n1[a][tc] = tile_zero();
#pragma unroll
          for (int b = tc; b < CT; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v)
              if (16 * b + 4 * v < NC) n1[a][tc] = tile(qm[b][a][v], gt[tc + b][v], n1[a][tc]);
        }
#pragma unroll
      for (int a = 0; a < CT; ++a)
#pragma unroll
        for (int b = 0; b <= a; ++b) {
          // dv z^T + z dv^T + qdd w^T + w qdd^T: one step
          pm[a][b] = tile(dv[NC * lg + 16 * a + lc], dv[NC * (lg ^ 1) + 16 * b + lc], tile_zero());
#pragma unroll
          for (int n = a; n < CT; ++n)
#pragma unroll
            for (int v = 0; v < 4; ++v)
              if (16 * n + 4 * v < NC) pm[a][b] = tile(gt[a + n][v], n1[n][b][v], pm[a][b]);
        }
    }
    // T = (S Z) G^T, Jbar = T + lambda z^T + ybar v*^T, signed and masked like J
    v4 jb[RT][CT];
    {
      const Lp<R> Tl = X;
      wsync();
#pragma unroll
      for (int rs = 0; rs < RT; ++rs)
#pragma unroll
        for (int q = 0; q < CT; ++q)
#pragma unroll
          for (int v = 0; v < 4; ++v) Tl[(16 * rs + 4 * v + lg) * ZS + 16 * q + lc] = tz[rs][q][v];
      wsync();
#pragma unroll
      for (int rs = 0; rs < RT; ++rs) {
        R tx[CT][4];
#pragma unroll
        for (int q = 0; q < CT; ++q)
#pragma unroll
          for (int v = 0; v < 4; ++v) tx[q][v] = Tl[(16 * rs + lc) * ZS + 16 * q + 4 * v + lg];
        const R ly = lg < 2 ? R(lamy[RC * min(lg, 1) + 16 * rs + lc]) : R(0);
#pragma unroll
        for (int tc = 0; tc < CT; ++tc) {
          jb[rs][tc] = tile(ly, lg == 0 ? R(z_[16 * tc + lc]) : R(vs[16 * tc + lc]), tile_zero());
#pragma unroll
          for (int n = tc; n < CT; ++n)
#pragma unroll
            for (int v = 0; v < 4; ++v)
              if (16 * n + 4 * v < NC) jb[rs][tc] = tile(tx[n][v], gt[tc + n][v], jb[rs][tc]);
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int r = 16 * rs + 4 * v + lg;
            const int on = __builtin_amdgcn_sbfe(rm[2 * r], 16 * tc + lc, 1), neg = __builtin_amdgcn_sbfe(rm[2 * r + 1], 16 * tc + lc, 1);
            const int hi = (__double2hiint(jb[rs][tc][v]) & (on | neg)) ^ (neg & (int)0x80000000);
            jb[rs][tc][v] = __hiloint2double(hi, __double2loint(jb[rs][tc][v]) & (on | neg));
          }
        }
      }
    }
    ADJ_PHASE(6);
    // ---------------------------------------------------- rows: axis adjoints of their columns, velocities under Jbar_r
    const Lp<R> rv = X;     // per row 6 words
    {
      wsync();
#pragma unroll
      for (int rs = 0; rs < RT; ++rs)
#pragma unroll
        for (int q = 0; q < CT; ++q)
#pragma unroll
          for (int v = 0; v < 4; ++v) X[(16 * rs + 4 * v + lg) * ZS + 16 * q + lc] = jb[rs][q][v];
      wsync();
      const int lw = min(lc, 5);
      v4 cs[CT];
#pragma unroll
      for (int q = 0; q < CT; ++q) cs[q] = tile_zero();
#pragma unroll
      for (int rs = 0; rs < RT; ++rs)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const R fr = rowf[6 * (16 * rs + 4 * v + lg) + lw];
#pragma unroll
          for (int q = 0; q < CT; ++q) cs[q] = tile(jb[rs][q][v], fr, cs[q]);
        }
      v4 vr[RT];
#pragma unroll
      for (int rs = 0; rs < RT; ++rs) vr[rs] = tile_zero();
#pragma unroll
      for (int k = 0; k < NC / 4; ++k) {
        const R s = S[6 * (4 * k + lg) + lw];
#pragma unroll
        for (int rs = 0; rs < RT; ++rs) vr[rs] = tile(X[(16 * rs + lc) * ZS + 4 * k + lg], s, vr[rs]);
      }
      wsync();
      if (lc < 6) {
#pragma unroll
        for (int rs = 0; rs < RT; ++rs)
#pragma unroll
          for (int v = 0; v < 4; ++v) rv[6 * (16 * rs + 4 * v + lg) + lc] = vr[rs][v];
#pragma unroll
        for (int q = 0; q < CT; ++q)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            if (16 * q + 4 * v < NC) sb[6 * (16 * q + 4 * v + lg) + lc] = cs[q][v];
      }
      // limit rows' bias adjoints, by column (lower, upper)
      if (lane < 32) u[lane] = u[32 + lane] = R(0);
      wsync();
      if (lane < nlim) u[(kind == 1 ? 0 : 32) + col] = (kind == 1 ? ybar : -ybar) * bc;
      // x_bar = d x w, d_bar = u of every contact row
      SV xd{zero3(), zero3()};
      if (own && kind >= 3) {
        const SV vv = ld6(rv + 6 * lane);
        const V3<R> x = ld3<R>(cx + 3 * (int)((unsigned)(lane - nlim) / 3u));
        xd = SV{cross(f.v, vv.w), add(vv.v, cross(vv.w, x))};
      }
      wsync();
      if (lane < RC) st6(rv + 6 * lane, xd);
      wsync();
    }
    // per contact (the lane of its normal row): see the general form
    {
      const Lp<R> ce = rowf;  // wrenches of bodies a, then b
      const int ce_n = (2 * n_contacts + 3) & ~3;
      SV wa{zero3(), zero3()}, wb = wa;
      const int ci = (int)((unsigned)(lane - nlim) / 3u);
      const bool normal = own && kind == 3;
      if (normal) {
        const auto sf = gp(P->m.sf) + (word >> 12) * SF_COLS;
        const R rad = sf[SF_R];
        const V3<R> n = f.v, c = add(ld3<R>(cx + 3 * ci), mul(n, rad));
        const SV r0 = ld6(rv + 6 * lane), r1 = ld6(rv + 6 * (lane + 1)), r2 = ld6(rv + 6 * (lane + 2));
        V3<R> cbar = add(add(r0.w, r1.w), r2.w);
        V3<R> nb = sub(r0.v, mul(cbar, rad));
        const R phib = ybar * bc;
        const int kb = ((word >> 6) & 63) - 1;
        if (kb < 0) {
          cbar.z += phib;
          wa = {cross(c, cbar), cbar};
        } else {
          nb = add(nb, tangents_adj(n, r1.v, r2.v));
          R Rb[9];
          const Lp<R> pb = pose + kDensePose * kb;
          quat_R(R(pb[0]), R(pb[1]), R(pb[2]), R(pb[3]), Rb);
          const V3<R> bcen = add(ld3<R>(pb + 4), mv(Rb, ld3<R>(sf + SF_BOXC)));
          R phi_, G[9];
          V3<R> n_;
          sphere_box(c, (const R*)Rb, bcen, ld3<R>(sf + SF_HALF), rad, phi_, n_, (R*)G);
          const V3<R> ub = add(mul(n, phib), mtv(G, nb));
          const V3<R> cab = add(cbar, ub);
          wa = {cross(c, cab), cab};
          wb = {sub(cross(n, nb), cross(c, ub)), mul(ub, R(-1))};
        }
      }
      wsync();
      if (normal) {
        const int a = word & 63, b = (word >> 6) & 63;
        st6(ce + 12 * ci, wa);
        st6(ce + 12 * ci + 6, wb);
        cel[2 * ci] = la[a];
        cel[2 * ci + 1] = b ? la[b - 1] : 0;
      }
      if (lane < ce_n - 2 * n_contacts) {
        st6(ce + 6 * (2 * n_contacts + lane), SV{zero3(), zero3()});
        cel[2 * n_contacts + lane] = 0;
      }
      // P into the work words
      wsync();
#pragma unroll
      for (int a = 0; a < CT; ++a)
#pragma unroll
        for (int b = 0; b <= a; ++b)
#pragma unroll
          for (int v = 0; v < 4; ++v) X[(16 * a + 4 * v + lg) * ZS + 16 * b + lc] = R(0.5) * pm[a][b][v];
      wsync();
    }
    ADJ_PHASE(4);
    Body body;  // the lane's link
    // ---------------------------------------------------- d tr(M P)/dq, weight -1
    {
      const int lw = min(lc, 5);
      auto keep = [](R x, int on) { return __hiloint2double(__double2hiint(x) & on, __double2loint(x) & on); };
      v4 y0 = tile_zero(), y1 = tile_zero(), e0 = tile_zero(), e1 = tile_zero();
      R pe0[NC / 4], pe1[NC / 4];
      {
        const int m0 = ccm[lc] >> lg, m1 = (16 + lc < NC ? ccm[min(16 + lc, NC - 1)] : 0) >> lg;
#pragma unroll
        for (int k = 0; k < NC / 4; ++k) {
          const int j = 4 * k + lg;
          const R s = S[6 * j + lw];
          // sum over the columns j at or before k on its path: P_kj s_j
          if (4 * k < 16) y0 = tile(keep(X[lc * ZS + j], __builtin_amdgcn_sbfe(m0, 4 * k, 1)), s, y0);
          if (NC > 16) y1 = tile(keep(X[(16 + lc) * ZS + j], __builtin_amdgcn_sbfe(m1, 4 * k, 1)), s, y1);
          // operands of the sum over the columns k below column j: P_kj F_k
          const int mj = ccm[j];
          pe0[k] = keep(X[j * ZS + lc], j > lc ? __builtin_amdgcn_sbfe(mj, lc, 1) : 0);
          pe1[k] = NC > 16 && 4 * k + 3 >= 16 ? keep(X[j * ZS + 16 + lc], j > 16 + lc ? __builtin_amdgcn_sbfe(mj, 16 + lc, 1) : 0) : R(0);
        }
      }
      const R pkk = lane < NC ? R(X[lane * ZS + lane]) : R(0);
      wsync();
      // velocities, accelerations, composite inertias and momenta again
      velocities();
      R I10[10];
      {
#pragma unroll
        for (int q = 0; q < 10; ++q) I10[q] = R(0);
        if (lk.is()) {
          const Lp<R> p = pose + kDensePose * lane;
          const R Q[4] = {p[0], p[1], p[2], p[3]};
          body = link_body(gp(P->m.lf) + lane * LF_COLS, Q, ld3<R>(p + 4));
          body.spatial(I10);
        }
        wsync();
        if (lane < NC) {
#pragma unroll
          for (int q = 0; q < 10; ++q) X[kDenseXStride * lane + q] = I10[q];
        }
        wsync();
        subtree_sum<NC>(X, la, lane, X, la, 0);
        const Lp<R> Y = X + kDenseXStride * cl.link();
#pragma unroll
        for (int q = 0; q < 10; ++q) I10[q] = Y[q];
        if (lane < NC) st6(Fm + 6 * lane, comp_mul(I10, ld6(S + 6 * lane)));
        wsync();
#pragma unroll
        for (int k = 0; k < NC / 4; ++k) {
          const R fm = Fm[6 * (4 * k + lg) + lw];
          e0 = tile(pe0[k], fm, e0);
          if (NC > 16 && 4 * k + 3 >= 16) e1 = tile(pe1[k], fm, e1);
        }
      }
      if (lc < 6) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          X[6 * (4 * v + lg) + lc] = y0[v];
          X[6 * NC + 6 * (4 * v + lg) + lc] = e0[v];
          if (16 + 4 * v < NC) {
            X[6 * (16 + 4 * v + lg) + lc] = y1[v];
            X[6 * NC + 6 * (16 + 4 * v + lg) + lc] = e1[v];
          }
        }
      }
      wsync();
      R w16[16];
#pragma unroll
      for (int q = 0; q < 16; ++q) w16[q] = R(0);
      if (cl.is()) {
        const SV s = ld6(S + 6 * lane), ya = ld6(X + 6 * lane), e = ld6(X + 6 * NC + 6 * lane);
        const SV Iy = comp_mul(I10, ya);
        st6(sb + 6 * lane, add6(ld6(sb + 6 * lane), mul6(add6(Iy, e), R(-2))));
        // y' = 2 y + P_kk s: -<s, I y'> per link below the column
        const SV yp = add6(mul6(ya, R(2)), mul6(s, -pkk));
        const V3<R> a = s.w, b = yp.w;
        w16[0] = R(2) * a.x * b.x; w16[1] = R(2) * a.y * b.y; w16[2] = R(2) * a.z * b.z;
        w16[3] = a.x * b.y + a.y * b.x; w16[4] = a.x * b.z + a.z * b.x; w16[5] = a.y * b.z + a.z * b.y;
        const V3<R> p = add(cross(yp.v, a), cross(s.v, b));
        w16[6] = p.x; w16[7] = p.y; w16[8] = p.z;
        const SV sw_ = mul6(s, R(w_[lane]));
        w16[9] = sw_.w.x; w16[10] = sw_.w.y; w16[11] = sw_.w.z; w16[12] = sw_.v.x; w16[13] = sw_.v.y; w16[14] = sw_.v.z;
      }
      wsync();
      if (lane < NC) {
#pragma unroll
        for (int q = 0; q < 16; ++q) X[kDenseXStride * lane + q] = w16[q];
      }
      wsync();
      // over the columns that move a link
      R b[NC / 4];
      const Lp<R> xb = X + kDenseXStride * lg + lc;
#pragma unroll
      for (int k = 0; k < NC / 4; ++k) b[k] = xb[4 * kDenseXStride * k];
      const int c0 = lcm[lc] >> lg, c1 = (16 + lc < NC ? lcm[min(16 + lc, NC - 1)] : 0) >> lg;
      v4 l0 = tile_zero(), l1 = tile_zero();
#pragma unroll
      for (int k = 0; k < NC / 4; ++k) {
        l0 = tile(bit01(c0, 4 * k), b[k], l0);
        if (NC > 16) l1 = tile(bit01(c1, 4 * k), b[k], l1);
      }
      wsync();
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        xb[4 * kDenseXStride * v] = l0[v];
        if (16 + 4 * v < NC) xb[4 * kDenseXStride * (4 + v)] = l1[v];
      }
      wsync();
    }
    ADJ_PHASE(5);
    // ---------------------------------------------------- per link: inertia adjoints, RNEA reverse (seed w)
    V3<R> cbl = zero3(), tI = zero3();
    SV Vb{zero3(), zero3()};
    {
      SV F{zero3(), zero3()}, Ab = F;
      V3<R> c_ = zero3();
      if (lk.is()) {
        const Lp<R> k = X + kDenseXStride * lane;
        const Body& b = body;
        const R q6[6] = {k[0], k[1], k[2], k[3], k[4], k[5]};
        const V3<R> c = b.c;
        c_ = c;
        const R tr = q6[0] + q6[1] + q6[2];
        const V3<R> Qc = mk(q6[0] * c.x + q6[3] * c.y + q6[4] * c.z, q6[3] * c.x + q6[1] * c.y + q6[5] * c.z,
                            q6[4] * c.x + q6[5] * c.y + q6[2] * c.z);
        cbl = mul(sub(add(ld3<R>(k + 6), mul(c, tr)), Qc), -b.m);
        // rows of I Q
        const V3<R> Qx = mk(q6[0], q6[3], q6[4]), Qy = mk(q6[3], q6[1], q6[5]), Qz = mk(q6[4], q6[5], q6[2]);
        const V3<R> ix = mk(b.I[0], b.I[3], b.I[4]), iy = mk(b.I[3], b.I[1], b.I[5]), iz = mk(b.I[4], b.I[5], b.I[2]);
        tI = mk(dot(iz, Qy) - dot(iy, Qz), dot(ix, Qz) - dot(iz, Qx), dot(iy, Qx) - dot(ix, Qy));
        const SV Wh = ld6(k + 9), vel = ld6(V + 6 * lane);
        SV acc = ld6(Acc + 6 * lane);
        acc.v = sub(acc.v, mk(R(P->gx), R(P->gy), R(P->gz)));
        const SV IV = b.mul6(vel);
        F = mul6(add6(b.mul6(acc), crf(vel, IV)), R(-1));
        Ab = mul6(b.mul6(Wh), R(-1));
        bil_neg(b, Wh, acc, cbl, tI);
        const SV Y = mul6(crm(vel, Wh), R(-1));
        bil_neg(b, Y, vel, cbl, tI);
        const SV cw = crf(Wh, IV), IY = b.mul6(Y);
        Vb = SV{sub(cw.w, IY.w), sub(cw.v, IY.v)};
      }
      // sums of F and Abar over the links below
      wsync();
      if (lane < NC) {
        const Lp<R> k = X + kDenseXStride * lane;
        st6(k, F);
        st6(k + 6, Ab);
      }
      wsync();
      subtree_sum<NC>(X, la, lane, X, la, 0);
      SV e{zero3(), zero3()};
      SV s = e;
      R nuc = R(0), wc = R(0);
      const int c = lk.root() ? max(lk.rootcol(), 0) : lk.col();
      const bool joint = lk.is() && !lk.root();
      if (lk.is()) {
        F = ld6(X + kDenseXStride * lane);
        Ab = ld6(X + kDenseXStride * lane + 6);
        if (joint) {
          s = ld6(S + 6 * c);
          nuc = nu[c];
          wc = w_[c];
          e = mul6(crf(s, Ab), nuc);
        }
      }
      wsync();
      if (lane < NC) {
        const Lp<R> k = X + kDenseXStride * lane;
        st6(k, Vb);
        st6(k + 6, e);
      }
      wsync();
      subtree_sum<NC>(X, la, lane, X, la, 0);
      SV own_w{zero3(), zero3()};  // the link's own wrench
      if (lk.is()) {
        // Vbar over the links below, and of every joint strictly below qd crf(s, Abar)
        const SV vsum = ld6(X + kDenseXStride * lane), esum = ld6(X + kDenseXStride * lane + 6);
        Vb = add6(vsum, SV{sub(esum.w, e.w), sub(esum.v, e.v)});
        if (joint) {
          const SV vel = ld6(V + 6 * lane);
          const SV Vp = add6(vel, mul6(s, -nuc));
          SV sbar = ld6(sb + 6 * c);
          sbar = add6(sbar, add6(mul6(F, wc), add6(mul6(crf(Vp, Ab), -nuc), mul6(Vb, nuc))));
          const auto lf = gp(P->m.lf) + lane * LF_COLS;
          nui[c] = vsb[c] - (h * R(lf[LF_KP]) + R(lf[LF_KD])) * wc + dot6(Ab, crm(Vp, s)) + dot6(s, Vb);
          own_w = crf(s, sbar);
        } else if (lk.rootcol() >= 0) {
          const V3<R> v = ld3<R>(nu + c), w = ld3<R>(nu + c + 3), ww = ld3<R>(w_ + c + 3);
          const V3<R> o = ld3<R>(pose + kDensePose * lane + 4);
          cbl = add(cbl, add(cross(ww, F.v), cross(w, Vb.v)));
          const V3<R> nvv = add(cross(w, Ab.v), Vb.v);
          const V3<R> nww = add(add(cross(Ab.v, v), Vb.w), cross(Vb.v, o));
          const R d6[6] = {nvv.x, nvv.y, nvv.z, nww.x, nww.y, nww.z};
#pragma unroll
          for (int q = 0; q < 6; ++q) nui[c + q] = vsb[c + q] + d6[q];
          // the rotation columns (e, o x e): o moves with the link
          V3<R> q3 = zero3();
#pragma unroll
          for (int q = 0; q < 3; ++q) q3 = add(q3, cross(mk(R(q == 0), R(q == 1), R(q == 2)), ld3<R>(sb + 6 * (c + 3 + q) + 3)));
          cbl = add(cbl, q3);
        }
        own_w = add6(own_w, SV{add(cross(c_, cbl), tI), cbl});
      }
      wsync();
      if (lane < NC) {
        const Lp<R> k = X + kDenseXStride * lane;
        st6(k, own_w);
      }
      wsync();
    }
    ADJ_PHASE(6);
    // ---------------------------------------------------- wrenches over the links below, contacts included
    subtree_sum<NC>(X, la, lane, rowf, cel, (2 * n_contacts + 3) & ~3);
    ADJ_PHASE(7);
    // ---------------------------------------------------- adjoint of the substep's start state
    if (cl.joint()) {
      const R wc = w_[lane];
      act_bar += wc;
      qbar += u[lane] + u[32 + lane] - kp * wc + dot6(ld6(S + 6 * lane), ld6(X + kDenseXStride * cl.link()));
      dbar[2 * cl.dof()] = qbar;
      dbar[2 * cl.dof() + 1] = nui[lane];
    }
    if (lk.is() && lk.root()) {
      const int a = lk.actor();
      const Lp<R> rb = rbar + 13 * a;
      if (lk.rootcol() < 0) {
        for (int k = 0; k < 13; ++k) rb[k] = R(0);
      } else {
        const SV Wc = ld6(X + kDenseXStride * lane);
        const V3<R> p0 = ld3<R>(pose + kDensePose * lane + 4);
        const V3<R> dth = sub(Wc.w, cross(p0, Wc.v));
        const R q[4] = {sin[13 * a + 3], sin[13 * a + 4], sin[13 * a + 5], sin[13 * a + 6]};
        const R nq = sqrt_(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3]);
        const R t4[4] = {dth.x, dth.y, dth.z, R(0)};
        const R qh[4] = {q[0] / nq, q[1] / nq, q[2] / nq, q[3] / nq};
        R o4[4];
        qmul(t4, qh, o4);
        rb[0] += Wc.v.x;
        rb[1] += Wc.v.y;
        rb[2] += Wc.v.z;
        for (int k = 0; k < 4; ++k) rb[3 + k] += R(2) * o4[k] / nq;
        for (int k = 0; k < 6; ++k) rb[7 + k] = nui[lk.rootcol() + k];
      }
    }
    wsync();
  }
  ADJ_PHASE(-1);
  if (!ok && P->retry) {  // more rows than this form holds: hand the environment to the larger one
    if (lane == 0) gp(P->retry)[atomicAdd((int*)P->retry_count, 1)] = env;
    return;
  }
  for (int k = lane; k < 13 * na; k += 64) gp(P->root_adj)[(long long)abase * 13 + k] = ok ? float(rbar[k]) : 0.0f;
  for (int k = lane; k < 2 * nd; k += 64) gp(P->dof_adj)[(long long)dbase * 2 + k] = ok ? float(dbar[k]) : 0.0f;
  if (cl.joint()) gp(P->act_adj)[dbase + cl.dof()] = ok ? float(act_bar) : 0.0f;
  if (P->status && lane == 0 && (!ok || !P->status_sticky)) gp(P->status)[env] = ok ? 0 : 1;
  if (P->cycles && lane == 0)
    for (int k = 0; k < kAdjPhases; ++k) gp(P->cycles)[(long long)env * kAdjPhases + k] = g_dadj_clock[k];
}

template <int NC, int RT>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(RT == 2 ? 2 : 1))) void dense_adjoint_kernel(AdjArgs, int) {
  struct Args {
    AdjArgs a;
    int n_envs;
  };
  const auto K = (Cp<Args>)__builtin_amdgcn_kernarg_segment_ptr();
  const int n_envs = K->n_envs;
  // the environments with many rows share their CUs with the others and finish last: highest issue priority
  if (RT == 4) __builtin_amdgcn_s_setprio(3);
  for (int ei = blockIdx.x; ei < n_envs; ei += gridDim.x) {
    if (K->a.list_count && ei >= __builtin_amdgcn_readfirstlane(gp(K->a.list_count)[0])) return;
    dense_adjoint_env<NC, RT>(&K->a, ei);
    __syncthreads();  // the next entry reuses the LDS
  }
}

template <int NC, int RT>
hipError_t launch_form(const AdjArgs& a, int n_envs, int grid, hipStream_t stream) {
  hipLaunchKernelGGL((dense_adjoint_kernel<NC, RT>), dim3(grid), dim3(64), (size_t)a.dd.total * sizeof(R), stream, a, n_envs);
  return hipGetLastError();
}
const void* adjoint_of(int nc, int big) {
  return nc == 16   ? (big ? (const void*)dense_adjoint_kernel<16, 4> : (const void*)dense_adjoint_kernel<16, 2>)
         : nc == 28 ? (big ? (const void*)dense_adjoint_kernel<28, 4> : (const void*)dense_adjoint_kernel<28, 2>)
                    : (big ? (const void*)dense_adjoint_kernel<32, 4> : (const void*)dense_adjoint_kernel<32, 2>);
}

}  // namespace

hipError_t launch_dense_adjoint(const AdjArgs& a, int nc, int big, int n_envs, hipStream_t stream, int grid) {
  if (n_envs <= 0) return hipSuccess;
  grid = (grid > 0 && grid < n_envs) ? grid : n_envs;
  if (nc == 16) return big ? launch_form<16, 4>(a, n_envs, grid, stream) : launch_form<16, 2>(a, n_envs, grid, stream);
  if (nc == 28) return big ? launch_form<28, 4>(a, n_envs, grid, stream) : launch_form<28, 2>(a, n_envs, grid, stream);
  return big ? launch_form<32, 4>(a, n_envs, grid, stream) : launch_form<32, 2>(a, n_envs, grid, stream);
}

hipError_t set_dense_adjoint_lds_limit(int nc, int big, size_t bytes) {
  return hipFuncSetAttribute(adjoint_of(nc, big), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

}  // namespace ags
