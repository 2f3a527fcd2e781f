// Resident CG family (Algorithms 2, 4 and 6, Section 2): see resident.hpp.
#include <type_traits>

#include "../../include/pbcgs.h"
#include "resident.hpp"

namespace pbcgs {

namespace {

// r = b - A x_0 for the setups: x in window w1, r to f(j, r_j).
template <class R, class F>
__device__ __forceinline__ bool res_residual(R& g, typename R::X& x, int w, F&& f) {
  g.load_x0(x, w);
  if (!g.barrier(w)) return false;
  g.product(w, [&](auto jc, D2 ax) {
    constexpr int j = decltype(jc)::value;
    f(jc, g.get(g.a.b, j) - ax);
  });
  return true;
}

// Algorithm 2: three exchanges per iteration, one of them a barrier only (p).
// Per row in registers: r, s and x ; u = M^{-1} r is formed where it is used.
// Window 0 holds p.  Measured per iteration at 128^3, streamed kernels / this
// one: 44.9 / 24.7 us.
template <int K, int ND, bool FAR, bool UNI, bool PC>
__global__ __launch_bounds__(kResT) void k_res_cg(ResOpT<ND> op, ResArgs a) {
  using R = Res<K, ND, FAR, UNI, PC, true>;
  constexpr int KP = R::KP;
  extern __shared__ __align__(16) double sm[];
  __shared__ typename R::Shared sh;
  R g(op, a, sh, sm, xcd_index());
  constexpr int P = 0, T = 1;

  D2 r[KP], s[KP];
  typename R::X x;
  State st = g.start();
  auto pre = [&](int j, D2 v) -> D2 {
    if constexpr (PC) return g.precond(j, v);
    else return v;
  };

  double g2[2];
  {
    typename R::template Tree<2> tr(sh);
    if (!res_residual(g, x, T, [&](auto jc, D2 v) {
          constexpr int j = decltype(jc)::value;
          r[j] = v;
          const D2 u = pre(j, v);
          g.put(P, j, u);
          double d[2] = {v.x * v.x + v.y * v.y, v.x * u.x + v.y * u.y};
          tr.template add<j>(d);
        }))
      return;
    if (!g.template exchange<2>(tr.top, g2, P)) return;
  }
  {
    st.relres = 1.0;
    if (a.hist && leader()) a.hist[0] = 1.0;
    const double rho0 = sqrt(g2[0]);
    st.rho0 = rho0;
    st.gamma = g2[1];
    if (!finite(rho0) || !finite(g2[1])) st.status = DS_NONFINITE;
    else if (rho0 == 0.0) { st.status = DS_SUCCESS; st.relres = 0.0; }
    uniform(st);
  }
  for (int64_t i = 0; st.status == DS_RUNNING && i < a.maxit; ++i) {
    {  // s = A p ; alpha
      typename R::template Tree<1> tr(sh);
      g.product(P, [&](auto jc, D2 v) {
        constexpr int j = decltype(jc)::value;
        s[j] = v;
        const D2 p = g.own(P, j);
        double d[1] = {v.x * p.x + v.y * p.y};
        tr.template add<j>(d);
      });
      double g1[1];
      if (!g.template exchange<1>(tr.top, g1, -1)) return;
      fin_cg_alpha(st, g1[0]);
      uniform(st);
      if (st.status != DS_RUNNING) break;
    }
    {  // x, r, u ; stop test, beta
      const double alpha = st.alpha;
      typename R::template Tree<2> tr(sh);
      each_pair<KP>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        g.set_x(x, j, g.get_x(x, j) + alpha * g.own(P, j));
        r[j] = r[j] - alpha * s[j];
        const D2 u = pre(j, r[j]);
        double d[2] = {r[j].x * u.x + r[j].y * u.y, r[j].x * r[j].x + r[j].y * r[j].y};
        tr.template add<j>(d);
      });
      if (!g.template exchange<2>(tr.top, g2, -1)) return;
      fin_cg_beta(st, a.hist, g2);
      uniform(st);
      if (st.status != DS_RUNNING) break;
    }
    const double beta = st.beta;
    g.next(P);
#pragma unroll
    for (int j = 0; j < KP; ++j) g.put(P, j, pre(j, r[j]) + beta * g.own(P, j));
    if (!g.barrier(P)) return;
  }
  g.finish(x, st);
}

// Algorithm 4: two exchanges per iteration, one of them a barrier only (u).
// Per row in registers: r, p, s, w and x.  Window 0 holds u.  At 128^3: 46.2 /
// 20.2 us.
template <int K, int ND, bool FAR, bool UNI, bool PC>
__global__ __launch_bounds__(kResT) void k_res_cgcg(ResOpT<ND> op, ResArgs a) {
  using R = Res<K, ND, FAR, UNI, PC, true>;
  constexpr int KP = R::KP;
  extern __shared__ __align__(16) double sm[];
  __shared__ typename R::Shared sh;
  R g(op, a, sh, sm, xcd_index());
  constexpr int U = 0, T = 1;

  D2 r[KP], p[KP], s[KP], w[KP];
  typename R::X x;
  State st = g.start();
  auto pre = [&](int j, D2 v) -> D2 {
    if constexpr (PC) return g.precond(j, v);
    else return v;
  };
  if (!res_residual(g, x, T, [&](auto jc, D2 v) {
        constexpr int j = decltype(jc)::value;
        const D2 zero = {0.0, 0.0};
        r[j] = v;
        p[j] = zero;
        s[j] = zero;
        g.put(U, j, pre(j, v));
      }))
    return;
  if (!g.barrier(U)) return;
  double g3[3];
  auto wsum = [&]() -> bool {  // w = A u with its three sums
    typename R::template Tree<3> tr(sh);
    g.product(U, [&](auto jc, D2 v) {
      constexpr int j = decltype(jc)::value;
      w[j] = v;
      const D2 u = g.own(U, j);
      double d[3] = {r[j].x * u.x + r[j].y * u.y, v.x * u.x + v.y * u.y, r[j].x * r[j].x + r[j].y * r[j].y};
      tr.template add<j>(d);
    });
    return g.template exchange<3>(tr.top, g3, -1);
  };
  if (!wsum()) return;
  int64_t i = 0;
  for (; i < a.maxit; ++i) {
    if (i == 0) fin_cgs_first(st, a.hist, g3);
    else fin_cgs_next(st, a.hist, g3);
    uniform(st);
    if (st.status != DS_RUNNING) break;
    st.iters += 1;  // the x update below
    const double alpha = st.alpha, beta = st.beta;
    g.next(U);
#pragma unroll
    for (int j = 0; j < KP; ++j) {
      p[j] = g.own(U, j) + beta * p[j];
      s[j] = w[j] + beta * s[j];
      g.set_x(x, j, g.get_x(x, j) + alpha * p[j]);
      r[j] = r[j] - alpha * s[j];
      g.put(U, j, pre(j, r[j]));
    }
    if (!g.barrier(U)) return;
    if (!wsum()) return;
  }
  if (st.status == DS_RUNNING && i == a.maxit) {
    if (i == 0) fin_cgs_first(st, a.hist, g3);
    else fin_cgs_next(st, a.hist, g3);
  }
  g.finish(x, st);
}

// Algorithm 6: one exchange per iteration; the gathered m = M^{-1} w (w
// without a preconditioner) alternates between the windows.  Per row in
// registers: r, p, s, z and x, with Jacobi also w, q and u.  At 128^3: 42.5 /
// 17.2 us.
template <int K, int ND, bool FAR, bool UNI, bool PC>
__global__ __launch_bounds__(kResT) void k_res_pcg(ResOpT<ND> op, ResArgs a) {
  using R = Res<K, ND, FAR, UNI, PC, true>;
  constexpr int KP = R::KP;
  extern __shared__ __align__(16) double sm[];
  __shared__ typename R::Shared sh;
  R g(op, a, sh, sm, xcd_index());

  D2 r[KP], p[KP], s[KP], z[KP];
  D2 w[PC ? KP : 1], q[PC ? KP : 1], u[PC ? KP : 1];
  typename R::X x;
  State st = g.start();
  // u_0 through window 1, then m_0 in window 0
  if (!res_residual(g, x, 0, [&](auto jc, D2 v) {
        constexpr int j = decltype(jc)::value;
        const D2 zero = {0.0, 0.0};
        r[j] = v;
        p[j] = zero;
        s[j] = zero;
        z[j] = zero;
        if constexpr (PC) {
          q[j] = zero;
          u[j] = g.precond(j, v);
          g.put(1, j, u[j]);
        } else {
          g.put(1, j, v);
        }
      }))
    return;
  if (!g.barrier(1)) return;
  double g3[3];
  {
    g.next(0);
    typename R::template Tree<3> tr(sh);
    g.product(1, [&](auto jc, D2 v) {
      constexpr int j = decltype(jc)::value;
      D2 uj;
      if constexpr (PC) {
        uj = u[j];
        w[j] = v;
        g.put(0, j, g.precond(j, v));
      } else {
        uj = r[j];
        g.put(0, j, v);
      }
      double d[3] = {r[j].x * uj.x + r[j].y * uj.y, v.x * uj.x + v.y * uj.y, r[j].x * r[j].x + r[j].y * r[j].y};
      tr.template add<j>(d);
    });
    if (!g.template exchange<3>(tr.top, g3, 0)) return;
  }
  int64_t i = 0;
  for (; i < a.maxit; ++i) {
    if (i == 0) fin_cgs_first(st, a.hist, g3);
    else fin_cgs_next(st, a.hist, g3);
    uniform(st);
    if (st.status != DS_RUNNING) break;
    st.iters += 1;  // the x update below
    const double alpha = st.alpha, beta = st.beta;
    const int cur = (int)(i & 1), nxt = cur ^ 1;
    g.next(nxt);
    typename R::template Tree<3> tr(sh);
    g.product(cur, [&](auto jc, D2 nv) {
      constexpr int j = decltype(jc)::value;
      const D2 m = g.own(cur, j);
      D2 wj, uj;
      if constexpr (PC) wj = w[j];
      else wj = m;
      z[j] = nv + beta * z[j];
      s[j] = wj + beta * s[j];
      if constexpr (PC) {
        q[j] = m + beta * q[j];
        p[j] = u[j] + beta * p[j];
      } else {
        p[j] = r[j] + beta * p[j];
      }
      g.set_x(x, j, g.get_x(x, j) + alpha * p[j]);
      r[j] = r[j] - alpha * s[j];
      const D2 wn = wj - alpha * z[j];
      if constexpr (PC) {
        u[j] = u[j] - alpha * q[j];
        uj = u[j];
        w[j] = wn;
        g.put(nxt, j, g.precond(j, wn));
      } else {
        uj = r[j];
        g.put(nxt, j, wn);
      }
      double d[3] = {r[j].x * uj.x + r[j].y * uj.y, wn.x * uj.x + wn.y * uj.y, r[j].x * r[j].x + r[j].y * r[j].y};
      tr.template add<j>(d);
    });
    if (!g.template exchange<3>(tr.top, g3, nxt)) return;
  }
  if (st.status == DS_RUNNING && i == a.maxit) {
    if (i == 0) fin_cgs_first(st, a.hist, g3);
    else fin_cgs_next(st, a.hist, g3);
  }
  g.finish(x, st);
}

}  // namespace

hipError_t res_launch_cg(const ResPlan& p, const ResOp& op, const ResJob& j, hipStream_t s) {
  if (j.variant == PBCGS_PIPE_CG)
    return res_dispatch<false>(p, op, j, [&](auto k, auto nd, auto far, auto uni, auto pc) -> hipError_t {
      constexpr int K = decltype(k)::value, ND = decltype(nd)::value;
      constexpr bool F = decltype(far)::value, U = decltype(uni)::value, C = decltype(pc)::value;
      return res_go<ND>(&k_res_pcg<K, ND, F, U, C>, K, p, op, j, s);
    });
  return res_dispatch<true>(p, op, j, [&](auto k, auto nd, auto far, auto uni, auto pc) -> hipError_t {
    constexpr int K = decltype(k)::value, ND = decltype(nd)::value;
    constexpr bool F = decltype(far)::value, U = decltype(uni)::value, C = decltype(pc)::value;
    if (j.variant == PBCGS_CG) return res_go<ND>(&k_res_cg<K, ND, F, U, C>, K, p, op, j, s);
    return res_go<ND>(&k_res_cgcg<K, ND, F, U, C>, K, p, op, j, s);
  });
}

}  // namespace pbcgs
