// Resident BiCGStab (Algorithms 7 and 10): see resident.hpp.
#include <type_traits>

#include "resident.hpp"

namespace pbcgs {

namespace {

// Five exchanges per iteration, two of them barriers only (q^ and p^ have to
// reach the other workgroups before their products).  Per row in registers:
// r0, r, s, y and x, with Jacobi also p and q.  Window 0 holds p^ (p), window
// 1 q^ (q).  Bound by its five exchanges; measured per iteration, streamed
// kernels / this one: 41^3 26.8 / 13.8 us, 64^3 27.7 / 16.4, 128^3 80.4 / 40.7.
template <int K, int ND, bool FAR, bool UNI, bool PC>
__device__ __forceinline__ void res_bicg_solve(const ResOpT<ND>& op, const ResArgs& a, int wg) {
  using R = Res<K, ND, FAR, UNI, PC, true>;
  constexpr int KP = R::KP;
  extern __shared__ __align__(16) double sm[];
  __shared__ typename R::Shared sh;
  R g(op, a, sh, sm, wg);
  constexpr int P = 0, Q = 1;

  D2 r0[KP], r[KP], s[KP], y[KP];
  D2 p[PC ? KP : 1], q[PC ? KP : 1];
  typename R::X x;
  State st = g.start();

  // r_0 = p_0 = b - A x_0
  g.load_x0(x, Q);
  if (!g.barrier(Q)) return;
  double g0[1];
  {
    typename R::template Tree<1> tr(sh);
    g.product(Q, [&](auto jc, D2 ax) {
      constexpr int j = decltype(jc)::value;
      const D2 v = g.get(a.b, j) - ax;
      r0[j] = v;
      r[j] = v;
      if constexpr (PC) {
        p[j] = v;
        g.put(P, j, g.precond(j, v));
      } else {
        g.put(P, j, v);
      }
      double d[1] = {v.x * v.x + v.y * v.y};
      tr.template add<j>(d);
    });
    if (!g.template exchange<1>(tr.top, g0, P)) return;
  }
  fin_setup_gamma(st, a.hist, g0[0]);
  uniform(st);
  for (int64_t i = 0; st.status == DS_RUNNING && i < a.maxit; ++i) {
    {  // s = A p^ ; alpha
      typename R::template Tree<1> tr(sh);
      g.product(P, [&](auto jc, D2 v) {
        constexpr int j = decltype(jc)::value;
        s[j] = v;
        double d[1] = {r0[j].x * v.x + r0[j].y * v.y};
        tr.template add<j>(d);
      });
      double g1[1];
      if (!g.template exchange<1>(tr.top, g1, -1)) return;
      fin_bicg_alpha(st, g1[0]);
      uniform(st);
      if (st.status != DS_RUNNING) break;
    }
    const double alpha = st.alpha;
    double g2[2];
    {  // q = r - alpha s ; y = A q^ ; omega
      g.next(Q);
#pragma unroll
      for (int j = 0; j < KP; ++j) {
        const D2 v = r[j] - alpha * s[j];
        if constexpr (PC) {
          q[j] = v;
          g.put(Q, j, g.precond(j, v));
        } else {
          g.put(Q, j, v);
        }
      }
      if (!g.barrier(Q)) return;
      typename R::template Tree<2> tr(sh);
      g.product(Q, [&](auto jc, D2 v) {
        constexpr int j = decltype(jc)::value;
        D2 qj;
        if constexpr (PC) qj = q[j];
        else qj = g.own(Q, j);
        y[j] = v;
        double d[2] = {qj.x * v.x + qj.y * v.y, v.x * v.x + v.y * v.y};
        tr.template add<j>(d);
      });
      if (!g.template exchange<2>(tr.top, g2, -1)) return;
    }
    const bool yz = uniform((int32_t)fin_omega(st, a.hist, g2[0], g2[1])) != 0;
    uniform(st);
    if (yz) {
#pragma unroll
      for (int j = 0; j < KP; ++j) g.set_x(x, j, g.get_x(x, j) + alpha * g.own(P, j));
      break;
    }
    if (st.status != DS_RUNNING) break;
    const double omega = st.omega;
    {  // x, r ; stop test, beta
      typename R::template Tree<2> tr(sh);
      each_pair<KP>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        const D2 qh = g.own(Q, j);
        D2 qj;
        if constexpr (PC) qj = q[j];
        else qj = qh;
        g.set_x(x, j, g.get_x(x, j) + alpha * g.own(P, j) + omega * qh);
        r[j] = qj - omega * y[j];
        double d[2] = {r0[j].x * r[j].x + r0[j].y * r[j].y, r[j].x * r[j].x + r[j].y * r[j].y};
        tr.template add<j>(d);
      });
      if (!g.template exchange<2>(tr.top, g2, -1)) return;
    }
    fin_bicg_beta(st, a.hist, g2[0], g2[1]);
    uniform(st);
    if (st.status != DS_RUNNING) break;
    const double beta = st.beta;
    g.next(P);
#pragma unroll
    for (int j = 0; j < KP; ++j) {
      D2 po;
      if constexpr (PC) po = p[j];
      else po = g.own(P, j);
      const D2 pn = r[j] + beta * (po - omega * s[j]);
      if constexpr (PC) {
        p[j] = pn;
        g.put(P, j, g.precond(j, pn));
      } else {
        g.put(P, j, pn);
      }
    }
    if (!g.barrier(P)) return;
  }
  g.finish(x, st);
}

template <int K, int ND, bool FAR, bool UNI, bool PC>
__global__ __launch_bounds__(kResT) void k_res_bicg(ResOpT<ND> op, ResArgs a) {
  res_bicg_solve<K, ND, FAR, UNI, PC>(op, a, xcd_index());
}

// Workgroup i of the launch (XCD-contiguous) belongs to system map[i].x and is
// its workgroup map[i].y.
template <int ND>
__global__ __launch_bounds__(kResT) void kb_res_bicg(const ResSys<ND>* __restrict__ sys, const int2* __restrict__ map) {
  const int i = xcd_index();
  const int k = uniform(map[i].x);
  const ResOpT<ND> op = sys[k].op;
  const ResArgs a = sys[k].a;
  res_bicg_solve<kResBatchK, ND, false, true, false>(op, a, uniform(map[i].y));
}

}  // namespace

hipError_t res_launch_bicg(const ResPlan& p, const ResOp& op, const ResJob& j, hipStream_t s) {
  return res_dispatch<false>(p, op, j, [&](auto k, auto nd, auto far, auto uni, auto pc) -> hipError_t {
    constexpr int K = decltype(k)::value, ND = decltype(nd)::value;
    return res_go<ND>(&k_res_bicg<K, ND, decltype(far)::value, decltype(uni)::value, decltype(pc)::value>, K, p, op, j,
                      s);
  });
}

hipError_t res_launch_batch_bicg(int nd, const void* sys, const int2* map, int workgroups, size_t lds, bool coop,
                                 hipStream_t s) {
  if (nd <= 5) return res_go_batch<5>(&kb_res_bicg<5>, sys, map, workgroups, lds, coop, s);
  return res_go_batch<7>(&kb_res_bicg<7>, sys, map, workgroups, lds, coop, s);
}

}  // namespace pbcgs
