// Resident p-BiCGStab (Algorithms 9 and 11), with or without residual
// replacement (Section 4.2): see resident.hpp.
#include <type_traits>

#include "resident.hpp"

namespace pbcgs {

namespace {

__device__ __forceinline__ bool res_rr_due(const ResArgs& a, int64_t i) {
  if (a.variant != 2 || a.rr_period <= 0 || i < 0) return false;
  if ((i + 1) % a.rr_period != 0) return false;
  const int64_t before = (i + 1) / a.rr_period - 1;
  return a.rr_max < 0 || before < a.rr_max;
}

// Per row in registers: r, s, p^, t / v (one slot: t is dead when v is made), x
// and r0 (the last two in memory for K = 16), with Jacobi also w, z, r^, s^.
// Window 0 holds w^ (w), window 1 z^ (z).  Two exchanges per iteration.  Bound
// by the exchange on small systems and by the vector ALUs (about 300
// instructions a pair and phase) and the far reads on large ones; measured per
// iteration, streamed kernels / this one: 64^2 14.6 / 6.8 us, 64^3 21.6 / 11,
// 100^3 47.9 / 23, 128^3 (folded Jacobi) 76.6 / 42.
template <int K, int ND, bool FAR, bool UNI, bool PC>
__device__ __forceinline__ void res_pipe_solve(const ResOpT<ND>& op, const ResArgs& a, int wg) {
  using R = Res<K, ND, FAR, UNI, PC, false>;
  constexpr int KP = R::KP;
  extern __shared__ __align__(16) double sm[];
  __shared__ typename R::Shared sh;
  R g(op, a, sh, sm, wg);
  constexpr int W = 0, Z = 1;
  typename R::X x, r0;
  D2 r[KP], s[KP], ph[KP], tv[KP];
  D2 w[PC ? KP : 1], z[PC ? KP : 1], rh[PC ? KP : 1], sh_[PC ? KP : 1];

  State st = g.start();

  // r_0 = b - A x_0 ; r^_0 (setup)
  double g5[5];
  g.load_x0(x, W);
  r0.v = 4;
  if (!g.barrier(W)) return;
  {
    typename R::template Tree<1> tr(sh);
    g.product(W, [&](auto jc, D2 ax) {
      constexpr int j = decltype(jc)::value;
      const D2 q = g.get(a.b, j) - ax;
      g.set_x(r0, j, q);
      r[j] = q;
      if constexpr (PC) rh[j] = g.precond(j, q);
      double d[1] = {q.x * q.x + q.y * q.y};
      tr.template add<j>(d);
    });
    __syncthreads();  // every wave has read x from the window
    g.next(W);
#pragma unroll
    for (int j = 0; j < KP; ++j) {
      if constexpr (PC) g.put(W, j, rh[j]);
      else g.put(W, j, r[j]);
    }
    double tot[1];
    if (!g.template exchange<1>(tr.top, tot, W)) return;
    fin_setup_gamma(st, a.hist, tot[0]);
    uniform(st);
  }
  double g1[1] = {0.0};
  if (st.status == DS_RUNNING) {  // w_0 = A r^_0
    typename R::template Tree<1> tr(sh);
    g.product(W, [&](auto jc, D2 y) {
      constexpr int j = decltype(jc)::value;
      tv[j] = y;
      const D2 q = g.get_x(r0, j);
      double d[1] = {q.x * y.x + q.y * y.y};
      tr.template add<j>(d);
    });
    __syncthreads();
    g.next(W);
#pragma unroll
    for (int j = 0; j < KP; ++j) {
      const D2 zero = {0.0, 0.0}, wn = tv[j];
      ph[j] = zero;
      s[j] = zero;
      tv[j] = zero;
      *reinterpret_cast<D2*>(&g.win(Z)[g.li0 + 128 * j]) = zero;
      if constexpr (PC) {
        w[j] = wn;
        z[j] = zero;
        sh_[j] = zero;
        g.put(W, j, g.precond(j, wn));
      } else {
        g.put(W, j, wn);
      }
    }
    if (!g.template exchange<1>(tr.top, g1, W)) return;
  }

  int64_t i = 0;
  for (; st.status == DS_RUNNING && i < a.maxit; ++i) {
    // reduction 2 of the previous iteration (alpha_0 in the first)
    if (i == 0) fin_setup_alpha(st, g1[0]);
    else fin_pipe_b(st, a.hist, g5, a.aform);
    uniform(st);
    if (st.status != DS_RUNNING) break;
    const double alpha = st.alpha, beta = st.beta;
    double g2[2];
    {
      const double omega = st.omega;
      typename R::template Tree<2> tr(sh);
      if (__builtin_expect(uniform((int32_t)res_rr_due(a, i - 1)) != 0, 0)) {
        // after a replacement: p^, then s = A p^ and z = A s^ from their definitions
        g.next(Z);
#pragma unroll
        for (int j = 0; j < KP; ++j) {
          if constexpr (PC) ph[j] = rh[j] + beta * (ph[j] - omega * sh_[j]);
          else ph[j] = r[j] + beta * (ph[j] - omega * s[j]);
          g.put(Z, j, ph[j]);
        }
        if (!g.barrier(Z)) return;
        g.product(W, [&](auto jc, D2 y) { tv[decltype(jc)::value] = y; });  // t = A w^
        g.product(Z, [&](auto jc, D2 y) { s[decltype(jc)::value] = y; });
        __syncthreads();
        g.next(Z);
#pragma unroll
        for (int j = 0; j < KP; ++j) {
          if constexpr (PC) {
            sh_[j] = g.precond(j, s[j]);
            g.put(Z, j, sh_[j]);
          } else {
            g.put(Z, j, s[j]);
          }
        }
        if (!g.barrier(Z)) return;
        D2 zn[R::kStash ? 1 : KP];
        g.product(Z, [&](auto jc, D2 y) {
          constexpr int j = decltype(jc)::value;
          if constexpr (R::kStash) {
            g.stash(j, y);
          } else {
            zn[j] = y;
          }
          D2 wj;
          if constexpr (PC) wj = w[j];
          else wj = g.own(W, j);
          const D2 q = r[j] - alpha * s[j], yy = wj - alpha * y;
          double d[2] = {q.x * yy.x + q.y * yy.y, yy.x * yy.x + yy.y * yy.y};
          tr.template add<j>(d);
        });
        __syncthreads();
        g.next(Z);
        if constexpr (R::kStash) {
          g.unstash(Z);
        } else {
#pragma unroll
          for (int j = 0; j < KP; ++j) {
            if constexpr (PC) {
              z[j] = zn[j];
              g.put(Z, j, g.precond(j, zn[j]));
            } else {
              g.put(Z, j, zn[j]);
            }
          }
        }
      } else {
        g.next(Z);
        g.product(W, [&](auto jc, D2 tj) {
          constexpr int j = decltype(jc)::value;
          D2 wj, zo, zn;
          const D2 so = s[j], v = tv[j];
          if constexpr (PC) {
            wj = w[j];
            zo = z[j];
            const D2 wh = g.own(W, j), zho = g.own(Z, j), sho = sh_[j];
            ph[j] = rh[j] + beta * (ph[j] - omega * sho);
            sh_[j] = wh + beta * (sho - omega * zho);
          } else {
            wj = g.own(W, j);
            zo = g.own(Z, j);
            ph[j] = r[j] + beta * (ph[j] - omega * so);
          }
          s[j] = wj + beta * (so - omega * zo);
          zn = tj + beta * (zo - omega * v);
          tv[j] = tj;
          const D2 q = r[j] - alpha * s[j], y = wj - alpha * zn;
          if constexpr (PC) {
            z[j] = zn;
            g.put(Z, j, g.precond(j, zn));
          } else {
            g.put(Z, j, zn);
          }
          double d[2] = {q.x * y.x + q.y * y.y, y.x * y.x + y.y * y.y};
          tr.template add<j>(d);
        });
      }
      if (!g.template exchange<2>(tr.top, g2, Z)) return;
    }
    const bool yz = uniform((int32_t)fin_omega(st, a.hist, g2[0], g2[1])) != 0;
    uniform(st);
    if (yz) {
#pragma unroll
      for (int j = 0; j < KP; ++j) g.set_x(x, j, g.get_x(x, j) + alpha * ph[j]);
      break;
    }
    if (st.status != DS_RUNNING) break;
    const double omega = st.omega;
    typename R::template Tree<5> tr(sh);
    if (__builtin_expect(uniform((int32_t)res_rr_due(a, i)) != 0, 0)) {
      // x, then r = b - A x, r^, w = A r^, w^ from their definitions
      g.next(W);
#pragma unroll
      for (int j = 0; j < KP; ++j) {
        D2 qh;
        if constexpr (PC) qh = rh[j] - alpha * sh_[j];
        else qh = r[j] - alpha * s[j];
        const D2 xj = g.get_x(x, j) + alpha * ph[j] + omega * qh;
        g.set_x(x, j, xj);
        g.put(W, j, xj);
      }
      if (!g.barrier(W)) return;
      g.product(W, [&](auto jc, D2 ax) {
        constexpr int j = decltype(jc)::value;
        r[j] = g.get(a.b, j) - ax;
        if constexpr (PC) rh[j] = g.precond(j, r[j]);
      });
      __syncthreads();
      g.next(W);
#pragma unroll
      for (int j = 0; j < KP; ++j) {
        if constexpr (PC) g.put(W, j, rh[j]);
        else g.put(W, j, r[j]);
      }
      if (!g.barrier(W)) return;
      st.n_rr += 1;
      g.product(W, [&](auto jc, D2 y) {
        constexpr int j = decltype(jc)::value;
        tv[j] = y;  // w (t and v are dead until the next iteration's t)
        D2 zj;
        if constexpr (PC) zj = z[j];
        else zj = g.own(Z, j);
        const D2 q = g.get_x(r0, j);
        double d[5] = {q.x * r[j].x + q.y * r[j].y, q.x * y.x + q.y * y.y, q.x * s[j].x + q.y * s[j].y,
                       q.x * zj.x + q.y * zj.y, r[j].x * r[j].x + r[j].y * r[j].y};
        tr.template add<j>(d);
      });
      __syncthreads();
      g.next(W);
#pragma unroll
      for (int j = 0; j < KP; ++j) {
        if constexpr (PC) {
          w[j] = tv[j];
          g.put(W, j, g.precond(j, tv[j]));
        } else {
          g.put(W, j, tv[j]);
        }
      }
    } else {
      g.next(W);
      D2 xl[KP], r0l[KP];
      auto load = [&](auto jc) {
        xl[decltype(jc)::value] = g.get_x(x, decltype(jc)::value);
        r0l[decltype(jc)::value] = g.get_x(r0, decltype(jc)::value);
      };
      g.product(Z, load, [&](auto jc, D2 v) {
        constexpr int j = decltype(jc)::value;
        D2 wj, zj;
        if constexpr (PC) {
          wj = w[j];
          zj = z[j];
        } else {
          wj = g.own(W, j);
          zj = g.own(Z, j);
        }
        const D2 q = r[j] - alpha * s[j], y = wj - alpha * zj;
        if constexpr (PC) {
          const D2 qh = rh[j] - alpha * sh_[j];
          g.set_x(x, j, xl[j] + alpha * ph[j] + omega * qh);
          rh[j] = qh - omega * (g.own(W, j) - alpha * g.own(Z, j));
        } else {
          g.set_x(x, j, xl[j] + alpha * ph[j] + omega * q);
        }
        const D2 rn = q - omega * y;
        const D2 wn = y - omega * (tv[j] - alpha * v);
        tv[j] = v;
        r[j] = rn;
        if constexpr (PC) {
          w[j] = wn;
          g.put(W, j, g.precond(j, wn));
        } else {
          g.put(W, j, wn);
        }
        const D2 r0j = r0l[j];
        double d[5] = {r0j.x * rn.x + r0j.y * rn.y, r0j.x * wn.x + r0j.y * wn.y, r0j.x * s[j].x + r0j.y * s[j].y,
                       r0j.x * zj.x + r0j.y * zj.y, rn.x * rn.x + rn.y * rn.y};
        tr.template add<j>(d);
      });
    }
    if (!g.template exchange<5>(tr.top, g5, W)) return;
  }
  // maxit reached: the reduction left pending
  if (st.status == DS_RUNNING && i == a.maxit) {
    if (i == 0) fin_setup_alpha(st, g1[0]);
    else fin_pipe_b(st, a.hist, g5, a.aform);
  }
  g.finish(x, st);
}

template <int K, int ND, bool FAR, bool UNI, bool PC>
__global__ __launch_bounds__(kResT) void k_res_pipe(ResOpT<ND> op, ResArgs a) {
  res_pipe_solve<K, ND, FAR, UNI, PC>(op, a, xcd_index());
}

// Workgroup i of the launch (XCD-contiguous) belongs to system map[i].x and is
// its workgroup map[i].y.
template <int ND>
__global__ __launch_bounds__(kResT) void kb_res_pipe(const ResSys<ND>* __restrict__ sys, const int2* __restrict__ map) {
  const int i = xcd_index();
  const int k = uniform(map[i].x);
  const ResOpT<ND> op = sys[k].op;
  const ResArgs a = sys[k].a;
  res_pipe_solve<kResBatchK, ND, false, true, false>(op, a, uniform(map[i].y));
}

}  // namespace

hipError_t res_launch_pipe(const ResPlan& p, const ResOp& op, const ResJob& j, hipStream_t s) {
  return res_dispatch<false>(p, op, j, [&](auto k, auto nd, auto far, auto uni, auto pc) -> hipError_t {
    constexpr int K = decltype(k)::value, ND = decltype(nd)::value;
    return res_go<ND>(&k_res_pipe<K, ND, decltype(far)::value, decltype(uni)::value, decltype(pc)::value>, K, p, op, j,
                      s);
  });
}

hipError_t res_launch_batch_pipe(int nd, const void* sys, const int2* map, int workgroups, size_t lds, bool coop,
                                 hipStream_t s) {
  if (nd <= 5) return res_go_batch<5>(&kb_res_pipe<5>, sys, map, workgroups, lds, coop, s);
  return res_go_batch<7>(&kb_res_pipe<7>, sys, map, workgroups, lds, coop, s);
}

}  // namespace pbcgs
