// Resident solvers: one cooperative launch runs a whole binary64 solve, the
// Krylov vectors held in registers and LDS from the setup to the last
// iteration.  Each workgroup owns a contiguous range of rows; per product it
// writes its part of the gathered vector to global memory once, and the
// workgroups meet at one grid-wide exchange per reduction phase.
//
// Why: an iteration through memory reads and writes every vector each time
// and pays two to five kernel boundaries; systems whose vectors fit the 256
// compute units' registers and LDS (up to 2^21 rows) need neither.  Per
// iteration only the gathered vectors cross memory (write-through stores, one
// or two reads per row), so the bounds are the exchange's latency on small
// systems and the gathered vectors' traffic and the vector ALUs on large ones.
//
// Rows and sums: thread t of a workgroup holds K rows as K / 2 pairs, pair j
// of lane l in wave w at row 64 K w + 128 j + 2 l of the workgroup's 512 K
// rows.  A pair's sum is the lowest level of the balanced tree over the row
// index, the wave's DPP sums, its K / 2 blocks, the 8 waves and the
// workgroups (padded with zeros to 256) are the levels above it: the same
// tree as the kernels in kernels.hpp, so the same bits.  The recurrences are
// those kernels' expressions in the same order.
//
// Exchange: data goes out with agent-scope (sc1, write-through) stores, then
// every wave waits for its stores and the workgroup publishes its partial
// sums, each double as two 64-bit words that carry the exchange's number
// beside one half of the value.  Every workgroup polls all partial sums until
// the numbers match: that is the barrier, and the sums are there with it.
// Data and words are read with agent-scope (sc1) loads, so no cache has to be
// written back or invalidated.  An agent-scope release fence per workgroup,
// which writes back a whole L2, cost 11 us a round on 256 workgroups where
// this exchange takes 3.4 (1.9 on 64).  With XCD-contiguous workgroup indices
// most of a workgroup's neighbours share its L2; without them the exchange
// takes 4.3 us and the gathered vectors' reads at 2^21 rows 7 instead of 6.
//
// Every wait is bounded: a workgroup that polls kResSpin times without success
// sets job.err and leaves, and so do the others in turn; the caller's x is not
// touched by this kernel (its history is: the entries of the iterations done).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "method.hpp"
#include "resident.h"

namespace pbcgs {

typedef unsigned long long u64;
typedef double D2 __attribute__((ext_vector_type(2)));
typedef double D2u __attribute__((ext_vector_type(2), aligned(8)));
typedef unsigned U4 __attribute__((ext_vector_type(4)));

constexpr int kResSpin = 1 << 19;  // polls before a wait gives up (0.07 s, measured)
constexpr int kResFront = 2;       // doubles before row 0 in an exchange buffer
constexpr int kSc1 = 16;           // buffer cache policy: agent scope

template <int ND>
struct ResOpT {
  const uint32_t* mask;
  const double* va;
  int32_t n, nd, ld, nx, ny, nz;
  int32_t off[ND];   // slot's offset (0 in an empty slot)
  int32_t vd[ND];    // slot's diagonal in the layout
  double c[ND];
};

struct ResArgs {
  int32_t G, H, reach, variant, rr_period, rr_max, maxit, aform, vec_dinv;
  double tol, dinv_s;
  const double* dinv;
  const double* b;
  const double* x0;
  double* hist;
  double* vecs;
  int64_t stride;
  u64* words;
  int32_t* err;
  DevState* st;
};

// f(j) for the pairs 0 .. N - 1 with j a compile-time constant.
template <int N, int J = 0, class F>
__device__ __forceinline__ void each_pair(F&& f) {
  if constexpr (J < N) {
    f(std::integral_constant<int, J>());
    each_pair<N, J + 1>(f);
  }
}

// A value every lane holds, in scalar registers.
__device__ __forceinline__ int32_t uniform(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ double uniform(double v) {
  return __hiloint2double(uniform((int32_t)__double2hiint(v)), uniform((int32_t)__double2loint(v)));
}
__device__ __forceinline__ void uniform(State& s) {
  s.alpha = uniform(s.alpha);
  s.beta = uniform(s.beta);
  s.omega = uniform(s.omega);
  s.gamma = uniform(s.gamma);
  s.rho0 = uniform(s.rho0);
  s.relres = uniform(s.relres);
  s.status = uniform(s.status);
  s.iters = uniform(s.iters);
}

// XCD-contiguous index of a launch's workgroup: workgroup b runs on XCD b % 8.
__host__ __device__ __forceinline__ int xcd_index(int b, int G) {
  const int q = G >> 3, r = G & 7, x = b & 7;
  return x * q + (x < r ? x : r) + (b >> 3);
}
__device__ __forceinline__ int xcd_index() { return xcd_index((int)blockIdx.x, (int)gridDim.x); }

// One system of a batched launch.
template <int ND>
struct ResSys {
  ResOpT<ND> op;
  ResArgs a;
};

// What the kernels of every method share: the thread's place, the windows in
// LDS, the exchange and the product.  KP = pairs per thread, NW = waves.
// NEAR: exchanges without sums are barriers among neighbours (the methods with
// such an exchange in every iteration; elsewhere the registers matter more).
template <int K, int ND, bool FAR, bool UNI, bool PC, bool NEAR>
struct Res {
  static constexpr int KP = K / 2;
  static constexpr int CJ = KP < 2 ? KP : 2;  // pairs whose far values are in flight (bounds the registers)
  static constexpr int NWAVE = kResT / 64;

  struct Shared {
    double red[2][5][NWAVE];
    double lvl[KP > 4 ? NWAVE : 1][3][5];
    double lw[2][4][5];
    int bad;
  };

  const ResOpT<ND>& op;
  const ResArgs& a;
  Shared& sh;
  double* sm;        // two windows: rows [base - H, base + 512 K + H) of two gathered vectors
  const int wg;      // the system's workgroup
  uint32_t ix;       // exchange buffer of each window's vector (bits 0-7, 8-15), then the spare one
  int32_t n, base, row0, li0;
  int lane, wave, t;
  unsigned epoch = 0;
  bool last_near = false;  // the latest exchange was among neighbours only
  // per pair: the diagonals its rows hold (row 0 in bits 0-7, row 1 in bits
  // 8-15; two pairs to a word), and those every row of its 128-row block holds
  // (uniform; four pairs to a word)
  uint32_t mk[(KP + 1) / 2];
  uint32_t all[(KP + 3) / 4];

  __device__ __forceinline__ Res(const ResOpT<ND>& op_, const ResArgs& a_, Shared& sh_, double* sm_, int wg_)
      : op(op_), a(a_), sh(sh_), sm(sm_), wg(wg_) {
    t = threadIdx.x;
    lane = t & 63;
    wave = t >> 6;
    n = op.n;
    base = wg * (kResT * K);
    row0 = base + wave * 64 * K + 2 * lane;
    li0 = a.H + wave * 64 * K + 2 * lane;
    ix = 0u | (1u << 8) | (2u << 16);
    if (t == 0) sh.bad = 0;
#pragma unroll
    for (int j = 0; j < KP; ++j) {
      const uint32_t m0 = row_mask(row0 + 128 * j), m1 = row_mask(row0 + 128 * j + 1);
      if (j % 2 == 0) mk[j / 2] = m0 | (m1 << 8);
      else mk[j / 2] |= (m0 | (m1 << 8)) << 16;
      uint32_t u = 0;
#pragma unroll
      for (int d = 0; d < ND; ++d)
        if (__ballot(((m0 & m1) >> d) & 1u) == ~0ull) u |= 1u << d;
      if (j % 4 == 0) all[j / 4] = u;
      else all[j / 4] |= u << (8 * (j % 4));
    }
  }

  static __device__ __forceinline__ uint32_t fresh_uniform(uint32_t v) {
    v = __builtin_amdgcn_readfirstlane(v);
    asm volatile("" : "+s"(v));
    return v;
  }
  // A value the compiler must recompute from: without it the addresses and
  // mask tests of every pair are hoisted out of the iteration loop into
  // registers the vectors need.
  template <class T>
  static __device__ __forceinline__ T fresh(T v) {
    asm volatile("" : "+v"(v));
    return v;
  }

  __device__ __forceinline__ double* win(int w) const { return sm + w * (kResT * K + 2 * a.H); }
  __device__ __forceinline__ int32_t row(int j) const { return row0 + 128 * j; }

  // slots of the diagonals row `i` holds
  __device__ __forceinline__ uint32_t row_mask(int32_t i) const {
    if (i >= n) return 0;
    if (op.mask) {
      const uint32_t m = op.mask[i];  // the last diagonal sits in the last slot
      const int l = op.nd - 1;
      return (m & ((1u << l) - 1u)) | (((m >> l) & 1u) << (ND - 1));
    }
    const int32_t x = i % op.nx, yz = i / op.nx;
    if constexpr (ND == 5) {
      return (yz > 0 ? 1u : 0u) | (x > 0 ? 2u : 0u) | 4u | (x < op.nx - 1 ? 8u : 0u) | (yz < op.ny - 1 ? 16u : 0u);
    } else {
      const int32_t y = yz % op.ny, z = yz / op.ny;
      return (z > 0 ? 1u : 0u) | (y > 0 ? 2u : 0u) | (x > 0 ? 4u : 0u) | 8u | (x < op.nx - 1 ? 16u : 0u) |
             (y < op.ny - 1 ? 32u : 0u) | (z < op.nz - 1 ? 64u : 0u);
    }
  }

  // Window w's exchange buffer as a bounded buffer: rows -2 .. n + 1; accesses outside
  // read 0 and write nothing.
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(int w) const {
    const uint32_t k = __builtin_amdgcn_readfirstlane((ix >> (8 * w)) & 0xffu);
    return __builtin_amdgcn_make_buffer_rsrc(a.vecs + (int64_t)k * a.stride, 0,
                                             (n + 2 * kResFront) * 8, 0x00020000);
  }
  static __device__ __forceinline__ D2 load2(__amdgpu_buffer_rsrc_t r, int32_t row) {
    return __builtin_bit_cast(D2, __builtin_amdgcn_raw_buffer_load_b128(r, (row + kResFront) * 8, 0, kSc1));
  }

  // Pair j of window w's vector: into the window and, for the other
  // workgroups, the exchange buffer chosen by next().
  __device__ __forceinline__ void put(int w, int j, D2 v) {
    *reinterpret_cast<D2*>(&win(w)[fresh(li0) + 128 * j]) = v;
    if (FAR || a.G > 1)
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(U4, v), rsrc(w),
                                             (fresh(row0) + 128 * j + kResFront) * 8, 0, kSc1);
  }
  __device__ __forceinline__ D2 own(int w, int j) const { return *reinterpret_cast<const D2*>(&win(w)[fresh(li0) + 128 * j]); }

  // Window w's next vector goes to the spare buffer.  Its last readers
  // gathered it before the latest exchange, and the buffer given up here may
  // still be read in this phase, so it is written no earlier than the next.
  __device__ __forceinline__ void next(int w) {
    const int b = 8 * w;
    const uint32_t k = (ix >> b) & 0xffu, sp = ix >> 16;
    ix = (ix & ~(0xffu << b) & 0xffffu) | (sp << b) | (k << 16);
  }

  // Publishes this workgroup's partial sums (lane 63 of each wave holds the
  // wave's in `part`) after its data, waits for every workgroup's, and returns
  // the totals in pairwise order "+ 0.0".  false: a wait timed out.
  //
  // The four waves that do not poll the sums fetch the rows around window w
  // (the vector the next product gathers) meanwhile: they wait for the
  // workgroups that hold those rows only.
  template <int NS>
  __device__ __forceinline__ bool exchange(const double (&part)[NS > 0 ? NS : 1], double (&tot)[NS > 0 ? NS : 1], int w) {
    constexpr int NWD = NS > 0 ? 2 * NS : 1;  // words per workgroup
    ++epoch;
    const int par = epoch & 1, slot = NEAR ? epoch & 3 : par;
    if constexpr (NS > 0) {
      if (lane == 63) {
#pragma unroll
        for (int k = 0; k < NS; ++k) sh.red[par][k][wave] = part[k];
      }
    }
    // this wave's exchange stores have reached their scope before the barrier
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    auto wg_sum = [&](int k) {
      const double* r = sh.red[par][k];
      return ((r[0] + r[1]) + (r[2] + r[3])) + ((r[4] + r[5]) + (r[6] + r[7]));
    };
    if (a.G == 1) {
#pragma unroll
      for (int k = 0; k < NS; ++k) tot[k] = uniform(wg_sum(k) + 0.0);
      return true;
    }
    // An exchange without sums is a barrier among neighbours, unless the one
    // before was: a workgroup then never runs more than two exchanges ahead of
    // any other, and four slots of words keep what the slowest still reads.
    const bool near = NEAR && NS == 0 && !last_near;
    if constexpr (NEAR) last_near = near;
    u64* words = a.words + (size_t)slot * (2 * 5 * kResMaxG);
    if (t < NWD) {
      u64 half = 0;
      if constexpr (NS > 0) {
        const u64 bits = (u64)__double_as_longlong(wg_sum(t >> 1));
        half = (t & 1) ? (bits >> 32) : (bits & 0xffffffffull);
      }
      __hip_atomic_store(&words[t * kResMaxG + wg], ((u64)epoch << 32) | half, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    }
    if (t < kResMaxG) {
      double v[NS > 0 ? NS : 1];
#pragma unroll
      for (int k = 0; k < NS; ++k) v[k] = 0.0;
      // a barrier only concerns the workgroups this one reads from or is read by
      bool mine = t < a.G;
      if constexpr (NEAR) mine = mine && (!near || (t >= wg - a.reach && t <= wg + a.reach));
      if (mine) {
        u64 w[NWD];
        bool ok;
        int spins = 0;
        do {
          ok = true;
#pragma unroll
          for (int k = 0; k < NWD; ++k)
            w[k] = __hip_atomic_load(&words[k * kResMaxG + t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
          for (int k = 0; k < NWD; ++k) ok = ok && (unsigned)(w[k] >> 32) == epoch;
        } while (!ok && ++spins < kResSpin);
        if (!ok) sh.bad = 1;
#pragma unroll
        for (int k = 0; k < NS; ++k)
          v[k] = __longlong_as_double((long long)((w[2 * k] & 0xffffffffull) | (w[2 * k + 1] << 32)));
      }
      if constexpr (NS > 0) {
        if (wave * 64 < a.G) {
          wave_sum63<NS, double>(v);
        }
        if (lane == 63) {
#pragma unroll
          for (int k = 0; k < NS; ++k) sh.lw[par][wave][k] = v[k];
        }
      }
    } else if (w >= 0 && a.H > 0) {
      // workgroups first .. last hold the H rows on either side
      constexpr int rows = kResT * K;
      const int reach = (a.H + rows - 1) / rows;
      for (int g = max(wg - reach, 0) + lane; g <= min(wg + reach, a.G - 1); g += 64) {
        int spins = 0;
        while ((unsigned)(__hip_atomic_load(&words[g], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> 32) != epoch) {
          if (++spins >= kResSpin) {
            sh.bad = 1;
            break;
          }
        }
      }
      asm volatile("" ::: "memory");
      halo(w);
    }
    __syncthreads();
    if (__builtin_amdgcn_readfirstlane(sh.bad)) {
      if (t == 0) atomicOr(a.err, 1);
      return false;
    }
    if constexpr (NS > 0) {
      const double(&l)[4][5] = sh.lw[par];
#pragma unroll
      for (int k = 0; k < NS; ++k) tot[k] = uniform(((l[0][k] + l[1][k]) + (l[2][k] + l[3][k])) + 0.0);
    }
    return true;
  }
  __device__ __forceinline__ bool barrier(int w) {
    double none[1];
    return exchange<0>(none, none, w);
  }

  // The rows around the workgroup's own in window w, by threads 256 ..  511;
  // rows outside [0, n) read 0 and belong to no entry.
  __device__ __forceinline__ void halo(int w) {
    const auto r = rsrc(w);
    const int h = a.H >> 1;
    auto at = [&](int p) { return p < h ? 2 * p : kResT * K + 2 * p; };  // window index: left rows, then right rows
    constexpr int kStep = kResT / 2, kAhead = 4;                       // loads in flight before the first is stored
    if (a.H <= kStep) {
      const int p = t - kStep;
      if (p < a.H) *reinterpret_cast<D2*>(&win(w)[at(p)]) = load2(r, base - a.H + at(p));
      return;
    }
#pragma unroll 1
    for (int p = t - kStep; p < a.H; p += kAhead * kStep) {
      D2 v[kAhead];
#pragma unroll
      for (int u = 0; u < kAhead; ++u)
        if (p + u * kStep < a.H) v[u] = load2(r, base - a.H + at(p + u * kStep));
#pragma unroll
      for (int u = 0; u < kAhead; ++u)
        if (p + u * kStep < a.H) *reinterpret_cast<D2*>(&win(w)[at(p + u * kStep)]) = v[u];
    }
  }

  // y = A v for every pair, v in window w, handed to f(j, y_j) with j a
  // compile-time constant; load(j) is called before pair j's arithmetic, to
  // issue loads f(j) needs.  Each row sums its present diagonals in ascending
  // order from 0.0.  The far diagonals' values are loaded CJ pairs ahead, into
  // the registers the pair before has just given up; the pairs themselves are
  // kept apart (one pair's temporaries at a time is what the registers hold
  // beside the vectors).
  template <class L, class F>
  __device__ __forceinline__ void product(int w, L&& load, F&& f) const {
    const int32_t r0 = fresh(row0);
    const double* const pw = win(w) + fresh(li0);
    D2 f0[CJ], f1[CJ];
    const auto ex = rsrc(w);
    if constexpr (FAR) {
#pragma unroll
      for (int j = 0; j < CJ; ++j) {
        f0[j] = load2(ex, r0 + 128 * j + op.off[0]);
        f1[j] = load2(ex, r0 + 128 * j + op.off[ND - 1]);
      }
    }
    each_pair<KP>([&](auto jc) {
      constexpr int j = decltype(jc)::value;
      __builtin_amdgcn_sched_barrier(0);
      load(jc);
      const double* p = pw + 128 * j;
      D2 xs[ND], vs[ND];
#pragma unroll
      for (int d = 0; d < ND; ++d) {
        if (FAR && d == 0) xs[d] = f0[j % CJ];
        else if (FAR && d == ND - 1) xs[d] = f1[j % CJ];
        else xs[d] = *reinterpret_cast<const D2u*>(p + op.off[d]);
      }
      if constexpr (!UNI) {
        const int32_t rv = min(r0 + 128 * j, (n - 1) & ~1);
#pragma unroll
        for (int d = 0; d < ND; ++d) vs[d] = *reinterpret_cast<const D2*>(&op.va[(int64_t)op.vd[d] * op.ld + rv]);
      }
      const uint32_t m = fresh(mk[j / 2]) >> (16 * (j % 2)), u = fresh_uniform(all[j / 4]) >> (8 * (j % 4));
      // Two forms: every row of the block holds all but the slots beside the
      // middle one (a grid's x neighbours, which the ends of a line miss), or
      // any slot may be missing.
      D2 acc = {0.0, 0.0};
      auto sum = [&](uint32_t test) {
#pragma unroll
        for (int d = 0; d < ND; ++d) {
          const double v0 = UNI ? op.c[d] : vs[d].x, v1 = UNI ? op.c[d] : vs[d].y;
          const double t0 = acc.x + v0 * xs[d].x, t1 = acc.y + v1 * xs[d].y;
          if ((test >> d) & 1u) {
            acc.x = ((m >> d) & 1u) ? t0 : acc.x;
            acc.y = ((m >> (8 + d)) & 1u) ? t1 : acc.y;
          } else {
            acc.x = t0;
            acc.y = t1;
          }
        }
      };
      constexpr uint32_t full = (1u << ND) - 1u, ends = 5u << (ND / 2 - 1);
      if (((u | ends) & full) == full) sum(ends);
      else sum(full);
      if constexpr (FAR && j + CJ < KP) {
        f0[j % CJ] = load2(ex, r0 + 128 * (j + CJ) + op.off[0]);
        f1[j % CJ] = load2(ex, r0 + 128 * (j + CJ) + op.off[ND - 1]);
      }
      __builtin_amdgcn_sched_barrier(0);
      f(jc, acc);
    });
  }
  template <class F>
  __device__ __forceinline__ void product(int w, F&& f) const {
    product(w, [](auto) {}, f);
  }

  // Caller vectors: pair j of v (8-byte aligned), 0 past n.
  __device__ __forceinline__ D2 get(const double* v, int j) const {
    D2 q;
    q.x = row(j) < n ? v[row(j)] : 0.0;
    q.y = row(j) + 1 < n ? v[row(j) + 1] : 0.0;
    return q;
  }
  // M^{-1} v at pair j
  __device__ __forceinline__ D2 precond(int j, D2 v) const {
    if (a.vec_dinv) return get(a.dinv, j) * v;
    return a.dinv_s * v;
  }

  // A vector only its rows' own threads touch: in registers (K <= 8), else in
  // global memory (x: vector 3, r0: vector 4; rows past n + 1 read 0 and are
  // not written).
  static constexpr bool kXReg = K <= 8;
  struct X {
    int v;
    D2 r[kXReg ? KP : 1];
  };
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_x(const X& x) const {
    return __builtin_amdgcn_make_buffer_rsrc(a.vecs + (int64_t)x.v * a.stride, 0, (n + 1) * 8, 0x00020000);
  }
  __device__ __forceinline__ D2 get_x(const X& x, int j) const {
    if constexpr (kXReg) return x.r[j];
    else return __builtin_bit_cast(D2, __builtin_amdgcn_raw_buffer_load_b128(rsrc_x(x), (fresh(row0) + 128 * j) * 8, 0, 0));
  }
  __device__ __forceinline__ void set_x(X& x, int j, D2 v) const {
    if constexpr (kXReg) x.r[j] = v;
    else __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(U4, v), rsrc_x(x), (fresh(row0) + 128 * j) * 8, 0, 0);
  }
  // x_0 into x and window w, for the setup's product
  __device__ __forceinline__ void load_x0(X& x, int w) {
    x.v = 3;
#pragma unroll
    for (int j = 0; j < KP; ++j) {
      const D2 v = get(a.x0, j);
      set_x(x, j, v);
      put(w, j, v);
    }
  }
  // the final x and state
  __device__ __forceinline__ void finish(const X& x, const State& st) const {
    if constexpr (kXReg) {
#pragma unroll
      for (int j = 0; j < KP; ++j)
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(U4, x.r[j]), rsrc_x(x), row(j) * 8, 0, 0);
    }
    if (wg == 0 && t == 0) store_state(a.st, st);
  }
  __device__ __forceinline__ State start() const {
    State st;
    st.alpha = 0.0; st.beta = 0.0; st.omega = 0.0; st.gamma = 0.0;
    st.rho0 = 0.0; st.relres = 1.0; st.tol = a.tol; st.result = 0.0;
    st.status = DS_RUNNING; st.iters = 0; st.n_rr = 0;
    return st;
  }

  // Sums of the thread's pairs as they are produced: `add` takes block j's
  // leaves, lane 63 ends with the wave's balanced tree in `top`.  Up to 4
  // blocks the tree's levels stay in registers; with 8 lane 63 keeps them in
  // LDS (they would take 30 registers of every lane).
  template <int NS>
  struct Tree {
    Shared& sh;
    double lvl[KP > 4 ? 1 : 3][NS];
    double top[NS];
    __device__ __forceinline__ explicit Tree(Shared& s) : sh(s) {}
    template <int J>
    __device__ __forceinline__ void add(double (&d)[NS]) {
      wave_sum63<NS, double>(d);
      constexpr int ones = (J & 1) ? ((J & 2) ? ((J & 4) ? 3 : 2) : 1) : 0;
      if constexpr (KP > 4) {
        if ((threadIdx.x & 63) == 63) {
          double(&lv)[3][5] = sh.lvl[threadIdx.x >> 6];
#pragma unroll
          for (int l = 0; l < ones; ++l) {
#pragma unroll
            for (int k = 0; k < NS; ++k) d[k] = lv[l][k] + d[k];
          }
          if constexpr (J + 1 < KP) {
#pragma unroll
            for (int k = 0; k < NS; ++k) lv[ones][k] = d[k];
          }
        }
      } else {
#pragma unroll
        for (int l = 0; l < ones; ++l) {
#pragma unroll
          for (int k = 0; k < NS; ++k) d[k] = lvl[l][k] + d[k];
        }
        if constexpr (J + 1 < KP) {
#pragma unroll
          for (int k = 0; k < NS; ++k) lvl[ones][k] = d[k];
        }
      }
      if constexpr (J + 1 == KP) {
#pragma unroll
        for (int k = 0; k < NS; ++k) top[k] = d[k];
      }
    }
  };

  // Pair j of window w's next vector, kept out of the window while other
  // waves still read it: it waits in its exchange buffer, which it has to
  // reach anyway, and unstash() moves it into the window after a barrier.
  // Used where no registers are left to hold it (K = 16; needs G > 1).
  static constexpr bool kStash = K > 8;
  __device__ __forceinline__ void stash(int j, D2 v) {  // before next(): into the spare buffer
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(U4, v), rsrc(2), (fresh(row0) + 128 * j + kResFront) * 8,
                                           0, kSc1);
  }
  __device__ __forceinline__ void unstash(int w) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const auto r = rsrc(w);
#pragma unroll
    for (int j = 0; j < KP; ++j)
      *reinterpret_cast<D2*>(&win(w)[fresh(li0) + 128 * j]) = load2(r, fresh(row0) + 128 * j);
  }
};

// The operator in ND slots: the last diagonal in the last slot (FAR reads the
// first and the last slot from memory), empty slots before it.
template <int ND>
inline ResOpT<ND> res_op(const ResOp& o) {
  ResOpT<ND> r = {};
  r.mask = o.mask;
  r.va = o.va;
  r.n = o.n;
  r.nd = o.nd;
  r.ld = o.ld;
  r.nx = o.nx;
  r.ny = o.ny;
  r.nz = o.nz;
  for (int d = 0; d < o.nd; ++d) {
    const int s = d == o.nd - 1 ? ND - 1 : d;
    r.off[s] = o.off[d];
    r.vd[s] = d;
    r.c[s] = o.c[d];
  }
  return r;
}

inline ResArgs res_args(const ResPlan& p, const ResJob& j) {
  ResArgs a = {};
  a.G = p.G + (j.give_up == 1 && p.G > 1 && p.G < kResMaxG ? 1 : 0);
  a.H = p.H;
  a.reach = p.reach;
  a.variant = j.variant;
  a.rr_period = j.rr_period;
  a.rr_max = j.rr_max;
  a.maxit = j.maxit;
  a.aform = j.aform;
  a.vec_dinv = j.dinv != nullptr ? 1 : 0;
  a.tol = j.tol;
  a.dinv_s = j.dinv_s;
  a.dinv = j.dinv;
  a.b = j.b;
  a.x0 = j.x0;
  a.hist = j.hist;
  a.vecs = j.vecs;
  a.stride = j.stride;
  a.words = j.words;
  a.err = j.err;
  a.st = j.st;
  return a;
}

// Dynamic LDS of a launch: the two windows.
inline size_t res_lds(int K, int H) { return 2 * (size_t)(kResT * K + 2 * H) * sizeof(double); }

template <int ND>
inline hipError_t res_go(void (*k)(ResOpT<ND>, ResArgs), int K, const ResPlan& p, const ResOp& op, const ResJob& j,
                         hipStream_t s) {
  ResOpT<ND> o = res_op<ND>(op);
  ResArgs a = res_args(p, j);
  const size_t lds = res_lds(K, p.H);
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)lds);
  if (e != hipSuccess) return e;
  void* args[] = {&o, &a};
  return hipLaunchCooperativeKernel(reinterpret_cast<const void*>(k), dim3((unsigned)p.G), dim3(kResT), args,
                                    (unsigned)lds, s);
}

template <int ND>
inline hipError_t res_go_batch(void (*k)(const ResSys<ND>*, const int2*), const void* sys, const int2* map, int workgroups,
                               size_t lds, bool coop, hipStream_t s) {
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)lds);
  if (e != hipSuccess) return e;
  const ResSys<ND>* p = static_cast<const ResSys<ND>*>(sys);
  void* args[] = {&p, &map};
  if (!coop)
    return hipLaunchKernel(reinterpret_cast<const void*>(k), dim3((unsigned)workgroups), dim3(kResT), args, lds, s);
  return hipLaunchCooperativeKernel(reinterpret_cast<const void*>(k), dim3((unsigned)workgroups), dim3(kResT), args,
                                    (unsigned)lds, s);
}

// Calls go<K, ND, FAR, UNI, PC>() for the plan's instance.
// PC16: the method has Jacobi instances with K = 16.
template <bool PC16, class L>
inline hipError_t res_dispatch(const ResPlan& p, const ResOp& op, const ResJob& j, L go) {
  const bool uni = op.va == nullptr;
  auto with_pc = [&](auto k, auto nd, auto far, auto u) -> hipError_t {
    constexpr int K = decltype(k)::value;
    if constexpr (K <= 8 || PC16) {
      if (j.pc) return go(k, nd, far, u, std::true_type());
    }
    if (j.pc) return hipErrorInvalidValue;
    return go(k, nd, far, u, std::false_type());
  };
  auto with_k = [&](auto nd) -> hipError_t {
    auto with_far = [&](auto k) -> hipError_t {
      if (p.far) return uni ? with_pc(k, nd, std::true_type(), std::true_type())
                            : with_pc(k, nd, std::true_type(), std::false_type());
      return uni ? with_pc(k, nd, std::false_type(), std::true_type())
                 : with_pc(k, nd, std::false_type(), std::false_type());
    };
    switch (p.K) {
      case 2: return with_far(std::integral_constant<int, 2>());
      case 4: return with_far(std::integral_constant<int, 4>());
      case 8: return with_far(std::integral_constant<int, 8>());
      case 16:
        // 2^20 rows and more: read the far diagonals from memory always; one
        // value per diagonal only (others would re-read the values)
        if (p.far && uni) return with_pc(std::integral_constant<int, 16>(), nd, std::true_type(), std::true_type());
        return hipErrorInvalidValue;
      default: return hipErrorInvalidValue;
    }
  };
  if (op.nd <= 5) return with_k(std::integral_constant<int, 5>());
  return with_k(std::integral_constant<int, 7>());
}

}  // namespace pbcgs
