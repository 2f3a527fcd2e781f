// Resident solves: the launch shape, the setup kernels and the dispatch per
// method (the kernels themselves: resident_pipe.hip, resident_bicg.hip,
// resident_cg.hip).
#include <algorithm>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "../../include/pbcgs.h"
#include "resident.hpp"

namespace pbcgs {

namespace {

// Rows around a workgroup's own in its windows, each side: beyond these the
// streamed kernels read such surroundings faster, from the caches.  60
// iterations, far diagonals beyond inner ones H rows away (ms, streamed /
// resident): p-BiCGStab on varying values, H = 3,000 / 3,500 / 4,000 / 4,400,
// 120,000 rows 1.07 / 1.05, 1.07 / 1.09, 1.08 / 1.11, 1.08 / 1.15, 250,000 rows
// 1.39 / 1.17, 1.39 / 1.23, 1.39 / 1.46, 1.39 / 1.56; BiCGStab on one value per
// diagonal, 250,000 rows, 3,500 / 4,000 / 4,400, 1.76 / 1.36, 1.72 / 1.79, 1.75 /
// 1.82.
constexpr int64_t kResMaxH = 3584;

// Rows per thread that `op` can run with, and its windows: the diagonals other
// than a far first and last one must lie within H rows, and two windows of
// 512 K + 2 H doubles must fit the 160 KB of LDS beside the kernel's 2.6 KB.
bool res_fit(const ResOp& op, int K, bool pc, bool pc16, int maxg, ResPlan* p) {
  if (K > 8 && ((pc && !pc16) || op.va != nullptr)) return false;
  const int64_t rows = (int64_t)kResT * K;
  const int64_t G = (op.n + rows - 1) / rows;
  if (G > maxg) return false;
  int64_t all = 0, inner = 0;
  for (int d = 0; d < op.nd; ++d) {
    const int64_t o = op.off[d] < 0 ? -(int64_t)op.off[d] : op.off[d];
    all = std::max(all, o);
    if (d > 0 && d < op.nd - 1) inner = std::max(inner, o);
  }
  // far diagonals cost two memory reads per row and product, a window's
  // surroundings 2 H per workgroup: far once H would pass half its rows
  const bool far = K > 8 || 2 * all > rows;
  const int64_t H = ((far ? inner : all) + 1) & ~1ll;
  if (K > 8 && G < 2) return false;
  if (H > kResMaxH) return false;
  if ((int64_t)res_lds(K, 0) + 4 * H * 8 > 160 * 1024 - 4096) return false;
  p->K = K;
  p->G = (int)G;
  p->H = (int)H;
  p->far = far;
  p->reach = (int)((all + rows - 1) / rows);
  return true;
}

struct MethodCost {
  int exchanges;   // per iteration
  double per_row;  // microseconds per row of a thread
  bool pc16;       // Jacobi instances with 16 rows per thread (the registers hold them)
};

MethodCost method_cost(int32_t variant) {
  switch (variant) {
    case PBCGS_BICGSTAB: return {5, 0.5, false};
    case PBCGS_CG: return {3, 0.23, true};
    case PBCGS_CGCG: return {2, 0.33, true};
    case PBCGS_PIPE_CG: return {1, 0.25, false};
    default: return {2, 0.9, false};
  }
}

}  // namespace

ResPlan res_plan(const ResOp& op, int32_t variant, bool pc, int cus) {
  ResPlan best;
  if (op.nd < 1 || op.nd > kResMaxND || op.n < 1) return best;
  const int maxg = std::min(cus, kResMaxG);
  const char* e = std::getenv("PBCGS_RESIDENT_ROWS");
  const int forced = e ? std::atoi(e) : 0;
  double cost = 0.0;
  const MethodCost m = method_cost(variant);
  for (int K = 2; K <= 16; K *= 2) {
    if (forced > 0 && K != forced) continue;
    ResPlan p;
    if (!res_fit(op, K, pc, m.pc16, maxg, &p)) continue;
    // Microseconds of an iteration that depend on the shape, fitted to runs
    // at 41^3, 64^3, 99^3, 100^3 and 150^2 (what fits is taken: 40 iterations,
    // ms, streamed / resident, of p-BiCGStab with Jacobi as written 64^3 1.16 /
    // 0.68, 81^3 2.18 / 1.67, 101^3 2.74 / 2.16, its eight-row kernel with 248 to
    // 298 spilled registers; on varying values 32^3 0.61 / 0.49, 48^3 0.72 / 0.55,
    // 63^3 0.98 / 0.69, CG with Jacobi 48^3 0.70 / 0.71, 63^3 0.91 / 0.77): an exchange takes 0.015 us more per
    // workgroup, a row per thread 0.23 us (CG) to 0.9 us (p-BiCGStab), twice
    // that with 16 rows (x, and r0, then come from memory).  At 64^3
    // p-BiCGStab takes 14.4 / 11.1 / 13.9 us with K = 2 / 4 / 8, BiCGStab
    // 29.5 / 18.8 / 16.4, CG 16.5 / 10.7 / 9.0, p-CG 6.2 / 5.1 / 6.0; at 100^3
    // p-BiCGStab 23.8 / 32.7 with K = 8 / 16.
    const double c = m.exchanges * 0.015 * p.G + (pc ? 1.3 : 1.0) * (K > 8 ? 2.0 : 1.0) * m.per_row * K;
    if (best.K == 0 || c < cost) {
      best = p;
      cost = c;
    }
  }
  return best;
}

// Clears the exchange words, the error word and the state's status (which a
// finished solve overwrites).
__global__ __launch_bounds__(256) void k_res_init(u64* words, int32_t* err, DevState* st, int32_t give_up) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < kResWords) words[i] = 0;
  if (i == 0) {
    *err = give_up == 2 ? 1 : 0;
    st->status = -1;
  }
}

namespace {

struct UniformArgs {
  const uint32_t* mask;
  const int32_t* rp;
  const int32_t* ci;
  const double* va;
  const double* dinv;
  double ds;
  u64* ref;
  int32_t* flag;
  int32_t n, nd, plain;
};

__device__ __forceinline__ u64 uniform_bits(const UniformArgs& u, int32_t k) {
  double v = u.va[k];
  if (!u.plain) v = v * (u.dinv ? u.dinv[u.ci[k]] : u.ds);
  return (u64)__double_as_longlong(v);
}

// Whether row i's entries equal their diagonals' reference values.
__device__ __forceinline__ bool same_row(const UniformArgs& u, int32_t i, const u64* ref) {
  const uint32_t m = u.mask[i];
  int32_t k = u.rp[i];
  bool same = true;
#pragma unroll
  for (int d = 0; d < kResMaxND; ++d) {
    if ((m >> d) & 1u) {
      same = same && uniform_bits(u, k) == ref[d];
      ++k;
    }
  }
  return same;
}

// Reference value of every diagonal: its first entry in the 8192 rows around
// the middle (a diagonal with none there counts as varying), and a first look
// at 1,024 of those rows: where values vary, they nearly always do there, and
// the check of the whole operator then ends at once.  64 rows tell whether a
// diagonal holds more values than a value code can name, which spares a
// streamed solve the search for them (7-point, random values, 40 iterations of
// p-BiCGStab at 64^3: 1.19 ms with the search, 1.21 with this question beside
// it, 0.99 with its answer taken).
__device__ __forceinline__ void uniform_ref(const UniformArgs& u) {
  __shared__ int first[kResMaxND];
  __shared__ u64 ref[kResMaxND];
  if (threadIdx.x < kResMaxND) first[threadIdx.x] = INT32_MAX;
  __syncthreads();
  const int32_t lo = max(u.n / 2 - 4096, 0), hi = min(u.n / 2 + 4096, u.n);
  for (int32_t base = lo; base < hi; base += 1024) {
    const int32_t i = base + (int32_t)threadIdx.x;
    const uint32_t m = i < hi ? u.mask[i] : 0;
    for (int d = 0; d < u.nd; ++d) {
      const u64 rows = __ballot((m >> d) & 1u);
      if (rows && (threadIdx.x & 63) == 0) atomicMin(&first[d], i + (int)__builtin_ctzll(rows));
    }
    __syncthreads();
    bool found = true;
    for (int d = 0; d < u.nd; ++d) found = found && first[d] != INT32_MAX;
    if (found) break;
    __syncthreads();
  }
  if (threadIdx.x == 0) *u.flag = 0;
  __syncthreads();
  const int d = threadIdx.x;
  if (d < u.nd) {
    const int32_t i = first[d];
    if (i == INT32_MAX) *u.flag = kResVaries;
    else u.ref[d] = ref[d] = uniform_bits(u, u.rp[i] + __builtin_popcount(u.mask[i] & ((1u << d) - 1u)));
  }
  __syncthreads();
  const int32_t i = lo + (int32_t)threadIdx.x;
  if (i < hi && !same_row(u, i, ref)) *u.flag = kResVaries;
  __syncthreads();
  // wave d: the different values of diagonal d in rows lo .. lo + 63
  const int wd = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (wd < u.nd && lo + lane < hi) {
    const uint32_t m = u.mask[lo + lane];
    const bool has = (m >> wd) & 1u;
    const u64 v = has ? uniform_bits(u, u.rp[lo + lane] + __builtin_popcount(m & ((1u << wd) - 1u))) : 0;
    const u64 rows = __ballot(has);
    bool fresh = has;  // no lane before holds the same
    for (int l = 0; l < 63; ++l) {
      const u64 w = (u64)__shfl((long long)v, l);
      if (l < lane && ((rows >> l) & 1u) && w == v) fresh = false;
    }
    if (__builtin_popcountll(__ballot(fresh)) > kResCodes + 1 && lane == 0) *u.flag = kResVaries | kResManyValues;
  }
}

// Every entry against its diagonal's reference.
__device__ __forceinline__ void uniform_check(const UniformArgs& u, int block, int blocks) {
  if (*u.flag) return;
  u64 ref[kResMaxND];
#pragma unroll
  for (int d = 0; d < kResMaxND; ++d) ref[d] = d < u.nd ? u.ref[d] : 0;
  bool same = true;
  for (int32_t i = block * 256 + threadIdx.x; i < u.n; i += blocks * 256) same = same && same_row(u, i, ref);
  if (!same) *u.flag = kResVaries;
}

__global__ __launch_bounds__(1024) void k_uniform_ref(UniformArgs u) { uniform_ref(u); }
__global__ __launch_bounds__(256) void k_uniform_check(UniformArgs u) {
  uniform_check(u, (int)blockIdx.x, (int)gridDim.x);
}

}  // namespace

hipError_t res_uniform(const ResOp& op, const int32_t* rp, const int32_t* ci, const double* va, const double* dinv,
                       bool plain, double ds, void* aux, hipStream_t s) {
  u64* ref = static_cast<u64*>(aux);
  const UniformArgs u = {op.mask, rp, ci, va, dinv, ds, ref, reinterpret_cast<int32_t*>(ref + kResMaxND), op.n, op.nd,
                         plain ? 1 : 0};
  k_uniform_ref<<<1, 1024, 0, s>>>(u);
  k_uniform_check<<<std::min((op.n + 255) / 256, 2048), 256, 0, s>>>(u);
  return hipGetLastError();
}

// ---- batches ----
namespace {

// Layout of a batch's tables: exchange words only for the `multi` systems of
// more than one workgroup (the others exchange nothing; 10,000 of them would
// hold 0.8 GB).
struct BatchTables {
  size_t uni, ref, err, words, sys, map, bytes;
  BatchTables(int nsys, int maps, int multi) {
    auto take = [this](size_t b) {
      const size_t at = bytes;
      bytes += (b + 255) & ~(size_t)255;
      return at;
    };
    bytes = 0;
    uni = take(sizeof(UniformArgs) * (size_t)nsys);
    ref = take(kResAux * (size_t)nsys);
    err = take(sizeof(int32_t));
    words = take(sizeof(u64) * (size_t)kResWords * multi);
    sys = take(sizeof(ResSys<7>) * (size_t)nsys);
    map = take(sizeof(int2) * (size_t)maps);
  }
};

__global__ __launch_bounds__(1024) void kb_uniform_ref(const UniformArgs* us) { uniform_ref(us[blockIdx.x]); }
__global__ __launch_bounds__(256) void kb_uniform_check(const UniformArgs* us) {
  uniform_check(us[blockIdx.x], (int)blockIdx.y, (int)gridDim.y);
}

template <int ND>
__global__ __launch_bounds__(256) void kb_res_init(const ResSys<ND>* sys, int32_t give_up) {
  const ResArgs& a = sys[blockIdx.x].a;
  const int i = blockIdx.y * 256 + threadIdx.x;
  if (a.G > 1 && i < kResWords) a.words[i] = 0;
  if (i == 0) {
    *a.err = give_up == 2 ? 1 : 0;
    a.st->status = -1;
  }
}

template <int ND>
__global__ __launch_bounds__(256) void kb_res_copy_x(const ResSys<ND>* sys) {
  const ResSys<ND>& y = sys[blockIdx.x];
  const double* v = y.a.vecs + 3 * y.a.stride;
  double* x = const_cast<double*>(y.a.x0);
  for (int i = blockIdx.y * 256 + threadIdx.x; i < y.op.n; i += gridDim.y * 256) x[i] = v[i];
}

template <int ND>
hipError_t batch_launch(const ResBatchPlan& p, const std::vector<ResBatchSys>& sys, const ResJob& opts, char* base,
                        const BatchTables& t, hipStream_t s) {
  const int nsys = (int)sys.size();
  std::vector<ResSys<ND>> h((size_t)nsys);
  size_t multi = 0;
  for (int k = 0; k < nsys; ++k) {
    const ResBatchSys& y = sys[(size_t)k];
    ResJob j = opts;
    j.pc = false;
    j.dinv = nullptr;
    j.dinv_s = 0.0;
    j.hist = nullptr;
    j.b = y.b;
    j.x0 = y.x0;
    j.vecs = y.vecs;
    j.stride = y.stride;
    j.words = reinterpret_cast<u64*>(base + t.words) + multi * kResWords;
    if (p.G[(size_t)k] > 1) ++multi;
    j.err = reinterpret_cast<int32_t*>(base + t.err);
    j.st = y.st;
    ResPlan q;
    q.K = kResBatchK;
    q.G = p.G[(size_t)k];
    q.H = p.H[(size_t)k];
    q.reach = (q.H + kResT * kResBatchK - 1) / (kResT * kResBatchK);
    h[(size_t)k].op = res_op<ND>(y.op);
    h[(size_t)k].a = res_args(q, j);
  }
  std::vector<int2> map;
  std::vector<size_t> first;
  auto list = [&](const std::vector<int>& l) {
    first.push_back(map.size());
    for (int k : l)
      for (int g = 0; g < p.G[(size_t)k]; ++g) map.push_back(int2{k, g});
  };
  for (const auto& l : p.launches) list(l);
  // in dispatch order, so that the largest start first on every XCD
  first.push_back(map.size());
  map.resize(map.size() + p.singles.size());
  const int ns = (int)p.singles.size();
  for (int b = 0; b < ns; ++b) map[first.back() + (size_t)xcd_index(b, ns)] = int2{p.singles[(size_t)b], 0};
  const ResSys<ND>* dsys = reinterpret_cast<const ResSys<ND>*>(base + t.sys);
  int2* dmap = reinterpret_cast<int2*>(base + t.map);
  hipError_t e = hipMemcpyAsync(base + t.sys, h.data(), sizeof(ResSys<ND>) * h.size(), hipMemcpyHostToDevice, s);
  if (e == hipSuccess) e = hipMemcpyAsync(dmap, map.data(), sizeof(int2) * map.size(), hipMemcpyHostToDevice, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);  // the host tables go away
  if (e != hipSuccess) return e;
  // the systems in x: y is limited to 65,536
  kb_res_init<ND><<<dim3((unsigned)nsys, (kResWords + 255) / 256), 256, 0, s>>>(dsys, opts.give_up);
  for (size_t l = 0; l <= p.launches.size(); ++l) {
    const bool coop = l < p.launches.size();
    int W = 0, H = 0;
    for (int k : coop ? p.launches[l] : p.singles) {
      W += p.G[(size_t)k];
      H = std::max(H, p.H[(size_t)k]);
    }
    if (W == 0) continue;
    const size_t lds = res_lds(kResBatchK, H);
    e = opts.variant == PBCGS_BICGSTAB ? res_launch_batch_bicg(ND, dsys, dmap + first[l], W, lds, coop, s)
                                       : res_launch_batch_pipe(ND, dsys, dmap + first[l], W, lds, coop, s);
    if (e != hipSuccess) return e;
  }
  return hipGetLastError();
}

}  // namespace

constexpr int64_t kResBatchMinRows = 1024;  // mean rows of a batch of many one-workgroup systems

// Largest systems first, each into the first launch with room: they iterate
// longest, and the small ones fill the workgroups beside them.  Systems of one
// workgroup exchange nothing, so those that find no room share one ordinary
// launch, whose workgroups start as others end; in cooperative launches of 256
// they waited for each launch's slowest system (400 of 64^2, 40 iterations:
// 4.7 ms, now 3.6, streamed 6.0).
//
// A batch with more of them than compute units and few rows a system streams:
// a workgroup's 4,096 rows are mostly empty then (ms, streamed / resident:
// 2,000 of 16^2 13.8 / 16.8, 500 of 16^2 solved to 1e-8 3.9 / 4.1, 1,000 of
// 32^2 8.4 / 8.3).  any_size: it does not.
ResBatchPlan res_batch_plan(const std::vector<ResBatchSys>& sys, int cus, bool any_size) {
  ResBatchPlan p;
  const int maxg = std::min(cus, kResMaxG);
  std::vector<int> order;
  int64_t rows = 0;
  p.nd = 5;
  for (size_t k = 0; k < sys.size(); ++k) {
    const ResOp& op = sys[k].op;
    if (op.nd < 1 || op.nd > kResMaxND || op.n < 1) return p;
    if (op.nd > 5) p.nd = 7;
    int64_t H = 0;
    for (int d = 0; d < op.nd; ++d) H = std::max(H, std::abs((int64_t)op.off[d]));
    H = (H + 1) & ~1ll;
    const int64_t G = (op.n + kResT * kResBatchK - 1) / (kResT * kResBatchK);
    if (G > maxg || (int64_t)res_lds(kResBatchK, 0) + 4 * H * 8 > 160 * 1024 - 4096) return p;
    p.G.push_back((int)G);
    p.H.push_back((int)H);
    order.push_back((int)k);
    rows += op.n;
  }
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return sys[(size_t)a].op.n > sys[(size_t)b].op.n; });
  std::vector<int> used;
  for (int k : order) {
    size_t l = 0;
    while (l < used.size() && used[l] + p.G[(size_t)k] > maxg) ++l;
    if (l == used.size()) {
      if (p.G[(size_t)k] == 1) {
        p.singles.push_back(k);
        continue;
      }
      used.push_back(0);
      p.launches.emplace_back();
    }
    used[l] += p.G[(size_t)k];
    p.launches[l].push_back(k);
  }
  if (!any_size && (int)p.singles.size() > maxg && rows < kResBatchMinRows * (int64_t)sys.size()) return p;
  p.ok = true;
  return p;
}

static BatchTables batch_tables(const ResBatchPlan& p) {
  int maps = 0, multi = 0;
  for (int g : p.G) {
    maps += g;
    multi += g > 1 ? 1 : 0;
  }
  return BatchTables((int)p.G.size(), maps, multi);
}

size_t res_batch_bytes(const ResBatchPlan& p) { return batch_tables(p).bytes; }

hipError_t res_batch_uniform(std::vector<ResBatchSys>& sys, void* tables, hipStream_t s, bool* uniform) {
  const int nsys = (int)sys.size();
  const BatchTables t(nsys, 0, 0);  // the two tables used here come first
  char* base = static_cast<char*>(tables);
  std::vector<UniformArgs> h((size_t)nsys);
  int32_t nmax = 0;
  for (int k = 0; k < nsys; ++k) {
    const ResBatchSys& y = sys[(size_t)k];
    u64* ref = reinterpret_cast<u64*>(base + t.ref + kResAux * (size_t)k);
    h[(size_t)k] = {y.op.mask, y.rp, y.ci, y.va, nullptr, 0.0, ref, reinterpret_cast<int32_t*>(ref + kResMaxND),
                    y.op.n, y.op.nd, 1};
    nmax = std::max(nmax, y.op.n);
  }
  std::vector<unsigned char> out(kResAux * (size_t)nsys);
  const UniformArgs* d = reinterpret_cast<const UniformArgs*>(base + t.uni);
  hipError_t e = hipMemcpyAsync(base + t.uni, h.data(), sizeof(UniformArgs) * h.size(), hipMemcpyHostToDevice, s);
  if (e != hipSuccess) return e;
  kb_uniform_ref<<<nsys, 1024, 0, s>>>(d);
  kb_uniform_check<<<dim3((unsigned)nsys, (unsigned)std::min((nmax + 1023) / 1024, 256)), 256, 0, s>>>(d);
  e = hipGetLastError();
  if (e == hipSuccess) e = hipMemcpyAsync(out.data(), base + t.ref, out.size(), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) return e;
  *uniform = true;
  for (int k = 0; k < nsys; ++k) {
    int32_t flag;
    std::memcpy(&flag, &out[kResAux * (size_t)k + 8 * kResMaxND], sizeof flag);
    *uniform = *uniform && flag == 0;
    std::memcpy(sys[(size_t)k].op.c, &out[kResAux * (size_t)k], sizeof(double) * kResMaxND);
  }
  return hipSuccess;
}

hipError_t res_batch_launch(const ResBatchPlan& p, const std::vector<ResBatchSys>& sys, const ResJob& opts, void* tables,
                            hipStream_t s, int32_t** err_word) {
  const BatchTables t = batch_tables(p);
  char* base = static_cast<char*>(tables);
  *err_word = reinterpret_cast<int32_t*>(base + t.err);
  if (p.nd <= 5) return batch_launch<5>(p, sys, opts, base, t, s);
  return batch_launch<7>(p, sys, opts, base, t, s);
}

hipError_t res_batch_copy_x(const ResBatchPlan& p, const std::vector<ResBatchSys>& sys, void* tables, hipStream_t s) {
  char* d = static_cast<char*>(tables) + batch_tables(p).sys;
  int32_t nmax = 0;
  for (const ResBatchSys& y : sys) nmax = std::max(nmax, y.op.n);
  const dim3 g((unsigned)sys.size(), (unsigned)std::min((nmax + 1023) / 1024, 64));
  if (p.nd <= 5) kb_res_copy_x<5><<<g, 256, 0, s>>>(reinterpret_cast<const ResSys<5>*>(d));
  else kb_res_copy_x<7><<<g, 256, 0, s>>>(reinterpret_cast<const ResSys<7>*>(d));
  return hipGetLastError();
}

bool res_method(int32_t variant) { return variant != PBCGS_CA_BICGSTAB; }

hipError_t res_launch(const ResPlan& p, const ResOp& op, const ResJob& j, hipStream_t s) {
  k_res_init<<<(kResWords + 255) / 256, 256, 0, s>>>(j.words, j.err, j.st, j.give_up);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  switch (j.variant) {
    case PBCGS_PBICGSTAB:
    case PBCGS_PBICGSTAB_RR: return res_launch_pipe(p, op, j, s);
    case PBCGS_BICGSTAB: return res_launch_bicg(p, op, j, s);
    case PBCGS_CG:
    case PBCGS_CGCG:
    case PBCGS_PIPE_CG: return res_launch_cg(p, op, j, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace pbcgs
