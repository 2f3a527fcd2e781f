// Host interface of the resident solvers (resident.hpp): one cooperative
// launch runs a whole binary64 solve with the Krylov vectors in registers and
// LDS.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

namespace pbcgs {

struct DevState;

constexpr int kResT = 512;          // threads per workgroup: 8 x wave64
constexpr int kResMaxG = 256;       // workgroups: one per compute unit
constexpr int kResMaxND = 7;        // diagonals
constexpr int kResVecs = 5;         // global vectors a launch needs (three exchange buffers, x and r0)
constexpr int kResWords = 4 * 2 * 5 * kResMaxG;  // tagged words of four exchanges
constexpr size_t kResAux = 64;      // bytes of res_uniform's result: one value per diagonal, then a flag word
constexpr size_t kResVecPad = 64;   // doubles a global vector holds beyond n

// Operator: at most kResMaxND diagonals, offsets ascending, a mask of the
// diagonals each row holds (a constant stencil derives its mask from the grid
// extents), and either one value per diagonal (va == nullptr) or the values of
// the diagonal layout.
struct ResOp {
  const uint32_t* mask;  // nullptr: a 5- or 7-point stencil on nx x ny x nz
  const double* va;      // values va[d * ld + row], or nullptr: c[d]
  int32_t n, nd, ld;
  int32_t nx, ny, nz;
  int32_t off[kResMaxND];
  double c[kResMaxND];
};

struct ResJob {
  int32_t variant, rr_period, rr_max, maxit, aform;
  int32_t give_up;       // test hook: 1: the workgroups wait for one that is not there and time out (about
                         // 0.07 s; needs 2 to 255 workgroups); 2: the solve counts as timed out at its end
  double tol;
  bool pc;               // Jacobi applied as the algorithms write it
  const double* dinv;    // its vector, or nullptr: the constant dinv_s
  double dinv_s;
  const double* b;
  const double* x0;
  double* hist;
  double* vecs;          // kResVecs vectors of `stride` doubles, 16-byte aligned
  int64_t stride;        // >= n + kResVecPad, even
  unsigned long long* words;  // kResWords
  int32_t* err;          // set to 1 when a wait timed out (of the caller's, only hist is written then)
  DevState* st;          // the final state
};

struct ResPlan {
  int K = 0;      // rows per thread; 0: the operator does not fit
  int G = 0;      // workgroups
  int reach = 0;  // workgroups on either side whose rows a product reads
  int H = 0;      // rows beyond the workgroup's own that its LDS windows hold, each side
  bool far = false;  // the first and last diagonal are read from the exchange buffers
};

// The launch shape for an operator on a device with `cus` compute units, or
// K = 0 where the resident form does not apply.
ResPlan res_plan(const ResOp& op, int32_t variant, bool pc, int cus);

// Whether the resident form implements a method (PBCGS_BICGSTAB ...).
bool res_method(int32_t variant);

// What res_uniform says of an operator (0: one value per diagonal).
// kResManyValues: some diagonal holds more than kResCodes values; not set, it
// may nevertheless.
constexpr int32_t kResVaries = 1, kResManyValues = 2;
constexpr int kResCodes = 16;  // values per diagonal of the value-indexed layout

// Writes to aux (kResAux device bytes) the value of each diagonal of the CSR
// operator (rp, ci, va; op.mask its diagonals) and after them a flag word.  plain: the stored values; else each times dinv of
// its column (one rounding), or times ds when dinv is nullptr.
hipError_t res_uniform(const ResOp& op, const int32_t* rp, const int32_t* ci, const double* va, const double* dinv,
                       bool plain, double ds, void* aux, hipStream_t s);

// x of the finished solve, inside job.vecs.
inline double* res_x(const ResJob& j) { return j.vecs + 3 * j.stride; }

hipError_t res_launch(const ResPlan& p, const ResOp& op, const ResJob& j, hipStream_t s);

// ---- batches ----
// A batched solve packs its systems into cooperative launches of at most one
// workgroup per compute unit (kResBatchK rows per thread, one value per
// diagonal, every diagonal within the windows).
struct ResBatchSys {  // what the caller knows of a system
  ResOp op;           // structure; c after res_batch_uniform
  const int32_t* rp;
  const int32_t* ci;
  const double* va;
  const double* b;
  const double* x0;
  double* vecs;       // kResBatchVecs vectors of `stride` doubles, 16-byte aligned
  int64_t stride;
  DevState* st;
};
constexpr int kResBatchVecs = 4;    // three exchange buffers and x
constexpr int kResBatchK = 8;       // rows per thread

// Launches of a batch: each a list of systems with their first workgroup.
struct ResBatchPlan {
  bool ok = false;
  int nd = 0;                       // slots: 5 or 7
  std::vector<std::vector<int>> launches;
  std::vector<int> singles;         // systems of one workgroup left over, one ordinary launch
  std::vector<int> G, H;            // per system
};
ResBatchPlan res_batch_plan(const std::vector<ResBatchSys>& sys, int cus, bool any_size);

// Device bytes of a batch's tables (descriptors, maps, words, uniform values).
size_t res_batch_bytes(const ResBatchPlan& p);

// Uploads the descriptors of res_uniform for every system, runs it and reads
// the values into sys[k].op.c; *uniform: every system has one value per
// diagonal.  Synchronises the stream.
hipError_t res_batch_uniform(std::vector<ResBatchSys>& sys, void* tables, hipStream_t s, bool* uniform);

// Queues the launches; *err_word receives the device address of the word that
// is nonzero afterwards when a wait timed out.  x of system k: its vecs + 3 stride.
hipError_t res_batch_launch(const ResBatchPlan& p, const std::vector<ResBatchSys>& sys, const ResJob& opts, void* tables,
                            hipStream_t s, int32_t** err_word);
// Queues the copies of every x to the caller's, after a launch without errors.
hipError_t res_batch_copy_x(const ResBatchPlan& p, const std::vector<ResBatchSys>& sys, void* tables, hipStream_t s);
// coop: a cooperative launch, every workgroup on the chip at once
hipError_t res_launch_batch_pipe(int nd, const void* sys, const int2* map, int workgroups, size_t lds, bool coop,
                                 hipStream_t s);
hipError_t res_launch_batch_bicg(int nd, const void* sys, const int2* map, int workgroups, size_t lds, bool coop,
                                 hipStream_t s);

// per method: its kernels live in a translation unit of their own
hipError_t res_launch_pipe(const ResPlan& p, const ResOp& op, const ResJob& j, hipStream_t s);
hipError_t res_launch_bicg(const ResPlan& p, const ResOp& op, const ResJob& j, hipStream_t s);
hipError_t res_launch_cg(const ResPlan& p, const ResOp& op, const ResJob& j, hipStream_t s);

}  // namespace pbcgs
