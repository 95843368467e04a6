// The lattice handle behind the C ABI and the launches that depend on its
// storage type, one translation unit per type (ops.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <memory>

#include "../../include/lbm.h"
#include "kernels.h"
#include "trace.h"

struct lbm_lattice {
  lbm_config cfg;
  int kind;  // 0 MRT Table 1, 1 MRT d'Humieres, 2 FCLB
  int Q;
  size_t N;
  size_t elem;  // bytes per stored value
  hipStream_t stream;
  // bound memory
  char* base = nullptr;
  size_t bytes = 0;
  size_t off_ghost = 0, off_partial = 0, off_result = 0, req = 0;
  size_t ghost_n_max = 0;
  size_t nblocks = 0;
  // state
  int64_t t = 0;
  int parity = 0;
  bool has_bc = false;
  bool solids = false;  // interior solid nodes set (general kernel only)
  // interpolated bounce-back links (caller-owned device buffers)
  const int32_t* link_nodes = nullptr;
  const float* link_q = nullptr;
  long long nlinks = 0;
  lbm::LatArgs args;
  dim3 grid, block;
  // odd steps with boundaries split into wall rows (x and y faces walls or
  // periodic, see pull_walls) and the rows on the other non-periodic faces
  bool split_odd = false;
  lbm::Rows rows_all, rows_odd;
  unsigned tiles_all = 0, tiles_inner = 0;  // workgroups of 256 nodes (FLAT)
  bool resident = false;  // populations fit the last-level cache
  // Streaming hint of the steps (see ld): on lattices larger than the
  // last-level cache, where populations (even steps, which run over them from
  // end to end) or rows (odd steps) are whole memory lines.
  bool nt_even = false, nt_odd = false;
  bool nt_read = false;  // of the readouts but populations (see with_read)
  // health check inside lbm_step (lbm_set_check)
  int64_t check_every = 0;
  double check_tol = -1.0, check_m0 = 0.0;
  // per-launch timing (LBM_TRACE=1 at creation)
  std::unique_ptr<lbm::Tracer> tracer = std::make_unique<lbm::Tracer>();
};

namespace lbm {

// f64: caller's field buffers are FP64, else FP32.
template <typename S>
struct Ops {
  static void step(const lbm_lattice* L, bool odd, long long t, void* rec);
  static void links(const lbm_lattice* L, bool after_odd);
  static void init_equilibrium(const lbm_lattice* L, const void* drho, const void* u, bool f64);
  static void set_populations(const lbm_lattice* L, const void* f, bool f64);
  static void get_populations(const lbm_lattice* L, void* f, bool f64);
  static void macroscopic(const lbm_lattice* L, void* rho, void* u, bool f64, int rho_mode);
  static void stats_accumulate(const lbm_lattice* L, double* sums);
  static void reduce_partial(const lbm_lattice* L, unsigned blocks, double* partial);
  static void probe(const lbm_lattice* L, int3 lo, int3 hi, double scale, void* lambda, bool f64,
                    double* partial);
};

}  // namespace lbm
