// Host runtime of the C ABI declared in include/lbm.h: validation, memory
// layout inside the caller's block and launch configuration. The launches
// that depend on the storage type are in ops.hip.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstring>
#include <memory>
#include <mutex>
#include <string>
#include <type_traits>

#include "../../include/lbm.h"
#include "adjoint.h"
#include "jetprofile.h"
#include "kernels.h"
#include "lattice.h"
#include "trace.h"

using namespace lbm;

namespace {

thread_local std::string g_hip_msg;

int hip_fail(hipError_t e) {
  g_hip_msg = std::string("HIP error: ") + hipGetErrorString(e);
  return LBM_EHIP;
}

size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

void launch_shape(lbm_lattice* L) {
  const int nx = L->cfg.nx, ny = L->cfg.ny, nz = L->cfg.nz;
  int bx = nx < 256 ? nx : 256;
  int by = 256 / bx;
  if (by > ny) by = ny;
  if (by < 1) by = 1;
  L->block = dim3(bx, by, 1);
  L->grid = dim3((nx + bx - 1) / bx, (ny + by - 1) / by, nz);
  L->nblocks = (size_t)L->grid.x * L->grid.y * L->grid.z;
}

// Slabs spanned by a population and its opposite (see max_opposite_distance).
double slab_span(int Q) {
  return 1.0 + (Q == 27 ? max_opposite_distance<27>() : max_opposite_distance<19>());
}

// Row sets of the split odd step for the current boundary description.
void plan_rows(lbm_lattice* L) {
  const int nx = L->cfg.nx, ny = L->cfg.ny, nz = L->cfg.nz;
  const uint32_t np = L->args.bc.nonper;
  Rows all{};
  all.y0 = 0;
  all.ny_in = ny;
  all.n0 = 0;
  all.n1 = (uint32_t)L->N;
  all.by_nx.set((uint32_t)nx);
  all.by_ny.set((uint32_t)ny);
  // Lattices that the last-level cache (256 MB) holds from step to step take
  // their tiles by XCD and no streaming hint; measured per step (even / odd
  // with walls), 96x112x224 MRT FP32 (183 MB): 54.0 / 56.5 us against 74.5 /
  // 67.4 with the hint in launch order. Beyond it the eight far apart ranges
  // cost more than the shared lines (256x256x512 FCLB FP32, 3.6 GB: 1296 /
  // 1514 against 1251 / 1396 us; all at five workgroups per CU) and the hint
  // pays (1251 against 1351 us),
  // where the accesses are whole lines: odd steps on 190-node rows (1.0 GB)
  // 440 us with it, 413 without; their even steps, whose slabs are aligned,
  // 361 and 393.
  const double bytes = (double)L->N * L->Q * (double)L->elem;
  L->resident = bytes <= 256.0 * 1048576.0;
  all.by_xcd = L->resident;
  L->nt_even = !L->resident && (L->N * L->elem) % 128 == 0;
  L->nt_odd = !L->resident && ((size_t)nx * L->elem) % 128 == 0;
  L->nt_read = bytes > 4.0 / 3.0 * 256.0 * 1048576.0;
  L->tiles_all = (unsigned)((L->N + 255) / 256);
  L->rows_all = all;
  const bool znp = (np & 48u) != 0;
  // y faces that are walls stay in the wall rows; other non-periodic y
  // faces go to the row list
  const bool ynp = (np & 12u) != 0 && (L->args.bc.wall & 12u) != 12u;
  Rows odd = all;
  int z0 = 0, nz_in = nz;
  if (ynp) {
    odd.y0 = 1;
    odd.ny_in = ny - 2;
    odd.yb_n = 2;
    odd.yb[0] = 0;
    odd.yb[1] = ny - 1;
  }
  if (znp) {
    z0 = 1;
    nz_in = nz - 2;
    odd.zb_n = 2;
    odd.zb[0] = 0;
    odd.zb[1] = nz - 1;
  }
  const size_t plane = (size_t)nx * ny;
  odd.n0 = (uint32_t)(z0 * plane);
  odd.n1 = odd.ny_in > 0 && nz_in > 0 ? odd.n0 + (uint32_t)(nz_in * plane) : odd.n0;
  L->tiles_inner = (odd.n1 - odd.n0 + 255) / 256;
  odd.zi0 = znp ? 1 : 0;
  const long long nrows =
      (long long)odd.zb_n * ny + (long long)odd.yb_n * (nz - odd.zb_n);
  const uint32_t xbits = np & 3u;
  const bool x_ok = (L->args.bc.inlet & 3u) == 0 && (xbits == 0 || (L->args.bc.wall & 3u) == 3u);
  // the wall rows address a population and its opposite from the lower
  // slab with 32-bit offsets: the span of slabs must stay below 4 GiB
  const bool span_ok = slab_span(L->Q) * (double)L->N * (double)L->elem < 4294967296.0;
  L->split_odd = L->has_bc && x_ok && nrows <= 65535 && span_ok;
  if (L->split_odd && nrows > 0) {
    odd.nlist = (uint32_t)(nrows * nx);
    // a multiple of eight: the wall rows' tiles behind them stay on the XCDs
    // of the even step's tiles
    odd.list_tiles = (odd.nlist + 2047) / 2048 * 8;
  }
  L->rows_odd = odd;
}

// Runs fn(a value of the lattice's storage type).
template <typename Fn>
void by_storage(const lbm_lattice* L, Fn&& fn) {
  switch (L->cfg.storage) {
    case LBM_F64: fn(double()); break;
    case LBM_F32: fn(float()); break;
    default: fn(_Float16()); break;
  }
}

int check_launch() {
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? LBM_OK : hip_fail(e);
}

bool valid_dtype(int d) { return d == LBM_DTYPE_F64 || d == LBM_DTYPE_F32; }

void default_bc(BcArgs& b) {
  std::memset(&b, 0, sizeof(b));
  b.inlet_axis = 2;
  b.ghost_n = 1;
}

// Blocks of a reduction: four per CU, each summing several tiles, so that the
// single block that adds up their rows has little to do. All of them run at
// once, except at odd parity with boundaries, where the general pull's
// registers leave room for two (D3Q27) or three (D3Q19) per CU.
constexpr unsigned kReduceBlocks = 1024;
unsigned reduce_blocks(const lbm_lattice* L) {
  return L->tiles_all < kReduceBlocks ? L->tiles_all : kReduceBlocks;
}

// FP64 sums of the current state (lbm_reduce's definition), blocking.
int reduce_now(lbm_lattice* L, double out[5]) {
  double* partial = (double*)(L->base + L->off_partial);
  double* result = (double*)(L->base + L->off_result);
  {
    TraceScope ts(L->tracer.get(), L->stream, "reduce_partial_kernel + reduce_final_kernel");
    const unsigned nb = reduce_blocks(L);
    by_storage(L, [&](auto s) { Ops<decltype(s)>::reduce_partial(L, nb, partial); });
    hipLaunchKernelGGL(reduce_final_kernel, dim3(1), dim3(256), 0, L->stream, partial,
                       (size_t)nb, result);
  }
  const int rc = check_launch();
  if (rc) return rc;
  hipError_t e = hipMemcpyAsync(out, result, 5 * sizeof(double), hipMemcpyDeviceToHost,
                                L->stream);
  if (e != hipSuccess) return hip_fail(e);
  e = hipStreamSynchronize(L->stream);
  if (e != hipSuccess) return hip_fail(e);
  for (int k = 0; k < 5; ++k)
    if (!std::isfinite(out[k])) return LBM_ENONFINITE;
  return LBM_OK;
}

// The check of lbm_set_check after a step.
int run_check(lbm_lattice* L) {
  double out[5];
  const int rc = reduce_now(L, out);
  if (rc) return rc;
  if (L->check_tol >= 0.0 && std::fabs(out[0] - L->check_m0) > L->check_tol)
    return LBM_EMASS;
  return LBM_OK;
}

}  // namespace

// Library-owned partial sums for lbm_reduce_static: one row of five per block
// of the reduce launch (kReduceBlocks at most). Each device holds its own copy
// for the life of the process; every call on a device shares it. The number of
// rows is the limit that the call documents for an x-y plane.
constexpr size_t kStaticPartials = 16384;
static __device__ __align__(256) double scratch[kStaticPartials * 5 + 8];
static_assert(kReduceBlocks <= kStaticPartials);

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_ptr[kMaxDevices] = {nullptr};

// The device address of the scratch array on the device that runs the
// lattice's stream (the current device for the null stream), looked up once
// per device with that device current (the array's name in host code is not
// a device address).
int static_scratch(hipStream_t stream, double** out) {
  int cur = 0, dev = 0;
  hipError_t e = hipGetDevice(&cur);
  if (e != hipSuccess) return hip_fail(e);
  dev = cur;
  if (stream) {
    e = hipStreamGetDevice(stream, &dev);
    if (e != hipSuccess) return hip_fail(e);
  }
  if (dev < 0 || dev >= kMaxDevices) return LBM_EINVAL;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    if (dev != cur && (e = hipSetDevice(dev)) != hipSuccess) return hip_fail(e);
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (dev != cur) (void)hipSetDevice(cur);
    if (e != hipSuccess) return hip_fail(e);
    g_scratch_ptr[dev] = (double*)ptr;
  }
  *out = g_scratch_ptr[dev];
  return LBM_OK;
}

}  // namespace

extern "C" {

const char* lbm_strerror(int status) {
  switch (status) {
    case LBM_OK: return "ok";
    case LBM_EINVAL: return "invalid argument or configuration";
    case LBM_ENOMEM: return "bound device block is smaller than required";
    case LBM_EUNBOUND: return "no device memory bound";
    case LBM_EHIP: return g_hip_msg.empty() ? "HIP error" : g_hip_msg.c_str();
    case LBM_ENONFINITE: return "non-finite global sum";
    case LBM_ESTATE: return "call not valid in the current lattice state";
    case LBM_EMASS: return "mass deviation drifted beyond the check tolerance";
    default: return "unknown status";
  }
}

int lbm_create_lattice(const lbm_config* cfg, lbm_lattice** out) {
  if (!cfg || !out) return LBM_EINVAL;
  const lbm_config& c = *cfg;
  if (c.model != LBM_D3Q19_MRT_LES && c.model != LBM_D3Q27_FCLB && c.model != LBM_D3Q27_CLB)
    return LBM_EINVAL;
  if (c.storage != LBM_F64 && c.storage != LBM_F32 && c.storage != LBM_F16) return LBM_EINVAL;
  if (c.nx < 1 || c.ny < 1 || c.nz < 1) return LBM_EINVAL;
  const double nnodes = (double)c.nx * c.ny * c.nz;
  if (nnodes >= 2147483648.0) return LBM_EINVAL;
  if (c.nz > 65535 || c.ny > 65535 * 256) return LBM_EINVAL;  // launch grid limits
  // one population slab (all nodes) below 4 GiB: the kernels address it with
  // 32-bit byte offsets
  const size_t elem_bytes = c.storage == LBM_F64 ? 8 : (c.storage == LBM_F32 ? 4 : 2);
  if (nnodes * (double)elem_bytes >= 4294967296.0) return LBM_EINVAL;
  if (!(c.nu > 0.0) || !std::isfinite(c.nu)) return LBM_EINVAL;
  if (!(c.cs_smag >= 0.0) || !std::isfinite(c.cs_smag)) return LBM_EINVAL;
  if (c.model == LBM_D3Q19_MRT_LES &&
      c.mrt_basis != LBM_BASIS_TABLE1 && c.mrt_basis != LBM_BASIS_DHUMIERES)
    return LBM_EINVAL;
  if (c.model == LBM_D3Q19_MRT_LES && !c.use_default_rates) {
    const int nr = c.mrt_basis == LBM_BASIS_TABLE1 ? 4 : 5;
    for (int k = 0; k < nr; ++k)
      if (!(c.rates[k] > 0.0 && c.rates[k] < 2.0)) return LBM_EINVAL;
  }
  lbm_lattice* L = new (std::nothrow) lbm_lattice();
  if (!L) return LBM_EINVAL;
  L->cfg = c;
  L->kind = c.model == LBM_D3Q27_FCLB ? 2
            : c.model == LBM_D3Q27_CLB  ? 3
                                        : (c.mrt_basis == LBM_BASIS_TABLE1 ? 0 : 1);
  L->Q = c.model == LBM_D3Q19_MRT_LES ? 19 : 27;
  L->N = (size_t)c.nx * c.ny * c.nz;
  L->elem = c.storage == LBM_F64 ? 8 : (c.storage == LBM_F32 ? 4 : 2);
  L->stream = (hipStream_t)c.stream;
  launch_shape(L);
  // memory layout: populations | outflow ghost plane (one z plane) |
  // reduction partials | result
  const size_t face = (size_t)c.nx * c.ny;
  L->ghost_n_max = face;
  L->off_ghost = align256(L->N * L->Q * L->elem);
  L->off_partial = L->off_ghost + align256(face * L->Q * L->elem);
  L->off_result = L->off_partial + align256(L->nblocks * 5 * sizeof(double));
  L->req = L->off_result + 256;
  // arguments
  LatArgs& a = L->args;
  std::memset(&a, 0, sizeof(a));
  a.nx = c.nx;
  a.ny = c.ny;
  a.nz = c.nz;
  a.N = (long long)L->N;
  const double tau0 = 3.0 * c.nu + 0.5;
  a.mrt.tau0 = tau0;
  a.mrt.cs18 = 18.0 * c.cs_smag * c.cs_smag;
  a.omega = 1.0 / tau0;
  if (c.model == LBM_D3Q19_MRT_LES) {
    if (c.use_default_rates) {
      const double t1[5] = {1.0, 1.0, 1.0, 1.0, 1.0};
      const double dh[5] = {1.19, 1.4, 1.2, 1.4, 1.98};
      for (int k = 0; k < 5; ++k)
        a.mrt.rates[k] = c.mrt_basis == LBM_BASIS_TABLE1 ? t1[k] : dh[k];
    } else {
      for (int k = 0; k < 5; ++k) a.mrt.rates[k] = c.rates[k];
    }
  }
  default_bc(a.bc);
  plan_rows(L);
  *out = L;
  return LBM_OK;
}

int lbm_required_bytes(const lbm_lattice* L, size_t* bytes) {
  if (!L || !bytes) return LBM_EINVAL;
  *bytes = L->req;
  return LBM_OK;
}

int lbm_bind_memory(lbm_lattice* L, void* dev, size_t bytes) {
  if (!L || !dev) return LBM_EINVAL;
  if (((uintptr_t)dev & 255) != 0) return LBM_EINVAL;
  if (bytes < L->req) return LBM_ENOMEM;
  L->base = (char*)dev;
  L->bytes = bytes;
  L->args.f = L->base;
  L->args.ghost = L->base + L->off_ghost;
  L->t = 0;
  L->parity = 0;
  return LBM_OK;
}

int lbm_set_stream(lbm_lattice* L, void* stream) {
  if (!L) return LBM_EINVAL;
  L->stream = (hipStream_t)stream;
  return LBM_OK;
}

int lbm_set_boundaries(lbm_lattice* L, const lbm_boundaries* bc) {
  if (!L || !bc) return LBM_EINVAL;
  if (L->parity != 0) return LBM_ESTATE;
  const int n3[3] = {L->cfg.nx, L->cfg.ny, L->cfg.nz};
  BcArgs b;
  default_bc(b);
  int n_inlet = 0, n_out = 0;
  for (int f = 0; f < 6; ++f) {
    const int ty = bc->face_type[f];
    if (ty < LBM_PERIODIC || ty > LBM_PRESSURE) return LBM_EINVAL;
    if (ty != LBM_PERIODIC) {
      b.nonper |= 1u << f;
      if (n3[f / 2] < 2) return LBM_EINVAL;
    }
    for (int k = 0; k < 3; ++k) {
      if (!std::isfinite(bc->face_u[f][k])) return LBM_EINVAL;
      b.face_u[f][k] = bc->face_u[f][k];
    }
    if (ty == LBM_WALL) b.wall |= 1u << f;
    if (ty == LBM_FREESLIP) b.freeslip |= 1u << f;
    if (ty == LBM_PRESSURE) {
      if (!std::isfinite(bc->face_drho[f]) || !(bc->face_drho[f] > -1.0)) return LBM_EINVAL;
      b.pressure |= 1u << f;
      b.face_drho[f] = bc->face_drho[f];
    }
    if (ty == LBM_INLET) {
      b.inlet |= 1u << f;
      b.inlet_axis = f / 2;
      ++n_inlet;
    }
    if (ty == LBM_OUTFLOW) {
      if (f / 2 != 2) return LBM_EINVAL;  // outflow faces are z faces
      b.outflow |= 1u << f;
      ++n_out;
    }
  }
  for (int d = 0; d < 3; ++d) {
    const bool lo = (b.nonper >> (2 * d)) & 1u, hi = (b.nonper >> (2 * d + 1)) & 1u;
    if (lo != hi) return LBM_EINVAL;  // faces of one axis: both periodic or neither
  }
  if (n_inlet > 1 || n_out > 1) return LBM_EINVAL;
  if (n_inlet) {
    if (!bc->inlet_u || !valid_dtype(bc->inlet_dtype)) return LBM_EINVAL;
    if (!std::isfinite(bc->inlet_amp)) return LBM_EINVAL;
    b.inlet_u = bc->inlet_u;
    b.inlet_f64 = bc->inlet_dtype == LBM_DTYPE_F64;
    b.inlet_mask = bc->inlet_mask;
    b.inlet_amp = bc->inlet_amp;
    b.seed = bc->seed;
    const int d = b.inlet_axis;
    b.inlet_na = n3[d == 0 ? 1 : 0];
    b.inlet_nb = n3[d == 2 ? 1 : 2];
    if (b.inlet_na >= 16384 || b.inlet_nb >= 16384) return LBM_EINVAL;
  }
  if (n_out) b.ghost_n = (long long)n3[0] * n3[1];
  fill_wall_terms(b, L->Q);
  L->args.bc = b;
  L->args.solid_nb = nullptr;  // new boundaries clear the solids and links
  L->solids = false;
  L->link_nodes = nullptr;
  L->link_q = nullptr;
  L->nlinks = 0;
  L->has_bc = b.nonper != 0;
  plan_rows(L);
  return LBM_OK;
}

int lbm_init_equilibrium(lbm_lattice* L, const void* drho, const void* u, int dtype,
                         int64_t t0) {
  if (!L || !drho || !u || !valid_dtype(dtype)) return LBM_EINVAL;
  if (!L->base) return LBM_EUNBOUND;
  by_storage(L, [&](auto s) {
    Ops<decltype(s)>::init_equilibrium(L, drho, u, dtype == LBM_DTYPE_F64);
  });
  const int rc = check_launch();
  if (rc) return rc;
  L->t = t0;
  L->parity = 0;
  return LBM_OK;
}

int lbm_set_populations(lbm_lattice* L, const void* f, int dtype, int64_t t0) {
  if (!L || !f || !valid_dtype(dtype)) return LBM_EINVAL;
  if (!L->base) return LBM_EUNBOUND;
  by_storage(L, [&](auto s) { Ops<decltype(s)>::set_populations(L, f, dtype == LBM_DTYPE_F64); });
  const int rc = check_launch();
  if (rc) return rc;
  L->t = t0;
  L->parity = 0;
  return LBM_OK;
}

int lbm_get_populations(lbm_lattice* L, void* f, int dtype) {
  if (!L || !f || !valid_dtype(dtype)) return LBM_EINVAL;
  if (!L->base) return LBM_EUNBOUND;
  by_storage(L, [&](auto s) { Ops<decltype(s)>::get_populations(L, f, dtype == LBM_DTYPE_F64); });
  return check_launch();
}

int lbm_step(lbm_lattice* L, int64_t n) {
  if (!L || n < 0) return LBM_EINVAL;
  if (!L->base) return LBM_EUNBOUND;
  for (int64_t k = 0; k < n; ++k) {
    by_storage(L, [&](auto s) {
      Ops<decltype(s)>::step(L, L->parity == 1, (long long)L->t, nullptr);
    });
    if (L->nlinks > 0)
      by_storage(L, [&](auto s) { Ops<decltype(s)>::links(L, L->parity == 1); });
    L->t += 1;
    L->parity ^= 1;
    if (L->check_every > 0 && L->t % L->check_every == 0) {
      const int rc = run_check(L);
      if (rc) return rc;
    }
  }
  return check_launch();
}

int lbm_step_record(lbm_lattice* L, void* rec, int dtype) {
  if (!L || !rec || !valid_dtype(dtype)) return LBM_EINVAL;
  if (!L->base) return LBM_EUNBOUND;
  if (L->kind > 2 || L->cfg.storage == LBM_F16 || L->solids || L->args.bc.freeslip ||
      L->args.bc.pressure)
    return LBM_EINVAL;
  if (dtype != (L->cfg.storage == LBM_F64 ? LBM_DTYPE_F64 : LBM_DTYPE_F32)) return LBM_EINVAL;
  by_storage(L, [&](auto s) {
    Ops<decltype(s)>::step(L, L->parity == 1, (long long)L->t, rec);
  });
  L->t += 1;
  L->parity ^= 1;
  return check_launch();
}

int lbm_get_macroscopic(lbm_lattice* L, void* rho, void* u, int dtype, int rho_mode) {
  if (!L || !valid_dtype(dtype)) return LBM_EINVAL;
  if (rho_mode != LBM_RHO_FULL && rho_mode != LBM_RHO_DEVIATION) return LBM_EINVAL;
  if (!L->base) return LBM_EUNBOUND;
  if (!rho && !u) return LBM_OK;
  by_storage(L, [&](auto s) {
    Ops<decltype(s)>::macroscopic(L, rho, u, dtype == LBM_DTYPE_F64, rho_mode);
  });
  return check_launch();
}

int lbm_set_solids(lbm_lattice* L, const uint8_t* solid, uint32_t* masks) {
  if (!L) return LBM_EINVAL;
  if (!L->base) return LBM_EUNBOUND;
  if (L->parity != 0) return LBM_ESTATE;
  L->args.solid_nb = nullptr;
  L->solids = false;
  L->link_nodes = nullptr;  // new solids clear the links
  L->link_q = nullptr;
  L->nlinks = 0;
  L->has_bc = L->args.bc.nonper != 0;
  if (solid) {
    if (!masks) return LBM_EINVAL;
    int* flag = (int*)(L->base + L->off_result);
    hipError_t e = hipMemsetAsync(flag, 0, sizeof(int), L->stream);
    if (e != hipSuccess) return hip_fail(e);
    if (L->Q == 27)
      hipLaunchKernelGGL((solid_mask_kernel<27>), L->grid, L->block, 0, L->stream, L->args, solid,
                         masks, flag);
    else
      hipLaunchKernelGGL((solid_mask_kernel<19>), L->grid, L->block, 0, L->stream, L->args, solid,
                         masks, flag);
    const int rc = check_launch();
    if (rc) return rc;
    int bad = 0;
    e = hipMemcpyAsync(&bad, flag, sizeof(int), hipMemcpyDeviceToHost, L->stream);
    if (e != hipSuccess) return hip_fail(e);
    e = hipStreamSynchronize(L->stream);
    if (e != hipSuccess) return hip_fail(e);
    if (bad) {
      plan_rows(L);
      return LBM_EINVAL;
    }
    L->args.solid_nb = masks;
    L->solids = true;
    L->has_bc = true;
  }
  plan_rows(L);
  return LBM_OK;
}

int lbm_set_links(lbm_lattice* L, const int32_t* nodes, const float* q, int64_t n) {
  if (!L || n < 0 || n >= ((int64_t)1 << 31)) return LBM_EINVAL;
  if (!L->base) return LBM_EUNBOUND;
  if (L->parity != 0) return LBM_ESTATE;
  if (n > 0 && (!nodes || !q || !L->solids)) return LBM_EINVAL;
  L->link_nodes = n > 0 ? nodes : nullptr;
  L->link_q = n > 0 ? q : nullptr;
  L->nlinks = n;
  return LBM_OK;
}

int lbm_stats_accumulate(lbm_lattice* L, double* sums) {
  if (!L || !sums) return LBM_EINVAL;
  if (!L->base) return LBM_EUNBOUND;
  by_storage(L, [&](auto s) { Ops<decltype(s)>::stats_accumulate(L, sums); });
  return check_launch();
}

int lbm_stats_finalize(const lbm_lattice* L, const double* sums, int64_t count, void* mean,
                       void* rms, void* ti, int dtype, int axis, int p0, int p1) {
  if (!L || !sums || !mean || !rms || !valid_dtype(dtype) || count < 1) return LBM_EINVAL;
  if (axis < 0 || axis > 2) return LBM_EINVAL;
  const int n3[3] = {L->cfg.nx, L->cfg.ny, L->cfg.nz};
  const int o0 = axis == 0 ? 1 : 0, o1 = axis == 2 ? 1 : 2;
  if (ti && (p0 < 0 || p0 >= n3[o0] || p1 < 0 || p1 >= n3[o1])) return LBM_EINVAL;
  const double inv = 1.0 / (double)count;
  if (dtype == LBM_DTYPE_F64)
    hipLaunchKernelGGL((stats_finalize_kernel<double>), L->grid, L->block, 0, L->stream, L->args,
                       sums, inv, (double*)mean, (double*)rms, (double*)ti, axis, p0, p1);
  else
    hipLaunchKernelGGL((stats_finalize_kernel<float>), L->grid, L->block, 0, L->stream, L->args,
                       sums, inv, (float*)mean, (float*)rms, (float*)ti, axis, p0, p1);
  return check_launch();
}

int lbm_jet_profile(const lbm_lattice* L, const void* mean, int dtype, int axis, double c0,
                    double c1, int ndir, double dr, int nr, double* um, double* re,
                    double* prof) {
  if (!L || !mean || !um || !re || !valid_dtype(dtype)) return LBM_EINVAL;
  if (axis < 0 || axis > 2 || ndir < 1 || ndir > 65536 || nr < 2 || nr > 65536) return LBM_EINVAL;
  if (!std::isfinite(dr) || !(dr > 0.0)) return LBM_EINVAL;
  const long long nx = L->cfg.nx, ny = L->cfg.ny, nz = L->cfg.nz;
  JetSections s{};
  s.comp = axis * nx * ny * nz;
  if (axis == 2) {
    s.sp = nx * ny, s.sa = 1, s.sb = nx, s.np = (int)nz, s.na = (int)nx, s.nb = (int)ny;
  } else if (axis == 1) {
    s.sp = nx, s.sa = 1, s.sb = nx * ny, s.np = (int)ny, s.na = (int)nx, s.nb = (int)nz;
  } else {
    s.sp = 1, s.sa = nx, s.sb = nx * ny, s.np = (int)nx, s.na = (int)ny, s.nb = (int)nz;
  }
  if (s.na < 2 || s.nb < 2) return LBM_EINVAL;
  if (!(c0 >= 0.0 && c0 <= s.na - 1 && c1 >= 0.0 && c1 <= s.nb - 1)) return LBM_EINVAL;
  if (dtype == LBM_DTYPE_F64)
    hipLaunchKernelGGL((jet_profile_kernel<double>), dim3(s.np), dim3(256), 0, L->stream,
                       (const double*)mean, s, c0, c1, ndir, dr, nr, um, re, prof);
  else
    hipLaunchKernelGGL((jet_profile_kernel<float>), dim3(s.np), dim3(256), 0, L->stream,
                       (const float*)mean, s, c0, c1, ndir, dr, nr, um, re, prof);
  return check_launch();
}

int lbm_jet_fit(const lbm_lattice* L, const double* um, const double* re, const double* prof,
                int np, int nr, double dr, double x0, double u0, double d, int p0, int p1,
                double* out) {
  if (!L || !um || !re || !prof || !out) return LBM_EINVAL;
  if (np < 1 || nr < 1 || p0 < 0 || p1 > np || p0 >= p1) return LBM_EINVAL;
  if (!std::isfinite(dr) || !(dr > 0.0) || !std::isfinite(x0) || !std::isfinite(u0) ||
      !(u0 != 0.0) || !std::isfinite(d) || !(d > 0.0))
    return LBM_EINVAL;
  hipLaunchKernelGGL(jet_fit_kernel, dim3(1), dim3(256), 0, L->stream, um, re, prof, np, nr, dr,
                     x0, u0, d, p0, p1, out);
  return check_launch();
}

int lbm_reduce(lbm_lattice* L, double out[5]) {
  if (!L || !out) return LBM_EINVAL;
  if (!L->base) return LBM_EUNBOUND;
  return reduce_now(L, out);
}

int lbm_set_check(lbm_lattice* L, int64_t every, double mass_tol) {
  if (!L || every < 0 || std::isnan(mass_tol)) return LBM_EINVAL;
  if (!L->base) return LBM_EUNBOUND;
  L->check_every = every;
  L->check_tol = mass_tol;
  L->check_m0 = 0.0;
  if (every > 0) {  // the current state is checked at once
    double out[5];
    const int rc = reduce_now(L, out);
    if (rc) {
      L->check_every = 0;
      return rc;
    }
    L->check_m0 = out[0];
  }
  return LBM_OK;
}

int lbm_reduce_static(lbm_lattice* L, double* out) {
  if (!L || !out) return LBM_EINVAL;
  if (!L->base) return LBM_EUNBOUND;
  const size_t plane = (size_t)L->grid.x * L->grid.y;
  if (plane > kStaticPartials) return LBM_EINVAL;
  double* partial = nullptr;
  int rc = static_scratch(L->stream, &partial);
  if (rc) return rc;
  const unsigned nb = reduce_blocks(L);
  by_storage(L, [&](auto s) { Ops<decltype(s)>::reduce_partial(L, nb, partial); });
  rc = check_launch();
  if (rc) return rc;
  hipLaunchKernelGGL(reduce_final_kernel, dim3(1), dim3(256), 0, L->stream, partial,
                     (size_t)nb, out);
  return check_launch();
}

int lbm_state_bytes(const lbm_lattice* L, size_t* bytes) {
  if (!L || !bytes) return LBM_EINVAL;
  *bytes = L->off_partial;
  return LBM_OK;
}

int lbm_save_state(lbm_lattice* L, void* dev, size_t bytes, int64_t* t, int32_t* parity) {
  if (!L || !dev) return LBM_EINVAL;
  if (!L->base) return LBM_EUNBOUND;
  if (bytes < L->off_partial) return LBM_ENOMEM;
  const hipError_t e =
      hipMemcpyAsync(dev, L->base, L->off_partial, hipMemcpyDeviceToDevice, L->stream);
  if (e != hipSuccess) return hip_fail(e);
  if (t) *t = L->t;
  if (parity) *parity = L->parity;
  return LBM_OK;
}

int lbm_load_state(lbm_lattice* L, const void* dev, size_t bytes, int64_t t, int32_t parity) {
  if (!L || !dev || (parity != 0 && parity != 1)) return LBM_EINVAL;
  if (!L->base) return LBM_EUNBOUND;
  if (bytes < L->off_partial) return LBM_ENOMEM;
  const hipError_t e =
      hipMemcpyAsync(L->base, dev, L->off_partial, hipMemcpyDeviceToDevice, L->stream);
  if (e != hipSuccess) return hip_fail(e);
  L->t = t;
  L->parity = parity;
  return LBM_OK;
}

int lbm_get_time(const lbm_lattice* L, int64_t* t) {
  if (!L || !t) return LBM_EINVAL;
  *t = L->t;
  return LBM_OK;
}

int lbm_destroy(lbm_lattice* L) {
  if (L) L->tracer->report("lattice");
  delete L;
  return LBM_OK;
}

int lbm_probe_ke(lbm_lattice* L, const int32_t lo[3], const int32_t hi[3], void* lambda,
                 int dtype, double* J) {
  if (!L || !lo || !hi || !J || !valid_dtype(dtype)) return LBM_EINVAL;
  if (!L->base) return LBM_EUNBOUND;
  const int n3[3] = {L->cfg.nx, L->cfg.ny, L->cfg.nz};
  for (int d = 0; d < 3; ++d)
    if (lo[d] < 0 || hi[d] > n3[d] || lo[d] >= hi[d]) return LBM_EINVAL;
  const double scale = 1.0 / ((double)(hi[0] - lo[0]) * (hi[1] - lo[1]) * (hi[2] - lo[2]));
  double* partial = (double*)(L->base + L->off_partial);
  double* result = (double*)(L->base + L->off_result);
  const int3 l3 = make_int3(lo[0], lo[1], lo[2]), h3 = make_int3(hi[0], hi[1], hi[2]);
  by_storage(L, [&](auto s) {
    Ops<decltype(s)>::probe(L, l3, h3, scale, lambda, dtype == LBM_DTYPE_F64, partial);
  });
  int rc = check_launch();
  if (rc) return rc;
  hipLaunchKernelGGL(reduce_final_kernel, dim3(1), dim3(256), 0, L->stream, partial,
                     L->nblocks, result);
  rc = check_launch();
  if (rc) return rc;
  hipError_t e = hipMemcpyAsync(J, result, sizeof(double), hipMemcpyDeviceToHost, L->stream);
  if (e != hipSuccess) return hip_fail(e);
  e = hipStreamSynchronize(L->stream);
  if (e != hipSuccess) return hip_fail(e);
  return std::isfinite(*J) ? LBM_OK : LBM_ENONFINITE;
}

int lbm_adjoint_step(lbm_lattice* L, const void* f_t, const void* lambda_next, void* lambda,
                     int dtype, double* grad_inlet) {
  if (!L || !f_t || !lambda_next || !lambda || !valid_dtype(dtype)) return LBM_EINVAL;
  if (L->kind > 2 || L->solids || L->args.bc.freeslip || L->args.bc.pressure)
    return LBM_EINVAL;
  if (lambda == lambda_next || lambda == f_t) return LBM_EINVAL;
  // the kernels address the adjoint arrays with 32-bit byte offsets: one
  // slab must stay below 4 GiB, and the wall rows (a population and its
  // opposite from the lower slab) need the whole span below 4 GiB, else the
  // general kernel takes every row
  const double rsz = dtype == LBM_DTYPE_F64 ? 8.0 : 4.0;
  if ((double)L->N * rsz >= 4294967296.0) return LBM_EINVAL;
  const int Q = L->kind == 2 ? 27 : 19;
  const bool split = L->split_odd && slab_span(Q) * (double)L->N * rsz < 4294967296.0;
  TraceScope ts(L->tracer.get(), L->stream, "adjoint step (adjoint_kernel launches)");
  auto run = [&](auto kind_c, auto real_tag) {
    constexpr int K = decltype(kind_c)::value;
    using R = typename decltype(real_tag)::type;
    const R* f = (const R*)f_t;
    const R* ln = (const R*)lambda_next;
    R* l = (R*)lambda;
    const dim3 block(256), all(L->tiles_all), both(L->rows_odd.list_tiles + L->tiles_inner);
    if (!L->has_bc) {
      hipLaunchKernelGGL((adjoint_kernel<K, R, BC_NONE, ROWS_FLAT>), all, block, 0, L->stream,
                         L->args, L->rows_all, f, ln, l, grad_inlet);
    } else if (!split) {
      hipLaunchKernelGGL((adjoint_kernel<K, R, BC_GENERAL, ROWS_FLAT>), all, block, 0, L->stream,
                         L->args, L->rows_all, f, ln, l, grad_inlet);
    } else {
      if constexpr (std::is_same_v<R, double>) {
        // Without listed rows FP64 leaves the general rules' registers out (64^3
        // channel FCLB 34.9 to 33.0 us, MRT 22.4 to 21.3, 94x73x33 33.8 to 31.0,
        // 21.8 to 20.6; from 128^3 on within 2 %). FP32 has room for them and is
        // slower apart (131x97x211 MRT 134 and 145 us).
        if (L->rows_odd.list_tiles == 0) {
          hipLaunchKernelGGL((adjoint_kernel<K, R, BC_WALLS, ROWS_FLAT>), dim3(L->tiles_inner),
                             block, 0, L->stream, L->args, L->rows_odd, f, ln, l, grad_inlet);
          return;
        }
      }
      hipLaunchKernelGGL((adjoint_kernel<K, R, BC_WALLS, ROWS_SPLIT>),
                         both, block, 0, L->stream,
                         L->args, L->rows_odd, f, ln, l, grad_inlet);
    }
  };
  auto by_type = [&](auto kind_c) {
    if (dtype == LBM_DTYPE_F64)
      run(kind_c, std::type_identity<double>{});
    else
      run(kind_c, std::type_identity<float>{});
  };
  switch (L->kind) {
    case 0: by_type(std::integral_constant<int, 0>{}); break;
    case 1: by_type(std::integral_constant<int, 1>{}); break;
    default: by_type(std::integral_constant<int, 2>{}); break;
  }
  return check_launch();
}

int lbm_stream_copy(void* dst, const void* src, size_t n, void* stream) {
  if (!dst || !src || (((uintptr_t)dst | (uintptr_t)src | n) & 15) != 0) return LBM_EINVAL;
  const size_t n16 = n / 16;
  if (n16 == 0) return LBM_OK;
  const size_t blocks = (n16 + 255) / 256;
  if (blocks > 0x7fffffffu) return LBM_EINVAL;
  hipLaunchKernelGGL(copy_kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream,
                     (u32x4*)dst, (const u32x4*)src, n16);
  return check_launch();
}

}  // extern "C"
