// Launches of the kernels that depend on the storage type of a lattice, over
// model x step parity x boundary handling. Compiled once per type, with
// LBM_STORAGE set to it.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>
#include <type_traits>

#include "adjoint.h"
#include "lattice.h"

using namespace lbm;

namespace {

// LDS requested by a step's workgroups beyond the last-level cache, only to
// limit how many run on a CU (160 KB). These steps are bound by HBM, two
// workgroups per CU already keep it busy, and the fewer nodes are in flight
// the fewer DRAM pages are open at once. FP32 256x256x512 by workgroups per
// CU 5 (registers) / 3 / 2, us: FCLB even 1274 / 1227 / 1185, odd 1361 / 1326
// / 1276, odd with walls 1381 / 1368 / 1499 (their address arithmetic needs
// the third); MRT even 863 / 825 / 849, odd 926 / 866 / 862, with walls 932 /
// 916 / 933. FP64 256^3: FCLB even 1282 / 1280 / 1246, odd 1408 / 1390 / 1365,
// with walls 1400 / 1386 / 1383; MRT 859 / 857 / 836, 949 / 940 / 920, 970 /
// 960 / 939. FP16 is bound by arithmetic: none (FCLB even 607 / 605 / 768, odd
// with walls 763 / 864 / 1152), and so are wall rows with solids (128x128x256
// FCLB FP32 159 / 178 us). Within the last-level cache nothing is gained.
template <int KIND, typename S, bool WALLS, bool SOLID>
unsigned lds_limit(const lbm_lattice* L) {
  if (std::is_same_v<S, _Float16> || L->resident || (WALLS && SOLID)) return 0;
  const bool two = std::is_same_v<S, double> || (KIND >= 2 && !WALLS);
  return (two ? 64u : 52u) * 1024u;
}

template <int KIND, typename S, bool ODD, int BCM, int ROWS, bool EXT, bool NT>
void launch_step(const lbm_lattice* L, dim3 grid, dim3 block, const Rows& r, long long t,
                 void* rec) {
  TraceScope ts(L->tracer.get(), L->stream, LBM_TRACE_LABEL("step_kernel"));
  hipLaunchKernelGGL((step_kernel<KIND, S, ODD, BCM, ROWS, EXT, NT>), grid, block,
                     (ROWS == ROWS_LIST ? 0u
                                        : lds_limit<KIND, S, BCM == BC_WALLS,
                                                    EXT && ROWS == ROWS_FLAT>(L)), L->stream,
                     L->args, r, t, (typename Compute<S>::type*)rec);
}

template <int KIND, typename S, bool EXT, bool NT>
void step_model_ext(const lbm_lattice* L, bool odd, long long t, void* rec) {
  const dim3 block(256), grid(L->tiles_all);
  if (!L->has_bc) {
    if (odd)
      launch_step<KIND, S, true, BC_NONE, ROWS_FLAT, false, NT>(L, grid, block, L->rows_all, t,
                                                                rec);
    else
      launch_step<KIND, S, false, BC_NONE, ROWS_FLAT, false, NT>(L, grid, block, L->rows_all, t,
                                                                 rec);
  } else if (!odd) {
    launch_step<KIND, S, false, BC_GENERAL, ROWS_FLAT, EXT, NT>(L, grid, block, L->rows_all, t,
                                                                rec);
  } else if (!L->split_odd) {
    launch_step<KIND, S, true, BC_GENERAL, ROWS_FLAT, EXT, false>(L, grid, block, L->rows_all, t,
                                                                  rec);
  } else {
    // One launch, except in FP16 (256x256x512 FCLB 805 us, apart 763 + 16) and
    // with the rules of EXT, whose registers spill beside the wall rows: they
    // win on a large lattice (96x112x224 MRT FP32 tank, ten steps 722 us against
    // 741) but cost on small ones (94x73x33, ten steps: FCLB 353 us against 192,
    // MRT 200 against 142). Without EXT one launch is the faster at every size
    // where rows are listed, though the wall rows keep three waves in FP32 and
    // two in FP64 beside the general rules and FCLB and CLB FP32 spill there too
    // (jet, us per step in one / two launches: 16^3 FCLB FP32 7.7 / 9.7, MRT
    // FP64 5.7 / 9.2, 64^3 FCLB FP32 13.7 / 14.0, FP64 20.7 / 25.6, MRT FP32 7.9
    // / 10.6, 131x97x211 110 / 115, 243 / 253, 62 / 67).
    // Where no row is listed the rules cost nothing to speak of (channel, with /
    // without them: 64^3 FCLB FP32 8.8 / 8.4, FP64 19.4 / 19.5, MRT FP32 8.2 /
    // 7.9; 100x75x110 29.1 / 28.9, 54.5 / 54.5, 21.3 / 21.0; 192x160x200 224 /
    // 225, 462 / 462, 150 / 151).
    const Rows& r = L->rows_odd;
    const dim3 inner(L->tiles_inner), list(r.list_tiles), both(r.list_tiles + L->tiles_inner);
    if constexpr (!EXT && !std::is_same_v<S, _Float16>) {
      launch_step<KIND, S, true, BC_WALLS, ROWS_SPLIT, false, NT>(L, both, block, r, t, rec);
    } else {
      if (inner.x > 0) {
        if (EXT && L->solids)
          launch_step<KIND, S, true, BC_WALLS, ROWS_FLAT, EXT, NT>(L, inner, block, r, t, rec);
        else
          launch_step<KIND, S, true, BC_WALLS, ROWS_FLAT, false, NT>(L, inner, block, r, t, rec);
      }
      if (list.x > 0)
        launch_step<KIND, S, true, BC_GENERAL, ROWS_LIST, EXT, false>(L, list, block, r, t, rec);
    }
  }
}

// Lattices without interior solids, FREESLIP or PRESSURE faces run the
// general kernel compiled without their rules. The even step touches only
// each node's own slots, which no other node reads: solid nodes may run it
// (their populations are never read) and free slip has no even-step rule,
// so there the rules are compiled in only for PRESSURE faces.
template <int KIND, typename S>
void step_model(const lbm_lattice* L, bool odd, long long t, void* rec) {
  const bool ext = odd ? (L->solids || L->args.bc.freeslip || L->args.bc.pressure)
                       : L->args.bc.pressure != 0;
  const bool nt = odd ? L->nt_odd : L->nt_even;
  if constexpr (std::is_same_v<S, _Float16>) {
    // FP16 even steps: two nodes per lane
    if (!odd && !ext && rec == nullptr && L->N % 2 == 0) {
      const dim3 block(256), grid((unsigned)((L->N / 2 + 255) / 256));
      const bool by_xcd = L->rows_all.by_xcd;
      TraceScope ts(L->tracer.get(), L->stream,
                    L->has_bc ? "step_even_pair_kernel (FP16, boundaries)"
                              : "step_even_pair_kernel (FP16)");
      auto go = [&](auto bc_c, auto nt_c) {
        hipLaunchKernelGGL((step_even_pair_kernel<KIND, decltype(bc_c)::value,
                                                  decltype(nt_c)::value>),
                           grid, block, 0, L->stream, L->args, by_xcd);
      };
      auto by_bc = [&](auto nt_c) {
        if (L->has_bc) go(std::true_type{}, nt_c);
        else go(std::false_type{}, nt_c);
      };
      if (nt) by_bc(std::true_type{});
      else by_bc(std::false_type{});
      return;
    }
  }
  auto by_nt = [&](auto ext_c) {
    if (nt)
      step_model_ext<KIND, S, decltype(ext_c)::value, true>(L, odd, t, rec);
    else
      step_model_ext<KIND, S, decltype(ext_c)::value, false>(L, odd, t, rec);
  };
  if (ext) by_nt(std::true_type{});
  else by_nt(std::false_type{});
}

// Runs fn<KIND, BC>() for the lattice's model.
template <typename Fn>
void with_model(const lbm_lattice* L, Fn&& fn) {
  auto by_bc = [&](auto kind_c) {
    if (L->has_bc)
      fn(kind_c, std::true_type{});
    else
      fn(kind_c, std::false_type{});
  };
  switch (L->kind) {
    case 0: by_bc(std::integral_constant<int, 0>{}); break;
    case 1: by_bc(std::integral_constant<int, 1>{}); break;
    case 3: by_bc(std::integral_constant<int, 3>{}); break;
    default: by_bc(std::integral_constant<int, 2>{}); break;
  }
}

// Runs fn(a value of the field type).
template <typename Fn>
void with_field(bool f64, Fn&& fn) {
  if (f64)
    fn(double());
  else
    fn(float());
}

// Runs fn(Q, odd parity, boundaries, streaming hint, ReadArgs) for a readout.
// The hint at even parity, whose accesses run from end to end, on lattices
// larger than the last-level cache: by `hint`, over a third larger except for
// the populations themselves. Up to there enough of them is still cached
// (density and velocity after two steps with / without it, us: 270 MiB MRT
// FP32 161x153x151 67.5 / 57.9, 304 MiB MRT FP64 128^3 68 / 55; 383 MiB FCLB
// FP32 161x153x151 71 / 118; statistics 129 / 115, 97 / 77; 134 / 192; the
// populations' copy 108 / 108, 96 / 101; 122 / 140). Workgroups per CU are not limited here: fewer
// cost (256x256x512 FCLB FP16, density and velocity: 382 us; 455 us with
// three).
template <typename Fn>
void with_read(const lbm_lattice* L, bool hint, Fn&& fn) {
  ReadArgs r;
  r.rows = L->rows_all;
  r.t = (long long)L->t;
  const BcArgs& bc = L->args.bc;
  r.general = L->split_odd ? bc.nonper & ~(bc.wall & 15u) : ALL_GENERAL;
  auto go = [&](auto q_c, auto odd_c, auto bc_c) {
    if constexpr (!decltype(odd_c)::value) {
      if (hint) {
        fn(q_c, odd_c, bc_c, std::true_type{}, r);
        return;
      }
    }
    fn(q_c, odd_c, bc_c, std::false_type{}, r);
  };
  auto by_bc = [&](auto q_c, auto odd_c) {
    if (L->has_bc) go(q_c, odd_c, std::true_type{});
    else go(q_c, odd_c, std::false_type{});
  };
  auto by_parity = [&](auto q_c) {
    if (L->parity) by_bc(q_c, std::true_type{});
    else by_bc(q_c, std::false_type{});
  };
  if (L->Q == 27) by_parity(std::integral_constant<int, 27>{});
  else by_parity(std::integral_constant<int, 19>{});
}

}  // namespace

namespace lbm {

template <typename S>
void Ops<S>::step(const lbm_lattice* L, bool odd, long long t, void* rec) {
  switch (L->kind) {
    case 0: step_model<0, S>(L, odd, t, rec); break;
    case 1: step_model<1, S>(L, odd, t, rec); break;
    case 3: step_model<3, S>(L, odd, t, rec); break;
    default: step_model<2, S>(L, odd, t, rec); break;
  }
}

// Interpolated bounce-back over the link list after a step.
template <typename S>
void Ops<S>::links(const lbm_lattice* L, bool after_odd) {
  const dim3 grid((unsigned)((L->nlinks + 7) / 8)), block(256);  // 32 lanes per node
  TraceScope ts(L->tracer.get(), L->stream, "link_kernel (interpolated bounce-back)");
  auto go = [&](auto q_c, auto odd_c) {
    constexpr int Q = decltype(q_c)::value;
    constexpr bool ODD = decltype(odd_c)::value;
    hipLaunchKernelGGL((link_kernel<Q, S, ODD>), grid, block, 0, L->stream, L->args,
                       L->link_nodes, L->link_q, L->nlinks);
  };
  if (L->Q == 27) {
    if (after_odd) go(std::integral_constant<int, 27>{}, std::true_type{});
    else go(std::integral_constant<int, 27>{}, std::false_type{});
  } else {
    if (after_odd) go(std::integral_constant<int, 19>{}, std::true_type{});
    else go(std::integral_constant<int, 19>{}, std::false_type{});
  }
}

template <typename S>
void Ops<S>::init_equilibrium(const lbm_lattice* L, const void* drho, const void* u, bool f64) {
  with_model(L, [&](auto kind_c, auto) {
    constexpr int KIND = decltype(kind_c)::value;
    with_field(f64, [&](auto v) {
      using O = decltype(v);
      hipLaunchKernelGGL((init_equilibrium_kernel<KIND, S, O>), L->grid, L->block, 0, L->stream,
                         L->args, (const O*)drho, (const O*)u);
    });
  });
}

template <typename S>
void Ops<S>::set_populations(const lbm_lattice* L, const void* f, bool f64) {
  with_field(f64, [&](auto v) {
    using O = decltype(v);
    if (L->Q == 27)
      hipLaunchKernelGGL((set_populations_kernel<27, S, O>), L->grid, L->block, 0, L->stream,
                         L->args, (const O*)f);
    else
      hipLaunchKernelGGL((set_populations_kernel<19, S, O>), L->grid, L->block, 0, L->stream,
                         L->args, (const O*)f);
  });
}

// The stores carry the streaming hint, except where lattice and output fit the
// last-level cache together and the output's slabs are not whole memory lines
// (a line that two waves write is then written once). Stores with / without
// it, us at even and odd parity: 111x93x121 FCLB FP16 (193 MiB) 49.5 / 34.8
// and 48.3 / 31.0, MRT FP32 (181 MiB) 30.5 / 28.8 and 32.6 / 28.9; whole lines,
// 64^3 FCLB FP32 7.3 / 10.4 and 9.2 / 9.2; 300 MiB, 90^3 FCLB FP64 45.9 / 53.5.
template <typename S>
void Ops<S>::get_populations(const lbm_lattice* L, void* f, bool f64) {
  const size_t osize = f64 ? 8 : 4;
  const bool keep = (L->N * osize) % 128 != 0 &&
                    (double)L->N * L->Q * (double)(sizeof(S) + osize) <= 256.0 * 1048576.0;
  with_read(L, !L->resident, [&](auto q_c, auto odd_c, auto bc_c, auto nt_c, const ReadArgs& r) {
    constexpr int Q = decltype(q_c)::value;
    constexpr bool BC = decltype(bc_c)::value, NT = decltype(nt_c)::value;
    auto by_field = [&](auto ont_c) {
      constexpr bool ONT = decltype(ont_c)::value;
      with_field(f64, [&](auto v) {
        using O = decltype(v);
        if constexpr (decltype(odd_c)::value) {
          hipLaunchKernelGGL((get_populations_kernel<Q, S, BC, O, ONT>), dim3(L->tiles_all),
                             dim3(256), 0, L->stream, L->args, r, (O*)f);
        } else {
          auto go = [&](auto solid_c) {
            constexpr bool HALF = std::is_same_v<S, _Float16>, SOLID = decltype(solid_c)::value;
            constexpr int G = HALF || (SOLID && Q == 19) ? (Q == 27 ? 9 : 19) : (SOLID ? 3 : 1);
            constexpr int U = HALF || G > 3 ? 1 : (SOLID ? 2 : (NT ? 8 : 4));
            const dim3 grid((unsigned)((L->N + 256 * U - 1) / (256 * U)), Q / G);
            hipLaunchKernelGGL((get_slabs_kernel<S, SOLID, O, G, U, NT, ONT>), grid, dim3(256), 0,
                               L->stream, L->args, (O*)f);
          };
          if constexpr (BC) {
            if (L->solids) {
              go(std::true_type{});
              return;
            }
          }
          go(std::false_type{});
        }
      });
    };
    if constexpr (!NT) {  // what fits together is not read with the hint
      if (keep) {
        by_field(std::false_type{});
        return;
      }
    }
    by_field(std::true_type{});
  });
}

template <typename S>
void Ops<S>::macroscopic(const lbm_lattice* L, void* rho, void* u, bool f64, int rho_mode) {
  with_read(L, L->nt_read, [&](auto q_c, auto odd_c, auto bc_c, auto nt_c, const ReadArgs& r) {
    with_field(f64, [&](auto v) {
      using O = decltype(v);
      hipLaunchKernelGGL((macroscopic_kernel<decltype(q_c)::value, S, decltype(odd_c)::value,
                                             decltype(bc_c)::value, O, decltype(nt_c)::value>),
                         dim3(L->tiles_all), dim3(256), 0, L->stream, L->args, r, (O*)rho,
                         (O*)u, rho_mode);
    });
  });
}

template <typename S>
void Ops<S>::stats_accumulate(const lbm_lattice* L, double* sums) {
  with_read(L, L->nt_read, [&](auto q_c, auto odd_c, auto bc_c, auto nt_c, const ReadArgs& r) {
    hipLaunchKernelGGL((stats_accumulate_kernel<decltype(q_c)::value, S, decltype(odd_c)::value,
                                                decltype(bc_c)::value, decltype(nt_c)::value>),
                       dim3(L->tiles_all), dim3(256), 0, L->stream, L->args, r, sums);
  });
}

template <typename S>
void Ops<S>::reduce_partial(const lbm_lattice* L, unsigned blocks, double* partial) {
  with_read(L, L->nt_read, [&](auto q_c, auto odd_c, auto bc_c, auto nt_c, const ReadArgs& r) {
    hipLaunchKernelGGL((reduce_partial_kernel<decltype(q_c)::value, S, decltype(odd_c)::value,
                                              decltype(bc_c)::value, decltype(nt_c)::value>),
                       dim3(blocks), dim3(256), 0, L->stream, L->args, r, partial);
  });
}

template <typename S>
void Ops<S>::probe(const lbm_lattice* L, int3 lo, int3 hi, double scale, void* lambda, bool f64,
                   double* partial) {
  with_model(L, [&](auto kind_c, auto bc_c) {
    constexpr int KIND = decltype(kind_c)::value;
    constexpr bool BC = decltype(bc_c)::value;
    with_field(f64, [&](auto v) {
      using O = decltype(v);
      hipLaunchKernelGGL((probe_kernel<KIND, S, BC, O>), L->grid, L->block, 0, L->stream, L->args,
                         L->parity, (long long)L->t, lo, hi, scale, (O*)lambda, partial);
    });
  });
}

template struct Ops<LBM_STORAGE>;

}  // namespace lbm
