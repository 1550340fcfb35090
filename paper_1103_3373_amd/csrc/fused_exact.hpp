// Launch helpers of the fused kernels with the exact Riemann solver, shared by
// the two files that instantiate them.  Ghosted groups only.  The paper-style
// kernel, one workgroup of 256 threads per group with its face states in global
// memory, took 1,136 us a call for 16 groups (MHM, PLM, FP64, ghost fill included)
// against 85 here (16 workgroups per group).
#pragma once

#include "fused_muscl.hpp"
#include "fused_vlpred.hpp"
#include "riemann_exact.hpp"

namespace hy {
namespace exact_launch {

template <typename T>
hipError_t go(void (*k)(FusedArgs<T>), int threads, size_t shm, std::atomic<unsigned long long>& lds_set,
              const FusedArgs<T>& a, int grid, hipStream_t st) {
  const hipError_t e = raise_lds_limit((const void*)k, shm, lds_set);
  if (e != hipSuccess) return e;
  k<<<dim3(grid), dim3(threads), shm, st>>>(a);
  return hipGetLastError();
}

// SCHEME 0 MHM, 1 the VL second stage, 2 CTU; ZR 1 a group, 0 a chunk.
template <typename T, int SCHEME, bool PPM, int ZR>
hipError_t solve(const FusedArgs<T>& a, int grid, hipStream_t st) {
  constexpr int W = sizeof(T) == 8 ? 2 : 4;
  static std::atomic<unsigned long long> lds_set{0};
  if constexpr (SCHEME == 2)
    return go<T>(ctu::ctu_fused_kernel<T, PPM, 3, W, false, ZR, true>, fz::kThreads, ctu::kLdsBytes(sizeof(T)), lds_set, a,
                 grid, st);
  else
    return go<T>(muscl::muscl_kernel<T, PPM, 3, W, SCHEME, false, ZR, true>, fz::kThreads, muscl::kLdsBytes(sizeof(T)),
                 lds_set, a, grid, st);
}

template <typename T, bool PPM> hipError_t predict(const FusedArgs<T>& a, const FusedCfg& cfg, hipStream_t st) {
  constexpr int G = PPM ? 4 : 3;
  static std::atomic<unsigned long long> lds_set{0};
  FusedArgs<T> p = a;
  p.zsplit = cfg.zsplit_pred > 0 ? cfg.zsplit_pred : 1;
  return go<T>(vlpred::vl_predict_kernel<T, G, 3>, vlpred::threads<G>(), vlpred::lds_elems<G>() * sizeof(T), lds_set,
               p, cfg.grid_pred > 0 ? cfg.grid_pred : cfg.grid, st);
}

template <typename T, int SCHEME, bool PPM>
hipError_t run(const FusedArgs<T>& a, const FusedCfg& cfg, hipStream_t st) {
  if constexpr (SCHEME == 1) {
    if (!a.wstar || a.wstar_box) return hipErrorInvalidValue;
    const hipError_t e = predict<T, PPM>(a, cfg, st);
    if (e != hipSuccess) return e;
  }
  return a.zsplit > 1 ? solve<T, SCHEME, PPM, 0>(a, cfg.grid, st) : solve<T, SCHEME, PPM, 1>(a, cfg.grid, st);
}

template <typename T>
hipError_t launch(const FusedArgs<T>& a, int scheme, int recon, const FusedCfg& cfg, hipStream_t st) {
  if (a.zrun != 1) return hipErrorInvalidValue;
  switch (scheme * 2 + recon) {
    case 0: return run<T, 0, false>(a, cfg, st);
    case 1: return run<T, 0, true>(a, cfg, st);
    case 2: return run<T, 1, false>(a, cfg, st);
    case 3: return run<T, 1, true>(a, cfg, st);
    case 4: return run<T, 2, false>(a, cfg, st);
    case 5: return run<T, 2, true>(a, cfg, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace exact_launch
}  // namespace hy
