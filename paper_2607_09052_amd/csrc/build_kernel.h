// The block statistics build kernels, per (batch row, KV head, block) of LB
// tokens: one 64-thread wave per block (block_stats_wave: L = 32 or 64, r <= 4,
// full-space or subspace factors) or one 256-thread workgroup per block
// (block_stats on 32 columns: r > 4, or L = 128, where the 128 x 128 Gram matrix
// of unstructured keys has a flat top).
#pragma once

#include "block_stats.h"
#include "block_stats_wave.h"
#include "cobs_kernels.h"

namespace cobs {

constexpr int kWgColumns = 32;           // power-iteration columns of the four-wave routine

// Workgroups per CU (waves per SIMD) that the registers are fitted to, by the
// LDS that a block takes.  A block's serial parts (Cholesky on one wave, Jacobi's
// rounds) leave the CU to the others: 2,048 blocks of 128 tokens (d = 128,
// r = 4, bf16 keys) take 1,350 us with four (128 registers, 200 spilled, mostly
// the Gram matrix across the Cholesky) and 1,461 with three (43 spilled); they
// took 3,534 with one, which 107 KB of LDS allowed.
template <int D, int LB, bool KF32, bool SS>
constexpr int wg_build_waves() {
  if (SS) return 1;
  if (LB == 128) return !KF32 ? 4 : (D == 128 ? 2 : 3);
  return 3;
}

template <int D, int LB, bool KF32, bool SS, int WAVES, int P = kWgColumns>
__global__ __launch_bounds__(kBuildThreads, WAVES) void build_stats_kernel(BuildParams p) {
  constexpr size_t kPool = stats_lds_bytes<D, P, LB, KF32, SS>();
  constexpr size_t kProj = SS ? sizeof(float) * kProjectLdsFloats : 0;
  __shared__ __align__(16) char pool[kPool > kProj ? kPool : kProj];
  const int b = blockIdx.z, h = blockIdx.y;
  // the decode step's build with subspace factors also projects the queries
  // (the grid is one workgroup per (b, h) then, the condition uniform)
  if constexpr (SS) {
    if (p.qt) project_unit<D, kBuildThreads>(p.q, p.basis, p.qt, b, h, p.hq, p.g, p.fd, reinterpret_cast<float*>(pool));
  }
  const int T = clamp_len(p.seq_lens[b], p.tmax);
  if (T <= 0) return;
  const int nb = (T + LB - 1) / LB;
  const int j = p.tail_mode ? (T - 1) / LB : p.first_block + (int)blockIdx.x;
  if (j < 0 || j >= nb) return;
  StatsArgs a;
  a.kv = p.kv;
  a.rec = p.rec;
  a.hkv = p.hkv;
  a.nbmax = p.nbmax;
  a.r = p.r;
  a.mdt = p.mdt;
  a.fdt = p.fdt;
  a.skew = p.skew;
  a.vmean = p.vmean;
  a.lay = p.lay;
  a.basis = p.basis;
  a.fd = SS ? p.fd : D;
  block_stats<D, P, LB, KF32, SS>(a, b, h, j, min(LB, T - j * LB), pool);
}

template <size_t A, size_t B>
constexpr size_t size_max() { return A > B ? A : B; }

// Waves per SIMD that the registers are fitted to: the routine is bound by the
// latencies of its serial parts, so more blocks in flight pay up to what LDS holds
// (eleven waves per CU at L = 64, sixteen at L = 32); subspace factors of fp32 keys
// hold too many projected keys for three.  The step's single newest block
// (NT = 256) has the SIMD to itself.
template <int D, int LB, bool KF32, int FD, int NT>
constexpr int wave_build_waves() {
  if (NT > 64) return 2;
  if (LB == 32) return FD < D ? 3 : 4;
  return (FD < D && KF32) ? 2 : 3;
}

// One wave per (batch row, KV head, block) of LB tokens: the configurations
// of block_stats_wave (FD < D: subspace factors).  NT = 256: the decode step's
// build with subspace factors, whose four waves first project the queries
// (project_unit); then a partial newest block's means by all of them
// (block_mean_wg, bitwise the wave routine's record), a full one by wave 0.
template <int D, int LB, bool KF32, int FD = D, int NT = 64>
__global__ __launch_bounds__(NT, (wave_build_waves<D, LB, KF32, FD, NT>())) void build_stats_wave_kernel(BuildParams p) {
  constexpr size_t kPool = wave_stats_lds_bytes<D, LB>();
  constexpr size_t kProj = NT > 64 ? size_max<sizeof(float) * kProjectLdsFloats, block_mean_lds_bytes<D>()>() : 0;
  __shared__ __align__(16) char pool[size_max<kPool, kProj>()];
  const int b = blockIdx.z, h = blockIdx.y;
  if constexpr (NT > 64) {
    if (p.qt) project_unit<D, NT>(p.q, p.basis, p.qt, b, h, p.hq, p.g, p.fd, reinterpret_cast<float*>(pool));
    __syncthreads();                     // every wave is done with the pool
  }
  const int T = clamp_len(p.seq_lens[b], p.tmax);
  if (T <= 0) return;
  const int nb = (T + LB - 1) / LB;
  const int j = p.tail_mode ? (T - 1) / LB : p.first_block + (int)blockIdx.x;
  if (j < 0 || j >= nb) return;
  StatsArgs a;
  a.kv = p.kv;
  a.rec = p.rec;
  a.hkv = p.hkv;
  a.nbmax = p.nbmax;
  a.r = p.r;
  a.mdt = p.mdt;
  a.fdt = p.fdt;
  a.skew = p.skew;
  a.vmean = p.vmean;
  a.lay = p.lay;
  a.basis = FD < D ? p.basis : nullptr;
  a.fd = FD;
  const int n = min(LB, T - j * LB);
  if constexpr (NT > 64) {
    if (n < LB && !KF32) {
      block_mean_wg<D, LB>(a, b, h, j, n, pool);
      return;
    }
    if (threadIdx.x >= 64) return;
  }
  block_stats_wave<D, LB, KF32, false, FD>(a, b, h, j, n, pool);
}

// Subspace factors of FD elements on one wave per block (L = 32 or 64, r <= 4).
template <int D, int FD>
hipError_t launch_build_wave_ss(const BuildParams& p, dim3 grid, hipStream_t st) {
  const bool proj = p.qt != nullptr;
#define COBS_WAVE_SS(LB, KF)                                                                                   \
  if (proj) hipLaunchKernelGGL((build_stats_wave_kernel<D, LB, KF, FD, 256>), grid, dim3(256), 0, st, p);     \
  else hipLaunchKernelGGL((build_stats_wave_kernel<D, LB, KF, FD, 64>), grid, dim3(64), 0, st, p);
  if (p.kv.lsh == 5) {
    if (p.kv_f32) { COBS_WAVE_SS(32, true) } else { COBS_WAVE_SS(32, false) }
  } else {
    if (p.kv_f32) { COBS_WAVE_SS(64, true) } else { COBS_WAVE_SS(64, false) }
  }
#undef COBS_WAVE_SS
  return hipGetLastError();
}

template <int D>
hipError_t launch_build_wave(const BuildParams& p, dim3 grid, hipStream_t st) {
  if (p.kv.lsh == 5) {
    if (p.kv_f32) hipLaunchKernelGGL((build_stats_wave_kernel<D, 32, true>), grid, dim3(64), 0, st, p);
    else hipLaunchKernelGGL((build_stats_wave_kernel<D, 32, false>), grid, dim3(64), 0, st, p);
  } else {
    if (p.kv_f32) hipLaunchKernelGGL((build_stats_wave_kernel<D, 64, true>), grid, dim3(64), 0, st, p);
    else hipLaunchKernelGGL((build_stats_wave_kernel<D, 64, false>), grid, dim3(64), 0, st, p);
  }
  return hipGetLastError();
}

// With no more blocks than the device has CUs each workgroup has a CU to itself,
// and nothing is gained by fewer registers: a decode step over four units with
// blocks of 128 tokens takes 35.4 us on the four-to-a-CU form, 30.3 on this one (387
// and 356 when it fills the blocks).
template <int D, int LB, bool KF32, bool SS>
void launch_build_wg_as(const BuildParams& p, dim3 grid, hipStream_t st) {
  if ((int64_t)grid.x * grid.y * grid.z <= device_cus())
    hipLaunchKernelGGL((build_stats_kernel<D, LB, KF32, SS, 1>), grid, dim3(kBuildThreads), 0, st, p);
  else
    hipLaunchKernelGGL((build_stats_kernel<D, LB, KF32, SS, wg_build_waves<D, LB, KF32, SS>()>), grid,
                       dim3(kBuildThreads), 0, st, p);
}

// Launch over `grid` for the block length of p.kv.
template <int D, bool SS>
hipError_t launch_build_wg(const BuildParams& p, dim3 grid, hipStream_t st) {
  switch (p.kv.lsh) {
    case 5:
      if (p.kv_f32) launch_build_wg_as<D, 32, true, SS>(p, grid, st);
      else launch_build_wg_as<D, 32, false, SS>(p, grid, st);
      break;
    case 7:
      if (p.kv_f32) launch_build_wg_as<D, 128, true, SS>(p, grid, st);
      else launch_build_wg_as<D, 128, false, SS>(p, grid, st);
      break;
    default:
      if (p.kv_f32) launch_build_wg_as<D, 64, true, SS>(p, grid, st);
      else launch_build_wg_as<D, 64, false, SS>(p, grid, st);
  }
  return hipGetLastError();
}

}  // namespace cobs
