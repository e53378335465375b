// Size-independent kernels and the dispatch from a run-time probe side to the
// per-side launchers (instantiated in kernels_m32.hip, kernels_m64.hip and
// kernels_m128.hip).
#include "kernels.hpp"

namespace emg {

extern template struct Launchers<32>;
extern template struct Launchers<64>;
extern template struct Launchers<128>;

__global__ __launch_bounds__(256) void k_sum_doubles(const double* in, int count, double* out) {
  __shared__ double redd[16];
  sum_doubles(in, count, out, redd, threadIdx.x);
}

__global__ __launch_bounds__(256) void k_zero_doubles(double* p, int count) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < count) p[i] = 0.0;
}

__global__ __launch_bounds__(64) void k_zero_u32(unsigned* p) { p[threadIdx.x] = 0u; }

__global__ __launch_bounds__(256) void k_slot_info(const int* idx, const int2* pos, int n_pos,
                                                   int4* slot, int count) {
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j >= count) return;
  const int k = min(max(idx[j], 0), n_pos - 1);
  const int2 p = pos[k];
  slot[j] = make_int4(k, p.x, p.y, 0);
}

__global__ __launch_bounds__(256) void k_fill_c64(float2* p, size_t count, float2 v) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < count) p[i] = v;
}

// No sequence number of an earlier launch may be found in the scratch (a captured launch is
// replayed with the same numbers).  The one worker of m = 32 and its summing workgroup use only
// the counters.
__global__ __launch_bounds__(256) void k_chain_clear(float4* p, int count, double* sampled) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < count) p[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  if (i == 0 && sampled) *sampled = 0.0;
}

hipError_t launch_chain_clear(int m, float2* scratch, double* sampled, hipStream_t s) {
  const size_t all = chain_clear_units(m), first = m == 32 ? all - kChainCounterUnits : 0;
  const int count = (int)(all - first);
  hipLaunchKernelGGL(k_chain_clear, dim3((count + 255) / 256), dim3(256), 0, s,
                     reinterpret_cast<float4*>(scratch) + first, count, sampled);
  return hipGetLastError();
}

hipError_t launch_slot_info(const int* idx, const int2* pos, int n_pos, int4* slot, int count,
                            hipStream_t s) {
  hipLaunchKernelGGL(k_slot_info, dim3((count + 255) / 256), dim3(256), 0, s, idx, pos, n_pos, slot,
                     count);
  return hipGetLastError();
}

hipError_t launch_zero_u32(unsigned* p, hipStream_t s) {
  hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(64), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_zero_doubles(double* p, int count, hipStream_t s) {
  hipLaunchKernelGGL(k_zero_doubles, dim3((count + 255) / 256), dim3(256), 0, s, p, count);
  return hipGetLastError();
}

hipError_t launch_sum_doubles(const double* in, int count, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_sum_doubles, dim3(1), dim3(256), 0, s, in, count, out);
  return hipGetLastError();
}

hipError_t launch_fill_c64(float2* p, size_t count, float2 v, hipStream_t s) {
  if (count == 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_c64, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, p, count, v);
  return hipGetLastError();
}

#define EMG_BY_M(m, CALL)                        \
  switch (m) {                                   \
    case 32: return Launchers<32>::CALL;         \
    case 64: return Launchers<64>::CALL;         \
    case 128: return Launchers<128>::CALL;       \
    case 256: return Launchers256::CALL;         \
    default: return hipErrorInvalidValue;        \
  }

hipError_t launch_patch_step(int m, int v, int L, const StepArgs& a, hipStream_t s, hipEvent_t e0,
                             hipEvent_t e1) {
  EMG_BY_M(m, patch_step(v, L, a, s, e0, e1));
}
hipError_t launch_finalize(int m, int f, const StepArgs& a, hipStream_t s, hipEvent_t e0,
                           hipEvent_t e1) {
  EMG_BY_M(m, finalize(f, a, s, e0, e1));
}
hipError_t launch_patch_step_multi(int m, int v, int L, bool phase, const StepArgs* args, const int2* work,
                                   int blocks, hipStream_t s) {
  EMG_BY_M(m, patch_step_multi(v, L, phase, args, work, blocks, s));
}
hipError_t launch_finalize_multi(int m, int f, const StepArgs* args, const int2* work, int blocks,
                                 hipStream_t s) {
  EMG_BY_M(m, finalize_multi(f, args, work, blocks, s));
}
hipError_t finalize_item_count(int m, int f, int nr, int nc, int pgroups, int* items) {
  EMG_BY_M(m, finalize_item_count(f, nr, nc, pgroups, items));
}
hipError_t launch_plain_step(int m, int v, int L, const StepArgs& a, hipStream_t s) {
  EMG_BY_M(m, plain_step(v, L, a, s));
}
hipError_t persistent_grid_size(int m, int v, int L, int num_cus, int* grid) {
  EMG_BY_M(m, persistent_grid_size(v, L, num_cus, grid));
}
hipError_t launch_persistent_epoch(int m, int v, int L, const StepArgs& a, int n_pos, int minibatch,
                                   int grid, unsigned* bar, unsigned bar_base, int* err,
                                   unsigned spin_limit, int* used_grid, hipStream_t s) {
  EMG_BY_M(m, persistent_epoch(v, L, a, n_pos, minibatch, grid, bar, bar_base, err, spin_limit,
                               used_grid, s));
}
hipError_t launch_layout_intensities(int m, int v, const float* d, float* dperm, int n_pos,
                                     double* pattern_sums, int* bad_flag, hipStream_t s) {
  EMG_BY_M(m, layout(v, d, dperm, n_pos, pattern_sums, bad_flag, s));
}
hipError_t launch_normalize_probe(int m, float2* probe, double dp_avg, int* zero_flag,
                                  hipStream_t s) {
  EMG_BY_M(m, normalize(probe, dp_avg, zero_flag, s));
}
hipError_t launch_misfit_terms(int m, int v, const float2* obj, int n, const float2* probe,
                               const float* dperm, const int2* pos, const int4* slot, int count,
                               const float2* tw, double* phi_out, int by_pattern, hipStream_t s) {
  EMG_BY_M(m, misfit(v, obj, n, probe, dperm, pos, slot, count, tw, phi_out, by_pattern, s));
}
hipError_t launch_revised_waves(int m, int v, const StepArgs& a, hipStream_t s) {
  EMG_BY_M(m, revised_waves(v, a, s));
}
hipError_t launch_numerators(int m, int v, int L, const StepArgs& a, hipStream_t s) {
  EMG_BY_M(m, numerators(v, L, a, s));
}
hipError_t launch_surrogate_terms(int m, int v, const StepArgs& a, double* terms, hipStream_t s) {
  EMG_BY_M(m, surrogate(v, a, terms, s));
}
hipError_t launch_chain_sweep(int m, int v, int L, const StepArgs& a, int n_steps, bool add,
                              const ChainSync& y, hipStream_t s) {
  EMG_BY_M(m, chain(v, L, a, n_steps, add, y, s));
}
hipError_t launch_grad(int m, int v, bool f64, const GradArgs& g, hipStream_t s) {
  EMG_BY_M(m, grad(v, f64, g, s));
}

}  // namespace emg
