// Probe side m = 256.  A 256 x 256 complex64 tile (512 KiB) exceeds a CU's LDS,
// so one patch runs as 16 row strips and 16 column blocks of 16 lines each, the
// tile passing through the per-minibatch stack buffer (L2/MALL resident) between
// them:
//   1. row strips:    psi = Q . z_k (Def. 2.1), forward row passes, strip maxima
//                     of |Q|^2 and |z_k|^2;
//   2. column blocks: forward column passes, the modulus projection between the
//                     last forward and the first inverse pass (as in the one-
//                     workgroup kernel), inverse column passes, partial misfits;
//   3. row strips:    inverse row passes, then the per-pixel surrogate algebra of
//                     the strip (multigrid blocks of 2 x 2 and 4 x 4 never cross a
//                     strip of 16 rows), numerators for the finalize.
// Every pass is 16 points per thread, and a strip goes through LDS only where its points
// change threads: the column blocks and the inverse row passes start from memory in registers,
// and every last pass writes from them.  The
// stack buffer keeps rows in natural order and columns in frequency order: transform
// position 16 k + j of the 16 x 16 split is frequency k + 16 j, so the lanes k of one output j
// write 16 neighbours, and a column block reads 16 neighbours of every row.  The measured
// intensities are laid out the same way (rows in transform order, columns in natural order).
// Measured (961 patterns of 256^2, minibatch 32): the sweep's stages 31.3 -> 29.9 us per
// minibatch against passes that all went through LDS; the full misfit, in chunks of up to 256
// patterns instead of a minibatch's, 555 -> 285 us.
// The finalize, layout and normalisation kernels are the shared templates.
#include "kernels.hpp"

namespace emg {

namespace big {
constexpr int M = 256, S = 16, NT = 256;
constexpr int R1 = Plan<256, 0>::R1, R2 = Plan<256, 0>::R2;
static_assert(R1 == 16 && R2 == 16, "16-point passes");
// LDS strides and padding without bank conflicts: a strip as rows of padded positions, a
// column block as positions of 17
constexpr int LSR = M + 16, LSC = S + 1;
__device__ __forceinline__ int pad(int p) { return p + p / 16; }

// The strided passes of group g.  The twiddles come from the table in LDS: 15 loads per
// thread from the global one, as many as the pass's data, cost 4-5% of a sweep.
__device__ __forceinline__ void twiddle_forward(cx<float>* v, const cx<float>* tws, int g) {
#pragma unroll
  for (int j = 1; j < 16; ++j) v[j] = mul_fma(tws[g * j], v[j]);
}
__device__ __forceinline__ void strided_inverse(cx<float>* v, const cx<float>* tws, int g) {
#pragma unroll
  for (int j = 1; j < 16; ++j) v[j] = mul_fma(conjg(tws[g * j]), v[j]);
  dft16<float, true>(v);
}

// thread's 2 x 2 blocks in a 16 x 256 strip: four rounds of 16 x 64 pixels side by
// side; four consecutive lanes own one 4 x 4 region
struct StripLayout {
  static constexpr int ROUNDS = 4;
  __device__ static void origin(int tid, int rd, int& r0, int& c0) {
    const int q = tid >> 2, sub = tid & 3;
    r0 = 4 * (q >> 4) + 2 * (sub >> 1);
    c0 = 4 * (q & 15) + 2 * (sub & 1) + 64 * rd;
  }
};
}  // namespace big

// Every kernel below runs (slot, strip) pairs strip-major: with nsl, the slot count a.b
// rounded up to a multiple of the XCD count, block i takes slot i mod nsl and strip i / nsl.
// All strips of a slot then run on one XCD (block i runs on XCD i mod 8), beside the
// slots listed next to it, and the overlapping windows' object rows and the slot's stack
// columns meet in that XCD's L2 (full misfit in chunks of 241 patterns: 303 us without the
// rounding, 279 us with it).  What the first loads need comes as leading arguments, in
// scalar registers at dispatch (see k_patch_step); a copy in the record is not used.
//
// 1. psi and forward row passes of strip rb of slot s (or of pattern k0 + s when
// a.slot is null: the misfit over all patterns)
__global__ __launch_bounds__(256) void k256_rows_fwd(int nsl, int b, const int4* slot, float2* obj, int n, float2* probe, StepArgs rec, int k0) {
  StepArgs a = rec;
  a.slot = slot;
  a.obj = obj;
  a.n = n;
  a.probe = probe;
  using namespace big;
  __shared__ cx<float> A[S * LSR];
  __shared__ cx<float> tws[M];
  __shared__ float redf[2 * NT / 64];
  const int tid = threadIdx.x, s = blockIdx.x % nsl, rb = blockIdx.x / nsl,
            row0 = rb * S;
  if (s >= b) return;
  int wr, wc;
  if (a.slot) {
    const int4 sl = a.slot[s];
    wr = sl.y;
    wc = sl.z;
  } else {
    const int2 p = a.pos[k0 + s];
    wr = p.x;
    wc = p.y;
  }
  const int row = tid / 16, g = tid % 16, ln = tid & 63, wave = tid >> 6;
  tws[tid] = ld(a.tw, tid);
  // Four rows per wave, loaded 64 pixels at a time: the window's alignment is arbitrary,
  // and runs of 16 pixels (the first pass's own points) would each cross a cache line.  The
  // wave's rows stay its own, so its passes need no block barrier between them.
  const float2* zwin = a.obj + (size_t)(wr + row0) * a.n + wc;
  float q2m = 0.f, z2m = 0.f;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int r = 4 * wave + i / 4, c = ln + 64 * (i % 4);
    const cx<float> q = ld(a.probe, (row0 + r) * M + c), z = ld(zwin, (size_t)r * a.n + c);
    q2m = fmaxf(q2m, norm2(q));
    z2m = fmaxf(z2m, norm2(z));
    A[r * LSR + pad(c)] = mul(q, z);
  }
  wave_order();
  cx<float> v[16];
  cx<float>* L = A + row * LSR;
#pragma unroll
  for (int j = 0; j < 16; ++j) v[j] = L[pad(g + 16 * j)];
  dft16<float, false>(v);
  __syncthreads();  // the table is staged
  twiddle_forward(v, tws, g);
#pragma unroll
  for (int j = 0; j < 16; ++j) L[pad(g + 16 * j)] = v[j];
  wave_order();
  // contiguous pass of run g; its output j is frequency g + 16 j
#pragma unroll
  for (int j = 0; j < 16; ++j) v[j] = L[pad(16 * g + j)];
  dft16<float, false>(v);
  wave_max2_to_lds<NT>(q2m, z2m, redf, tid);
  const __amdgpu_buffer_rsrc_t out = through_buffer(a.stack + (size_t)s * M * M + (size_t)row0 * M, S * M);
#pragma unroll
  for (int j = 0; j < 16; ++j) st_through(out, row * M + g + 16 * j, v[j]);
  __syncthreads();
  if (tid == 0) {
    float qm, zm;
    lds_max2<NT>(redf, qm, zm);
    a.part_q[s * S + rb] = qm;
    a.part_z[s * S + rb] = zm;
  }
}

// 2. column block cb of slot s: forward column passes, then in the pair pass the
// modulus projection (kColsStep), only the misfit terms (kColsMisfit), or the Fourier
// residual of the gradient (kColsGrad: Psi - Psi' = (|Psi| - a) Psi / |Psi|, or -a
// where Psi = 0, scaled by 1/m^2, with the misfit terms of the gradient's own
// arithmetic); inverse column passes (kColsStep, kColsGrad)
constexpr int kColsMisfit = 0, kColsStep = 1, kColsGrad = 2;
// PH: the step keeps a phase memory (compiled without it, two more workgroups fit a CU)
template <int MODE, bool PH = false>
__global__ __launch_bounds__(256) void k256_cols(int nsl, int b, const int4* slot, float2* stack, const float2* tw, const float* dperm,
                                                 StepArgs rec, int k0) {
  StepArgs a = rec;
  a.slot = slot;
  a.stack = stack;
  a.tw = tw;
  a.dperm = dperm;
  constexpr bool STEP = MODE == kColsStep, INVERSE = MODE != kColsMisfit;
  using namespace big;
  __shared__ cx<float> A[M * LSC];
  __shared__ cx<float> tws[M];
  __shared__ double redd[NT / 64];
  const int tid = threadIdx.x, s = blockIdx.x % nsl, cb = blockIdx.x / nsl,
            col0 = cb * S;
  if (s >= b) return;
  const int k = a.slot ? a.slot[s].x : k0 + s;
  // item tid of every pass: column line, group (or run) g
  const int line = tid % S, g = tid / S;
  float2* blk = a.stack + (size_t)s * M * M + col0;
  cx<float> v[16];
#pragma unroll
  for (int j = 0; j < 16; ++j) v[j] = ld(blk, (g + 16 * j) * M + line);
  float amp[16];
  tws[tid] = ld(a.tw, tid);
  const float* dk = a.dperm + (size_t)k * M * M;
#pragma unroll
  for (int j = 0; j < 16; ++j) amp[j] = dk[(16 * g + j) * M + col0 + line];
  dft16<float, false>(v);
  __syncthreads();  // the table is staged
  twiddle_forward(v, tws, g);
#pragma unroll
  for (int j = 0; j < 16; ++j) A[(g + 16 * j) * LSC + line] = v[j];
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 16; ++j) v[j] = A[(16 * g + j) * LSC + line];
  dft16<float, false>(v);
  double acc = 0.0;
  float2* ph = PH ? a.phase + (size_t)k * M * M : nullptr;
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    if constexpr (STEP) {
      float2* pe = PH ? ph + (16 * g + e) * M + col0 + line : nullptr;
      acc += (double)project_amp<M>(v[e], amplitude(amp[e]), pe, a.phase_write != 0);
    } else if constexpr (MODE == kColsGrad) {
      const float am = sqrtf(fmaxf(amp[e], 0.f));
      const float mag = sqrtf(norm2(v[e]));
      const float diff = mag - am;
      acc += (double)diff * (double)diff;
      const cx<float> E = mag > 0.f ? scale(v[e], diff / mag) : cx<float>{-am, 0.f};
      v[e] = scale(E, 1.f / float(M * M));
    } else {
      cx<float> t = v[e];
      acc += (double)project_amp<M>(t, amplitude(amp[e]));
    }
  }
  if constexpr (INVERSE) {
    dft16<float, true>(v);
    // back where the thread read them
#pragma unroll
    for (int j = 0; j < 16; ++j) A[(16 * g + j) * LSC + line] = v[j];
  }
  acc = wave_sum(acc);
  if ((tid & 63) == 0) redd[tid >> 6] = acc;
  __syncthreads();
  if constexpr (INVERSE) {
#pragma unroll
    for (int j = 0; j < 16; ++j) v[j] = A[(g + 16 * j) * LSC + line];
    strided_inverse(v, tws, g);
    const __amdgpu_buffer_rsrc_t out = through_buffer(blk, M * M - col0);
#pragma unroll
    for (int j = 0; j < 16; ++j) st_through(out, (g + 16 * j) * M + line, v[j]);
  }
  if (tid == 0) a.part_phi[s * S + cb] = lds_sum<NT>(redd);
}

// the inverse row passes of a strip (rows of the stack buffer at `in`): thread (row, g) ends
// with the natural-order points g + 16 j of its row
__device__ __forceinline__ void rows_inverse(const float2* in, const float2* tw, cx<float>* A,
                                             cx<float>* tws, int tid, cx<float>* v) {
  using namespace big;
  const int row = tid / 16, g = tid % 16;
#pragma unroll
  for (int j = 0; j < 16; ++j) v[j] = ld(in, row * M + g + 16 * j);
  tws[tid] = ld(tw, tid);
  dft16<float, true>(v);
  cx<float>* L = A + row * LSR;
#pragma unroll
  for (int j = 0; j < 16; ++j) L[pad(16 * g + j)] = v[j];
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 16; ++j) v[j] = L[pad(g + 16 * j)];
  strided_inverse(v, tws, g);
}

// 3. inverse row passes of strip rb of slot s and the strip's per-pixel algebra;
// with STORE_R the revised exit wave R_k of the strip also goes back to the stack
// buffer (the descent check keeps it, frozen, for the surrogate after the step)
template <int L, bool STORE_R = false>
__global__ __launch_bounds__(256) void k256_rows_inv(int nsl, int b, const int4* slot, float2* stack, const float2* tw, float2* probe,
                                                     StepArgs rec) {
  StepArgs a = rec;
  a.slot = slot;
  a.stack = stack;
  a.tw = tw;
  a.probe = probe;
  using namespace big;
  __shared__ cx<float> A[S * LSR];
  __shared__ cx<float> tws[M];
  const int tid = threadIdx.x, s = blockIdx.x % nsl, rb = blockIdx.x / nsl,
            row0 = rb * S;
  if (s >= b) return;
  const int4 sl = a.slot[s];
  float2* strip = a.stack + (size_t)s * M * M + (size_t)row0 * M;
  const int row = tid / 16, g = tid % 16;
  cx<float> v[16];
  rows_inverse(strip, a.tw, A, tws, tid, v);
  // max |Q|^2 and max |z_k|^2 over the whole patch, from the strip maxima
  float qqmax = a.part_q[s * S], zmax = a.part_z[s * S];
#pragma unroll
  for (int i = 1; i < S; ++i) {
    qqmax = fmaxf(qqmax, a.part_q[s * S + i]);
    zmax = fmaxf(zmax, a.part_z[s * S + i]);
  }
  if (rb == 0 && tid == 0 && a.phi) {
    double t = a.part_phi[s * S];
    for (int i = 1; i < S; ++i) t += a.part_phi[s * S + i];
    a.phi[s] = t / (2.0 * M * M);
  }
#pragma unroll
  for (int j = 0; j < 16; ++j) A[row * LSR + pad(g + 16 * j)] = v[j];
  if constexpr (STORE_R) {
#pragma unroll
    for (int j = 0; j < 16; ++j) st(strip, row * M + g + 16 * j, v[j]);
  }
  __syncthreads();
  const size_t n = (size_t)a.n;
  const float2* zwin = a.obj + (size_t)sl.y * n + sl.z;
  pixel_update_ly<M, StripLayout, L>(
      a, s, tid, row0,
      [&](int rd, int r0, int c0, cx<float>* q, cx<float>* zz, cx<float>* Rv) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          ld_pair(a.probe, (size_t)(r0 + i) * M + c0, q[2 * i], q[2 * i + 1]);
          zz[2 * i] = ld(zwin, (size_t)(r0 + i) * n + c0);
          zz[2 * i + 1] = ld(zwin, (size_t)(r0 + i) * n + c0 + 1);
          Rv[2 * i] = A[(r0 - row0 + i) * LSR + pad(c0)];
          Rv[2 * i + 1] = A[(r0 - row0 + i) * LSR + pad(c0) + 1];
        }
      },
      qqmax, zmax);
}

// per-pattern terms from the 16 partial sums of its column blocks (or strips), in
// block order, times `scale`
__global__ __launch_bounds__(256) void k256_phi_reduce(const double* part_phi, int count,
                                                       double* phi_out, double scale) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= count) return;
  double t = part_phi[i * big::S];
  for (int c = 1; c < big::S; ++c) t += part_phi[i * big::S + c];
  phi_out[i] = t * scale;
}

// gradient: inverse row passes of strip rb of pattern k0 + s turn the Fourier residual
// into e_k = Q z_k - R_k; the strip's slot terms conj(Q) e_k (object) and conj(z_k) e_k
// (probe) go to the gradient slots, for the shared reductions of k_grad_reduce
__global__ __launch_bounds__(256) void k256_rows_grad(int nsl, int b, const int2* pos, float2* stack, const float2* tw, float2* probe,
                                                      StepArgs rec, int k0, float2* gz, float2* gq) {
  StepArgs a = rec;
  a.pos = pos;
  a.stack = stack;
  a.tw = tw;
  a.probe = probe;
  using namespace big;
  __shared__ cx<float> A[S * LSR];
  __shared__ cx<float> tws[M];
  const int tid = threadIdx.x, s = blockIdx.x % nsl, rb = blockIdx.x / nsl,
            row0 = rb * S;
  if (s >= b) return;
  const int2 p = a.pos[k0 + s];
  const int row = tid / 16, g = tid % 16;
  cx<float> v[16];
  rows_inverse(a.stack + (size_t)s * M * M + (size_t)row0 * M, a.tw, A, tws, tid, v);
  const float2* zrow = a.obj + (size_t)(p.x + row0 + row) * a.n + p.y + g;
  const float2* qrow = a.probe + (row0 + row) * M + g;
  const size_t base = (size_t)s * M * M + (size_t)(row0 + row) * M + g;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    st(gz, base + 16 * j, cmulc(ld(qrow, 16 * j), v[j]));
    st(gq, base + 16 * j, cmulc(ld(zrow, 16 * j), v[j]));
  }
}

// descent check: 1/2 ||Q . z_k - R_k||^2 (Eq. 3 with R_k frozen in the stack buffer) of
// strip rb of slot s at the current state; FP32 differences, FP64 sum -> part_phi
__global__ __launch_bounds__(256) void k256_surrogate_strips(int nsl, int b, StepArgs rec) {
  StepArgs a = rec;
  using namespace big;
  __shared__ double redd[NT / 64];
  const int tid = threadIdx.x, s = blockIdx.x % nsl, rb = blockIdx.x / nsl,
            row0 = rb * S;
  if (s >= b) return;
  const int4 sl = a.slot[s];
  const size_t n = (size_t)a.n;
  const float2* zwin = a.obj + (size_t)(sl.y + row0) * n + sl.z;
  const float2* Rg = a.stack + (size_t)s * M * M + (size_t)row0 * M;
  double acc = 0.0;
#pragma unroll
  for (int r = 0; r < S; ++r) {
    const cx<float> d = sub(mul(ld(a.probe, (size_t)(row0 + r) * M + tid), ld(zwin, (size_t)r * n + tid)),
                            ld(Rg, (size_t)r * M + tid));
    acc += (double)d.re * (double)d.re + (double)d.im * (double)d.im;
  }
  const double tot = block_sum<NT>(acc, redd, tid);
  if (tid == 0) a.part_phi[s * S + rb] = tot;
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
static int slots_up(int b) { return (b + kDispatchXcds - 1) / kDispatchXcds * kDispatchXcds; }
static void launch_rows_fwd(const StepArgs& a, int k0, hipStream_t s) {
  const int nsl = slots_up(a.b);
  hipLaunchKernelGGL(k256_rows_fwd, dim3(nsl * big::S), dim3(big::NT), 0, s, nsl, a.b, a.slot, a.obj, a.n,
                     a.probe, a, k0);
}
template <int MODE, bool PH = false>
static void launch_cols(const StepArgs& a, int k0, hipStream_t s) {
  const int nsl = slots_up(a.b);
  hipLaunchKernelGGL((k256_cols<MODE, PH>), dim3(nsl * big::S), dim3(big::NT), 0, s, nsl, a.b, a.slot,
                     a.stack, a.tw, a.dperm, a, k0);
}
template <int L, bool STORE_R>
static void launch_rows_inv(const StepArgs& a, hipStream_t s) {
  const int nsl = slots_up(a.b);
  hipLaunchKernelGGL((k256_rows_inv<L, STORE_R>), dim3(nsl * big::S), dim3(big::NT), 0, s, nsl, a.b, a.slot,
                     a.stack, a.tw, a.probe, a);
}
// the three stages of a step
template <bool STORE_R>
static void launch_step(const StepArgs& a, int L, hipStream_t s) {
  launch_rows_fwd(a, 0, s);
  if (a.phase) launch_cols<kColsStep, true>(a, 0, s);
  else launch_cols<kColsStep>(a, 0, s);
  switch (L) {
    case 1: launch_rows_inv<1, STORE_R>(a, s); break;
    case 2: launch_rows_inv<2, STORE_R>(a, s); break;
    default: launch_rows_inv<3, STORE_R>(a, s); break;
  }
}

hipError_t Launchers256::patch_step(int v, int L, const StepArgs& a, hipStream_t s, hipEvent_t e0,
                                    hipEvent_t e1) {
  if (v != 0 || L < 1 || L > 3 || !a.part_q || !a.slot) return hipErrorInvalidValue;
  hipError_t e;
  if (e0 && (e = hipEventRecord(e0, s)) != hipSuccess) return e;
  launch_step<false>(a, L, s);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (e1 && (e = hipEventRecord(e1, s)) != hipSuccess) return e;
  return hipSuccess;
}

hipError_t launch_misfit256(const StepArgs& a, int n_pos, int chunk, double* phi_out, hipStream_t s) {
  if (!a.part_q || n_pos < 1 || chunk < 1) return hipErrorInvalidValue;
  StepArgs x = a;
  x.slot = nullptr;
  for (int k0 = 0; k0 < n_pos; k0 += chunk) {
    x.b = min(chunk, n_pos - k0);
    x.part_phi = a.part_phi + (size_t)k0 * big::S;
    launch_rows_fwd(x, k0, s);
    launch_cols<kColsMisfit>(x, k0, s);
  }
  hipLaunchKernelGGL(k256_phi_reduce, dim3((n_pos + 255) / 256), dim3(256), 0, s,
                     (const double*)a.part_phi, n_pos, phi_out, 1.0 / (2.0 * big::M * big::M));
  return hipGetLastError();
}

hipError_t launch_grad256(const StepArgs& a, const GradArgs& g, hipStream_t s) {
  constexpr int M = 256;
  if (!a.part_q || g.chunk < 1) return hipErrorInvalidValue;
  StepArgs x = a;
  x.slot = nullptr;
  for (int k0 = 0; k0 < g.n_pos; k0 += g.chunk) {
    const int cnt = min(g.chunk, g.n_pos - k0);
    x.b = cnt;
    const int nsl = slots_up(cnt);
    x.part_phi = a.part_phi + (size_t)k0 * big::S;
    launch_rows_fwd(x, k0, s);
    launch_cols<kColsGrad>(x, k0, s);
    hipLaunchKernelGGL(k256_rows_grad, dim3(nsl * big::S), dim3(big::NT), 0, s, nsl, cnt, x.pos, x.stack,
                       x.tw, x.probe, x, k0, static_cast<float2*>(g.gz_slots),
                       static_cast<float2*>(g.gq_slots));
    if (k0 + cnt == g.n_pos)  // the terms are complete: the last reduction adds them
      hipLaunchKernelGGL(k256_phi_reduce, dim3((g.n_pos + 255) / 256), dim3(256), 0, s,
                         (const double*)a.part_phi, g.n_pos, g.phi_all, 1.0 / (2.0 * M * M));
    const hipError_t e = launch_grad_reduce<float, M>(g, k0, cnt, cnt, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_check256(const StepArgs& a, int levels, int finalize_shape, double* out3,
                           hipStream_t s) {
  if (!a.part_q || !a.slot || levels < 1 || levels > 3) return hipErrorInvalidValue;
  // the step, keeping the revised waves R_k of the state before it in the stack buffer
  launch_step<true>(a, levels, s);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  StepArgs f = a;
  f.sampled = out3;  // [0] += sum_k Phi_k at the state before the step
  if ((e = Launchers256::finalize(finalize_shape, f, s, nullptr, nullptr)) != hipSuccess) return e;
  // [1] surrogate of Eq. 3 at the new state against the frozen R_k
  const int nsl = slots_up(a.b);
  hipLaunchKernelGGL(k256_surrogate_strips, dim3(nsl * big::S), dim3(big::NT), 0, s, nsl, a.b, a);
  hipLaunchKernelGGL(k256_phi_reduce, dim3((a.b + 255) / 256), dim3(256), 0, s,
                     (const double*)a.part_phi, a.b, a.phi, 0.5);
  if ((e = launch_sum_doubles(a.phi, a.b, out3 + 1, s)) != hipSuccess) return e;
  // [2] Phi_B at the new state: the batch's misfit terms through the strip kernels
  launch_rows_fwd(a, 0, s);
  launch_cols<kColsMisfit>(a, 0, s);
  hipLaunchKernelGGL(k256_phi_reduce, dim3((a.b + 255) / 256), dim3(256), 0, s,
                     (const double*)a.part_phi, a.b, a.phi, 1.0 / (2.0 * big::M * big::M));
  if ((e = hipGetLastError()) != hipSuccess) return e;
  return launch_sum_doubles(a.phi, a.b, out3 + 2, s);
}

hipError_t Launchers256::finalize(int f, const StepArgs& a, hipStream_t s, hipEvent_t e0,
                                  hipEvent_t e1) {
  constexpr int M = 256;
  return with_fin(f, [&](auto fc) {
    constexpr int F = decltype(fc)::value, FNT = FinShape<F>::FNT, T = FinShape<F>::T;
    int ntiles;
    const int items = finalize_items<M, FNT, T>(a.nr, a.n, a.pgroups, &ntiles);
    if (e0) {
      StepArgs aa = a;
      const int4* sl = a.slot;
      float2* ob = a.obj;
      int n = a.n, b = a.b;
      void* args[] = {&sl, &ob, &n, &b, &aa, &ntiles};
      return hipExtLaunchKernel((const void*)k_finalize<M, F>, dim3(items), dim3(FNT), args, 0, s,
                                e0, e1, 0);
    }
    hipLaunchKernelGGL((k_finalize<M, F>), dim3(items), dim3(FNT), 0, s, a.slot, a.obj, a.n, a.b,
                       a, ntiles);
    return hipGetLastError();
  });
}

hipError_t Launchers256::finalize_item_count(int f, int nr, int nc, int pgroups, int* items) {
  return with_fin(f, [&](auto fc) {
    constexpr int F = decltype(fc)::value;
    int ntiles = 0;
    *items = finalize_items<256, FinShape<F>::FNT, FinShape<F>::T>(nr, nc, pgroups, &ntiles);
    return hipSuccess;
  });
}

hipError_t Launchers256::layout(int v, const float* d, float* dperm, int n_pos, double* sums,
                                int* bad, hipStream_t s) {
  if (v != 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL((k_layout<256, 0>), dim3(n_pos), dim3(256), 0, s, d, dperm, sums, bad);
  return hipGetLastError();
}

hipError_t Launchers256::normalize(float2* probe, double dp_avg, int* flag, hipStream_t s) {
  hipLaunchKernelGGL(k_normalize<256>, dim3(1), dim3(256), 0, s, probe, dp_avg, flag);
  return hipGetLastError();
}

hipError_t Launchers256::persistent_grid_size(int, int, int, int* grid) {
  *grid = 0;  // no persistent form at this size
  return hipSuccess;
}

// no m = 256 form (the host rejects these requests before they reach here)
hipError_t Launchers256::patch_step_multi(int, int, bool, const StepArgs*, const int2*, int, hipStream_t) {
  return hipErrorInvalidValue;
}
hipError_t Launchers256::finalize_multi(int, const StepArgs*, const int2*, int, hipStream_t) {
  return hipErrorInvalidValue;
}
hipError_t Launchers256::plain_step(int, int, const StepArgs&, hipStream_t) { return hipErrorInvalidValue; }
hipError_t Launchers256::persistent_epoch(int, int, const StepArgs&, int, int, int, unsigned*, unsigned,
                                          int*, unsigned, int*, hipStream_t) {
  return hipErrorInvalidValue;
}
hipError_t Launchers256::misfit(int, const float2*, int, const float2*, const float*, const int2*,
                                const int4*, int, const float2*, double*, int, hipStream_t) {
  return hipErrorInvalidValue;
}
hipError_t Launchers256::revised_waves(int, const StepArgs&, hipStream_t) { return hipErrorInvalidValue; }
hipError_t Launchers256::numerators(int, int, const StepArgs&, hipStream_t) { return hipErrorInvalidValue; }
hipError_t Launchers256::surrogate(int, const StepArgs&, double*, hipStream_t) { return hipErrorInvalidValue; }
hipError_t Launchers256::grad(int, bool, const GradArgs&, hipStream_t) { return hipErrorInvalidValue; }
hipError_t Launchers256::chain(int, int, const StepArgs&, int, bool, const ChainSync&, hipStream_t) {
  return hipErrorInvalidValue;
}

}  // namespace emg
