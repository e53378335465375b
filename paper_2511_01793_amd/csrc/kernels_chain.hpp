// The sequential sweep (minibatch 1: the paper's literal order) of one patch spread over
// several workgroups, one launch for the whole sweep.
//
// A step is a dependent chain of transforms of one m x m patch.  One workgroup per step
// took 29.4 us at m = 128 and 8.1 us at m = 64 (one CU's VALU, then LDS and load latency).
// Here m^2 / 1024 workgroups of 256 threads share a step, each owning LINES rows of the
// patch and LINES columns of the spectrum, 4 points per thread.  Per step:
//   1. row phase: exit wave psi = Q . z_k and the forward row passes;
//   2. column phase: forward column passes, modulus projection, inverse column passes;
//   3. row phase: inverse row passes, the per-pixel update, the new object window.
// What bounds a step is the latency of its three exchanges between workgroups, so there is no
// barrier: every exchanged value travels as a 16-byte packet {re, n, im, n} with the
// step's number n, each 8-byte half written and read whole, and its reader polls the packet
// itself until both halves carry the number.  An exchange costs one store and one load latency
// (a counter barrier of 16 workgroups with drained stores cost 1.5 us, three per step:
// 8.7 us per step with the same 4 points per thread).  The packet is the low-latency line known
// from collective libraries, which carries data and a sequence number in one store.  The
// workgroups are blocks 0, 8, 16, ... of the launch, which run on one
// XCD and share its L2: the packets stay there (0.78 us per exchange of 16 workgroups, 4
// packets per thread) and are read past the L1s.  Where their XCDs differ the packets are
// written through to memory (1.5 us; a step of m = 128 then takes 7.4 us instead of 6.4).
//
// Waiting for each other's data is sound only among workgroups that are all running, and an
// ordinary launch does not promise that: sweeps on several streams or of several processes, or
// any other kernel, may hold the places.  So nobody waits for data before a roll call (roll_call)
// has found every workgroup of the launch started.  Where that takes too long the first to
// give up calls the sweep off for all: those started leave, those that start later leave at
// once, nothing has been written, and k_sweep_one, launched behind, does the whole sweep in one
// workgroup, which waits for nobody.  The decision is one atomic word's, so all take the same.
//
// A packet is overwritten one step later by its writer, which by then has received data that
// every reader sends only after reading it (each phase needs data of all workgroups
// in the phase before).  The object itself is written beside the packets of the window; the
// stores of step s are complete before their writer sends its column-phase data of step
// s + 1, so from then on (the start of row phase 3) the pixels of the window of step
// s + 2 outside that of step s + 1 are loaded ahead, and only the overlap is polled.
// The rows of the probe a workgroup owns stay in its LDS for the whole sweep.  The probe update
// of a step runs while the new window travels; the next step's intensities
// and window corner are loaded a step ahead.
//
// The DFTs, twiddle products, projection and per-pixel arithmetic are those of patch_step,
// operand for operand, so object and probe are bitwise those of every other path.  The
// sampled misfit is summed by one more workgroup, up to kChainTermSteps steps behind, from
// every point's term, in the order of the plan's patch kernel.
#pragma once

namespace emg {

template <int M, int V>
struct Chain {
  static constexpr int R1 = Plan<M, V>::R1, R2 = Plan<M, V>::R2;
  static constexpr int NT = 256, WAVES = NT / 64;
  static constexpr int LINES = 4 * NT / M;  // rows, and columns, of a workgroup
  static constexpr int Workers = M / LINES;
  // m = 32 is one workgroup's work: the tile stays in its LDS, where the other sides' columns
  // and window travel as packets
  static constexpr bool SOLO = Workers == 1;
  // LDS row stride: at most two-way bank conflicts in any pass (m = 32: four-way in one)
  static constexpr int LS = SOLO ? M + 4 : M + 2;
  // order of a block's LINES columns in the exchanged tile: where a lane pair holds two
  // neighbouring points of two groups (8-point runs, 16 lines), those four lie together
  __device__ static int slot(int c) {
    return R1 == 8 && LINES == 16 ? ((c >> 1) & 3) * 4 + (c >> 3) * 2 + (c & 1) : c;
  }
  __device__ static int column(int s) {
    return R1 == 8 && LINES == 16 ? ((s >> 1) & 1) * 8 + (s >> 2) * 2 + (s & 1) : s;
  }
};

// A wait that gives up raises the error flag and marks its workgroup, which leaves the
// sweep at the next block barrier; the others' waits then give up too.
struct ChainWait {
  unsigned limit;
  int* err;
  int* dead;  // LDS
  __device__ __forceinline__ bool give_up(unsigned& polls) const {
    if (++polls <= limit) return false;
    __hip_atomic_store(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    *dead = 1;
    return true;
  }
  // until *counter >= target
  __device__ __forceinline__ void counter(unsigned* c, unsigned target) const {
    unsigned polls = 0;
    while ((int)(__hip_atomic_load(c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - target) < 0)
      if (give_up(polls)) break;
  }
};

// Roll call of a launch, one word: six bits per XCD with the workers that started there, from
// bit kRollCount the workgroups that started, and kRollOff once one has given up on the others.
constexpr int kRollXcdBits = 6, kRollCount = 54;
constexpr unsigned long long kRollOff = 1ull << 63;
// Looks at the word before giving up, each 0.16 us: 2.6 ms, longer than the tail of most kernels
// that are making room, and less than the sweeps that sharing pays for.
constexpr unsigned kRollPolls = 1u << 14;
__device__ __forceinline__ void roll_answer(unsigned long long* word, bool worker, unsigned xcd) {
  const unsigned long long place = worker && xcd < kDispatchXcds ? 1ull << (kRollXcdBits * xcd) : 0ull;
  (void)__hip_atomic_fetch_add(word, (1ull << kRollCount) + place, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// the word with all `parties` started, or with kRollOff: which of the two comes first is final
__device__ __forceinline__ unsigned long long roll_call(unsigned long long* word, unsigned parties) {
  unsigned long long w = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  for (unsigned polls = 0; !(w & kRollOff) && (unsigned)(w >> kRollCount) < parties; ++polls) {
    if (polls < kRollPolls) {
      __builtin_amdgcn_s_sleep(1);
      w = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else if (__hip_atomic_compare_exchange_strong(word, &w, w | kRollOff, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_AGENT)) {
      w |= kRollOff;
    }  // else another has started or given up meanwhile, and w is the word now
  }
  return w;
}

typedef int chain_packet __attribute__((ext_vector_type(4)));
// N packets; shared_l2: every reader is on this XCD, so the packets may stay in its L2
template <int N>
__device__ __forceinline__ void send(__amdgpu_buffer_rsrc_t r, const int* at, const cx<float>* v,
                                     unsigned n, bool shared_l2) {
  chain_packet p[N];
#pragma unroll
  for (int j = 0; j < N; ++j)
    p[j] = chain_packet{__float_as_int(v[j].re), (int)n, __float_as_int(v[j].im), (int)n};
  if (shared_l2) {
#pragma unroll
    for (int j = 0; j < N; ++j) __builtin_amdgcn_raw_buffer_store_b128(p[j], r, at[j] * 16, 0, 0);
  } else {
#pragma unroll
    for (int j = 0; j < N; ++j)
      __builtin_amdgcn_raw_buffer_store_b128(p[j], r, at[j] * 16, 0, kCachePolicyThrough);
  }
}
// v[j] <- packet at[j] once it carries n, for every j with want[j] (its others keep v[j])
template <int N>
__device__ __forceinline__ void receive(__amdgpu_buffer_rsrc_t r, const int* at, const bool* want,
                                        cx<float>* v, unsigned n, const ChainWait& w) {
  unsigned polls = 0;
  for (;;) {
    chain_packet p[N];
#pragma unroll
    for (int j = 0; j < N; ++j)
      p[j] = __builtin_amdgcn_raw_buffer_load_b128(r, at[j] * 16, 0, kCachePolicyThrough);
    bool all = true;
#pragma unroll
    for (int j = 0; j < N; ++j) all = all && (!want[j] || (p[j][1] == (int)n && p[j][3] == (int)n));
    if (all || w.give_up(polls)) {
#pragma unroll
      for (int j = 0; j < N; ++j) {
        v[j].re = want[j] ? __int_as_float(p[j][0]) : v[j].re;
        v[j].im = want[j] ? __int_as_float(p[j][2]) : v[j].im;
      }
      return;
    }
    asm volatile("" ::: "memory");  // the next poll loads again
  }
}
__device__ __forceinline__ cx<float> ld_agent(__amdgpu_buffer_rsrc_t r, int i) {
  const auto v = __builtin_amdgcn_raw_buffer_load_b64(r, i * (int)sizeof(float2), 0, kCachePolicyThrough);
  return cx<float>{__int_as_float(v[0]), __int_as_float(v[1])};
}

// One pass of R points (4, 8 or 16) over the workgroup's 1024, 4 points per thread: a DFT
// takes R / 4 lanes of a wave, which differ in lane bit 4 (h0) and, for R = 16, bit 5 (h1).  The even
// inputs lie in the lanes with one of these bits clear, so each lane runs the 4-point DFTs and
// twiddles of dft8 / dft16 on its own inputs, and each butterfly across lanes is one lane
// swap and one fused add (the same operations on the same operands as dft8 / dft16).
// F (R = 16): the lane bit of the inputs' last bit, h1 (F = 0) or h0 (F = 1); the other one
// is that of their second bit.
struct PassPlace {
  int line, g, h0, h1;
};
// input and output index of a thread's value i in its DFT
template <int R, int F = 0>
__device__ __forceinline__ int pass_in(int i, const PassPlace& p) {
  return R == 4 ? i : R == 8 ? 2 * i + p.h0 : F == 0 ? 4 * i + 2 * p.h0 + p.h1 : 4 * i + 2 * p.h1 + p.h0;
}
template <int R, int F = 0>
__device__ __forceinline__ int pass_out(int i, const PassPlace& p) {
  return R == 4 ? i : R == 8 ? 4 * p.h0 + i : F == 0 ? 8 * p.h1 + 4 * p.h0 + i : 8 * p.h0 + 4 * p.h1 + i;
}
// the thread's part of an item, and its item of the pass
template <int R>
__device__ __forceinline__ int pass_item(int t, PassPlace& p) {
  p.h0 = R >= 8 ? (t >> 4) & 1 : 0;
  p.h1 = R == 16 ? (t >> 5) & 1 : 0;
  if (R == 4) return t;
  return (t & 15) | (R == 16 ? (t >> 6) << 4 : (t >> 5) << 4);
}

// v[i] <- e_i + t_i in the lanes with `upper` clear, e_i - t_i in the others, where e is
// the lower lane's v and t the upper lane's t; D the lane distance
template <int D>
__device__ __forceinline__ void cross_butterfly(cx<float>* v, const cx<float>* t, bool upper) {
  const float sg = upper ? -1.f : 1.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    cx<float> e{upper ? t[i].re : v[i].re, upper ? t[i].im : v[i].im}, o = e;
    xl_exchange<D>(e, o);
    v[i] = axpy(sg, o, e);  // e + t, e - t: the product is exact
  }
}

template <int R, bool INV, int F = 0>
__device__ __forceinline__ void group_dft(cx<float>* v, const PassPlace& p) {
  const bool second = R == 8 || F == 0 ? p.h0 != 0 : p.h1 != 0;
  dft4<float, INV>(v[0], v[1], v[2], v[3]);
  if constexpr (R == 4) return;
  cx<float> t[4];
  twiddle8<float, INV>(v, t);
  cross_butterfly<(R == 8 || F == 0) ? 16 : 32>(v, t, second);
  if constexpr (R == 16) {
    // W16^k of dft16 at k = i, or 4 + i
    const float c1 = 0.92387953251128675612818318939678828682f;  // cos(pi / 8)
    const float s1 = 0.38268343236508977172845998403039886676f;  // sin(pi / 8)
    const float h = 0.70710678118654752440084436210484903928f;
    const float sg = INV ? 1.f : -1.f;
    const cx<float> r = rot90<float, INV>(v[0]);
    t[0] = cx<float>{second ? r.re : v[0].re, second ? r.im : v[0].im};
    t[1] = mul(cx<float>{second ? -s1 : c1, sg * (second ? c1 : s1)}, v[1]);
    const float ps = h * (v[2].re + v[2].im),
                ms = INV ? h * (v[2].re - v[2].im) : h * (v[2].im - v[2].re);
    t[2] = INV ? cx<float>{second ? -ps : ms, second ? ms : ps}
               : cx<float>{second ? ms : ps, second ? -ps : ms};
    t[3] = mul(cx<float>{second ? -c1 : s1, sg * (second ? s1 : c1)}, v[3]);
    cross_butterfly<F == 0 ? 32 : 16>(v, t, F == 0 ? p.h1 != 0 : p.h0 != 0);
  }
}

// the outputs of a pass (F = 0) to the order of the inputs of the next (F = 1): lane bits
// and register bits exchanged
template <int R>
__device__ __forceinline__ void outputs_to_inputs(cx<float>* v) {
  if constexpr (R == 4) return;
  xl_exchange<16>(v[0], v[1]);
  xl_exchange<16>(v[2], v[3]);
  if constexpr (R == 16) {
    xl_exchange<32>(v[0], v[2]);
    xl_exchange<32>(v[1], v[3]);
  } else {
    const cx<float> t = v[1];
    v[1] = v[2];
    v[2] = t;
  }
}

// the workgroup's 2 x 2 blocks in its LINES x m rows, one per thread
template <int M>
struct ChainRows {
  static constexpr int ROUNDS = 1;
  __device__ static void origin(int t, int, int& r0, int& c0) {
    const int q = t >> 2;
    r0 = 4 * (q / (M / 4)) + 2 * ((t >> 1) & 1);
    c0 = 4 * (q % (M / 4)) + 2 * (t & 1);
  }
};

// New window values to the object and to the next step (as packets, or in the one workgroup's
// LDS); new probe values to the rows in LDS.
template <int M, int LS, bool SOLO>
struct ChainSink {
  static constexpr bool direct = true;
  __amdgpu_buffer_rsrc_t win, packets;
  int n, row0;
  unsigned number;
  bool shared_l2;
  cx<float>*q, *z;
  __device__ __forceinline__ void object(int r, int c, cx<float> v, bool changed) const {
    const int at = r * M + c;
    if constexpr (SOLO) z[r * LS + c] = v;
    else send<1>(packets, &at, &v, number, shared_l2);
    if (changed) st_through(win, r * n + c, v);
  }
  __device__ __forceinline__ void probe(int r, int c, cx<float> v) const { q[(r - row0) * LS + c] = v; }
};

// hwreg(HW_REG_XCC_ID, 0, 4), the number of the XCD a wave runs on
constexpr int kHwRegXccId = 20 | (0 << 6) | ((4 - 1) << 11);

// counters of a launch: steps whose terms a workgroup has stored (summed over them), and
// steps the summing workgroup is done with
constexpr int kChainStored = 0, kChainSummed = 32;

// The sampled misfit of every step: the terms at [column * m + row] in transform order, added
// as the plan's patch kernel adds them (each thread its points in order, the wave sum, the
// waves in order), then the finalize's additions.
template <int M, int V>
__device__ __forceinline__ void chain_account(const StepArgs& a, int n_steps, float* terms,
                                              unsigned* counters, const ChainWait& wait, unsigned skew) {
  using C = Chain<M, V>;
  using CP = ColPass<M, V>;
  constexpr int NTV = Plan<M, V>::NT, IT = NTV / C::NT;
  static_assert(IT * C::NT == NTV, "the plan's threads in whole rounds");
  __shared__ double redd[16];
  const int tid = threadIdx.x;
  double sampled = tid == 0 ? *a.sampled : 0.0;
  for (int step = 0; step < n_steps; ++step) {
    if (tid == 0) wait.counter(counters + kChainStored, (unsigned)(step + 1) * C::Workers + skew);
    __syncthreads();
    if (*wait.dead) break;
    const __amdgpu_buffer_rsrc_t tr = through_buffer(
        reinterpret_cast<float2*>(terms + (size_t)(step % kChainTermSteps) * M * M), M * M / 2);
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      const int t = tid + i * C::NT;
      double acc = 0.0;
      auto add_run = [&](int line, int g) {
        cx<float> v[C::R1 / 2];
#pragma unroll
        for (int j = 0; j < C::R1 / 2; j += 2) {
          const auto x = __builtin_amdgcn_raw_buffer_load_b128(tr, (line * M + C::R1 * g + 2 * j) * 4, 0,
                                                               kCachePolicyThrough);
          v[j] = cx<float>{__int_as_float(x[0]), __int_as_float(x[1])};
          v[j + 1] = cx<float>{__int_as_float(x[2]), __int_as_float(x[3])};
        }
#pragma unroll
        for (int j = 0; j < C::R1 / 2; ++j) {
          acc += (double)v[j].re;
          acc += (double)v[j].im;
        }
      };
      if constexpr (Plan<M, V>::XL != 0) {
        if (t < 512) add_run(8 * (t >> 6) + (t & 7), (t & 63) >> 3);
      } else {
#pragma unroll
        for (int it = 0; it < CP::IT; ++it) {
          const int w = t + it * NTV;
          if (CP::ITEMS < NTV && w >= CP::ITEMS) break;
          add_run(w % M, w / M);
        }
      }
      acc = wave_sum(acc);
      if ((t & 63) == 0) redd[t >> 6] = acc;
    }
    __syncthreads();
    if (tid == 0) {
      __hip_atomic_store(counters + kChainSummed, (unsigned)(step + 1), __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
      double t = 0.0;
      t += lds_sum<NTV>(redd) / (2.0 * M * M);
      sampled += t;
    }
  }
  if (tid == 0) *a.sampled = sampled;
}

template <int M, int V, int L, bool PH>
__global__ __launch_bounds__((Chain<M, V>::NT)) void k_chain(StepArgs a, int n_steps,
                                                                      ChainSync y) {
  using C = Chain<M, V>;
  constexpr int R1 = C::R1, R2 = C::R2, LINES = C::LINES, LS = C::LS, NT = C::NT;
  constexpr int WAVES = C::WAVES * C::Workers;
  static_assert(WAVES <= 64, "one packet of maxima per lane");
  constexpr bool SOLO = C::SOLO;
  __shared__ alignas(16) cx<float> Q[LINES * LS], Z2[(SOLO ? 2 : 1) * LINES * LS], W[LINES * LS];
  __shared__ float redf[2 * NT / 64];
  __shared__ int dead;
  __shared__ unsigned long long rolled;
  if (blockIdx.x % kDispatchXcds != 0) return;
  const int tid = threadIdx.x, ln = tid & 63, party = blockIdx.x / kDispatchXcds;
  const unsigned parties = C::Workers + (a.sampled ? 1 : 0);
  unsigned long long* roll = reinterpret_cast<unsigned long long*>(y.scratch + 2 * chain_clear_units(M)) - 1;
  const unsigned xcd = __builtin_amdgcn_s_getreg(kHwRegXccId) & 15u;
  if (tid == 0) {
    dead = 0;
    if (parties > 1) roll_answer(roll, party < C::Workers, xcd);
  }
  const ChainWait wait{y.spin_limit, y.err, &dead};
  // the scratch in packets: the tile after the row and after the column phase, the
  // new window, the maxima, the counters, the terms
  float2* tile1 = y.scratch;
  float2 *tile2 = tile1 + 2 * M * M, *window = tile2 + 2 * M * M, *maxima = window + 2 * M * M;
  unsigned* counters = reinterpret_cast<unsigned*>(maxima + 2 * 64);
  constexpr size_t kTermsAt = 2 * chain_clear_units(M);
  float* terms = reinterpret_cast<float*>(y.scratch + kTermsAt);
  if (party == C::Workers) {
    if (tid == 0) rolled = roll_call(roll, parties + y.absent);
    __syncthreads();
    if (rolled & kRollOff) return;
    chain_account<M, V>(a, n_steps, terms, counters, wait, y.skew);
    return;
  }
  const __amdgpu_buffer_rsrc_t b1 = through_buffer(tile1, 2 * M * M), b2 = through_buffer(tile2, 2 * M * M),
                               bw = through_buffer(window, 2 * M * M), bm = through_buffer(maxima, 2 * 64),
                               cb = through_buffer(reinterpret_cast<float2*>(counters), 32);
  const int line0 = party * LINES;  // its rows, and columns
  // places in the passes.  Strided row passes: lanes of a row beside each other (window
  // rows are read that way).  The others: lanes of one position beside each other (the
  // order of the exchanged tile and of the intensities).  The one workgroup of m = 32: every
  // pass with whole lines in a wave, so that only the turns between rows and columns and
  // the new window need a block barrier.
  PassPlace sr, sc, ct;
  const int ir = pass_item<R2>(tid, sr), ic = pass_item<R1>(tid, ct);
  sc = sr;
  sr.line = ir / R1;
  sr.g = ir % R1;
  sc.line = SOLO ? ir / R1 : C::column(ir % LINES);
  sc.g = SOLO ? ir % R1 : ir / LINES;
  ct.line = SOLO ? ic / R2 : ic % LINES;
  ct.g = SOLO ? ic % R2 : ic / LINES;
  // packet of the tile's element (row, p): blocks of LINES transform-order columns
  auto at = [](int row, int p) { return ((p / LINES) * M + row) * LINES + C::slot(p % LINES); };
  int at_row[4], at_col_in[4], at_col_out[4], at_row_in[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    at_row[i] = at(line0 + ct.line, R1 * ct.g + pass_in<R1, 1>(i, ct));
    at_row_in[i] = at(line0 + ct.line, R1 * ct.g + pass_in<R1>(i, ct));
    at_col_in[i] = at(sc.g + R1 * pass_in<R2>(i, sc), line0 + sc.line);
    at_col_out[i] = at(sc.g + R1 * pass_out<R2>(i, sc), line0 + sc.line);
  }
  const bool every[4] = {true, true, true, true};

  // twiddles W^(g j) of the strided passes: forward on the outputs, inverse on the inputs
  cx<float> wrf[4], wri[4], wcf[4], wci[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    wrf[i] = ld(a.tw, sr.g * pass_out<R2>(i, sr));
    wri[i] = conjg(ld(a.tw, sr.g * pass_in<R2>(i, sr)));
    wcf[i] = ld(a.tw, sc.g * pass_out<R2>(i, sc));
    wci[i] = conjg(ld(a.tw, sc.g * pass_in<R2>(i, sc)));
  }
  // v[i] <- w[i] v[i], the value of index 0 (value 0 of the lanes with h0 = h1 = 0) as it is
  const bool first = sr.h0 == 0 && sr.h1 == 0;
  auto twiddle = [&](cx<float>* v, const cx<float>* w) {
    const cx<float> t = mul_fma(w[0], v[0]);
    v[0] = cx<float>{first ? v[0].re : t.re, first ? v[0].im : t.im};
#pragma unroll
    for (int i = 1; i < 4; ++i) v[i] = mul_fma(w[i], v[i]);
  };
  // the values of a pass in W: points g + R1 j (strided) or R1 g + j (contiguous) of a
  // line, a column's in a row of W of their own or (the one workgroup) down W.  An item's lanes lie in one wave, so an item goes back to where it was read
  // without a block barrier; wave_order keeps the compiler from moving the accesses.
  auto line_sync = [&]() {
    if constexpr (SOLO) wave_order();
    else __syncthreads();
  };
  auto in_row = [](int line, int p) { return line * LS + p; };
  auto in_column = [](int line, int p) { return SOLO ? p * LS + line : line * LS + p; };
  auto put_strided = [&](auto in, const cx<float>* v, const PassPlace& s) {
#pragma unroll
    for (int i = 0; i < 4; ++i) W[in(s.line, s.g + R1 * pass_out<R2>(i, s))] = v[i];
  };
  auto get_strided = [&](auto in, cx<float>* v, const PassPlace& s) {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = W[in(s.line, s.g + R1 * pass_in<R2>(i, s))];
  };
  auto put_contiguous = [&](auto in, const cx<float>* v) {
#pragma unroll
    for (int i = 0; i < 4; ++i) W[in(ct.line, R1 * ct.g + pass_out<R1>(i, ct))] = v[i];
  };
  auto get_contiguous = [&](auto in, cx<float>* v) {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = W[in(ct.line, R1 * ct.g + pass_in<R1>(i, ct))];
  };

  for (int e = tid; e < LINES * M; e += NT) Q[(e / M) * LS + e % M] = ld(a.probe, (size_t)line0 * M + e);
  // a thread's outputs of a contiguous pass (F = 0) are positions trow .. trow + 3 of its line
  const int trow = R1 * ct.g + pass_out<R1>(0, ct), tline = line0 + ct.line;
  float d_next[4];
  auto load_intensities = [&](int k) {
    const float* dk = a.dperm + (size_t)k * M * M;
#pragma unroll
    for (int i = 0; i < 4; ++i) d_next[i] = dk[(trow + i) * M + tline];
  };
  auto uniform = [](int4 s) {
    return make_int4(__builtin_amdgcn_readfirstlane(s.x), __builtin_amdgcn_readfirstlane(s.y),
                     __builtin_amdgcn_readfirstlane(s.z), 0);
  };
  auto window_of = [&](const int4& s) {
    return through_buffer(a.obj + (size_t)s.y * a.n + s.z, (M - 1) * a.n + M);
  };
  // the thread's pixels of a window in the strided row pass
  auto load_window = [&](const int4& s, cx<float>* z) {
    const __amdgpu_buffer_rsrc_t w = window_of(s);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      z[i] = ld_agent(w, (line0 + sr.line) * a.n + sr.g + R1 * pass_in<R2>(i, sr));
  };
  // slots run a step ahead of the window they give: no step waits for its slot's load
  int4 sl = uniform(a.slot[0]), before = sl, ahead = a.slot[min(1, n_steps - 1)];
  cx<float> z[4];
  load_window(sl, z);
  load_intensities(sl.x);
  if (parties > 1 && tid == 0) rolled = roll_call(roll, parties + y.absent);
  __syncthreads();
  // all workers on this one's XCD
  bool shared_l2 = false;
  if (parties > 1) {
    const unsigned long long w = rolled;
    if (w & kRollOff) return;
    shared_l2 = !y.apart && xcd < kDispatchXcds &&
                (int)((w >> (kRollXcdBits * (xcd % kDispatchXcds))) & ((1 << kRollXcdBits) - 1)) == C::Workers;
    shared_l2 = __builtin_amdgcn_readfirstlane(shared_l2);
  }

  for (int step = 0; step < n_steps; ++step) {
    const unsigned sent = (unsigned)step + 1, n = sent + y.skew;  // packets' numbers: sent, awaited
    const int4 next = uniform(ahead);
    ahead = a.slot[min(step + 2, n_steps - 1)];
    cx<float>* Z = Z2 + (SOLO && (step & 1) ? LINES * LS : 0);
    cx<float> v[4];
    float d[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) d[i] = d_next[i];

    // 1. exit wave and forward row passes
    {
      if (step > 0) {  // the pixels that the previous step updated
        const int dr = line0 + sr.line + sl.y - before.y, dc = sl.z - before.z;
        int from[4];
        bool in[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int c = sr.g + R1 * pass_in<R2>(i, sr) + dc;
          in[i] = (unsigned)dr < (unsigned)M && (unsigned)c < (unsigned)M;
          from[i] = in[i] ? dr * (SOLO ? LS : M) + c : 0;
        }
        if constexpr (SOLO) {
          const cx<float>* Zp = Z2 + (step & 1 ? 0 : LINES * LS);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            cx<float> t = Zp[from[i]];
            asm("" : "+v"(t.re), "+v"(t.im));  // loaded by every lane, not behind a branch
            z[i] = cx<float>{in[i] ? t.re : z[i].re, in[i] ? t.im : z[i].im};
          }
        } else if (in[0] || in[1] || in[2] || in[3]) {
          receive<4>(bw, from, in, z, n - 1, wait);
        }
      }
      float q2m = 0.f, z2m = 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int o = sr.line * LS + sr.g + R1 * pass_in<R2>(i, sr);
        const cx<float> q = Q[o];
        Z[o] = z[i];
        q2m = fmaxf(q2m, norm2(q));
        z2m = fmaxf(z2m, norm2(z[i]));
        v[i] = mul(q, z[i]);
      }
      load_intensities(next.x);
      group_dft<R2, false>(v, sr);
      twiddle(v, wrf);
      put_strided(in_row, v, sr);
      if constexpr (SOLO) wave_max2_to_lds<NT>(q2m, z2m, redf, tid);
      line_sync();
      get_contiguous(in_row, v);
      group_dft<R1, false>(v, ct);
      if constexpr (SOLO) {
        wave_order();
        put_contiguous(in_row, v);
      } else {
        outputs_to_inputs<R1>(v);
        send<4>(b1, at_row, v, sent, shared_l2);
        q2m = wave_max(q2m);
        z2m = wave_max(z2m);
        if (ln == 0) {
          const int to = party * C::WAVES + (tid >> 6);
          const cx<float> m{q2m, z2m};
          send<1>(bm, &to, &m, sent, shared_l2);
        }
      }
    }

    // 2. forward column passes, projection, inverse column passes
    // a look at the summing workgroup's progress (in a vector register, so it is not waited for
    // before its use)
    int summed = 0, lane0 = 0;
    asm("" : "+v"(lane0));
    if (a.sampled)
      summed = __builtin_amdgcn_raw_buffer_load_b32(cb, lane0 + kChainSummed * 4, 0, kCachePolicyThrough);
    float t[4];
    cx<float> pm{0.f, 0.f};
    if constexpr (SOLO) {
      __syncthreads();
      get_strided(in_column, v, sc);
    } else {
      receive<4>(b1, at_col_in, every, v, n, wait);
    }
    group_dft<R2, false>(v, sc);
    twiddle(v, wcf);
    if constexpr (SOLO) wave_order();
    else __syncthreads();  // every wave has read its row items
    put_strided(in_column, v, sc);
    if constexpr (!SOLO) {
      const int from = ln % WAVES;
      receive<1>(bm, &from, every, &pm, n, wait);
    }
    // the stores of the step before (object, terms) are complete: said to the summing
    // workgroup, and implied by what this one sends from here on
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    // `dead` is looked at where no wave can set it between this barrier and the next, so that
    // all waves see the same: here, or where one workgroup has no barrier before its wait for
    // the summing one below, after the barrier that follows that
    if constexpr (!SOLO)
      if (dead) break;
    if (a.sampled && tid == 0 && step > 0)
      __hip_atomic_fetch_add(counters + kChainStored, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    get_contiguous(in_column, v);
    group_dft<R1, false>(v, ct);
    {
      float2* ph =
          (PH && a.phase) ? a.phase + (size_t)sl.x * M * M + (size_t)trow * M + tline : nullptr;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        t[i] = project_amp<M>(v[i], amplitude(d[i]), (PH && ph) ? ph + i * M : nullptr, a.phase_write != 0);
    }
    outputs_to_inputs<R1>(v);
    group_dft<R1, true, 1>(v, ct);
    wave_order();
#pragma unroll
    for (int i = 0; i < 4; ++i) W[in_column(ct.line, R1 * ct.g + pass_out<R1, 1>(i, ct))] = v[i];
    line_sync();
    get_strided(in_column, v, sc);
    twiddle(v, wci);
    group_dft<R2, true>(v, sc);
    if constexpr (SOLO) {
      wave_order();
      put_strided(in_column, v, sc);
    } else {
      send<4>(b2, at_col_out, v, sent, shared_l2);
    }
    if (a.sampled) {
      if (step >= kChainTermSteps && (int)((unsigned)summed + kChainTermSteps - n) < 0)
        wait.counter(counters + kChainSummed, n - kChainTermSteps);
      st_pair_through(through_buffer(reinterpret_cast<float2*>(
                                         terms + (size_t)(step % kChainTermSteps) * M * M), M * M / 2),
                      (tline * M + trow) / 2, cx<float>{t[0], t[1]}, cx<float>{t[2], t[3]});
    }

    // 3. inverse row passes, then the update of the workgroup's rows
    float qqmax, zmax;
    if constexpr (SOLO) {
      __syncthreads();
      if (dead) break;
      get_contiguous(in_row, v);
      group_dft<R1, true>(v, ct);
      lds_max2<NT>(redf, qqmax, zmax);
      wave_order();
    } else {
      qqmax = wave_max(pm.re);
      zmax = wave_max(pm.im);
      receive<4>(b2, at_row_in, every, v, n, wait);
      group_dft<R1, true>(v, ct);
      __syncthreads();  // every wave has read its column items, and received: from all workgroups
    }
    load_window(next, z);  // current outside this step's window
    put_contiguous(in_row, v);
    line_sync();
    get_strided(in_row, v, sr);
    twiddle(v, wri);
    group_dft<R2, true>(v, sr);
    wave_order();
    put_strided(in_row, v, sr);
    line_sync();
    cx<float> qb[4], zb[4], rb[4];
    int r0, c0;
    ChainRows<M>::origin(tid, 0, r0, c0);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int o = (r0 + (e >> 1)) * LS + c0 + (e & 1);
      qb[e] = Q[o];
      zb[e] = Z[o];
      rb[e] = W[o];
    }
    auto load = [&](int, int, int, cx<float>* q, cx<float>* zz, cx<float>* Rv) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        q[e] = qb[e];
        zz[e] = zb[e];
        Rv[e] = rb[e];
      }
    };
    const ChainSink<M, LS, SOLO> sink{window_of(sl), bw, a.n, line0, sent, shared_l2, Q, Z};
    if constexpr (SOLO) {
      pixel_update_body<M, ChainRows<M>, L, false>(a, 0, tid, line0, load, qqmax, zmax, sink);
    } else {
      pixel_update_body<M, ChainRows<M>, L, false, kObject>(a, 0, tid, line0, load, qqmax, zmax, sink);
      pixel_update_body<M, ChainRows<M>, L, false, kProbe>(a, 0, tid, line0, load, qqmax, zmax, sink);
    }
    __syncthreads();  // the probe rows are written, Z and W read
    before = sl;
    sl = next;
  }
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (a.sampled && tid == 0)
    __hip_atomic_fetch_add(counters + kChainStored, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (a.update_probe)
    for (int e = tid; e < LINES * M; e += NT) st(a.probe, (size_t)line0 * M + e, Q[(e / M) * LS + e % M]);
}

// The sweep in one workgroup: of few steps, or (roll) one that the launch before called off.
// Every step touches only its own window and the probe, and the workgroup barrier at its end
// orders it before the next.  3.8 us per step at m = 32, 8 at m = 64, 28 at m = 128.
template <int M, int V, int L, bool PH>
__global__ __launch_bounds__((Plan<M, V>::NT)) void k_sweep_one(StepArgs a, int n_steps,
                                                               const unsigned long long* roll) {
  __shared__ cx<float> A[M * lds_stride<M>()];
  __shared__ cx<float> tws[M];
  __shared__ float redf[32];
  __shared__ double redd[16];
  if (roll && !(*roll & kRollOff)) return;
  const int tid = threadIdx.x;
  stage_twiddles<M, Plan<M, V>::NT>(a.tw, tws, tid);
  __syncthreads();
  // the finalize's additions
  double sampled = (tid == 0 && a.sampled) ? *a.sampled : 0.0;
  for (int step = 0; step < n_steps; ++step) {
    StepArgs x = a;
    x.slot = a.slot + step;
    x.b = 1;
    double t = 0.0;
    t += patch_step<M, V, L, false, PH, InPlace>(x, 0, A, tws, redf, redd, tid);
    sampled += t;
  }
  if (tid == 0 && a.sampled) *a.sampled = sampled;
}

}  // namespace emg
