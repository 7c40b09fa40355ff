// Per-lane steps of the fused overlap-and-save kernel (sec. 3.2, Alg. 2):
// segment load with zero fill, spectrum product, discard-and-store.  Shared by
// the device kernels and by the host emulator used in CPU tests.
#pragma once

#include <type_traits>

#include "ols_fft.hpp"

namespace ols {

// Raw buffers of the device code.  Loads and stores of a wave that holds one
// segment (G >= 64) go through a buffer resource over exactly the elements
// that exist: the hardware range check returns zero for the loads outside it
// and drops the stores (a negative offset wraps to a huge unsigned one), with
// no per-lane compare, branch or zero fill and 32-bit offsets.
#if defined(__HIP_DEVICE_COMPILE__)
constexpr int CPOL_NT = 2;  // cache-policy operand of the buffer builtins: nt

// Raw buffer over [base, base + bytes).
template <class P>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(P base, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, bytes, 0x00020000);
}

// Element at byte offset off (zero outside the buffer).
__device__ __forceinline__ float2 buffer_load_c64(__amdgpu_buffer_rsrc_t rs, int off) {
  typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
  const u32x2 d = __builtin_amdgcn_raw_buffer_load_b64(rs, off, 0, 0);
  return make_float2(__uint_as_float(d.x), __uint_as_float(d.y));
}
__device__ __forceinline__ float buffer_load_f32(__amdgpu_buffer_rsrc_t rs, int off) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0));
}

// Hides how a lane offset was computed, so that the sixteen offsets derived from
// it are added again at each use instead of held in registers over a loop.
__device__ __forceinline__ void opaque(int& v) { asm volatile("" : "+v"(v)); }

// Buffer over the elements of window [start, start + len) of an array of n that
// exist, and the number of the window's elements before the first of them.
// start is the same in every lane.
struct WindowBuffer {
  __amdgpu_buffer_rsrc_t rs;
  int skip;
};
template <class P>
__device__ __forceinline__ WindowBuffer window_buffer(P src, int64_t start, int len, int64_t n, int el) {
  const int64_t before = start < 0 ? -start : 0;
  const int skip = before < len ? (int)before : len;
  const int64_t first = start + skip, rem = n - first;  // first >= 0, or the window is empty
  const int count = rem <= 0 ? 0 : (rem < len - skip ? (int)rem : len - skip);
  return WindowBuffer{make_rsrc(wave_uniform_ptr(src + (count > 0 ? first : 0)),
                                __builtin_amdgcn_readfirstlane(count * el)),
                      __builtin_amdgcn_readfirstlane(skip)};
}
#endif

// Segment j covers signal samples start .. start + N - 1 with
// start = j*H - D (D >= M-1 samples of history, sec. 3.2); samples outside
// [0, N_s) read as zero.  Register reg of lane g receives the sample at
// position g + time_pos_const(reg) of the segment.
template <int N, class P>
OLS_HD void load_segment(float2 (&x)[16], P __restrict__ s, int64_t Ns, int64_t start, int g) {
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (Geo<N>::G >= 64) {
    const WindowBuffer w = window_buffer(s, start, N, Ns, 8);
#pragma unroll
    for (int reg = 0; reg < 16; ++reg)
      x[reg] = buffer_load_c64(w.rs, (g + time_pos_const<N>(reg) - w.skip) * 8);
    return;
  }
#endif
  // valid positions p satisfy lo <= p < hi (clamped into [0, N])
  const int64_t lo64 = -start, hi64 = Ns - start;
  const int lo = lo64 <= 0 ? 0 : (lo64 >= N ? N : (int)lo64);
  const int hi = hi64 <= 0 ? 0 : (hi64 >= N ? N : (int)hi64);
#pragma unroll
  for (int reg = 0; reg < 16; ++reg) {
    const int p = g + time_pos_const<N>(reg);
    x[reg] = (p >= lo && p < hi) ? load_c64(s, start + p) : make_float2(0.f, 0.f);
  }
}

// Filter r zero padded to N (plan step, Fig. 1 / Alg. 2): register reg of
// lane g receives tap g + time_pos_const(reg) - shift if that is in [0, M)
// (shift > 0 delays the filter by that many samples; see row_shift).
template <int N>
OLS_HD void load_filter(float2 (&x)[16], const float2* __restrict__ h, int M, bool valid, int g, int shift = 0) {
#pragma unroll
  for (int reg = 0; reg < 16; ++reg) {
    const int p = g + time_pos_const<N>(reg) - shift;
    x[reg] = (valid && p >= 0 && p < M) ? h[p] : make_float2(0.f, 0.f);
  }
}

// Filter r followed by a first difference, h'[k] = h[k] - h[k-1] for
// k = 0 .. M (h[-1] = h[M] = 0): y' = y * [1, -1] is the derivative of the
// convolved signal (sec. 4, non-local post-processing) and, being a
// convolution, it folds into the filter spectrum at no cost per segment.
template <int N>
OLS_HD void load_filter_diff(float2 (&x)[16], const float2* __restrict__ h, int M, bool valid, int g, int shift = 0) {
#pragma unroll
  for (int reg = 0; reg < 16; ++reg) {
    const int p = g + time_pos_const<N>(reg) - shift;
    const float2 a = (valid && p >= 0 && p < M) ? h[p] : make_float2(0.f, 0.f);
    const float2 b = (valid && p >= 1 && p <= M) ? h[p - 1] : make_float2(0.f, 0.f);
    x[reg] = csub(a, b);
  }
}

// Real filter r (R2R plans) as complex taps with zero imaginary part,
// optionally followed by the first difference of load_filter_diff.
template <int N>
OLS_HD void load_filter_real(float2 (&x)[16], const float* __restrict__ h, int M, bool valid, bool diff, int g,
                             int shift = 0) {
#pragma unroll
  for (int reg = 0; reg < 16; ++reg) {
    const int p = g + time_pos_const<N>(reg) - shift;
    float a = (valid && p >= 0 && p < M) ? h[p] : 0.f;
    if (diff) a -= (valid && p >= 1 && p <= M) ? h[p - 1] : 0.f;
    x[reg] = make_float2(a, 0.f);
  }
}

// Two real segments in one complex transform (R2R): segment 2q in the real
// part, segment 2q+1 in the imaginary part.  With real filters the product
// of their joint spectrum with a filter spectrum transforms back to the two
// real convolutions in the real and imaginary parts, so the pair costs one
// complex FFT of length N and needs no split of the spectra.  start is the
// window start of segment 2q; segment 2q+1 starts H samples later.
template <int N, class P>
OLS_HD void load_segment_pair(float2 (&x)[16], P __restrict__ s, int64_t Ns, int64_t start, int H, int g) {
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (Geo<N>::G >= 64) {
    const WindowBuffer a = window_buffer(s, start, N, Ns, 4), b = window_buffer(s, start + H, N, Ns, 4);
#pragma unroll
    for (int reg = 0; reg < 16; ++reg) {
      const int p = g + time_pos_const<N>(reg);
      x[reg] = make_float2(buffer_load_f32(a.rs, (p - a.skip) * 4), buffer_load_f32(b.rs, (p - b.skip) * 4));
    }
    return;
  }
#endif
  const int64_t lo0 = -start, hi0 = Ns - start;
  const int lo_a = lo0 <= 0 ? 0 : (lo0 >= N ? N : (int)lo0);
  const int hi_a = hi0 <= 0 ? 0 : (hi0 >= N ? N : (int)hi0);
  const int64_t lo1 = lo0 - H, hi1 = hi0 - H;
  const int lo_b = lo1 <= 0 ? 0 : (lo1 >= N ? N : (int)lo1);
  const int hi_b = hi1 <= 0 ? 0 : (hi1 >= N ? N : (int)hi1);
  const P sa = s + start;
  const P sb = sa + H;
#pragma unroll
  for (int reg = 0; reg < 16; ++reg) {
    const int p = g + time_pos_const<N>(reg);
    x[reg] = make_float2((p >= lo_a && p < hi_a) ? sa[p] : 0.f, (p >= lo_b && p < hi_b) ? sb[p] : 0.f);
  }
}

// Spectra are stored in the order the forward transform leaves them in
// registers, two registers of a lane side by side: F[r][reg/2][g][reg%2].
// Each lane then loads its 16 values with 8 16-byte loads, and a wave reads
// 1 KB contiguous per load (half the load instructions of 8-byte loads;
// 3-6 % faster forward kernels).
template <int N>
OLS_HD int spectrum_offset(int reg, int g) { return (((reg >> 1) * Geo<N>::G + g) << 1) + (reg & 1); }

template <int N, bool LEAN = false, class P>
OLS_HD void load_spectrum(float2 (&f)[16], P __restrict__ F, int r, int g) {
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (N == 2048 || LEAN) {
    // One lane offset and scalar strides instead of eight 64-bit lane
    // addresses: 2^23 x 32 431.5 -> 428.9 us, its power 377 -> 370.5.  At N =
    // 1024 and 4096 level or slower (2^18 x 16, N = 4096: 16.1 -> 17.4).
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(wave_uniform_ptr(F + (int64_t)r * N), N * 8);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
      const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, g * 16, j * Geo<N>::G * 16, 0);
      f[2 * j] = make_float2(__uint_as_float(v.x), __uint_as_float(v.y));
      f[2 * j + 1] = make_float2(__uint_as_float(v.z), __uint_as_float(v.w));
    }
    return;
  }
#endif
  const auto Fr = rebind_ptr<const f32x4>(F + (int64_t)r * N);
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const f32x4 v = Fr[j * Geo<N>::G + g];
    f[2 * j] = make_float2(v.x, v.y);
    f[2 * j + 1] = make_float2(v.z, v.w);
  }
}

template <int N>
OLS_HD void store_spectrum(const float2 (&x)[16], float2* __restrict__ F, int r, int g, float scale = 1.0f) {
  float2* Fr = F + (int64_t)r * N;
#pragma unroll
  for (int reg = 0; reg < 16; ++reg) Fr[spectrum_offset<N>(reg, g)] = cscale(x[reg], scale);
}

// x = A * f (point-wise product in the permuted frequency order, sec. 3.4)
OLS_HD void spectrum_product(float2 (&x)[16], const float2 (&A)[16], const float2 (&f)[16]) {
#pragma unroll
  for (int reg = 0; reg < 16; ++reg) x[reg] = cmul(A[reg], f[reg]);
}

// Output stores.  Forward outputs are written once and never read back by
// the kernel, so they take the non-temporal (streaming) cache policy, which
// measured ~7 % faster than default stores on the filter-bank benchmark.
// When a transform spans whole waves (G >= 64) a wave's segment and output
// row are wave-uniform, so the stores go through a buffer resource covering
// exactly the kept outputs: the hardware range check drops the aliased and
// past-the-end positions (a negative offset wraps to a huge unsigned one),
// with no per-lane compare or branch.  Smaller transforms share a wave
// between segments and use per-lane predicates.
//
// Non-temporal stores only pay for whole 64-byte granules.  A granule that
// one store instruction covers only in part (rows of complex outputs whose
// length N_s is not a multiple of 8 start off the 64-byte grid; so can a
// segment edge) is written with the default policy instead, so that its two
// partial writes can merge in L2 before they go to HBM: with non-temporal
// partial writes the forward kernel ran 1.5-1.75x slower when its rows were
// off the grid, with the split policy 1.15x.  The batched kernel uses the
// split policy too (its rows, of arbitrary length, are mostly off the grid;
// the uneven batch ran 13 % faster with every row on the grid).
// How a kernel writes its outputs: plain per-lane predicated stores,
// non-temporal predicated stores, or non-temporal stores for whole granules
// only (buffer stores when G >= 64, predicated ones otherwise), or plain stores
// through a buffer when G >= 64.  Kernels near the register limit keep the
// cheaper forms.
enum StoreMode { STORE_PLAIN = 0, STORE_NT = 1, STORE_NT_WHOLE = 2, STORE_BUFFER = 3 };

// P: float* or gptr<float> (float2* or gptr<float2> for the complex form)
template <int MODE, typename P>
OLS_HD void out_store(P p, float v) {
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (MODE != STORE_PLAIN) {
    __builtin_nontemporal_store(v, p);
    return;
  }
#endif
  *p = v;
}

template <int MODE, typename P>
OLS_HD void out_store(P p, float2 v) {
  out_store<MODE>(&p->x, v.x);
  out_store<MODE>(&p->y, v.y);
}

// Vector elements (packed stencil phases): one store of the whole vector.
template <int MODE, typename P>
OLS_HD void out_store(P p, f32x2 v) {
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (MODE != STORE_PLAIN) {
    __builtin_nontemporal_store(v, p);
    return;
  }
#endif
  *p = v;
}

template <int MODE, typename P>
OLS_HD void out_store(P p, f32x4 v) {
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (MODE != STORE_PLAIN) {
    __builtin_nontemporal_store(v, p);
    return;
  }
#endif
  *p = v;
}

#if defined(__HIP_DEVICE_COMPILE__)
template <int CPOL>
__device__ __forceinline__ void buffer_store(float2 v, __amdgpu_buffer_rsrc_t rs, int off) {
  typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
  u32x2 d;
  d.x = __float_as_uint(v.x);
  d.y = __float_as_uint(v.y);
  __builtin_amdgcn_raw_buffer_store_b64(d, rs, off, 0, CPOL);
}

template <int CPOL>
__device__ __forceinline__ void buffer_store(float v, __amdgpu_buffer_rsrc_t rs, int off) {
  __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rs, off, 0, CPOL);
}

template <int CPOL>
__device__ __forceinline__ void buffer_store(f32x2 v, __amdgpu_buffer_rsrc_t rs, int off) {
  buffer_store<CPOL>(make_float2(v.x, v.y), rs, off);
}

template <int CPOL>
__device__ __forceinline__ void buffer_store(f32x4 v, __amdgpu_buffer_rsrc_t rs, int off) {
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  u32x4 d;
  d.x = __float_as_uint(v.x);
  d.y = __float_as_uint(v.y);
  d.z = __float_as_uint(v.z);
  d.w = __float_as_uint(v.w);
  __builtin_amdgcn_raw_buffer_store_b128(d, rs, off, 0, CPOL);
}
#endif

// Number of outputs a segment whose first output is out0 keeps: min(H, N_s - out0), >= 0.
OLS_HD int kept_count(int64_t Ns, int64_t out0, int H) {
  const int64_t rem = Ns - out0;
  return rem >= H ? H : (rem < 0 ? 0 : (int)rem);
}

// Position of an element inside its 64-byte granule, in elements.
template <typename T>
OLS_HD int granule_phase(const T* p) {
  return (int)(((uintptr_t)p / sizeof(T)) & (64 / sizeof(T) - 1));
}

// Stores of one segment's kept outputs.  After the inverse transform register
// reg of lane g holds circular position p = g + time_pos_const(reg); positions
// D .. D+H-1 are unaliased (D >= M-1, sec. 3.2) and go to outputs
// out0 + p - D, out0 = j*H; outputs >= N_s are not written.  val(reg) gives
// the value stored from register reg.
//
// STORE_NT_WHOLE: one store instruction writes C = min(G, 64) consecutive
// positions of a segment (lane l = g mod C of a chunk that starts on a
// multiple of C; time_pos_const is a multiple of G, and of LS, the outputs
// per 64-byte granule).  The phase c of a lane's output inside its granule
// is therefore the same in every register, so whether the chunk holds the
// lane's whole granule (l - c >= 0 and l - c + LS <= C) is a property of the
// lane: those lanes store non-temporally, the others (the partial granules
// at the two ends of each chunk when the row is off the 64-byte grid) with
// the default policy.  The first and last granule of a segment are partial
// when they share a granule with the neighbouring segment; the chunk test
// sees that exactly when the segment's kept positions start and end on chunk
// boundaries (D a multiple of C, and D + H = N as with the default hop),
// otherwise its head and tail granules may go non-temporal, two granules in
// H / LS.  The choice of policy never changes what is written.
// Registers R0 .. R0 + NR - 1 only (callers that produce the values in parts).
template <int N, int MODE, int R0 = 0, int NR = 16, typename T, typename V>
OLS_HD void store_segment(T* __restrict__ yrow, int64_t Ns, int64_t out0, int D, int H, int g, V val) {
  // T is float2 or float, with the pointer's address space (gptr) if any
  constexpr int LS = 64 / (int)sizeof(T);                // outputs per 64-byte granule
  constexpr int C = Geo<N>::G < 64 ? Geo<N>::G : 64;     // positions per store instruction
  static_assert(C % LS == 0, "chunks hold whole granules");
  const int cnt = kept_count(Ns, out0, H);
  const int l = g & (C - 1);
  const int c = (granule_phase(yrow + out0) + g - D) & (LS - 1);
  const bool whole = l >= c && l - c + LS <= C;
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (MODE == STORE_NT_WHOLE && Geo<N>::G >= 64) {
    // a wave holds one segment here, so its row, first output and count are
    // wave-uniform; saying so keeps the descriptor in scalar registers (the
    // compiler cannot always prove it, and would loop over the lanes)
    const __amdgpu_buffer_rsrc_t rs =
        make_rsrc(wave_uniform_ptr(yrow + out0), __builtin_amdgcn_readfirstlane(cnt * (int)sizeof(T)));
    if (whole) {
#pragma unroll
      for (int reg = R0; reg < R0 + NR; ++reg)
        buffer_store<CPOL_NT>(val(reg), rs, (g + time_pos_const<N>(reg) - D) * (int)sizeof(T));
    } else {
#pragma unroll
      for (int reg = R0; reg < R0 + NR; ++reg)
        buffer_store<0>(val(reg), rs, (g + time_pos_const<N>(reg) - D) * (int)sizeof(T));
    }
    return;
  }
#endif
#if defined(__HIP_DEVICE_COMPILE__)
  // the adjoint's windows (2^22 x 16: N = 1024 222.5 -> 220, N = 2048 264 -> 261.5 us;
  // at N = 8192 more spills, 212 -> 217)
  if constexpr ((MODE == STORE_BUFFER || (MODE == STORE_PLAIN && N <= 2048)) && Geo<N>::G >= 64) {
    const __amdgpu_buffer_rsrc_t rs =
        make_rsrc(wave_uniform_ptr(yrow + out0), __builtin_amdgcn_readfirstlane(cnt * (int)sizeof(T)));
#pragma unroll
    for (int reg = R0; reg < R0 + NR; ++reg)
      buffer_store<0>(val(reg), rs, (g + time_pos_const<N>(reg) - D) * (int)sizeof(T));
    return;
  }
#endif
  T* base = yrow + (out0 - D);
  if (MODE == STORE_NT || (MODE == STORE_NT_WHOLE && whole)) {
#pragma unroll
    for (int reg = R0; reg < R0 + NR; ++reg) {
      const int p = g + time_pos_const<N>(reg);
      if (p >= D && p < D + cnt) out_store<STORE_NT>(base + p, val(reg));
    }
  } else {
#pragma unroll
    for (int reg = R0; reg < R0 + NR; ++reg) {
      const int p = g + time_pos_const<N>(reg);
      if (p >= D && p < D + cnt) out_store<STORE_PLAIN>(base + p, val(reg));
    }
  }
}

// F maps the transform value to the stored one (the identity, or the power
// epilogue of sec. 4 with a float output).
template <int N, int MODE, typename T, typename F>
OLS_HD void store_kept(const float2 (&x)[16], T* __restrict__ yrow, int64_t Ns, int64_t out0, int D, int H, int g,
                       F f) {
  store_segment<N, MODE>(yrow, Ns, out0, D, H, g, [&](int reg) { return f(x[reg]); });
}

struct Identity {
  OLS_HD float2 operator()(float2 v) const { return v; }
};
// Per-element post-processing at the store (sec. 4): the power |y|^2 as
// float32, half the output bytes of complex64.
struct Power {
  OLS_HD float operator()(float2 v) const { return fmaf(v.x, v.x, v.y * v.y); }
};

template <int N, int MODE = STORE_PLAIN, class P>
OLS_HD void store_valid(const float2 (&x)[16], P yrow, int64_t Ns, int64_t out0, int D, int H, int g) {
  store_kept<N, MODE>(x, yrow, Ns, out0, D, H, g, Identity());
}

template <int N, int MODE = STORE_PLAIN, class P>
OLS_HD void store_valid_power(const float2 (&x)[16], P yrow, int64_t Ns, int64_t out0, int D, int H, int g) {
  store_kept<N, MODE>(x, yrow, Ns, out0, D, H, g, Power());
}

// ---------------------------------------------------------------------------
// Non-local post-processing (sec. 4: an output may depend on its neighbours,
// the paper's examples being the numerical derivative and interpolation).
// After the inverse transform the segment's outputs are written to LDS in
// natural order; each kept position p then combines the outputs at p - L ..
// p + R into J values by a stencil with real weights and J outputs (phases) per sample,
//     z[J n + j] = sum_{d=-L}^{R} w[j][d + L] * y[n + d],   n = out0 + p - D,
// optionally followed by the power.  The kept positions must see unaliased
// neighbours: D >= M - 1 + L and D + H + R <= N (stencil_delay), so the last
// segment also reads samples past N_s, which the zero-filled segment load
// makes eq. (1)'s tail.  Any hop up to N - D - R gives the same result.
// ---------------------------------------------------------------------------
constexpr int STENCIL_MAX_PHASES = 4;  // J: outputs per sample
constexpr int STENCIL_MAX_TAPS = 8;    // T = L + 1 + R
constexpr int STENCIL_PAD = 8;         // staged slots before and after a segment (>= max L, R)

struct Stencil {
  int J;       // phases, 1 .. STENCIL_MAX_PHASES
  int L;       // taps before the sample
  int T;       // taps, L + 1 + R
  int packed;  // the output is aligned to J elements: J <= 2 takes stage_store_packed
  float w[STENCIL_MAX_PHASES][STENCIL_MAX_TAPS];  // w[j][d + L]; zero past T and J
};

// A stencil with one output per sample is a convolution: it multiplies the
// segment's spectrum by its transfer function
//     S(k) = sum_d w[d] exp(+2 pi i k d / N),   d = -L .. T-1-L,
// once per segment instead of staging every filter's output.  Circularly it
// shifts by up to L back and R ahead, which the kept window leaves room for
// (stencil_delay), so the outputs are those of the staged stencil, and the
// power, R2R and row re-alignment apply as to a plain forward.  The function
// stays in registers for all of a workgroup's segments.  N = 8192 has none left
// and would gather it for every segment (2^24 samples, one filter: 146 us
// against 97 staged), so it stages.
OLS_HD constexpr bool fold_stencil(int N) { return N <= 4096; }
struct Response {
  int T;  // taps; 0: no stencil
  int L;  // taps before the sample
  float w[STENCIL_MAX_TAPS];
};
// Phases of a delay by d samples (of an advance for d < 0) at lane g's
// frequencies: register reg holds frequency k0 + reg * N / 16, so one root per
// lane and a step that all lanes share give all sixteen,
//     exp(-2 pi i d k / N) = z * u^reg,  z = root[k0 d mod N],  u = root[d N / 16 mod N],
// where a table read per frequency is sixteen loads whose lanes meet as many
// cache lines (the order of k0 over the lanes is digit reversed).  In float64:
// the product's rounding is far below the one to float32 that follows.
// root[m] = exp(-2 pi i m / N).
template <int N, class P>
OLS_HD double2 delay_root(P root, int k0, int d) { return load_c128(root, (k0 * d) & (N - 1)); }
template <int N, class P>
OLS_HD double2 delay_step(P root, int d) { return load_c128(root, (d * (N / 16)) & (N - 1)); }

// x times the phases of a delay by d samples.
template <int N, class P>
OLS_HD void delay_spectrum(float2 (&y)[16], const float2 (&x)[16], P root, int d, int g) {
  double2 z = delay_root<N>(root, spectrum_index<N>(g, 0), d);
  const double2 u = delay_step<N>(root, d);
#pragma unroll
  for (int reg = 0; reg < 16; ++reg) {
    y[reg] = cmul(x[reg], make_float2((float)z.x, (float)z.y));
    z = cmul64(z, u);
  }
}

// S(k) for lane g's frequencies, summed in float64 and rounded once.  Tap t
// advances by d = t - L.  Of its sixteen phases z u^reg only z u^a, a < 4, are
// formed: u^4 = (-i)^d, so the taps of equal t mod 4 share the rest, a radix-4
// step with a rotation by i^(bL) for b = reg / 4.  The roots of all taps load
// together.  One tap's phases from the table, sixteen loads at a time, held up
// the start of every workgroup (us, staged / that / this: 8 taps, 3000000 x 1 x
// 64, N = 4096 19.4 / 39.4 / 17.1; 100001 x 4 x 64, N = 512 9.3 / 10.8 / 8.8; two
// taps, 100001 x 4 x 64, N = 4096 8.9 / 9.8 / 8.9).
template <int N, class P>
OLS_HD void stencil_response(float2 (&S)[16], P root, const Response& st, int g) {
  const int k0 = spectrum_index<N>(g, 0);
  double2 z[STENCIL_MAX_TAPS], u[STENCIL_MAX_TAPS];
#pragma unroll
  for (int t = 0; t < STENCIL_MAX_TAPS; ++t) {
    if (t < st.T) {
      z[t] = delay_root<N>(root, k0, t - st.L);
      u[t] = delay_step<N>(root, t - st.L);
    }
  }
  // C[e][a]: sum over the taps with t mod 4 = e of w z u^a
  double2 C[4][4];
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int a = 0; a < 4; ++a) C[e][a] = make_double2(0.0, 0.0);
#pragma unroll
  for (int t = 0; t < STENCIL_MAX_TAPS; ++t) {
    if (t < st.T) {
      const double w = st.w[t];
      double2 v = z[t];
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        double2& c = C[t & 3][a];
        c = make_double2(fma(w, v.x, c.x), fma(w, v.y, c.y));
        if (a < 3) v = cmul64(v, u[t]);
      }
    }
  }
  // register a + 4 b: conj(i^(bL) sum_e (-i)^(be) C[e][a])  (the weights are real)
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    const double2 c0 = C[0][a], c1 = C[1][a], c2 = C[2][a], c3 = C[3][a];
    const double2 p = make_double2(c0.x + c2.x, c0.y + c2.y), m = make_double2(c0.x - c2.x, c0.y - c2.y);
    const double2 q = make_double2(c1.x + c3.x, c1.y + c3.y), n = make_double2(c1.x - c3.x, c1.y - c3.y);
    const double2 y[4] = {make_double2(p.x + q.x, p.y + q.y), make_double2(m.x + n.y, m.y - n.x),
                          make_double2(p.x - q.x, p.y - q.y), make_double2(m.x - n.y, m.y + n.x)};
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int r = (b * st.L) & 3;  // turns by i
      const float re = (float)y[b].x, im = (float)y[b].y;
      const float x = (r & 1) ? -im : re, v = (r & 1) ? re : im;
      S[a + 4 * b] = (r & 2) ? make_float2(-x, v) : make_float2(x, -v);
    }
  }
}

// LDS slots of one staged segment: position p at STENCIL_PAD + p, so every
// tap of every position of the transform stays inside its own segment slots.
template <int N>
constexpr int stage_stride() { return N + 2 * STENCIL_PAD; }

// First kept position of a plan whose stencil reaches L back and R ahead
// (Meff: taps of the filter as applied): the default_delay rounding when
// D + R <= N - 1 still holds, else exactly Meff - 1 + L.  The hop may reach
// N - D - R.
OLS_HD int stencil_delay(int N, int Meff, int L, int R) {
  const int lo = Meff - 1 + L;
  const int d = (lo + 15) / 16 * 16;
  return d + R <= N - 1 ? d : lo;
}

// Default hop with a stencil: N - D - R, rounded down to a multiple of 16
// samples when it is at least 16, so that segments keep starting on the
// 128-byte output grid (as the plain default hop does).
OLS_HD int stencil_hop(int N, int D, int R) {
  const int h = N - D - R;
  return h >= 16 ? h & ~15 : h;
}

// The transform output of lane g (register reg = circular position
// g + time_pos_const(reg)) into the segment's LDS slots.
template <int N>
OLS_HD void stage_write(float2* __restrict__ region, const float2 (&x)[16], int g) {
#pragma unroll
  for (int reg = 0; reg < 16; ++reg) region[STENCIL_PAD + g + time_pos_const<N>(reg)] = x[reg];
}

// Phase j of the stencil at the 16 positions of lane g.  The tap loop runs T
// times (wave-uniform); position p + d - L is read for tap d, inside the
// segment's slots for every p (|d - L| <= STENCIL_PAD), from staged outputs
// for every kept p.
template <int N, class S>
OLS_HD void stage_phase(float2 (&acc)[16], const float2* __restrict__ region, const S& st, int j, int g) {
#pragma unroll
  for (int reg = 0; reg < 16; ++reg) acc[reg] = make_float2(0.f, 0.f);
  const float2* src = region + STENCIL_PAD + g - st.L;
  for (int d = 0; d < st.T; ++d) {
    const float wd = st.w[j][d];
#pragma unroll
    for (int reg = 0; reg < 16; ++reg) {
      const float2 v = src[d + time_pos_const<N>(reg)];
      acc[reg].x = fmaf(wd, v.x, acc[reg].x);
      acc[reg].y = fmaf(wd, v.y, acc[reg].y);
    }
  }
}

// Store of phase j of a segment's kept positions: position p (D <= p <
// D + cnt) goes to element J * (out0 + p - D) + j of the row.  Rows with
// J > 1 are written J elements apart by each instruction, so the default
// cache policy lets the phases of a granule merge in L2.  A wave-wide
// transform (G >= 64) stores through a buffer resource over exactly the
// segment's J * cnt elements, whose range check drops the other positions.
template <int N, typename T, typename V>
OLS_HD void store_phase(T* __restrict__ yrow, int64_t Ns, int64_t out0, int D, int H, int g, int J, int j, V val) {
  const int cnt = kept_count(Ns, out0, H);
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (Geo<N>::G >= 64) {
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(wave_uniform_ptr(yrow + (int64_t)J * out0),
                                               __builtin_amdgcn_readfirstlane(J * cnt * (int)sizeof(T)));
#pragma unroll
    for (int reg = 0; reg < 16; ++reg)
      buffer_store<0>(val(reg), rs, ((g + time_pos_const<N>(reg) - D) * J + j) * (int)sizeof(T));
    return;
  }
#endif
  T* base = yrow + (int64_t)J * out0;
#pragma unroll
  for (int reg = 0; reg < 16; ++reg) {
    const int p = g + time_pos_const<N>(reg);
    if (p >= D && p < D + cnt) out_store<STORE_PLAIN>(base + (p - D) * J + j, val(reg));
  }
}

// All JC phases at positions R0 .. R0 + NR - 1 of lane g (acc[j][reg - R0]),
// each tap read from LDS once.
template <int N, int JC, int R0, int NR, class S>
OLS_HD void stage_phases(float2 (&acc)[JC][NR], const float2* __restrict__ region, const S& st, int g) {
#pragma unroll
  for (int j = 0; j < JC; ++j)
#pragma unroll
    for (int i = 0; i < NR; ++i) acc[j][i] = make_float2(0.f, 0.f);
  const float2* src = region + STENCIL_PAD + g - st.L;
  for (int d = 0; d < st.T; ++d) {
    float wd[JC];
#pragma unroll
    for (int j = 0; j < JC; ++j) wd[j] = st.w[j][d];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const float2 v = src[d + time_pos_const<N>(R0 + i)];
#pragma unroll
      for (int j = 0; j < JC; ++j) {
        acc[j][i].x = fmaf(wd[j], v.x, acc[j][i].x);
        acc[j][i].y = fmaf(wd[j], v.y, acc[j][i].y);
      }
    }
  }
}

// One (JC = 1) or two phases per position written as one element: a float2,
// float or the vector of the two phases, so that each store instruction
// covers consecutive positions whole and the store policy of store_segment
// (non-temporal for whole 64-byte granules) applies as to a plain row.
// yrow must be aligned to the element (Stencil::packed).
// The positions go in parts of STAGE_PART registers, which bounds the live
// accumulators.
constexpr int STAGE_PART = 4;
template <int N, int JC, bool POWER, bool REAL, int SMODE, int R0, class S, class P>
OLS_HD void stage_store_packed_part(const float2* __restrict__ region, const S& st, P yrow, int64_t Ns, int64_t out0,
                                    int D, int H, int g) {
  constexpr int NR = STAGE_PART;
  float2 acc[JC][NR];
  stage_phases<N, JC, R0, NR>(acc, region, st, g);
  if constexpr (REAL || POWER) {
    // float rows: component c of each phase (REAL) or the power (POWER)
    auto val = [&](int reg, int c) {
      float v[JC];
#pragma unroll
      for (int j = 0; j < JC; ++j) {
        const float2 a = acc[j][reg - R0];
        v[j] = REAL ? (c == 0 ? (POWER ? a.x * a.x : a.x) : (POWER ? a.y * a.y : a.y)) : Power()(a);
      }
      if constexpr (JC == 1) return v[0];
      else return f32x2{v[0], v[1]};
    };
    using V = typename std::conditional<JC == 1, float, f32x2>::type;
    const auto yv = rebind_ptr<V>(yrow);
    store_segment<N, SMODE, R0, NR>(yv, Ns, out0, D, H, g, [&](int reg) { return val(reg, 0); });
    if constexpr (REAL)
      store_segment<N, SMODE, R0, NR>(yv, Ns, out0 + H, D, H, g, [&](int reg) { return val(reg, 1); });
  } else if constexpr (JC == 1) {
    store_segment<N, SMODE, R0, NR>(yrow, Ns, out0, D, H, g, [&](int reg) { return acc[0][reg - R0]; });
  } else {
    const auto yv = rebind_ptr<f32x4>(yrow);
    store_segment<N, SMODE, R0, NR>(yv, Ns, out0, D, H, g, [&](int reg) {
      const float2 a = acc[0][reg - R0], b = acc[1][reg - R0];
      return f32x4{a.x, a.y, b.x, b.y};
    });
  }
}

template <int N, int JC, bool POWER, bool REAL, int SMODE, class S, class P>
OLS_HD void stage_store_packed(const float2* __restrict__ region, const S& st, P yrow, int64_t Ns, int64_t out0,
                               int D, int H, int g) {
  static_assert(JC == 1 || JC == 2, "one or two phases per element");
  stage_store_packed_part<N, JC, POWER, REAL, SMODE, 0>(region, st, yrow, Ns, out0, D, H, g);
  stage_store_packed_part<N, JC, POWER, REAL, SMODE, STAGE_PART>(region, st, yrow, Ns, out0, D, H, g);
  if constexpr (STAGE_PART < 8) {
    stage_store_packed_part<N, JC, POWER, REAL, SMODE, 2 * STAGE_PART>(region, st, yrow, Ns, out0, D, H, g);
    stage_store_packed_part<N, JC, POWER, REAL, SMODE, 3 * STAGE_PART>(region, st, yrow, Ns, out0, D, H, g);
  }
}

// Every phase of the stencil for one filter's staged segment, stored to row
// yrow (J * N_s elements; float for POWER or REAL).  REAL: the staged values
// hold segment 2q in the real part and 2q + 1 in the imaginary part (R2R
// pairs), stored from out0 and out0 + H.  J <= 2 with an aligned output takes
// the packed form; otherwise each phase is computed and stored on its own,
// J elements apart.
template <int N, bool POWER, bool REAL, int SMODE = STORE_PLAIN, class S, class P>
OLS_HD void stage_store(const float2* __restrict__ region, const S& st, P yrow, int64_t Ns, int64_t out0, int D,
                        int H, int g) {
  if constexpr (!fold_stencil(N)) {
    if (st.packed && st.J == 1) {
      stage_store_packed<N, 1, POWER, REAL, SMODE>(region, st, yrow, Ns, out0, D, H, g);
      return;
    }
  }
  if (st.packed && st.J == 2) {
    stage_store_packed<N, 2, POWER, REAL, SMODE>(region, st, yrow, Ns, out0, D, H, g);
    return;
  }
  for (int j = 0; j < st.J; ++j) {
    float2 acc[16];
    stage_phase<N>(acc, region, st, j, g);
    if constexpr (REAL) {
      store_phase<N>(yrow, Ns, out0, D, H, g, st.J, j,
                     [&](int reg) { return POWER ? acc[reg].x * acc[reg].x : acc[reg].x; });
      store_phase<N>(yrow, Ns, out0 + H, D, H, g, st.J, j,
                     [&](int reg) { return POWER ? acc[reg].y * acc[reg].y : acc[reg].y; });
    } else if constexpr (POWER) {
      store_phase<N>(yrow, Ns, out0, D, H, g, st.J, j, [&](int reg) { return Power()(acc[reg]); });
    } else {
      store_phase<N>(yrow, Ns, out0, D, H, g, st.J, j, [&](int reg) { return acc[reg]; });
    }
  }
}

// ---------------------------------------------------------------------------
// Adjoint (gradient) helpers.  For the adjoint, segment j's window starts at
// j*H (no delay): the correlation with conj(h) uses future samples, so the
// aliased positions are at the end of the window and positions 0 .. H-1 are
// exact for H <= N - M + 1 (footnote to eq. 2).
// ---------------------------------------------------------------------------

// x[reg] = src[start + p] for p = g + time_pos_const(reg) < lim and
// start + p < N_s (start >= 0); zero elsewhere.
template <int N, bool LEAN = false>
OLS_HD void load_window(float2 (&x)[16], const float2* __restrict__ src, int64_t Ns, int64_t start, int lim, int g) {
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (Geo<N>::G >= 64) {
    const WindowBuffer w = window_buffer(src, start, lim, Ns, 8);
    int go = g * 8;
    if constexpr (LEAN) opaque(go);
#pragma unroll
    for (int reg = 0; reg < 16; ++reg) x[reg] = buffer_load_c64(w.rs, go + time_pos_const<N>(reg) * 8);
    return;
  }
#endif
  const int64_t rem = Ns - start;
  const int hi = rem <= 0 ? 0 : (rem >= lim ? lim : (int)rem);
#pragma unroll
  for (int reg = 0; reg < 16; ++reg) {
    const int p = g + time_pos_const<N>(reg);
    x[reg] = p < hi ? src[start + p] : make_float2(0.f, 0.f);
  }
}

// A = conj(x) * scale
OLS_HD void conj_scaled(float2 (&A)[16], const float2 (&x)[16], float scale) {
#pragma unroll
  for (int i = 0; i < 16; ++i) A[i] = make_float2(x[i].x * scale, -x[i].y * scale);
}

// acc += G * conj(F)
OLS_HD void acc_conj_product(float2 (&acc)[16], const float2 (&G)[16], const float2 (&F)[16]) {
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = cfma<true>(G[i], F[i], acc[i]);
}

// Lags 0 .. M-1 of a time-domain result: part[p] += x[reg] for p < M.  Every
// lag is always owned by the same lane, so the read-modify-write needs no
// synchronisation.
// LEAN (here, in load_window and load_spectrum): for a kernel without registers
// for sixteen addresses and masks; through buffers, with offsets made again.
template <int N, bool LEAN = false>
OLS_HD void add_lags(float2* __restrict__ part, const float2 (&x)[16], int M, int g) {
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (LEAN) {
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(wave_uniform_ptr(part), __builtin_amdgcn_readfirstlane(M * 8));
    int go = g * 8;
    opaque(go);
    float2 old[4];
#pragma unroll
    for (int reg = 0; reg < 4; ++reg) old[reg] = buffer_load_c64(rs, go + time_pos_const<N>(reg) * 8);
#pragma unroll
    for (int reg = 0; reg < 4; ++reg) buffer_store<0>(cadd(old[reg], x[reg]), rs, go + time_pos_const<N>(reg) * 8);
#pragma unroll
    for (int q = 1; q < 4; ++q) {
      if (time_pos_const<N>(4 * q) < M) {
#pragma unroll
        for (int k = 0; k < 4; ++k) old[k] = buffer_load_c64(rs, go + time_pos_const<N>(4 * q + k) * 8);
#pragma unroll
        for (int k = 0; k < 4; ++k)
          buffer_store<0>(cadd(old[k], x[4 * q + k]), rs, go + time_pos_const<N>(4 * q + k) * 8);
      }
    }
    return;
  }
#endif
#pragma unroll
  for (int reg = 0; reg < 16; ++reg) {
    const int p = g + time_pos_const<N>(reg);
    if (p < M) part[p] = cadd(part[p], x[reg]);
  }
}

// The same for a workgroup's first unit of a filter: stored, nothing to add to.
template <int N, bool LEAN = false>
OLS_HD void store_lags(float2* __restrict__ part, const float2 (&x)[16], int M, int g) {
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (LEAN) {
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(wave_uniform_ptr(part), __builtin_amdgcn_readfirstlane(M * 8));
    int go = g * 8;
    opaque(go);
#pragma unroll
    for (int reg = 0; reg < 16; ++reg)
      if (time_pos_const<N>(reg) < M) buffer_store<0>(x[reg], rs, go + time_pos_const<N>(reg) * 8);
    return;
  }
#endif
#pragma unroll
  for (int reg = 0; reg < 16; ++reg) {
    const int p = g + time_pos_const<N>(reg);
    if (p < M) part[p] = x[reg];
  }
}

// Store of a segment pair (R2R): the real part holds segment 2q's output,
// written from out0 = 2q*H, the imaginary part segment 2q+1's, written from
// out0 + H; each with its own end bound.  POWER squares each sample.
template <int N, bool POWER, int MODE = STORE_PLAIN, class P>
OLS_HD void store_valid_pair(const float2 (&x)[16], P yrow, int64_t Ns, int64_t out0, int D, int H, int g) {
  store_segment<N, MODE>(yrow, Ns, out0, D, H, g,
                         [&](int reg) { return POWER ? x[reg].x * x[reg].x : x[reg].x; });
  store_segment<N, MODE>(yrow, Ns, out0 + H, D, H, g,
                         [&](int reg) { return POWER ? x[reg].y * x[reg].y : x[reg].y; });
}

// Workgroup rows of the spectra launch, which share out a bank's delays: enough
// for two workgroups per CU, at most one row per delay.
OLS_HD int delay_rows(int blocks, int delays, int cus) {
  const int rows = (2 * cus + blocks - 1) / blocks;
  return rows < delays ? rows : delays;
}

// Filters per work unit of the forward kernels: two interleaved transforms
// when a transform spans several waves (N = 2048, 4096: the pair shares each
// exchange's barriers), registers allow it and the filter count wastes little
// on a padded last group.  Single-wave transforms (N <= 1024) exchange
// without barriers and measured as fast or faster with one filter per unit.
constexpr int BATCH_NF2_MAX_N = 2048;
OLS_HD int choose_nf(int N, int K) { return (N >= 2048 && N <= 4096 && (K % 2 == 0 || K >= 9)) ? 2 : 1; }
// The batched kernel's registers are set by its largest branch, so one filter
// per unit saves nothing there, and two measured faster up to N = 1024 (64
// uneven signals: 723 against 749 us).  At N = 2048 so too when tiles are dealt
// whole (513 against 534), but not in shares, where one filter cuts finer (30
// signals: 42.6 against 43.9; see batch_shares).
OLS_HD int choose_nf_batched(int N, int K, bool shares) {
  return (N <= (shares ? 1024 : BATCH_NF2_MAX_N) && (K % 2 == 0 || K >= 9)) ? 2 : 1;
}
// R2R (segment pairs) needs a few more registers per transform: two filters
// per unit only up to N = 2048 as well.
OLS_HD int choose_nf_real(int N, int K) { return N <= BATCH_NF2_MAX_N ? choose_nf(N, K) : 1; }

// ---------------------------------------------------------------------------
// Segment geometry and FFT-length choice, shared by the host plan code and the
// device-side batch setup so that both always reach the same answer.
// ---------------------------------------------------------------------------
// First kept circular position: M - 1 rounded up to a multiple of 16 samples
// (128-byte aligned output windows) when that still leaves room, else M - 1.
OLS_HD int default_delay(int N, int M) {
  const int d = ((M - 1) + 15) / 16 * 16;
  return d <= N - 1 ? d : M - 1;
}

// Cost model for N = 0: transform work per kept output sample, about
// (K + 1) * 3.2 N log2 N + K * 4 N flops per segment over K * H kept samples,
// among N >= cost_model_min_n(K).  Compared as exact integers (5x the work,
// cross-multiplied by the hops) so that the host and the device pick the same
// N.  Lengths whose measured time per output is worse than their flop count
// says are left out:
//   * N = 256 and 512: their transforms are narrower than a wave and measured
//     10-24 % slower per output than N = 1024 on every cell of the
//     2^25-sample sweep where both fit, although they need up to ~10 % fewer
//     flops;
//   * N = 1024 for K >= COST_MODEL_WIDE_K filters: with the inverse
//     transforms dominating, N = 2048 measured 1-12 % faster per output
//     (K = 24 .. 64, M = 32, 128, 256, 2^25 samples) although it needs ~7 %
//     more flops; at K = 8 N = 1024 is 6-7 % faster, as the flops say.
// Returns 0 if no length in [cost_model_min_n(K), max_n] holds M taps.
constexpr int COST_MODEL_MIN_N = 1024;
constexpr int COST_MODEL_WIDE_K = 24;
OLS_HD int cost_model_min_n(int K) { return K >= COST_MODEL_WIDE_K ? 2 * COST_MODEL_MIN_N : COST_MODEL_MIN_N; }
OLS_HD int cost_model_fft_length(int K, int M, int max_n) {
  int best = 0;
  unsigned __int128 best_w = 0, best_h = 1;
  for (int n = cost_model_min_n(K); n <= max_n; n *= 2) {
    if (n < M) continue;
    const int h = n - default_delay(n, M);
    if (h < 1) continue;
    const unsigned __int128 w = (unsigned __int128)(K + 1) * 16u * (unsigned)n * (unsigned)ilog2(n) +
                                (unsigned __int128)K * 20u * (unsigned)n;
    if (best == 0 || w * best_h < best_w * (unsigned)h) {
      best = n;
      best_w = w;
      best_h = (unsigned)h;
    }
  }
  return best;
}

// Batched items: validation of one item (the checks ols_batch_plan and the
// workspace sizing do on the host, repeated by the device-side setup of
// ols_batched) and its FFT length.  Returns an ols_status_t value (0 = valid).
constexpr int BATCH_MIN_N = 256, BATCH_MAX_N = 4096;
OLS_HD int batch_item_check(const void* s, int64_t Ns, const void* h, int K, int M, int N, const void* y,
                            int* N_out) {
  if (K < 1 || M < 1 || Ns < 0) return 1;
  if (!h || (Ns > 0 && (!s || !y))) return 1;
  if (((uintptr_t)s | (uintptr_t)y | (uintptr_t)h) % 8) return 1;
  if (Ns > ((int64_t)1 << 56) / 8 / K) return 1;
  if (Ns > 0) {
    const uintptr_t s0 = (uintptr_t)s, s1 = s0 + (uintptr_t)Ns * 8;
    const uintptr_t y0 = (uintptr_t)y, y1 = y0 + (uintptr_t)Ns * 8 * (uintptr_t)K;
    if (s0 < y1 && y0 < s1) return 1;  // y overlaps s
  }
  int n = N;
  if (n == 0) {
    n = cost_model_fft_length(K, M, BATCH_MAX_N);
    if (n == 0) return 2;  // filter longer than the largest batched length
  }
  if (n < BATCH_MIN_N || n > BATCH_MAX_N || (n & (n - 1))) return 2;
  if (M > n) return 1;
  *N_out = n;
  return 0;
}

// Output rows off the 128-byte grid (the L2 line).  A row that starts off
// the grid (y not 128-byte aligned, or N_s not a multiple of LS, the outputs
// per line: 16 complex64 or 32 float32) would have every store
// instruction's run of consecutive outputs straddle two partly written
// lines.  For such a call each filter r is delayed by row_delay samples in
// its spectrum, which moves row r's outputs that many circular positions
// later: with the hop a multiple of LS, every store instruction then starts
// on a line (runs start at circular positions that are multiples of 64, or
// of the transform's G lanes), and only the two ends of each segment's kept
// window are partial.  The kept positions move with the filter (D + delay),
// so the hop must leave room for a delay of LS - 1.
struct RowShift {
  int H;     // hop the call runs with
  int mask;  // LS - 1 when the rows are shifted, else 0
};
constexpr int SHIFT_LINE = 128;  // bytes
// H: the plan's hop; el: bytes per output; allowed: the kernel supports it.
// The hop the call runs with is H rounded down to a multiple of LS, and no
// more than the room the delay leaves (N - D - (LS - 1), rounded down too);
// below LS the rows stay as they are.
OLS_HD RowShift row_shift_geometry(const void* y, int64_t Ns, int N, int D, int H, int el, bool allowed) {
  const int LS = SHIFT_LINE / el;
  const bool off = ((uintptr_t)y & (SHIFT_LINE - 1)) != 0 || (Ns & (LS - 1)) != 0;
  if (!allowed || !off) return RowShift{H, 0};
  const int room = (N - D - (LS - 1)) & ~(LS - 1);
  const int hs = (H & ~(LS - 1)) < room ? (H & ~(LS - 1)) : room;
  return hs >= LS ? RowShift{hs, LS - 1} : RowShift{H, 0};
}
// Delay of row r (0 .. mask): output n of row r is element r*N_s + n of y
// (el bytes each), and circular position p of segment j holds
// n = j*H - D + p - delay, so the line phase of a position p on the LS-sample
// grid is (y/el + r*N_s - D - delay) mod LS, which this delay makes 0.
OLS_HD int row_delay(const void* y, int el, int64_t Ns, int D, int r, int mask) {
  return (int)((((uintptr_t)y / (uintptr_t)el) + (uint64_t)r * (uint64_t)Ns - (uint64_t)D) & (uint64_t)mask);
}
// Batched items (complex64 rows, the default hop).
OLS_HD RowShift batch_row_shift(const void* y, int64_t Ns, int N, int D) {
  return row_shift_geometry(y, Ns, N, D, N - D, 8, true);
}

// ---------------------------------------------------------------------------
// How one forward call runs: filters per unit and threads per workgroup.  A
// choice of the call's size and the plan's occupancy, not of the grid set by
// ols_plan_set_tiling.
// ---------------------------------------------------------------------------
// Threads per workgroup.  One transform, or one wave of narrower ones, is the
// smallest (narrow).  A unit then holds one segment, so short calls spread over
// more CUs, long ones end more evenly, and a barrier joins only the waves of one
// transform.  Measured against 256 threads (us, complex, one GPU): N = 1024,
// 2^20 x 1 8.0 -> 7.0, 2^13 x 4 6.2 -> 4.9, 2^22 x 64 438 -> 427; N = 2048, 2^18
// x 7 11.4 -> 10.4, 2^21 x 7 33.9 -> 31.1, 2^23 x 32 (one filter per unit) 447 ->
// 433.  Long calls keep 256 threads (base) where the spectra are loaded without
// prefetch or fit in L1, because the segments of such a workgroup read each
// spectrum through one L1 at the same time: two filters per unit at N = 2048
// (2^23 x 32: 441 against 452 with 128), R2R at N = 1024 (2^23 x 16: 114.5
// against 120.7), and N <= 512 (2^22 x 8, N = 512: 57.1 against 61.4).
OLS_HD constexpr int base_threads(int N) { return N / 16 >= 256 ? N / 16 : 256; }
OLS_HD constexpr int narrow_threads(int N) { return N / 16 <= 64 ? 64 : N / 16; }
OLS_HD constexpr int wide_threads(int N, int nf, bool real) {
  return (N <= 512 || (N == 1024 && real) || (N == 2048 && nf == 2)) ? base_threads(N) : narrow_threads(N);
}
struct ForwardShape {
  int nf, wg;
};
struct ForwardCall {
  int N, K, H;         // H: the call's hop
  int nf;              // the plan's filters per unit
  bool nf_auto;        // they are the library's choice
  bool real, power;
  bool on_grid;        // output rows on the 128-byte grid
  bool realigned;      // off it, with delayed filters (row_shift_geometry)
  int64_t ntrans;      // transforms: segments, or segment pairs (R2R)
  int64_t full;        // workgroups of base_threads at full occupancy
  // Workgroups of wg threads that fill the device, and the units they share.
  OLS_HD int64_t slots(int wg) const { return full * (base_threads(N) / wg); }
  OLS_HD int64_t units(ForwardShape s) const {
    const int segs = s.wg / (N / 16);
    return (ntrans + segs - 1) / segs * ((K + s.nf - 1) / s.nf);
  }
  // Units of the longest workgroup.
  OLS_HD int64_t longest(ForwardShape s) const { return (units(s) + slots(s.wg) - 1) / slots(s.wg); }
  OLS_HD bool at_least(ForwardShape s, int per_workgroup) const { return units(s) >= per_workgroup * slots(s.wg); }
  // Times that the device reads the bank's spectra, as long as its workgroups keep
  // step: a tile starts slots / tiles workgroups after the one before, and
  // where that is a multiple of the 8 XCDs, which take the workgroups in turn,
  // both tiles read the same spectra through the same L2.
  OLS_HD int64_t bank_reads(ForwardShape s) const {
    const int segs = s.wg / (N / 16);
    const int64_t tiles = (ntrans + segs - 1) / segs;
    int64_t a = tiles, b = slots(s.wg) / 8;
    while (b != 0) {
      const int64_t r = a % b;
      a = b;
      b = r;
    }
    return a > 0 ? tiles / a : 0;
  }
};
OLS_HD ForwardShape forward_shape(const ForwardCall& c) {
  const int N = c.N, narrow = narrow_threads(N), base = base_threads(N);
  ForwardShape s{c.nf, narrow};
  const ForwardShape one{1, narrow}, two{2, narrow};
  // Plans that leave the tiling to the library: one filter per unit, with
  // prefetched spectra and twice the units (us, two -> one filter, workgroups of
  // one transform: N = 2048, 2^18 x 32 24.6 -> 20.5, 2^20 x 32 65.2 -> 58.7; N =
  // 4096, 2^15 x 16 9.1 -> 7.3, 2^18 x 16 19.3 -> 16.9), except where two
  // filters give every workgroup one unit and one filter does not (2^16 x 32, N
  // = 2048: 10.0 against 12.6; N = 8192, whose pair kernel has no prefetched
  // spectra and is 3-30 % slower elsewhere: 2^20 x 2 18.3 -> 14.4, 2^18 x 8
  // 17.8 -> 14.4).
  const bool one_unit = c.units(one) > c.slots(narrow) && c.units(two) <= c.slots(narrow);
  if (c.nf_auto && c.nf == 2 && N == 2048 && !one_unit) s.nf = 1;
  if (c.nf_auto && c.nf == 2 && N == 4096) {
    // a pair costs 1.86 single units (us, one / two filters: 1290944 x 4 x
    // 1300, 4 and 2 units 20.9 / 18.2, x 60, 3 and 2 units 17.7 / 20.6; 1710519
    // x 4 x 1571, 6 and 3 units 28.6 / 25.1), and from N4096_NF2_UNITS units per
    // workgroup the pair's shared barriers count (2^23 x 32: 446 against 457)
    constexpr int N4096_NF2_UNITS = 8;
    if (15 * c.longest(two) > 8 * c.longest(one) && !c.at_least(one, N4096_NF2_UNITS)) s.nf = 1;
  }
  if (c.nf_auto && N == 8192 && !c.real && one_unit) s.nf = 2;
  // base_threads, where they pay, from 8 (N <= 512) or 4 units each on (N = 512,
  // 2^20 x 8: 4.3 units, 20.7 against 20.1 us with 64 threads; R2R N = 1024, 2^19
  // x 8: 2.1 units, 12.3 against 11.9, 2^21 x 8: 4.1 units, 20.6 against 21.5; N =
  // 2048, two filters, 2^18 x 32: 2.3 units, 26.0 against 24.6, 2^19 x 32: 4.6
  // units, 36.9 against 37.5)
  const ForwardShape w{s.nf, wide_threads(N, s.nf, c.real)}, b{s.nf, base};
  if (w.wg != narrow && c.at_least(w, N <= 512 ? 8 : 4)) s = w;
  const int64_t bank = (int64_t)c.K * N * 8;  // bytes of spectra; an XCD's L2 holds 4 MiB
  const int aliased = N - c.H;
  if (N == 1024) {
    // Banks that the L2 does not hold, and many rows off the grid (whose spectra
    // lie delay by delay): a spectrum read by four segments at once, unless the
    // longest workgroup gets many more units by it.  us, 64 -> 256 threads: 10080 x
    // 512 x 200 17.2 -> 14.8, 23168 x 1024 x 200 64 -> 42, 92672 x 1024 x 19 201 ->
    // 164, power 18240 x 1300 x 19 47 -> 33, two filters per unit 17888 x 1182 x 133
    // 60 -> 50; off the grid 40337 x 128 x 19 17.6 -> 14.7, 370721 x 64 x 19 53.3 ->
    // 49.9.  Fewer filters are level or slower (on the grid 20160 x 256 x 19 14.5
    // against 15.1, off it 215153 x 24 x 19 16.1 against 16.0), and so are fewer
    // units (5040 x 1024 x 19: 3 units and 4, 14.2 against 14.9; 80673 x 64 x 19,
    // off the grid: 3 and 3, 15.6 against 16.2).  Banks of more than twice the L2
    // are worth a third more units (8000 x 1300 x 60, 6 and 8: 32.3 -> 26.3, x 2000, 9
    // and 12: 46.7 -> 34.7, R2R 5040 x 2000 19.6 -> 16.1; 5040 x 1300, 4 and 6: 18.4
    // against 20.1), not with the power, whose narrow workgroups are three waves
    // per SIMD (8000 x 2000 30.0 against 33.1).
    const ForwardShape narrowest{s.nf, narrow};
    const int64_t n = c.longest(narrowest), m = c.longest(b);
    const bool rows = c.realigned && (c.K >= 128 || (c.K >= 64 && n >= 8));
    const bool twice = bank >= ((int64_t)10 << 20) && !c.power;
    if ((bank >= ((int64_t)4 << 20) || rows) && n >= 2 && (twice ? 3 * m <= 4 * n : 4 * m <= 5 * n)) s = b;
  }
  if (N == 2048 && s.nf == 1) {
    // Two segments per workgroup; complex outputs with their waves in step
    // (step_forward).  us, 128 -> 256 threads:
    //   - banks of many short filters on the grid, which write as fast as the HBM
    //     takes it: 2^22 x 32 x 64 226 -> 204, 2^23 x 32 x 32 438 -> 416, 3000000 x
    //     32 x 112 170 -> 168, 2^19 x 32 x 32 36.6 -> 35.5.  Not from 128 aliased
    //     samples on (2^23 x 32: M = 128 415 against 423, M = 256 427 against 444),
    //     with fewer filters (2^22 x 16 x 64 109.7 against 111.6, 2^23 x 8 x 64 113
    //     against 120) or few units (2^18 x 32 x 64, 4 units: 21.4 against 22.1; 6
    //     units: 28.7 -> 27.5);
    //   - re-aligned rows the other way round: long filters, 741441 x 32 x 400 52.4
    //     -> 48.5, 1482897 x 64 x 400 179 -> 166, not short ones (2^23 + 1 x 32 x 64
    //     485 against 492) nor fewer rows (5931633 x 16 x 400 171 against 182);
    //   - banks of twice the L2, one segment at a time up to 6 TB/s of spectra:
    //     39537 x 600 x 400 67 -> 60, 72993 x 1300 x 400 (no delayed spectra) 250 ->
    //     204, power 51616 x 1300 x 60 133 -> 96, R2R 111841 x 600 x 60 85 -> 70;
    //     complex on the grid, of four times (23168 x 1024 x 400 70 -> 48; 158176 x
    //     600 x 400 157 against 168).  Where neighbouring workgroups happen to work
    //     on the same filters the L2 serves them either way, and the narrow ones
    //     are up to 10 % faster (power 39536 x 600 x 400 38 against 42).
    constexpr int STEP_ALIASED = 128, STEP_UNITS = 6;
    const bool shorts = aliased < STEP_ALIASED, complex = !c.real && !c.power;
    const bool step = complex && ((c.on_grid && shorts && c.K >= 24) || (c.realigned && !shorts && c.K >= 32));
    const bool large = bank >= ((int64_t)(complex && c.on_grid ? 16 : 8) << 20);
    if ((step || large) && c.at_least(b, STEP_UNITS)) s = b;
    // Banks over the L2: pairs of filters and of segments where the spectra read
    // less often outweigh what pairs add to the longest workgroup (a unit is worth
    // 32 MiB of spectra), up to READS_UNITS units per workgroup, beyond which the
    // workgroups no longer keep step; and for re-aligned rows of few units in place
    // of two segments, where pairs add nothing (us, one filter -> two: 10001 x 512 x
    // 400, 7 reads to 1, 22.9 -> 16.7, power 20.3 -> 15.7; 5040 x 1500 x 60 27.4 -> 22.4;
    // 130000 x 511 x 461, 83 reads to 21, 168 -> 128, R2R 101 -> 73; 264947 x 473 x 60 263
    // -> 242; re-aligned 10001 x 2000 x 400 59.8 -> 50.9, 14001 x 1500 x 60 49.7 -> 43.3.
    // Against: 8000 x 512 x 60 18.2 and 19.5, 10001 x 512 x 60, 3 reads and 3, 16.3 and
    // 19.9, 264960 x 473 x 461, 21 and 21, 220 and 231; re-aligned 39033 x 562 x 400 46.7
    // and 47.4).
    constexpr int READS_UNITS = 96, ROWS_UNITS = 16;
    const ForwardShape pair{2, base};
    if (c.nf_auto && c.nf == 2 && bank >= ((int64_t)4 << 20)) {
      const int64_t n = c.longest(s), p = c.longest(pair);
      const int64_t less = c.bank_reads(s) - c.bank_reads(pair);
      const bool rows = c.realigned && s.wg == base && n < ROWS_UNITS && 2 * p <= n;
      const bool reads = less > 0 && n <= READS_UNITS && 8 * less * bank > ((int64_t)32 << 20) * (15 * p - 8 * n);
      if (rows || reads) s = pair;
    }
  }
  return s;
}

// Classes of batched items, (N, filters per unit): the kernel takes the items
// class by class (stable within a class), so that each workgroup meets each
// class in one run of tiles.
constexpr int BATCH_CLASSES = 10;
OLS_HD constexpr int batch_class(int N, int nf) { return 2 * (ilog2(N) - 8) + (nf - 1); }

// Schedule of the batched kernel (the device kernel and the host emulator
// both walk it through these functions).  Tiles of all items, numbered in the
// kernel's item order, are dealt to the P persistent workgroups round-robin:
// workgroup b takes tiles b, b + P, b + 2P, ..., so the grid as a whole works
// on a window of neighbouring tiles of one or two items (whose filter spectra
// then stay in L2).  Dealing chunks of 2-8 consecutive tiles instead measured
// 4-18 % slower on the uneven batch.
OLS_HD int64_t first_batch_tile(int64_t b) { return b; }
OLS_HD int64_t next_batch_tile(int64_t t, int64_t P) { return t + P; }
// Dealing whole tiles suits batches of many tiles per workgroup.  With few,
// the tiles' uneven cost (one transform of the segments and one per filter)
// leaves workgroups idle: then workgroup b instead takes the b-th of P equal
// shares of the batch's weight, contiguous in the kernel's item order, cut at
// units; a tile cut between workgroups is transformed by each.  Weights count
// transforms per lane.  Past BATCH_SHARE_WEIGHT transforms per workgroup the
// spread of the shares over all items costs more spectrum reads than the
// balance saves.  Measured, us, dealt -> shared, by transforms per workgroup: 6
// 61 -> 34, 17 116 -> 87, 24 99.5 -> 86, 51 202 -> 168, 73 286 -> 252, 86 308 -> 291,
// 95 327 -> 373, 193 722 -> 807.
constexpr int BATCH_SHARE_WEIGHT = 88;
OLS_HD int64_t batch_item_weight(int64_t ntiles, int K) { return ntiles * (1 + (int64_t)K); }
OLS_HD bool batch_shares(int64_t total_weight, int64_t P) { return total_weight < BATCH_SHARE_WEIGHT * P; }
// Unit of an item that weight off falls in (0 <= off <= the item's weight, which
// gives the item's units; within the shared batches' bounds the product stays
// small).
OLS_HD int64_t batch_unit_at(int64_t off, int64_t units, int64_t weight) {
  return weight > 0 ? off * units / weight : 0;
}
// Workgroup index b of launch index blk: the hardware deals workgroups to the
// 8 XCDs round-robin by launch index, so consecutive b (consecutive chunks of
// a round, which share overlap samples and spectra) are put on one XCD and
// its L2.  A permutation of [0, P).
OLS_HD int64_t batch_workgroup_order(int64_t blk, int64_t P) {
  return P % 8 == 0 ? (blk % 8) * (P / 8) + blk / 8 : blk;
}

// dh reduction order: the per-slot partial lags are summed in chunks of
// DH_CHUNK consecutive slots (each chunk in slot order, one thread per lag
// and chunk), then the chunk sums in chunk order.  Fixed order, no atomics.
constexpr int DH_CHUNK = 16;
OLS_HD int64_t dh_chunks(int64_t nslots) { return (nslots + DH_CHUNK - 1) / DH_CHUNK; }

// Walk of one workgroup over its units [u0, u1) of a single signal: unit u is
// filter group u mod KG of tile u / KG (a tile's groups in order, then the
// next tile).  The forward kernels and the host emulator both walk with it.
struct UnitWalk {
  int64_t tile;
  int rg;  // filter group within the tile; KG once the tile is done
  OLS_HD UnitWalk(int64_t u0, int KG) : tile(u0 / KG), rg((int)(u0 - (u0 / KG) * KG)) {}
  // At the start of a unit: past the tile's last group the unit starts the
  // next tile (new segments to transform).
  OLS_HD bool tile_done(int KG) const { return rg == KG; }
  OLS_HD void next_tile() {
    rg = 0;
    ++tile;
  }
  OLS_HD int next_group(int KG) const { return rg + 1 == KG ? 0 : rg + 1; }  // group of the unit after this one
  OLS_HD void leave() { ++rg; }
};

// Partition arithmetic shared by the persistent kernels: workgroup b of P
// owns units [first_unit(b), first_unit(b+1)); owner(u) inverts it.
OLS_HD int64_t first_unit(int64_t U, int64_t P, int64_t b) { return U * b / P; }
OLS_HD int64_t owner_of_unit(int64_t U, int64_t P, int64_t u) { return ((u + 1) * P + U - 1) / U - 1; }

// ---------------------------------------------------------------------------
// Tail of the adjoint: split tiles' ds windows and the dh slots.
// ---------------------------------------------------------------------------
// Unit `unit` of the ds part: a tile whose filters are split between
// workgroups blo .. bhi, or none (t < 0).  A unit is a tile, or the boundary
// between workgroups unit and unit + 1, of which the first inside a tile
// stands for it.
struct SplitTile {
  int64_t t, blo, bhi;
};
OLS_HD SplitTile split_tile(int64_t U, int64_t P, int64_t upt, bool by_tile, int64_t unit) {
  int64_t t = unit;
  if (!by_tile) {
    const int64_t ub = first_unit(U, P, unit + 1);
    t = ub / upt;
    if (ub == t * upt || first_unit(U, P, unit) > t * upt) return SplitTile{-1, 0, 0};
  }
  const int64_t blo = owner_of_unit(U, P, t * upt), bhi = owner_of_unit(U, P, (t + 1) * upt - 1);
  return SplitTile{blo == bhi ? -1 : t, blo, bhi};
}

// Which slots hold lags of filter r: those of the workgroups with a unit of it,
// and of the groups that collect its parity in the paired adjoint.  The others
// are not written, and a call of few units per workgroup (K filters, one unit
// each, and K M values per slot) would otherwise spend its time clearing and
// reading them.
struct DhSlots {
  int64_t U, P;  // units and workgroups of the adjoint kernel
  int upt;       // units per tile
  int fpu;       // filters per unit
  int M;
};
// here[w]: workgroup b + w has a unit of filter r.
template <int NW>
OLS_HD void dh_workgroups(bool (&here)[NW], const DhSlots& sl, int64_t b, int r) {
  // workgroups own base or base + 1 consecutive units
  const int64_t base = sl.U / sl.P, rem = sl.U - base * sl.P;
  const bool all = base >= sl.upt;  // every workgroup has a unit of every filter
  const int q = r / sl.fpu;
  // first unit of workgroup b: its place in its tile, and what is left of
  // the division (carried from one workgroup to the next)
  const int64_t u0 = first_unit(sl.U, sl.P, b);
  int64_t left = sl.U * b - u0 * sl.P;
  int m = (int)(u0 % sl.upt);
#pragma unroll
  for (int w = 0; w < NW; ++w, ++b) {
    left += rem;
    const bool more = left >= sl.P;
    left -= more ? sl.P : 0;
    const int len = (int)(base < sl.upt ? base : sl.upt) + (more ? 1 : 0);
    const int d = q >= m ? q - m : q - m + sl.upt;
    here[w] = b < sl.P && (all || d < len);
    m += len;
    m -= m >= sl.upt ? sl.upt : 0;
  }
}
// Group `group` of a workgroup collects filter r.
template <bool PAIRED>
OLS_HD bool dh_group(int group, int r) { return !PAIRED || ((group ^ r) & 1) == 0; }

// How the tail's work is cut, for latency: a lane waits in turn for each of
// its ds outputs (their windows load together) and for each round of chunks of
// its dh lag.
//   ds   nfix units (split_tile), the tiles where they are fewer than the
//        boundaries, none where every tile has one workgroup, with `split`
//        workgroups each: at least four, eight for windows of more than 16
//        outputs per lane, and as many as a launch of TAIL_FIX_GROUPS allows (a
//        thousand workgroups that find nothing to do take 1.4 us), up to one
//        output per lane.
//   dh   2^lags_log2 lags per workgroup: 128 bytes of each slot where a
//        workgroup of the adjoint has one slot (2^22 x 16 x 512: 265 -> 259 us
//        against 64 bytes), 64 where it has several (2^18 x 16, N = 1024: 39
//        against 43), fewer while the chunks take several rounds and the launch
//        has not TAIL_DH_GROUPS workgroups.
// Four workgroups per boundary and the full width throughout (us, adjoint,
// that / this): many workgroups per tile, 4356 x 59 x 1, N = 4096, ds 29.7 / 15.0;
// many segments per tile, 2882696 x 6 x 3, N = 256, ds 57.7 / 43.2; many slots,
// 2628819 x 1 x 12, N = 256, dh 47.2 / 34.5.
constexpr int TAIL_THREADS = 256;
constexpr int64_t TAIL_FIX_GROUPS = 1024, TAIL_DH_GROUPS = 512;
struct TailShape {
  int64_t nfix, ndh;  // units of the ds part, workgroups of the dh part (a multiple of the 8 XCDs)
  int split, by_tile, lags_log2;
};
OLS_HD TailShape tail_shape(int segs, int H, int64_t ntiles, int64_t upt, int64_t grid, int64_t KM, bool ds, bool dh) {
  TailShape t{0, 0, 1, 0, 0};
  if (ds && grid > 1 && upt > 1 && ntiles % grid != 0) {
    t.by_tile = ntiles < grid - 1;
    t.nfix = t.by_tile ? ntiles : grid - 1;
    const int64_t one = ((int64_t)segs * H + TAIL_THREADS - 1) / TAIL_THREADS;  // one output per lane
    int64_t split = TAIL_FIX_GROUPS / t.nfix;
    const int least = one > 16 ? 8 : 4;
    split = split < least ? least : split;
    t.split = (int)(split < one ? split : one);
  }
  if (dh) {
    t.lags_log2 = segs == 1 ? 4 : 3;
    const int64_t chunks = dh_chunks(grid * segs);
    while (t.lags_log2 > 1 && chunks > (TAIL_THREADS >> t.lags_log2) && (KM >> t.lags_log2) < TAIL_DH_GROUPS)
      --t.lags_log2;
    const int64_t lags = (int64_t)1 << t.lags_log2;
    t.ndh = ((KM + lags - 1) / lags + 7) / 8 * 8;
  }
  return t;
}

}  // namespace ols
