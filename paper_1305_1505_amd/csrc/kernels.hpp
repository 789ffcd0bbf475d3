// HIP kernels of the collapse-time path for one grid size N and one precision.
//
// Layouts (C order, z fastest):
//   user half spectrum dk   [N][N][N/2+1] complex
//   half slot               [N][N][N/2]   complex -- the kz = N/2 (Nyquist) plane is zero by
//                                                    construction and is not stored
//   packed z slot           [N][N][N]     complex -- for one pair of real outputs (A, B), the
//       full-length z spectrum C = A + iB of each (x, y) line, stored as
//         P[k]       = C[k]       k in [0, N/2)
//         P[N/2 + k] = C[N - k]   k in [1, N/2)     (= conj(A[k]) + i conj(B[k]))
//       (P[N/2], the Nyquist term, is zero and is neither written nor read), so that both halves
//       are written as aligned runs by the y pass and the z pass loads each element once.  A slot
//       of one real output (B = 0) holds the first half only.
//   real field              [N][N][N]
//
// Inverse 3D transform of the six Hessian components with shared prefixes.  With
// g = M W dk / f^2 (M zeroes Nyquist modes, W the Gaussian window, f the integer wavevector),
// component (a, b, c) with a + b + c = 2 is the inverse transform of fx^a fy^b fz^c g, and the
// factors fx^a, fy^b, fz^c commute with the other axes' transforms:
//   x pass:  X_a = IFFT_x[fx^a g]                      a = 0, 1, 2         (1 -> 3 half slots)
//   y pass:  S_abc = IFFT_y[fy^b X_a] fz^c, written in pairs of components (3 -> 3 packed slots)
//   z pass:  IFFT_z of each packed pair gives two real components per complex transform; the six
//            real values of a point stay in registers for the per-point epilogue (collapse,
//            store, or the 2LPT source).
// Gradients (displacements) use the same passes with a + b + c = 1 and g = i c M dk / f^2.
// Every kernel first stages the twiddles it needs in LDS, laid out per FFT stage.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "collapse_dev.hpp"
#include "fft_core.hpp"
#include "host_math.hpp"
#include "ops.hpp"

namespace pin {

// ---------------------------------------------------------------------------------------------
// Tile shapes
// Tuning constants (measured at 512^3 on MI355X): 128-byte z rows for the strided passes; the z
// pass keeps one transform of 4 lines in LDS at a time (its three transforms run in turn), which
// keeps its LDS below 25 KB so that VGPRs, not LDS, bound its occupancy.
constexpr int kRowBytes = 128;
constexpr bool kZSequential = true;
constexpr int kZWaves = 4;
template <typename R> struct Tile {
  using V = typename Cplx<R>::type;
  static constexpr int PS = kRowBytes / (int)sizeof(V);   // strided passes: rows of z
};

// Blocks are dealt round-robin to the 8 XCDs (block b runs on XCD b mod 8).  The strided passes
// give XCD k the contiguous tile range [k G/8, (k+1) G/8): the tiles in flight on one XCD then
// cover whole rows of the same slabs, which spreads them over the L2 and lets the per-transform
// re-reads of an input tile (x and y passes) hit there.
__device__ __forceinline__ int xcd_tile(int b, int nblocks) {
  if (nblocks % 8 != 0) return b;
  return (b & 7) * (nblocks >> 3) + (b >> 3);
}

constexpr int round_up64(int x) { return (x + 63) / 64 * 64; }
// one butterfly a thread up to 1024; above, the most threads that share the butterflies evenly
// (1536 at N = 384 and 768: 768 threads with two each, not 1024 of which half have two)
constexpr int strided_threads(int nb0) {
  const int turns = (nb0 + 1023) / 1024;
  return round_up64((nb0 + turns - 1) / turns);
}
constexpr int pow2_floor(int x) {
  int p = 1;
  while (p * 2 <= x) p *= 2;
  return p;
}

// Strided passes (x, y): a workgroup owns PS consecutive z (one 128-byte row) of one pencil set
// and all N elements along the transform axis.
template <typename R, int N, int DIR>
struct Strided {
  using V = typename Cplx<R>::type;
  static constexpr int PS = Tile<R>::PS;
  static constexpr int HZ = N / 2;
  static constexpr int NZT = (HZ + PS - 1) / PS;
  using E0 = Engine<V, N, PS, 1, true, 64, DIR>;
  static constexpr int T = strided_threads(E0::nb(E0::R0));
  using E = Engine<V, N, PS, 1, true, T, DIR>;
  // occupancy target (least waves per SIMD), float32 tiles of at most 8 values a thread at either
  // end: two workgroups per CU (8 waves per SIMD of 64 VGPRs at 1024 threads, 6 of 80 at 768: with
  // one workgroup of 1024, 384^3 took 0.235 ms in the x and 0.532 in the y pass, 0.213 and 0.450
  // with two of 768); otherwise 4 (float64 tiles are LDS-bound there)
  static constexpr int WPE = sizeof(V) != 8 || !E::SAME ? 4 : E::max_held() <= 8 ? 8 : E::K0 > 1 && E::K0 * E::R0 <= 8 ? T / 128 : 4;
  // the float64 x pass keeps three outputs' multipliers and a transform live: held to 4 waves per
  // SIMD it spilled with masked stages, so 2 are asked for; without the masks it needs 108 VGPRs and
  // runs 4 (512^3: 1.20 ms at 2, 0.84 at 4).  The float32 Hessian x pass of workgroups
  // under 1024 threads (64^3, 256^3: 64 bytes a lane at 64 VGPRs, which made the 256^3 pass
  // fetch 5.6x its input) gets 6 waves per SIMD (80 VGPRs; three 512-thread workgroups a CU).
  static constexpr int XWPE = sizeof(V) == 16 ? 2 : (WPE == 8 && T < 1024 ? 6 : WPE);
  // float32 tiles of more than 8 values a thread (768^3) leave room for one workgroup per CU, whose
  // loads, transforms and stores nothing else overlaps: the y pass then holds a pair's input in
  // registers for both its transforms and loads the next one while the second runs (768^3: 4.36 ->
  // 4.05 ms; the x pass, bound by its strided writes, gained nothing from holding its input).
  // 1024 threads have no registers left for it (1024^3: 52 spilled).
  static constexpr bool HOLD = sizeof(V) == 8 && E::K0 * E::R0 > 8 && T < 1024;
  // small grids: the x pass's outputs and the y pass's pairs are workgroups of their own
  // (blockIdx.z) instead of one's turns, of which each waits for its loads and barriers (32^3
  // float32, 8 radii: x pass 10.9 -> 7.0 us, y pass 9.2 -> 6.6; at 64^3 the launches are full
  // without it: 183 us against 186 with it for 16 float64 radii)
  static constexpr bool SPLIT = N <= 48;
  static constexpr int GRID = N * NZT;
  static constexpr size_t HSLOT = (size_t)N * N * HZ;
};

// z pass: P lines per workgroup so that T = P * N/R0 threads (<= 64 kZWaves) and the LDS tile
// stays within 96 KB.
template <typename R, int N, int Q> struct ZTile {
  using V = typename Cplx<R>::type;
  static constexpr int R0 = factorize(N).r[0];
  static constexpr int M0 = N / R0;
  static constexpr int NPAD = N + N / 16 + 1;
  static constexpr int QL = kZSequential ? 1 : Q;   // transforms resident in LDS at once
  static constexpr int P_by_threads = pow2_floor((kZWaves * 64) / M0 > 0 ? (kZWaves * 64) / M0 : 1);
  static constexpr int P_by_lds = pow2_floor((96 * 1024) / (QL * NPAD * (int)sizeof(V)) > 0
                                                 ? (96 * 1024) / (QL * NPAD * (int)sizeof(V)) : 1);
  static constexpr int P0 = P_by_threads < P_by_lds ? P_by_threads : P_by_lds;
  static constexpr int P = P0 < 2 ? 2 : P0;   // even: the 2LPT epilogue pairs lines
  static constexpr int T = P * M0;
};

// The prepared half slot g0 (k_prep's output, read only by the Hessian x pass): tiled where W
// divides N/2, so that an x-pass workgroup (one y, W consecutive z, all x) reads one contiguous
// block of N W elements instead of W elements every 1 MB at 512^3 (x pass 0.494 -> 0.463 ms);
// rows (x, y, z) otherwise.
template <typename R, int N> struct PrepLayout {
  static constexpr int W = Tile<R>::PS;
  static constexpr int HZ = N / 2;
  static constexpr bool TILED = HZ % W == 0;
  __device__ static __forceinline__ size_t index(int x, int y, int z) {
    if constexpr (TILED) {
      return (((size_t)y * (HZ / W) + z / W) * N + x) * W + z % W;
    } else {
      return ((size_t)x * N + y) * HZ + z;
    }
  }
};

// Packed z lines, the y pass's output and the z pass's input: N lines of N complex per x-plane,
// element n of line (x, y) at `index(x, y, n)`.  Tiled where the widths allow: positions in
// groups of W (one y-pass tile row, 128 bytes), and for each x and group the N lines' W elements
// one after another.  A y-pass workgroup then writes whole contiguous blocks (N W elements per
// group) instead of W elements every line (y pass 1.02 -> 0.96 ms at 512^3), and a z-pass wave
// still reads W consecutive elements per group.  The z pass steps through its elements
// M0 = N/R0 positions apart, which must stay in the same column of a group.
template <typename R, int N> struct PackedLayout {
  static constexpr int W = Tile<R>::PS;
  static constexpr int M0 = N / factorize(N).r[0];
  static constexpr bool TILED = (N / 2) % W == 0 && M0 % W == 0;
  // elements between positions n and n + M0 of a line
  static constexpr size_t STEP = TILED ? (size_t)(M0 / W) * N * W : (size_t)M0;
  // affine in n (also for n outside [0, N), so that offsets can be formed from a base)
  __device__ static __forceinline__ long long index(int x, int y, int n) {
    if constexpr (TILED) {
      const int g = n >= 0 ? n / W : -((W - 1 - n) / W);
      return (((long long)x * (N / W) + g) * N + y) * W + (n - g * W);
    } else {
      return ((long long)x * N + y) * N + n;
    }
  }
};

__device__ __forceinline__ int ifreq(int i, int n) { return i < (n >> 1) ? i : i - n; }

template <typename R> __device__ __forceinline__ R powf_int(R f, int e) {
  return e == 0 ? R(1) : (e == 1 ? f : f * f);
}

// Streaming store: the line is not retained in the caches.  Used for every output that the next
// pass reads only after much other traffic: plain stores would leave dirty lines that evict the
// tiles a pass re-reads, or that the next pass has to write back while it runs.
template <typename V> __device__ __forceinline__ void st_stream(V* p, V v) {
  using R = decltype(v.x);
  typedef R R2 __attribute__((ext_vector_type(2)));
  R2 w;
  w.x = v.x;
  w.y = v.y;
  __builtin_nontemporal_store(w, reinterpret_cast<R2*>(p));
}

// Whether `count` half slots fit the last-level cache (256 MB), and how often.
template <typename R, int N> constexpr int slots_fit(int count) {
  return (int)(((size_t)256 << 20) / (count * (size_t)N * N * (N / 2) * 2 * sizeof(R)));
}

// Store into a slot between two passes: plain where the SLOTS half slots that matter to its next
// reader fit the last-level cache, streamed past the caches otherwise.  x-pass outputs count their
// own 3, the forward y pass's and the 2LPT source's 2, the prepared input itself and the x pass's
// outputs.  Measured: x-pass outputs plain at 256^3 float32 (3 fit, 9 do not), x pass 63 -> 59 us,
// y pass 139 -> 112, z pass 100 -> 121 (it waits for their write-back), collapse over 20 radii
// 5.98 -> 5.78 ms, with v_max 8.49 -> 8.01; at 512^3 streaming is the faster (y pass 1.04 -> 1.01).
template <typename R, int N, int SLOTS, typename V> __device__ __forceinline__ void st_slot(V* p, V v) {
  if constexpr (slots_fit<R, N>(SLOTS) > 0) *p = v; else st_stream(p, v);
}
// The packed y pass's outputs, counting a radius's 9 half slots (13 with v_max): plain only in
// float32 with two radii's worth in the cache.  y and z pass, streamed / plain: 128^3 float32 (three
// radii a launch) 34.1 + 50.9 / 36.4 + 46.9 us, 192^3 float32 (one radius's 9 just fit) 44.3 + 52.3 /
// 60.0 + 48.4, 96^3 float64 (four a launch) 47.0 + 95.1 / 57.2 + 89.0, 128^3 float64 25.6 + 43.0 /
// 28.7 + 40.0; 64^3 float64 in range calls of one radius each, 16 radii: 577 / 597 us.
template <typename R, int N, int SLOTS, typename V> __device__ __forceinline__ void st_yout(V* p, V v) {
  if constexpr (sizeof(R) == 4 && slots_fit<R, N>(SLOTS) > 1) *p = v; else st_stream(p, v);
}

// Streaming load, for the last read of a tile (its lines need not stay in L2).
template <typename V> __device__ __forceinline__ V ld_stream(const V* p) {
  using R = decltype(p->x);
  typedef R R2 __attribute__((ext_vector_type(2)));
  const R2 w = __builtin_nontemporal_load(reinterpret_cast<const R2*>(p));
  return V{w.x, w.y};
}

template <int N, int T, typename V>
__device__ __forceinline__ void load_twiddles(V* __restrict__ s_tw, const V* __restrict__ tw, int t) {
  load_stage_twiddles<N, T>(s_tw, tw, t);
}

// ---------------------------------------------------------------------------------------------
// Radius-independent part of the Hessian multiplier, once per call: g0 = M dk scale / f^2 into
// a half slot in the x pass's tile order (PrepLayout; the user spectrum's rows of N/2+1 complex
// are neither aligned nor in that order), so the per-radius x pass reads contiguous blocks.
template <typename R, int N>
__global__ void k_prep(const typename Cplx<R>::type* __restrict__ dk, typename Cplx<R>::type* __restrict__ g0,
                       R scale) {
  using V = typename Cplx<R>::type;
  constexpr int HZ = N / 2, NH = N / 2 + 1;
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (size_t)N * N * HZ) return;
  const int z = (int)(i % HZ);
  const int y = (int)((i / HZ) % N);
  const int x = (int)(i / ((size_t)HZ * N));
  V out = V{R(0), R(0)};
  if (x != N / 2 && y != N / 2) {
    const int fx = ifreq(x, N), fy = ifreq(y, N);
    const R f2 = R(fx * fx + fy * fy + z * z);
    if (f2 > R(0)) {
      const V d = dk[((size_t)x * N + y) * NH + z];
      const R m = scale / f2;
      out = V{d.x * m, d.y * m};
    }
  }
  st_slot<R, N, 4>(&g0[PrepLayout<R, N>::index(x, y, z)], out);
}

// ---------------------------------------------------------------------------------------------
// x pass.  MODE 0 (Hessian): input g0 (k_prep's tiled half slot), 3 outputs, multiplier
// W(x)W(y)W(z) from the window row wtab (never null; a row of ones for no smoothing).  MODE 1
// (gradient): input the user half spectrum, 2 outputs, multiplier i * scale / f^2 (wtab
// unused).  Outputs: half slots.  blockIdx.y is the radius within a batch (MODE 0): its window row
// follows the first one's, its three outputs the previous radius's.  Loads are unconditional (lanes without an element read an
// in-bounds address and discard it): a load under a per-lane branch would make the compiler
// wait for each one before issuing the next.
template <typename R, int N, int MODE>
__global__ void __launch_bounds__((Strided<R, N, +1>::T))
__attribute__((amdgpu_waves_per_eu(Strided<R, N, +1>::XWPE)))
k_xpass(const typename Cplx<R>::type* __restrict__ in, typename Cplx<R>::type* __restrict__ out,
        const R* __restrict__ wtab, const typename Cplx<R>::type* __restrict__ tw, R scale) {
  using S = Strided<R, N, +1>;
  using V = typename S::V;
  using E = typename S::E;
  constexpr int PS = S::PS, HZ = S::HZ, NH = N / 2 + 1, NA = MODE == 0 ? 3 : 2, M = N / E::R0;
  __shared__ V lds[E::LDS_ELEMS];
  __shared__ V s_tw[tw_elems(N)];
  const int t = threadIdx.x;
  if constexpr (MODE == 0) {
    wtab += (size_t)blockIdx.y * N;
    out += (size_t)blockIdx.y * 3 * S::HSLOT;
  }
  load_twiddles<N, S::T>(s_tw, tw, t);
  const int bt = xcd_tile(blockIdx.x, S::GRID);
  const int zt = bt % S::NZT;
  const int y = bt / S::NZT;
  const int fy = ifreq(y, N);
  const int a0 = S::SPLIT ? blockIdx.z : 0, a1 = S::SPLIT ? a0 + 1 : NA;   // this workgroup's outputs
  if constexpr (MODE == 0 && E::K0 == 1) {
    // Hessian, one butterfly per thread: same values as the general form below, in a form whose
    // schedule (data loads batched, the window loads kept out of that batch) measured 13% faster
    // at 512^3.  wtab is never null here; the test only shapes that schedule.
    int q, p, j;
    bool ok;
    E::first_layout(t, 0, q, p, j, ok);
    const int z = zt * PS + p;
    ok = ok && z < HZ;
    const R wyz = ok ? wtab[y] * wtab[z] : R(1);
#pragma unroll 1
    for (int a = a0; a < a1; ++a) {
      V u[1][E::R0];
#pragma unroll
      for (int s = 0; s < E::R0; ++s) {
        const int n = j + s * M;
        V val = V{R(0), R(0)};
        if (ok) {
          val = in[PrepLayout<R, N>::index(n, y, z)];
          if (wtab != nullptr) val = cscale(val, wtab[n] * wyz);
        }
        u[0][s] = cscale(val, powf_int(R(ifreq(n, N)), a));
      }
      E::run(u, lds, s_tw, t);
      // streamed past the caches on large grids (st_slot): left there, their dirty lines would be
      // written back while the y pass runs
      if (ok) {
#pragma unroll
        for (int s = 0; s < E::R0; ++s) st_slot<R, N, 3>(out + a * S::HSLOT + ((size_t)(j + s * M) * N + y) * HZ + z, u[0][s]);
      }
    }
    return;
  }
  int zz[E::K0], jj[E::K0];
  bool ok[E::K0];
  R wyz[E::K0];
#pragma unroll
  for (int k = 0; k < E::K0; ++k) {
    int q, p, j;
    E::first_layout(t, k, q, p, j, ok[k]);
    const int z = zt * PS + p;
    ok[k] = ok[k] && z < HZ;
    zz[k] = ok[k] ? z : 0;   // lanes without an element read (and never write) z = 0
    jj[k] = j;
    if constexpr (MODE == 0) wyz[k] = wtab[y] * wtab[zz[k]];
  }
  // One output at a time: the input tile is read again for each output (an L2 hit after the
  // first), so that only one transform's data is live and two workgroups fit on a CU.
#pragma unroll 1
  for (int a = a0; a < a1; ++a) {
    V u[E::K0][E::R0];
#pragma unroll
    for (int k = 0; k < E::K0; ++k) {
      // opaque copies: addresses and multipliers are computed per output, not hoisted
      int jv = jj[k], z = zz[k];
      asm volatile("" : "+v"(jv), "+v"(z));
#pragma unroll
      for (int s = 0; s < E::R0; ++s) {
        const int n = jv + s * M;
        const R fa = powf_int(R(ifreq(n, N)), a);
        V val;
        if constexpr (MODE == 0) {
          // no mask: a lane without an element never writes its values (to LDS or out)
          val = cscale(in[PrepLayout<R, N>::index(n, y, z)], wtab[n] * wyz[k] * fa);
        } else {
          const V d = in[((size_t)n * N + y) * NH + z];
          const int fx = ifreq(n, N);
          const int f2 = fx * fx + fy * fy + z * z;
          const bool keep = ok[k] && n != N / 2 && y != N / 2 && f2 > 0;
          const R m = keep ? scale / R(f2) * fa : R(0);
          val = V{-d.y * m, d.x * m};
        }
        u[k][s] = val;
      }
    }
    E::run(u, lds, s_tw, t);
#pragma unroll
    for (int k = 0; k < E::K0; ++k)
      if (ok[k]) {
#pragma unroll
        for (int s = 0; s < E::R0; ++s)
          st_slot<R, N, 3>(out + a * S::HSLOT + ((size_t)(jj[k] + s * M) * N + y) * HZ + zz[k], u[k][s]);
      }
  }
}

// ---------------------------------------------------------------------------------------------
// Fused forward-x / inverse-x pass of a second-order source: reads the (z-forward, y-forward)
// transformed source from a half slot and completes the forward transform along x.  Gradient
// form (HESS false, the 2LPT displacement): multiplies by i * scale * M / f^2 and runs the two
// inverse x transforms of fx^a (a = 0, 1).  Hessian form (HESS true, the second-order tensor of
// the third-order displacement): multiplies by scale * M / f^2 and runs the three inverse x
// transforms of fx^a (a = 0, 1, 2), the outputs of the Hessian x pass.  Outputs: half slots.
template <typename R, int N, bool HESS>
__global__ void __launch_bounds__((Strided<R, N, +1>::T))
k_xpass_fwdinv(const typename Cplx<R>::type* __restrict__ in, typename Cplx<R>::type* __restrict__ out,
               const typename Cplx<R>::type* __restrict__ tw, R scale) {
  using S = Strided<R, N, +1>;
  using V = typename S::V;
  using E = typename S::E;
  using EF = Engine<V, N, S::PS, 1, true, S::T, -1>;
  constexpr int PS = S::PS, HZ = S::HZ, M = N / E::R0;
  __shared__ V lds[E::LDS_ELEMS];
  __shared__ V s_tw[tw_elems(N)];
  const int t = threadIdx.x;
  load_twiddles<N, S::T>(s_tw, tw, t);
  const int bt = xcd_tile(blockIdx.x, S::GRID);
  const int zt = bt % S::NZT;
  const int y = bt / S::NZT;
  const int fy = ifreq(y, N);
  V v[E::K0][E::R0];
  int zz[E::K0], jj[E::K0];
  bool ok[E::K0];
#pragma unroll
  for (int k = 0; k < E::K0; ++k) {
    int q, p, j;
    E::first_layout(t, k, q, p, j, ok[k]);
    const int z = zt * PS + p;
    ok[k] = ok[k] && z < HZ;
    zz[k] = z;
    jj[k] = j;
#pragma unroll
    for (int s = 0; s < E::R0; ++s)
      v[k][s] = ok[k] ? in[((size_t)(j + s * M) * N + y) * HZ + z] : V{R(0), R(0)};
  }
  EF::run(v, lds, s_tw, t);
#pragma unroll
  for (int k = 0; k < E::K0; ++k)
#pragma unroll
    for (int s = 0; s < E::R0; ++s) {
      const int n = jj[k] + s * M;
      const int fx = ifreq(n, N);
      const R f2 = R(fx * fx + fy * fy + zz[k] * zz[k]);
      const bool keep = ok[k] && n != N / 2 && y != N / 2 && f2 > R(0);
      const R m = keep ? scale / f2 : R(0);
      const V d = v[k][s];
      v[k][s] = HESS ? V{d.x * m, d.y * m} : V{-d.y * m, d.x * m};
    }
#pragma unroll 1
  for (int a = 0; a < (HESS ? 3 : 2); ++a) {
    V u[E::K0][E::R0];
#pragma unroll
    for (int k = 0; k < E::K0; ++k)
#pragma unroll
      for (int s = 0; s < E::R0; ++s) u[k][s] = cscale(v[k][s], powf_int(R(ifreq(jj[k] + s * M, N)), a));
    E::run(u, lds, s_tw, t);
#pragma unroll
    for (int k = 0; k < E::K0; ++k)
      if (ok[k]) {
#pragma unroll
        for (int s = 0; s < E::R0; ++s)
          st_slot<R, N, 3>(out + a * S::HSLOT + ((size_t)(jj[k] + s * M) * N + y) * HZ + zz[k], u[k][s]);
      }
  }
}

// ---------------------------------------------------------------------------------------------
// Fused forward-x / inverse-x pass of the third-order displacement: four half slots in, the
// (z-forward, y-forward) transforms of the divergence source s and of the transverse source
// c = (cx, cy, cz); forward transforms along x; per mode
//     psi_a = i scale M / f^2 (-f_a S + f_b C_d - f_d C_b),   (a, b, d) cyclic,
// and the three inverse x transforms of psi_a into half slots (the y and z passes finish them).
template <typename R, int N>
__global__ void __launch_bounds__((Strided<R, N, +1>::T))
k_xpass_lpt3(const typename Cplx<R>::type* __restrict__ in, typename Cplx<R>::type* __restrict__ out,
             const typename Cplx<R>::type* __restrict__ tw, R scale) {
  using S = Strided<R, N, +1>;
  using V = typename S::V;
  using E = typename S::E;
  using EF = Engine<V, N, S::PS, 1, true, S::T, -1>;
  constexpr int PS = S::PS, HZ = S::HZ, M = N / E::R0;
  __shared__ V lds[E::LDS_ELEMS];
  __shared__ V s_tw[tw_elems(N)];
  const int t = threadIdx.x;
  load_twiddles<N, S::T>(s_tw, tw, t);
  const int bt = xcd_tile(blockIdx.x, S::GRID);
  const int zt = bt % S::NZT;
  const int y = bt / S::NZT;
  const R fy = R(ifreq(y, N));
  V v[4][E::K0][E::R0];
  int zz[E::K0], jj[E::K0];
  bool ok[E::K0];
#pragma unroll
  for (int k = 0; k < E::K0; ++k) {
    int q, p, j;
    E::first_layout(t, k, q, p, j, ok[k]);
    const int z = zt * PS + p;
    ok[k] = ok[k] && z < HZ;
    zz[k] = z;
    jj[k] = j;
  }
  // each source is loaded just before its forward transform (all four in flight at once would
  // exceed the register budget of a 1024-thread workgroup)
#pragma unroll
  for (int c = 0; c < 4; ++c) {
#pragma unroll
    for (int k = 0; k < E::K0; ++k)
#pragma unroll
      for (int s = 0; s < E::R0; ++s)
        v[c][k][s] = ok[k] ? in[c * S::HSLOT + ((size_t)(jj[k] + s * M) * N + y) * HZ + zz[k]] : V{R(0), R(0)};
    EF::run(v[c], lds, s_tw, t);
  }
  // psi3 components in place of (S, cx, cy), element by element
#pragma unroll
  for (int k = 0; k < E::K0; ++k)
#pragma unroll
    for (int s = 0; s < E::R0; ++s) {
      const int n = jj[k] + s * M;
      const R fx = R(ifreq(n, N)), fz = R(zz[k]);
      const R f2 = fx * fx + fy * fy + fz * fz;
      const bool keep = ok[k] && n != N / 2 && y != N / 2 && f2 > R(0);
      const R m = keep ? scale / f2 : R(0);
      const V sk = v[0][k][s], cx = v[1][k][s], cy = v[2][k][s], cz = v[3][k][s];
      // i m (-f_a S + f_b c_d - f_d c_b): w = the bracket, then times i m
      const V wx = V{fy * cz.x - fz * cy.x - fx * sk.x, fy * cz.y - fz * cy.y - fx * sk.y};
      const V wy = V{fz * cx.x - fx * cz.x - fy * sk.x, fz * cx.y - fx * cz.y - fy * sk.y};
      const V wz = V{fx * cy.x - fy * cx.x - fz * sk.x, fx * cy.y - fy * cx.y - fz * sk.y};
      v[0][k][s] = V{-wx.y * m, wx.x * m};
      v[1][k][s] = V{-wy.y * m, wy.x * m};
      v[2][k][s] = V{-wz.y * m, wz.x * m};
    }
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    E::run(v[a], lds, s_tw, t);
#pragma unroll
    for (int k = 0; k < E::K0; ++k)
      if (ok[k]) {
#pragma unroll
        for (int s = 0; s < E::R0; ++s)
          st_slot<R, N, 3>(out + a * S::HSLOT + ((size_t)(jj[k] + s * M) * N + y) * HZ + zz[k], v[a][k][s]);
      }
  }
}

// ---------------------------------------------------------------------------------------------
// y pass, packed output.  Packed component c of the recipe is (a, b, cz): input half slot a,
// fy^b before the transform, fz^cz after it; components (2q, 2q+1) go to packed slot q as
// C = A + iB.  The Hessian pairs are ordered so that each pair reads as few inputs as possible
// (pair 0 reads X_1 only, pair 1 X_0 only), which lets X_2 be fetched while pair 1 runs:
//   Hessian (RECIPE 0), packed order xy xz | yy yz | xx zz:
//       (1,1,0) (1,0,1) | (0,2,0) (0,1,1) | (2,0,0) (0,0,2)
//   gradient (RECIPE 1), packed order x y | z:  (1,0,0) (0,1,0) | (0,0,1)
//   three finished components (RECIPE 4, the third-order displacement), packed order x y | z:
//       (0,0,0) (1,0,0) | (2,0,0)
//   Hessian and v_max gradient in one pass (RECIPE 5): RECIPE 0's pairs, then RECIPE 1's components
//       times i, which the gradient x pass applies itself but the Hessian x pass does not (TI), into a
//       second output (pairs from SPLIT on), so the Hessian x-pass outputs are read once
// The z pass maps the packed order back to (xx, xy, xz, yy, yz, zz) and (x, y, z).
// STREAM: the last transform that reads an input tile streams it (its lines need not stay in L2).
template <int RECIPE> struct YRecipe;
template <> struct YRecipe<0> {
  static constexpr bool STREAM = true;
  static constexpr int NIN = 3, NC = 6, Q = 3, SPLIT = 0;
  static constexpr int A[6] = {1, 1, 0, 0, 2, 0}, B[6] = {1, 0, 2, 1, 0, 0}, C[6] = {0, 1, 0, 1, 0, 2};
  static constexpr bool ti(int) { return false; }
};
template <> struct YRecipe<1> {
  static constexpr bool STREAM = false;
  static constexpr int NIN = 2, NC = 3, Q = 2, SPLIT = 0;
  static constexpr int A[3] = {1, 0, 0}, B[3] = {0, 1, 0}, C[3] = {0, 0, 1};
  static constexpr bool ti(int) { return false; }
};
template <> struct YRecipe<4> {
  static constexpr bool STREAM = true;
  static constexpr int NIN = 3, NC = 3, Q = 2, SPLIT = 0;
  static constexpr int A[3] = {0, 1, 2}, B[3] = {0, 0, 0}, C[3] = {0, 0, 0};
  static constexpr bool ti(int) { return false; }
};
template <> struct YRecipe<5> {
  static constexpr bool STREAM = true;
  static constexpr int NIN = 3, NC = 9, Q = 5, SPLIT = 3;
  static constexpr int A[9] = {1, 1, 0, 0, 2, 0, 1, 0, 0}, B[9] = {1, 0, 2, 1, 0, 0, 0, 1, 0},
                       C[9] = {0, 1, 0, 1, 0, 2, 0, 0, 1};
  static constexpr bool ti(int c) { return c >= 6; }
};

// Pair of the last transform that reads input slot `a` under recipe RC.
template <class RC> constexpr int last_pair(int a) {
  int q = -1;
  for (int c = 0; c < RC::NC; ++c)
    if (RC::A[c] == a) q = c / 2;
  return q;
}

template <typename R, int N, int RECIPE>
__global__ void __launch_bounds__((Strided<R, N, +1>::T))
__attribute__((amdgpu_waves_per_eu(Strided<R, N, +1>::WPE)))
k_ypass_packed(const typename Cplx<R>::type* __restrict__ in, typename Cplx<R>::type* __restrict__ out,
               const typename Cplx<R>::type* __restrict__ tw, typename Cplx<R>::type* __restrict__ out2) {
  using S = Strided<R, N, +1>;
  using RC = YRecipe<RECIPE>;
  using V = typename S::V;
  using E = typename S::E;
  constexpr int PS = S::PS, HZ = S::HZ, M = N / E::R0;
  constexpr size_t PSLOT = (size_t)N * N * N;
  constexpr int SLOTS = RC::SPLIT > 0 ? 13 : 9;
  __shared__ V lds[E::LDS_ELEMS];
  __shared__ V s_tw[tw_elems(N)];
  const int t = threadIdx.x;
  // blockIdx.y: the radius within a batch, its slots behind the previous radius's
  in += (size_t)blockIdx.y * RC::NIN * S::HSLOT;
  out += (size_t)blockIdx.y * (RC::SPLIT > 0 ? RC::SPLIT : RC::Q) * PSLOT;
  if constexpr (RC::SPLIT > 0) out2 += (size_t)blockIdx.y * (RC::Q - RC::SPLIT) * PSLOT;
  load_twiddles<N, S::T>(s_tw, tw, t);
  const int bt = xcd_tile(blockIdx.x, S::GRID);
  const int zt = bt % S::NZT;
  const int x = bt / S::NZT;
  int zz[E::K0], jj[E::K0];
  bool ok[E::K0];
#pragma unroll
  for (int k = 0; k < E::K0; ++k) {
    int q, p, j;
    E::first_layout(t, k, q, p, j, ok[k]);
    const int z = zt * PS + p;
    ok[k] = ok[k] && z < HZ;
    zz[k] = z;
    jj[k] = j;
  }
  // HOLD: the pair's first input stays in registers for both signs, and the next pair's is loaded
  // while the pair's last transform runs
  constexpr bool HOLD = S::HOLD;
  V held[HOLD ? E::K0 : 1][HOLD ? E::R0 : 1];
  auto hold = [&](int q) {
    if constexpr (HOLD) {
#pragma unroll
      for (int k = 0; k < E::K0; ++k) {
        unsigned off = (unsigned)(jj[k] * HZ + (ok[k] ? zz[k] : 0));
        asm volatile("" : "+v"(off));
#pragma unroll
        for (int s = 0; s < E::R0; ++s) {
          const V* p = in + RC::A[2 * q] * S::HSLOT + ((size_t)x * N + s * M) * HZ + off;
          held[k][s] = RC::STREAM && q == last_pair<RC>(RC::A[2 * q]) ? ld_stream(p) : *p;
        }
      }
    }
  };
  hold(0);
  // One transform per (pair, sign): u = fy^bA fz^cA X_aA + sgn i fy^bB fz^cB X_aB.  By
  // linearity sgn = +1 gives C[kz] = A + iB and sgn = -1 gives conj(C[N - kz]) = A - iB.  Each
  // transform reads its inputs itself (L2 hits after the first read of a tile) so that only one
  // transform's data is live and two workgroups fit on a CU; outputs as st_yout says.
#pragma unroll
  for (int q = 0; q < RC::Q; ++q) {
    if (S::SPLIT && q != (int)blockIdx.z) continue;
    const int ca = 2 * q, cb = 2 * q + 1;
    const bool has_b = cb < RC::NC;
    const int aa = RC::A[ca];
    const int ab = RC::A[has_b ? cb : ca];
    V* dst = (RC::SPLIT > 0 && q >= RC::SPLIT) ? out2 + (size_t)(q - RC::SPLIT) * PSLOT : out + (size_t)q * PSLOT;
#pragma unroll
    for (int sgn = 1; sgn >= -1; sgn -= 2) {
      if (!has_b && sgn < 0) break;   // B = 0: C[N - kz] = conj(C[kz]), formed by the z pass
      // opaque copies of the indices: the compiler would otherwise compute every transform's
      // multipliers and addresses up front and keep them live across all of them
      int jv[E::K0], zv[E::K0];
#pragma unroll
      for (int k = 0; k < E::K0; ++k) {
        jv[k] = jj[k];
        zv[k] = zz[k];
        asm volatile("" : "+v"(jv[k]), "+v"(zv[k])::"memory");
      }
      V u[E::K0][E::R0];
#pragma unroll
      for (int k = 0; k < E::K0; ++k) {
        const R fz = R(zv[k]);
#pragma unroll
        for (int s = 0; s < E::R0; ++s) {
          const R fy = R(ifreq(jv[k] + s * M, N));
          const size_t ubase = ((size_t)x * N + s * M) * HZ;   // uniform part of the address
          const unsigned off = (unsigned)(jv[k] * HZ + zv[k]);
          // the last transform that reads a tile streams it (Hessian: X_1 after pair 0, X_0 and
          // X_2 after pair 2)
          const bool final_sgn = sgn < 0 || !has_b;
          const bool last_a = RC::STREAM && final_sgn && q == last_pair<RC>(aa);
          const bool last_b = RC::STREAM && final_sgn && q == last_pair<RC>(ab);
          const V* pa = in + aa * S::HSLOT + ubase + off;
          V xa;
          if constexpr (HOLD)
            xa = held[k][s];
          else
            xa = ok[k] ? (last_a ? ld_stream(pa) : *pa) : V{R(0), R(0)};
          V ta = cscale(xa, powf_int(fy, RC::B[ca]) * powf_int(fz, RC::C[ca]));
          if (RC::ti(ca)) ta = V{-ta.y, ta.x};
          if (has_b) {
            const V* pb = in + ab * S::HSLOT + ubase + off;
            const V xb = ab == aa ? xa : (ok[k] ? (last_b ? ld_stream(pb) : *pb) : V{R(0), R(0)});
            V tb = cscale(xb, powf_int(fy, RC::B[has_b ? cb : ca]) * powf_int(fz, RC::C[has_b ? cb : ca]));
            if (RC::ti(cb)) tb = V{-tb.y, tb.x};
            u[k][s] = sgn > 0 ? V{ta.x - tb.y, ta.y + tb.x} : V{ta.x + tb.y, ta.y - tb.x};
          } else {
            u[k][s] = ta;
          }
        }
      }
      if (HOLD && q + 1 < RC::Q && (sgn < 0 || !has_b)) hold(q + 1);
      E::run(u, lds, s_tw, t);
#pragma unroll
      for (int k = 0; k < E::K0; ++k)
        if (ok[k]) {
#pragma unroll
          for (int s = 0; s < E::R0; ++s) {
            // x-plane base (uniform) + 32-bit byte offsets within the plane
            using L = PackedLayout<R, N>;
            char* plane = reinterpret_cast<char*>(dst + (size_t)x * N * N);
            V* first = reinterpret_cast<V*>(plane + (unsigned)L::index(0, jv[k] + s * M, zv[k]) * (unsigned)sizeof(V));
            V* second =
                reinterpret_cast<V*>(plane + (unsigned)L::index(0, jv[k] + s * M, zv[k] + HZ) * (unsigned)sizeof(V));
            if (sgn > 0) {
              st_yout<R, N, SLOTS>(first, u[k][s]);
              // the conjugate that a slot of one component leaves to the z pass stays an operand:
              // without it the last butterfly's products would be contracted into its sums where
              // they were not, and the gradient would round differently
              if (!has_b && zv[k] > 0) {
                const V w = conj(u[k][s]);
                asm volatile("" ::"v"(w.x), "v"(w.y));
              }
            } else if (zv[k] > 0) {
              st_yout<R, N, SLOTS>(second, conj(u[k][s]));
            }
          }
        }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Forward y pass of the 2LPT source: half slot -> half slot, no multiplier.
template <typename R, int N>
__global__ void __launch_bounds__((Strided<R, N, -1>::T))
k_ypass_fwd(const typename Cplx<R>::type* __restrict__ in, typename Cplx<R>::type* __restrict__ out,
            const typename Cplx<R>::type* __restrict__ tw) {
  using S = Strided<R, N, -1>;
  using V = typename S::V;
  using E = typename S::E;
  constexpr int PS = S::PS, HZ = S::HZ, M = N / E::R0;
  __shared__ V lds[E::LDS_ELEMS];
  __shared__ V s_tw[tw_elems(N)];
  const int t = threadIdx.x;
  load_twiddles<N, S::T>(s_tw, tw, t);
  const int bt = xcd_tile(blockIdx.x, S::GRID);
  const int zt = bt % S::NZT;
  const int x = bt / S::NZT;
  V v[E::K0][E::R0];
  int zz[E::K0], jj[E::K0];
  bool ok[E::K0];
#pragma unroll
  for (int k = 0; k < E::K0; ++k) {
    int q, p, j;
    E::first_layout(t, k, q, p, j, ok[k]);
    const int z = zt * PS + p;
    ok[k] = ok[k] && z < HZ;
    zz[k] = z;
    jj[k] = j;
#pragma unroll
    for (int s = 0; s < E::R0; ++s)
      v[k][s] = ok[k] ? in[((size_t)x * N + j + s * M) * HZ + z] : V{R(0), R(0)};
  }
  E::run(v, lds, s_tw, t);
#pragma unroll
  for (int k = 0; k < E::K0; ++k)
    if (ok[k]) {
#pragma unroll
      for (int s = 0; s < E::R0; ++s) st_slot<R, N, 2>(out + ((size_t)x * N + jj[k] + s * M) * HZ + zz[k], v[k][s]);
    }
}

// ---------------------------------------------------------------------------------------------
// z pass: inverse transform along z of Q packed slots (two real components each) and the
// per-point epilogue.
enum ZEpi { EPI_STORE = 1, EPI_MU2 = 2, EPI_LPT3 = 4 };

template <typename R, int N, int Q, int EPI>
struct ZPass {
  using V = typename Cplx<R>::type;
  using ZT = ZTile<R, N, Q>;
  static constexpr int P = ZT::P;
  static constexpr int T = ZT::T;
  static constexpr int HZ = N / 2;
  using E = Engine<V, N, P, ZT::QL, false, T, +1>;
  static constexpr int LINES = N * N;
  static constexpr int GRID = (LINES + P - 1) / P;
  static_assert(E::K0 == ZT::QL, "z pass: one butterfly per transform per thread");
};

// One thread's elements of packed z lines: n = j + s N/R0, s < R0, of line `line`.
//
// Packed storage of C[n]: P[n] for n < N/2, P[3N/2 - n] for n > N/2; R0 is even, so elements
// s < R0/2 are the first kind and s >= R0/2 the second.  Loads are unconditional (the caller
// passes a line in range); the Nyquist element n = N/2 (lane j = 0, s = R0/2) reads P[N/2], which
// is never written, and is replaced by zero.  Offsets of element j + s M0, of the Nyquist slot and
// of element 3N/2 - j - s M0 = (3N/2 - j) - s M0 are the same for every slot.  A workgroup's lines
// share one x-plane when P divides N: the plane's base is then uniform and the offsets within it
// (bytes) fit 32 bits, so each load adds one 32-bit offset to a scalar base.
template <typename R, int N, int P> struct ZLoader {
  using V = typename Cplx<R>::type;
  using L = PackedLayout<R, N>;
  static constexpr int R0 = factorize(N).r[0];
  static constexpr int M0 = N / R0, HZ = N / 2;
  static constexpr bool PLANE = N % P == 0;
  static constexpr unsigned STEPB = (unsigned)(L::STEP * sizeof(V));
  static_assert(R0 % 2 == 0 && M0 * (R0 / 2) == HZ, "z pass: the first half of the elements is n < N/2");
  static_assert((size_t)3 * N * N * sizeof(V) < ((size_t)1 << 32), "z pass: plane offsets must fit 32 bits");
  size_t plane;
  unsigned o_lo, o_ny, o_hi, o_rev;
  bool ny;

  __device__ __forceinline__ ZLoader(int line, int j) {
    const int ly = line % N;
    const int lx = PLANE ? (int)(blockIdx.x * P / N) : line / N;
    plane = (size_t)lx * N * N;
    o_lo = (unsigned)L::index(0, ly, j) * (unsigned)sizeof(V);
    o_ny = (unsigned)L::index(0, ly, j == 0 ? HZ : N - j) * (unsigned)sizeof(V);
    o_hi = (unsigned)L::index(0, ly, 3 * HZ - j) * (unsigned)sizeof(V);
    o_rev = (unsigned)L::index(0, ly, M0 - j) * (unsigned)sizeof(V);
    ny = j == 0;
  }
  // A slot of one real component: C[N - k] = conj(C[k]), so only the first half is there, and the
  // second, n = N - ((R0 - s) M0 - j), is the first read backwards from the same cache lines.
  __device__ __forceinline__ void load_one(const V* slot, V (&dst)[R0]) const {
    const char* base = reinterpret_cast<const char*>(slot + plane);
#pragma unroll
    for (int s = 0; s < R0 / 2; ++s) dst[s] = *reinterpret_cast<const V*>(base + (o_lo + s * STEPB));
#pragma unroll
    for (int s = R0 / 2; s < R0; ++s) {
      const V x = *reinterpret_cast<const V*>(base + (o_rev + (R0 - 1 - s) * STEPB));
      // opaque: the transform then takes the sign as it takes any loaded value, and contracts and
      // rounds as it does for a slot of two components
      R y = -x.y;
      asm("" : "+v"(y));
      dst[s] = s == R0 / 2 && ny ? V{R(0), R(0)} : V{x.x, y};
    }
  }
  __device__ __forceinline__ void load(const V* slot, V (&dst)[R0]) const {
    const char* base = reinterpret_cast<const char*>(slot + plane);
#pragma unroll
    for (int s = 0; s < R0 / 2; ++s) dst[s] = *reinterpret_cast<const V*>(base + (o_lo + s * STEPB));
    {
      const V x = *reinterpret_cast<const V*>(base + o_ny);
      dst[R0 / 2] = ny ? V{R(0), R(0)} : x;
    }
#pragma unroll
    for (int s = R0 / 2 + 1; s < R0; ++s) dst[s] = *reinterpret_cast<const V*>(base + (o_hi - s * STEPB));
  }
};

struct ZArgs {
  int nc;           // EPI_STORE: number of real components to store (<= 2Q)
  void* out;        // EPI_STORE: [nc][N^3] real; EPI_MU2: one half slot (complex)
  void* t6;         // EPI_MU2: when not null, the six components are stored to t6[6][N^3] (R);
                    // EPI_LPT3: the first-order tensor T1 [6][N^3] read at each point
};

// Sources of the third-order displacement at one point from the first-order tensor a and the
// second-order tensor b (xx, xy, xz, yy, yz, zz): the divergence
//     sl = det(a) / 3 - (10/21) ((tr a)(tr b) - tr(a b)) / 2
// and the curl c_i = eps_ijk (a b)_jk / 7.
template <typename R>
__device__ __forceinline__ void lpt3_sources(const R (&a)[6], const R (&b)[6], R& sl, R& cx, R& cy, R& cz) {
  const R axx = a[0], axy = a[1], axz = a[2], ayy = a[3], ayz = a[4], azz = a[5];
  const R bxx = b[0], bxy = b[1], bxz = b[2], byy = b[3], byz = b[4], bzz = b[5];
  const R det = axx * (ayy * azz - ayz * ayz) - axy * (axy * azz - ayz * axz) + axz * (axy * ayz - ayy * axz);
  const R trab = axx * bxx + ayy * byy + azz * bzz + R(2) * (axy * bxy + axz * bxz + ayz * byz);
  const R mixed = R(0.5) * ((axx + ayy + azz) * (bxx + byy + bzz) - trab);
  sl = det * R(1.0 / 3.0) - mixed * R(10.0 / 21.0);
  cx = (axy * bxz + ayy * byz + ayz * bzz - axz * bxy - ayz * byy - azz * byz) * R(1.0 / 7.0);
  cy = (axz * bxx + ayz * bxy + azz * bxz - axx * bxz - axy * byz - axz * bzz) * R(1.0 / 7.0);
  cz = (axx * bxy + axy * byy + axz * byz - axy * bxx - ayy * bxy - ayz * bxz) * R(1.0 / 7.0);
}

template <typename R, int N, int Q, int EPI>
__global__ void __launch_bounds__((ZPass<R, N, Q, EPI>::T))
k_zpass(const typename Cplx<R>::type* __restrict__ in, const typename Cplx<R>::type* __restrict__ tw, ZArgs args) {
  using Z = ZPass<R, N, Q, EPI>;
  using V = typename Z::V;
  using E = typename Z::E;
  constexpr int P = Z::P, HZ = Z::HZ, R0 = E::R0, M0 = N / R0;
  constexpr size_t PSLOT = (size_t)N * N * N;
  __shared__ V lds[E::LDS_ELEMS];
  __shared__ V s_tw[tw_elems(N)];
  const int t = threadIdx.x;
  load_twiddles<N, Z::T>(s_tw, tw, t);
  // thread t owns pencil position (p, j) of every transform q
  const int j = t % M0;
  const int p = t / M0;
  const int line = blockIdx.x * P + p;
  const bool line_ok = Z::LINES % P == 0 || line < Z::LINES;
  V v[Q][R0];
  const int lineL = line_ok ? line : Z::LINES - 1;
  const ZLoader<R, N, P> ld(lineL, j);
#pragma unroll
  for (int q = 0; q < Q; ++q)
    if (Q == 2 && q == 1)
      ld.load_one(in + (size_t)q * PSLOT, v[q]);   // x y | z
    else
      ld.load(in + (size_t)q * PSLOT, v[q]);
  if constexpr (Z::ZT::QL == Q) {
    E::run(v, lds, s_tw, t);
  } else {
#pragma unroll
    for (int q = 0; q < Q; ++q) E::run(*reinterpret_cast<V(*)[1][R0]>(&v[q]), lds, s_tw, t);
  }
  // v[q][s] = (packed component 2q) + i (packed component 2q+1) at n = j + s*M0 of line `line`;
  // comp(c, s) is the canonical component c (Hessian xx xy xz yy yz zz; gradient x y z).
  auto comp = [&](int c, int s) -> R {
    if constexpr (Q == 3) {
      return c == 0 ? v[2][s].x : c == 1 ? v[0][s].x : c == 2 ? v[0][s].y : c == 3 ? v[1][s].x
                                                                 : c == 4 ? v[1][s].y : v[2][s].y;
    } else {
      return c == 0 ? v[0][s].x : c == 1 ? v[0][s].y : v[1][s].x;
    }
  };
  if constexpr (EPI == EPI_STORE) {
    R* out = static_cast<R*>(args.out);
    constexpr size_t VOL = (size_t)N * N * N;
    if (line_ok) {
#pragma unroll
      for (int s = 0; s < R0; ++s) {
        const size_t idx = (size_t)line * N + j + s * M0;
#pragma unroll
        for (int c = 0; c < 2 * Q; ++c)
          if (c < args.nc) __builtin_nontemporal_store(comp(c, s), &out[(size_t)c * VOL + idx]);
      }
    }
  } else if constexpr (EPI == EPI_LPT3) {
    static_assert(Q == 3, "third-order sources need the six components of T2");
    // sources of the third-order displacement at each point from T2 (this pass) and T1 (read),
    // packed (sl + i cx), (cy + i cz) and transformed forward along z; the two real spectra of
    // each packed line are separated and written to four half slots (sl, cx, cy, cz)
    using EF = Engine<V, N, P, 1, false, Z::T, -1>;
    static_assert(EF::K0 == 1 && EF::LDS_ELEMS <= E::LDS_ELEMS, "forward z tile: the inverse one's layout");
    const R* t1 = static_cast<const R*>(args.t6);
    constexpr size_t VOL = (size_t)N * N * N;
    V w[2][R0];
#pragma unroll
    for (int s = 0; s < R0; ++s) {
      const size_t idx = (size_t)lineL * N + j + s * M0;
      R a6[6], b6[6];
#pragma unroll
      for (int c = 0; c < 6; ++c) {
        a6[c] = t1[c * VOL + idx];
        b6[c] = comp(c, s);
      }
      R sl, cx, cy, cz;
      lpt3_sources(a6, b6, sl, cx, cy, cz);
      w[0][s] = V{sl, cx};
      w[1][s] = V{cy, cz};
    }
    V* out = static_cast<V*>(args.out);
    constexpr size_t HSLOT = (size_t)N * N * HZ;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      EF::run(*reinterpret_cast<V(*)[1][R0]>(&w[q]), lds, s_tw, t);
#pragma unroll
      for (int s = 0; s < R0; ++s) lds[EF::lds_index(0, p, j + s * M0)] = w[q][s];
      __syncthreads();
#pragma unroll
      for (int s = 0; s < R0 / 2; ++s) {
        const int k = j + s * M0;
        const V zk = lds[EF::lds_index(0, p, k)];
        const V zn = lds[EF::lds_index(0, p, (N - k) % N)];
        const V A = V{R(0.5) * (zk.x + zn.x), R(0.5) * (zk.y - zn.y)};   // (Z_k + conj Z_{N-k})/2
        const V B = V{R(0.5) * (zk.y + zn.y), R(0.5) * (zn.x - zk.x)};   // (Z_k - conj Z_{N-k})/(2i)
        if (line_ok) {
          out[(size_t)(2 * q) * HSLOT + (size_t)line * HZ + k] = A;
          out[(size_t)(2 * q + 1) * HSLOT + (size_t)line * HZ + k] = B;
        }
      }
      __syncthreads();
    }
  } else {
    static_assert(EPI == EPI_MU2 && Q == 3, "2LPT source needs the six components");
    // mu2 at each point, then a forward real-to-complex transform along z of line pairs
    // (2u, 2u+1) packed as one complex line, written to a half slot.
    using EF = Engine<V, N, P / 2, 1, false, Z::T, -1>;
    static_assert(EF::LDS_ELEMS <= E::LDS_ELEMS, "forward z tile fits the LDS of the inverse one");
#pragma unroll
    for (int s = 0; s < R0; ++s) {
      const int n = j + s * M0;
      const R xx = comp(0, s), xy = comp(1, s), xz = comp(2, s), yy = comp(3, s), yz = comp(4, s), zz = comp(5, s);
      const R mu2 = line_ok ? (xx * yy + xx * zz + yy * zz - xy * xy - xz * xz - yz * yz) : R(0);
      if (args.t6 != nullptr && line_ok) {
        R* t6 = static_cast<R*>(args.t6);
        constexpr size_t VOL = (size_t)N * N * N;
        const size_t idx = (size_t)line * N + n;
        t6[idx] = xx;
        t6[VOL + idx] = xy;
        t6[2 * VOL + idx] = xz;
        t6[3 * VOL + idx] = yy;
        t6[4 * VOL + idx] = yz;
        t6[5 * VOL + idx] = zz;
      }
      reinterpret_cast<R*>(&lds[EF::lds_index(0, p >> 1, n)])[p & 1] = mu2;
    }
    __syncthreads();
    static_assert(EF::K0 == 1, "forward z: one butterfly per thread");
    V w[1][R0];
    {
      int q2, p2, j2;
      bool ok2;
      EF::first_layout(t, 0, q2, p2, j2, ok2);
#pragma unroll
      for (int s = 0; s < R0; ++s) w[0][s] = ok2 ? lds[EF::lds_index(0, p2, j2 + s * M0)] : V{R(0), R(0)};
      __syncthreads();
      EF::run(w, lds, s_tw, t);
      if (ok2) {
#pragma unroll
        for (int s = 0; s < R0; ++s) lds[EF::lds_index(0, p2, j2 + s * M0)] = w[0][s];
      }
    }
    __syncthreads();
    V* out = static_cast<V*>(args.out);
    constexpr int NOUT = (P / 2) * HZ;
    for (int o = t; o < NOUT; o += Z::T) {
      const int u = o / HZ, k = o % HZ;
      const V zk = lds[EF::lds_index(0, u, k)];
      const V zn = lds[EF::lds_index(0, u, (N - k) % N)];
      const V a = V{R(0.5) * (zk.x + zn.x), R(0.5) * (zk.y - zn.y)};   // (Z_k + conj Z_{N-k})/2
      const V b = V{R(0.5) * (zk.y + zn.y), R(0.5) * (zn.x - zk.x)};   // (Z_k - conj Z_{N-k})/(2i)
      const int l0 = blockIdx.x * P + 2 * u;
      if (l0 < Z::LINES) st_slot<R, N, 2>(out + (size_t)l0 * HZ + k, a);
      if (l0 + 1 < Z::LINES) st_slot<R, N, 2>(out + (size_t)(l0 + 1) * HZ + k, b);
    }
  }
}

// ---------------------------------------------------------------------------------------------
// z pass with the collapse epilogue: inverse transforms along z of the three packed slots of each
// radius of a batch, the collapse model per point, and the running maximum over the radii.
//
// Order of the radii.  A whole call (WHOLE) takes the radii from the last (the smallest) to the
// first: F grows towards small radii at most points, so the maximum is nearly final after a few
// radii and few points change later (5.8% of the points per radius against 67% in increasing
// index, counted over 40 radii on a 2 Mpc/h grid).  Ties then go to the radius taken last, which is
// the smaller index, as in increasing order, where they go to the first.  A range call has to be
// the next part of a walk in increasing order, whatever its state holds, and takes its radii so.
//
// Points that cannot change are left out of a whole call.  For every symmetric tensor T,
// F(T) > 0 implies
//     F <= delta / 2 + 0.6915 |T|,   delta = tr T, |T| = sqrt(sum T_ij^2)
// (both sides scale with T; the constant is the largest value of (F - delta/2)/|T| over all
// eigenvalue directions, sampled at a million points of the ordered ones), so a point whose
// running maximum f has f - delta/2 > 0.7 |T| keeps it: the 1.2% of slack covers the float32
// rounding of T's norm and of F.  21% of the points are left for the model (counted as above), too
// spread out for whole waves to skip it (68% of the 64-point rows hold one), so each wave gathers
// those of its points in LDS and evaluates them densely, 64 at a time.  With the model in place at
// every point its 1230 of 1879 VALU instructions per wave bounded the pass (512^3 float32: 0.91 ms);
// now its loads do: 0.75 ms averaged over 40 radii, 0.62 at the last, 5.4 TB/s (float64: 2.28 ->
// 1.68 ms; 256^3 float32 with v_max: 0.222 -> 0.150 ms).  Nothing may spill: 32 bytes a lane of
// scratch wrote 0.5 GB per launch at 512^3 and cost the whole gain (0.96 ms).
struct ZCollapseArgs {
  const void* F;       // running F_max (R) before this batch
  void* Fout;          // F_max after it; with groups, [groups][N^3]
  uint8_t* ridx;       // radius index of F_max; with groups, [groups][N^3]
  int r0;              // radius index of the batch's first slots
  int nb;              // radii in the batch
  bool fresh;          // no state before this batch: F, ridx (v_max) are written at every point
  CollapseConst cc;
  const void* gin;     // v_max: the packed gradient slots (y-pass recipe 5), two per radius
  void* vout;          // v_max [3][N^3] (R)
  double vscale;       // v_max: L / 2 pi
};

template <typename R> __device__ __forceinline__ R collapse_of(R xx, R xy, R xz, R yy, R yz, R zz, const CollapseConst& cc) {
  if constexpr (sizeof(R) == 4) {
    return collapse_point_mixed(xx, xy, xz, yy, yz, zz, (float)cc.sphere_gain);
  } else {
    return collapse_point(xx, xy, xz, yy, yz, zz, cc);
  }
}

// Whether a point with tensor T could reach the running maximum f.  The computed F follows the bound
// only while the sixth powers of |T| in its discriminant neither overflow nor lose bits to underflow
// (in float32 F is infinite from |T| = 2.6e6 at some points), so points with |T| above 1.4e6 (float64
// 1.4e40) are kept, and the term added to |T|^2 keeps those below 1e-4 (1e-40); a NaN keeps its point.
template <typename R> __device__ __forceinline__ bool may_reach(R xx, R xy, R xz, R yy, R yz, R zz, R f) {
  const R off = xy * xy + xz * xz + yz * yz;
  const R norm2 = (sizeof(R) == 4 ? R(1e-8) : R(1e-80)) + R(0.49) * (xx * xx + yy * yy + zz * zz + R(2) * off);
  const R h = f - R(0.5) * (xx + yy + zz);
  return !(h > R(0) && h * h > norm2 && norm2 < (sizeof(R) == 4 ? R(1e12) : R(1e80)));
}

// Place of this lane among the lanes of mask m, counted from first.
__device__ __forceinline__ unsigned lane_rank(unsigned long long m, unsigned first) {
  return __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, first));
}

// Radii that share a launch of the collapse passes.  The launches of a small grid are short (at
// 64^3 a pass over one radius took 8-9 us, of which its data needs 1-2), so as many radii share one
// as keep the slots between the passes, 9 half slots a radius, within the last-level cache.  At
// 128^3 float32, 32 radii: 2 radii a launch 1.24 ms, 3 (this rule) 1.13, 4 1.25; 96^3 float64, 24
// radii: 2 a launch 1.29 ms, 4 (this rule) 1.05, 5 0.99 (one launch of each pass fewer).
template <typename R, int N> struct BatchRule {
  static constexpr int most(int fit) { return fit < 1 ? 1 : fit < 16 ? fit : 16; }
  static constexpr int RADII = most(slots_fit<R, N>(9));
  static constexpr int RADII_V = most(slots_fit<R, N>(13));   // with v_max: 4 half slots more
  static constexpr bool MANY = RADII > 1;
};

// Points of one wave gathered at a time: half of its 64 R0.
template <int R0> constexpr int kGather = 32 * R0;

template <typename R, int N, bool VEL, bool WHOLE>
struct ZCollapse {
  using V = typename Cplx<R>::type;
  using ZT = ZTile<R, N, 3>;
  static constexpr int P = ZT::P;
  static constexpr int T = ZT::T;
  using E = Engine<V, N, P, 1, false, T, +1>;
  static constexpr int LINES = N * N;
  static constexpr int GRID = (LINES + P - 1) / P;
  static constexpr int WAVES = (T + 63) / 64;
  static constexpr int GATHER = kGather<E::R0>;
  static constexpr size_t GATHER_BYTES = WHOLE ? (size_t)WAVES * GATHER * 6 * sizeof(R) : 0;
  static constexpr size_t LDS_BYTES = E::LDS_ELEMS * sizeof(V) > GATHER_BYTES ? E::LDS_ELEMS * sizeof(V) : GATHER_BYTES;
  static_assert(E::K0 == 1 && ZT::QL == 1, "z pass: one butterfly per transform per thread");
  static_assert(T % 64 == 0, "z pass: gathered points are evaluated 64 at a time by whole waves");
  // least waves per SIMD: the most that hold one radius's three transforms with few registers spilled
  // (float32: 110 VGPRs at 512^3; lines with a radix-3 stage hold 9 values a thread, 138).  Launches
  // of several radii hold more: up to 33 spilled in float64 range calls at 64^3.
  static constexpr int WPE = sizeof(R) == 8 ? (VEL ? 1 : 2) : (VEL || E::max_held() > 8 ? 3 : 4);
};

// MANY: the launch takes several radii.  A launch of one stores its results as they come and holds
// the running maximum in registers: eight range calls of one radius each, 64^3 float64 327 us with the
// kernel of several radii (33 registers spilled) and 301 with its own, 96^3 float64 581 and 539.
template <typename R, int N, bool VEL, bool WHOLE, bool MANY>
__global__ void __launch_bounds__((ZCollapse<R, N, VEL, WHOLE>::T))
__attribute__((amdgpu_waves_per_eu(ZCollapse<R, N, VEL, WHOLE>::WPE)))
k_zcollapse(const typename Cplx<R>::type* __restrict__ in, const typename Cplx<R>::type* __restrict__ tw,
            ZCollapseArgs args) {
  using Z = ZCollapse<R, N, VEL, WHOLE>;
  using V = typename Z::V;
  using E = typename Z::E;
  constexpr int P = Z::P, R0 = E::R0, M0 = N / R0;
  constexpr size_t VOL = (size_t)N * N * N, PSLOT = VOL;
  __shared__ __align__(16) unsigned char lds_bytes[Z::LDS_BYTES];
  __shared__ V s_tw[tw_elems(N)];
  V* lds = reinterpret_cast<V*>(lds_bytes);
  const int t = threadIdx.x;
  load_twiddles<N, Z::T>(s_tw, tw, t);
  const int line = blockIdx.x * P + t / M0;
  const bool line_ok = Z::LINES % P == 0 || line < Z::LINES;
  const int lineL = line_ok ? line : Z::LINES - 1;
  // this group's radii of the batch, every groups-th from its own (one group: all of them), and
  // its outputs
  const int groups = gridDim.y, g = blockIdx.y;
  const int turns = (args.nb - g + groups - 1) / groups;
  const bool dense = args.fresh || groups > 1;   // every point is written
  R* F = static_cast<R*>(args.Fout) + (size_t)g * VOL;
  uint8_t* ridx = args.ridx + (size_t)g * VOL;
  const size_t at = (size_t)lineL * N + t % M0;
  R* q = reinterpret_cast<R*>(lds_bytes) + (size_t)(t >> 6) * (Z::GATHER * 6);
  // the running maximum of this thread's points: in registers, or in LDS where several radii share
  // the launch (held across the transforms of a radius it would spill)
  R fold[MANY ? 1 : R0];
  __shared__ R s_fold[MANY ? R0 * Z::T : 1];
  auto best = [&](int s) -> R& { return MANY ? s_fold[s * Z::T + t] : fold[MANY ? 0 : s]; };
  // several radii a launch: index of the one that set fold, a byte per point, 255: none; stored
  // at the end.  One radius: stored as it comes.  Streamed: read again only after other passes.
  uint32_t rset[(R0 + 3) / 4];
#pragma unroll
  for (int s = 0; s < R0; ++s) best(s) = args.fresh ? R(0) : static_cast<const R*>(args.F)[at + s * M0];
#pragma unroll
  for (int s = 0; s < (R0 + 3) / 4; ++s) rset[s] = ~0u;
#pragma unroll 1
  for (int i = 0; i < (MANY ? turns : 1); ++i) {
    const int b = WHOLE ? args.nb - 1 - g - i * groups : g + i * groups;
    // an opaque copy: every address made from it would otherwise be computed ahead of the loop and
    // held across the epilogue (33 spilled registers at 512^3)
    int tt = t;
    if constexpr (MANY) asm volatile("" : "+v"(tt));
    const ZLoader<R, N, P> ld(line_ok ? blockIdx.x * P + tt / M0 : Z::LINES - 1, tt % M0);
    V v[3][R0];
#pragma unroll
    for (int c = 0; c < 3; ++c) ld.load(in + (size_t)(3 * b + c) * PSLOT, v[c]);
    if (i > 0) __syncthreads();   // the gathered points of the radius before are read
#pragma unroll
    for (int c = 0; c < 3; ++c) E::run(*reinterpret_cast<V(*)[1][R0]>(&v[c]), lds, s_tw, tt);
    // v[c][s] = (packed component 2c) + i (packed component 2c + 1): xy xz | yy yz | xx zz
    bool upd[R0];
    auto take = [&](int s, R fr) {
      const R f = best(s);
      upd[s] = line_ok && (fr > f || (WHOLE && fr == f && fr > R(0)));
      if constexpr (MANY) {
        if (upd[s]) best(s) = fr;
        const uint32_t set = (rset[s / 4] & ~(0xFFu << (8 * (s % 4)))) | ((uint32_t)(args.r0 + b) << (8 * (s % 4)));
        rset[s / 4] = upd[s] ? set : rset[s / 4];
      } else if (upd[s] || (dense && line_ok)) {
        __builtin_nontemporal_store(upd[s] ? fr : R(0), &F[at + s * M0]);
        __builtin_nontemporal_store(upd[s] ? (uint8_t)args.r0 : (uint8_t)255, &ridx[at + s * M0]);
      }
    };
    if constexpr (WHOLE) {
      const unsigned long long me = 1ull << (t & 63);
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        constexpr int H = R0 / 2;
        unsigned long long left[H];   // the lanes whose point is left for the model
        unsigned total = 0;
#pragma unroll
        for (int h = 0; h < H; ++h) {
          const int s = half * H + h;
          const bool need = line_ok && may_reach(v[2][s].x, v[0][s].x, v[0][s].y, v[1][s].x, v[1][s].y, v[2][s].y, best(s));
          left[h] = __ballot(need);
          if (need) {
            R* e = q + lane_rank(left[h], total);
            e[0] = v[2][s].x;
            e[Z::GATHER] = v[0][s].x;
            e[2 * Z::GATHER] = v[0][s].y;
            e[3 * Z::GATHER] = v[1][s].x;
            e[4 * Z::GATHER] = v[1][s].y;
            e[5 * Z::GATHER] = v[2][s].y;
          }
          total += (unsigned)__popcll(left[h]);
        }
        // one wave's own part of LDS: its lanes run in step, so only the compiler has to be held
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll 1
        for (unsigned k = t & 63; k < total; k += 64) {
          R* e = q + k;
          e[0] = collapse_of<R>(e[0], e[Z::GATHER], e[2 * Z::GATHER], e[3 * Z::GATHER], e[4 * Z::GATHER],
                                e[5 * Z::GATHER], args.cc);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        total = 0;
#pragma unroll
        for (int h = 0; h < H; ++h) {
          unsigned long long m = left[h];
          asm volatile("" : "+s"(m));   // ranked again: kept from above, the ranks would hold H registers
          R fr = R(0);                  // a point left out changes nothing
          if (m & me) fr = q[lane_rank(m, total)];
          take(half * H + h, fr);
          total += (unsigned)__popcll(m);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
      }
    } else {
#pragma unroll
      for (int s = 0; s < R0; ++s)
        take(s, collapse_of<R>(v[2][s].x, v[0][s].x, v[0][s].y, v[1][s].x, v[1][s].y, v[2][s].y, args.cc));
    }
    if constexpr (VEL) {
      // v_max: the smoothed gradient at this radius, transformed only now (the Hessian data is
      // dead); in a whole call only where a line of this workgroup has a point that changed
      R* vout = static_cast<R*>(args.vout);
      const bool all = args.fresh && i == 0;
      bool any = !WHOLE || all;
#pragma unroll
      for (int s = 0; s < R0; ++s) any = any || upd[s];
      if (!WHOLE || __syncthreads_or(any)) {
        const V* gin = static_cast<const V*>(args.gin) + (size_t)2 * b * PSLOT;
        V w[2][R0];
        ld.load(gin, w[0]);
        ld.load_one(gin + PSLOT, w[1]);
#pragma unroll
        for (int c = 0; c < 2; ++c) E::run(*reinterpret_cast<V(*)[1][R0]>(&w[c]), lds, s_tw, tt);
        const R vs = (R)args.vscale;
#pragma unroll
        for (int s = 0; s < R0; ++s) {
          if (upd[s] || (all && line_ok)) {
            __builtin_nontemporal_store(upd[s] ? w[0][s].x * vs : R(0), &vout[at + s * M0]);
            __builtin_nontemporal_store(upd[s] ? w[0][s].y * vs : R(0), &vout[VOL + at + s * M0]);
            __builtin_nontemporal_store(upd[s] ? w[1][s].x * vs : R(0), &vout[2 * VOL + at + s * M0]);
          }
        }
      }
    }
  }
  if constexpr (MANY) {
#pragma unroll
    for (int s = 0; s < R0; ++s) {
      const uint8_t r = (uint8_t)(rset[s / 4] >> (8 * (s % 4)));
      if (line_ok && (r != 255 || dense)) {
        __builtin_nontemporal_store(best(s), &F[at + s * M0]);
        __builtin_nontemporal_store(r, &ridx[at + s * M0]);
      }
    }
  }
}

// Groups' results [groups][VOL] into the running state: the largest F, of equal ones the smallest
// radius index.  The state before the batch holds larger indices in a whole call and smaller ones
// otherwise.
template <typename R>
__global__ void k_merge(const R* __restrict__ Fg, const uint8_t* __restrict__ rg, int groups, size_t vol, R* __restrict__ F,
                        uint8_t* __restrict__ ridx, bool whole, bool fresh) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= vol) return;
  R f = fresh ? R(0) : F[i];
  const int before = whole ? 256 : -1;
  int r = before;
  // eight groups' values at a time, all loaded before any is compared
  for (int k0 = 0; k0 < groups; k0 += 8) {
    R fk[8];
    int rk[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const size_t e = (size_t)(k0 + k < groups ? k0 + k : groups - 1) * vol + i;
      fk[k] = Fg[e];
      rk[k] = rg[e];   // 255: this group left the state as it was
    }
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (rk[k] != 255 && (fk[k] > f || (fk[k] == f && rk[k] < r))) {
        f = fk[k];
        r = rk[k];
      }
  }
  if (r != before || fresh) {
    F[i] = f;
    ridx[i] = (uint8_t)(r != before ? r : 255);
  }
}

// ---------------------------------------------------------------------------------------------
// Per-point collapse model on caller-given tensors T6 [6][count] (xx, xy, xz, yy, yz, zz): the
// same device functions as the z pass epilogue.
template <typename R>
__global__ void k_collapse_points(const R* __restrict__ t6, size_t count, R* __restrict__ F, CollapseConst cc) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const R xx = t6[i], xy = t6[count + i], xz = t6[2 * count + i];
  const R yy = t6[3 * count + i], yz = t6[4 * count + i], zz = t6[5 * count + i];
  if constexpr (sizeof(R) == 4) {
    F[i] = collapse_point_mixed(xx, xy, xz, yy, yz, zz, (float)cc.sphere_gain);
  } else {
    F[i] = collapse_point(xx, xy, xz, yy, yz, zz, cc);
  }
}

// ---------------------------------------------------------------------------------------------
// Running-maximum reset: F = 0, ridx = 255.
template <typename R>
__global__ void k_reset(R* __restrict__ F, uint8_t* __restrict__ ridx, size_t count) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) {
    F[i] = R(0);
    ridx[i] = 255;
  }
}

// ---------------------------------------------------------------------------------------------
// Collapse redshift: z_c with D(z_c) = 1/F, D the growing mode normalised to 1 at z = 0,
// tabulated (float64) on y = ln a at m nodes y0 + i h with D and dD/dy.  F <= 0, or 1/F beyond the
// last node (a > 1e6), gives z_c = -1.
//
// 1 + z_c is read from a polynomial per bucket of 1/32 octave of F, or of e = F - 1/D_inf towards
// the no-collapse limit, whose coefficients the host fits to the table's inverse (float64): an
// index from the variable's leading bits, 64 bytes of coefficients from LDS, 7 fused multiply-adds.
// Values outside the buckets take the search: the interval holding 1/F by bisection on the monotone
// D, then y by Newton steps on the cubic Hermite interpolant of D(y) there; below the first node
// D = a (1 - (2/11)(Lambda/Om) a^3 + ...) / a_per_D is inverted directly.  The search for every
// value (a chain of dependent loads, three float64 divisions and an exponential) took 179 us for
// the 256^3 values of a float32 grid, 0.75 TB/s of its 8 bytes a value; with the buckets 42 us,
// 3.2 TB/s.
// z_c by search, for f >= f_none
__device__ __forceinline__ double redshift_search(const GrowthArgs& g, double f) {
  const double t = 1.0 / f;
  if (t < g.d[0]) {
    const double a0 = t * g.a_per_D;
    const double a = a0 * (1.0 + (2.0 / 11.0) * g.lambda_over_m * a0 * a0 * a0);
    return 1.0 / a - 1.0;
  }
  if (!(t < g.d[g.m - 1])) return -1.0;
  // the bucket of t in log2 narrows the node search to a few steps; the bounds are checked
  // against t so that a bucket taken one off by rounding only widens the search
  int b = (int)((__log2f((float)t) - g.l0) * g.inv);
  b = min(max(b, 0), g.k - 2);
  int lo = g.guide[b], hi = min(g.guide[b + 1] + 1, g.m - 1);   // d[lo] <= t < d[hi]
  if (!(g.d[lo] <= t)) lo = 0;
  if (!(t < g.d[hi])) hi = g.m - 1;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (g.d[mid] <= t) lo = mid; else hi = mid;
  }
  const double d0 = g.d[lo], d1 = g.d[hi], m0 = g.dd[lo] * g.h, m1 = g.dd[hi] * g.h;
  // Newton on the cubic Hermite segment from the chord: the chord is within h/4 of the root
  // in s, and each step squares the error times about h, so three steps reach rounding
  double s = (t - d0) / (d1 - d0);
#pragma unroll
  for (int it = 0; it < 3; ++it) {
    const double s2 = s * s, s3 = s2 * s;
    const double hv = (2 * s3 - 3 * s2 + 1) * d0 + (s3 - 2 * s2 + s) * m0 + (-2 * s3 + 3 * s2) * d1 + (s3 - s2) * m1;
    const double hp = (6 * s2 - 6 * s) * d0 + (3 * s2 - 4 * s + 1) * m0 + (-6 * s2 + 6 * s) * d1 + (3 * s2 - 2 * s) * m1;
    s = fmin(1.0, fmax(0.0, s - (hv - t) / hp));
  }
  return exp(-(g.y0 + (lo + s) * g.h)) - 1.0;
}

// z_c from the buckets' polynomials, or by search for values outside them
__device__ __forceinline__ double redshift_of(const GrowthArgs& g, const double* poly, double f) {
  if (!(f >= g.f_none)) return -1.0;
  // bucket of F, else of e
  const double e = f - g.f_inf;
  const unsigned bf = (unsigned)(__double2hiint(f) >> (20 - kBucketBits)) - (unsigned)g.f_base;
  const unsigned be = (unsigned)(__double2hiint(e) >> (20 - kBucketBits)) - (unsigned)g.e_base;
  const bool in_f = bf < (unsigned)g.f_count, in_e = be < (unsigned)g.e_count;
  double out = __builtin_nan("");
  if (in_f || in_e) {
    const double x = in_f ? f : e;
    const double* c = poly + kBucketStride * (in_f ? bf : g.f_count + be);
    const int hi = (__double2hiint(x) & 0xFFFFF) | 0x3FF00000;
    const double mid = __hiloint2double((hi & ~((1 << (20 - kBucketBits)) - 1)) | (1 << (19 - kBucketBits)), 0);
    const double u = __hiloint2double(hi, __double2loint(x)) - mid;
    double v = c[kBucketCoefs - 1];
#pragma unroll
    for (int j = kBucketCoefs - 2; j >= 0; --j) v = fma(v, u, c[j]);
    out = v - 1.0;
  }
  return out == out ? out : redshift_search(g, f);
}

constexpr int kRedshiftThreads = 1024;   // two workgroups a CU: 64 KB of LDS and 64 VGPRs a thread
constexpr int kRedshiftValues = 4;       // a thread's values in flight, a workgroup's apart

template <typename R>
__global__ void __launch_bounds__(kRedshiftThreads)
__attribute__((amdgpu_waves_per_eu(8)))
k_redshift(const R* __restrict__ F, size_t count, const GrowthTables* __restrict__ t, R* __restrict__ z) {
  __shared__ double s_poly[kMaxBuckets * kBucketStride];
  for (int i = threadIdx.x; i < kMaxBuckets * kBucketStride; i += kRedshiftThreads) s_poly[i] = t->poly[i];
  const GrowthArgs g = t->args;
  __syncthreads();
  constexpr int SPAN = kRedshiftThreads * kRedshiftValues;
#pragma unroll 1
  for (size_t i0 = (size_t)blockIdx.x * SPAN + threadIdx.x; i0 < count; i0 += (size_t)gridDim.x * SPAN) {
    R f[kRedshiftValues];
#pragma unroll
    for (int k = 0; k < kRedshiftValues; ++k) {
      const size_t i = i0 + k * kRedshiftThreads;
      f[k] = F[i < count ? i : i0];
    }
#pragma unroll
    for (int k = 0; k < kRedshiftValues; ++k) {
      const double out = redshift_of(g, s_poly, (double)f[k]);
      const size_t i = i0 + k * kRedshiftThreads;
      if (i < count) z[i] = (R)out;
    }
  }
}

// Few values: coefficients from memory, no fill of LDS to wait for.  float32, one call of many in a
// graph, this / the kernel above: 1 value 1.6 / 3.0 us, 2^16 2.0 / 5.0, 2^19 5.4 / 6.9, 2^20 7.6 / 7.6,
// 2^21 11.6 / 10.3 (the search for every value: 2.2, 4.0, 7.8, 12.3, 21.0).
constexpr size_t kRedshiftFew = 1 << 19;
template <typename R>
__global__ void __launch_bounds__(256)
k_redshift_few(const R* __restrict__ F, size_t count, const GrowthTables* __restrict__ t, R* __restrict__ z) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < count) z[i] = (R)redshift_of(t->args, t->poly, (double)F[i]);
}

template <typename R>
__global__ void k_zero(R* __restrict__ p, size_t count) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) p[i] = R(0);
}

}  // namespace pin
