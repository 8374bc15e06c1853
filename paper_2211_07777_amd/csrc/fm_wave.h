// Per-wavefront form of the fused pass (forward FFT along the last axis, spectral
// multiply, inverse FFT) for complex lines of a power-of-two length.
//
// One line of M points is spread over P = M / E lanes of a 64-lane wavefront; lane j of
// the line holds points j + P m (m < E) in registers.  This is the layout of the input
// as loaded from HBM (consecutive lanes read consecutive points), of the spectrum after
// the forward transform and of the output before the store, so the forward transform,
// the multiplication by the Green's spectrum (or the spectral curl) and the inverse
// transform follow each other in registers.  The FFT is a Stockham radix schedule: the
// first stage is a radix-E butterfly over a lane's own registers, the later stages take
// their inputs from the other lanes of the line through a per-wave LDS buffer, and the
// last stage leaves the outputs in natural order in the lane layout above.  Nothing is
// shared between wavefronts, so there is no workgroup barrier: the LDS exchanges are
// ordered within the wave only.  L = 64 / P lines share a wavefront, W wavefronts a
// workgroup (one tile of W * L lines).  The three-component (curl) form gives each
// component its own wavefront (wave_curl_tile).
#pragma once
#include "fm_device.h"

namespace fm {

template <typename T, int M, int E_>
struct WaveShape {
  static constexpr int E = E_;
  static constexpr int P = M / E;
  static constexpr int L = 64 / P;
};

// LDS ordering between the lanes of one wavefront: every LDS access of the wave issued
// before the call is performed before any issued after it (LDS operations of a
// wavefront are performed in order; the fences keep the compiler from moving accesses
// across).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The same pointer (uniform) or lane index (per lane), whose value the compiler cannot
// connect with the original.  The forward and the inverse transform read the same twiddles,
// and the groups of a tile the same tables: kept in registers from one to the other, those
// loads and their addresses held up to 5 E registers across the whole tile, where reading
// them again costs cache hits that hide behind the exchanges.
template <class P>
__device__ __forceinline__ P unlinked(P p) {
#ifdef __HIP_DEVICE_COMPILE__
  asm volatile("" : "+s"(p));
#endif
  return p;
}
__device__ __forceinline__ int unlinked_lane(int j) {
#ifdef __HIP_DEVICE_COMPILE__
  asm volatile("" : "+v"(j));
#endif
  return j;
}

// Nothing is scheduled across: holds a phase of an unrolled loop to its registers.
__device__ __forceinline__ void sched_fence() {
#ifdef __HIP_DEVICE_COMPILE__
  __builtin_amdgcn_sched_barrier(0);
#endif
}

// Folded spectral index min(k, M - k) of point k = j + P m of a line (j < P, so k < M / 2
// for the first half of a lane's points): one of two addresses plus a constant.
template <int M, int E>
__device__ __forceinline__ int wave_fold(int j, int m) {
  constexpr int P = M / E;
  return m < E / 2 ? j + P * m : (M - P * m) - j;
}

// Stage s of the wave FFT (sign S) and all later stages.  Before the stage, v[i R + r]
// holds input r of the lane's butterfly i (t = j + P i), i.e. point t + r M / R; the
// first stage's inputs are the lane layout itself (one butterfly, t = j).  After the
// last stage v[m] holds output j + P m.
template <typename T, int M, int E, int s, int S, class TW>
__device__ __forceinline__ void wave_stages(cpx<T> (&v)[E], int j, cpx<T>* buf, TW tw) {
  constexpr int P = M / E;
  constexpr int R = wave_radix(M, s, E);
  if constexpr (R != 0) {
    constexpr int Ns = wave_ns(M, s, E);
    constexpr int NB = E / R;  // butterflies per lane
    if constexpr (s > 0) {
      // W_{Ns R}^{k r}, k = t mod Ns (table: offset + (r - 1) Ns + k)
      constexpr int off = wave_tw_offset(M, s, E);
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const int k = (j + P * i) & (Ns - 1);
#pragma unroll
        for (int r = 1; r < R; ++r) {
          const auto& g = tw[off + (r - 1) * Ns + k];
          const cpx<T> w = {g.x, S > 0 ? -g.y : g.y};
          v[i * R + r] = cmul(v[i * R + r], w);
        }
      }
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) SmallDft<R, S, T>::run(&v[i * R]);
    constexpr int R2 = wave_radix(M, s + 1, E);
    if constexpr (R2 == 0) {
      // last stage: output q of butterfly i is point t + q Ns = j + P (i + NB q)
      cpx<T> nat[E];
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int q = 0; q < R; ++q) nat[i + NB * q] = v[i * R + q];
#pragma unroll
      for (int e = 0; e < E; ++e) v[e] = nat[e];
    } else {
      // exchange through the wave's LDS line: output q of butterfly t goes to
      // (t - k) R + k + q Ns; the next stage reads point t' + r M / R2
      constexpr int NB2 = E / R2;
      constexpr int MR2 = M / R2;
      wave_lds_sync();  // the previous exchange's reads are done
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const int t = j + P * i;
        const int k = t & (Ns - 1);
        const int base = (t - k) * R + k;
#pragma unroll
        for (int q = 0; q < R; ++q) buf[pad16(base + q * Ns)] = v[i * R + q];
      }
      wave_lds_sync();
#pragma unroll
      for (int i = 0; i < NB2; ++i) {
        const int t = j + P * i;
#pragma unroll
        for (int r = 0; r < R2; ++r) v[i * R2 + r] = buf[pad16(t + r * MR2)];
      }
      wave_stages<T, M, E, s + 1, S, TW>(v, j, buf, tw);
    }
  }
}

// One tile of the scalar fused pass (Poisson: times the Green's spectrum): W wavefronts of
// L lines each.
template <typename T, int M, int EV>
__device__ __forceinline__ void wave_tile(const PassDesc& d, const void* in, void* out, char* smem,
                                          int tile) {
  using WS = WaveShape<T, M, EV>;
  constexpr int E = WS::E, P = WS::P, L = WS::L;
  const int wave = (int)threadIdx.x >> 6, lane = (int)threadIdx.x & 63;
  const int j = lane % P;
  const int l = wave * L + lane / P;  // line of the tile
  const TileIdx ti = tile_index(d, tile);
  if (l >= ti.nl) return;  // no workgroup barrier follows
  cpx<T>* buf = reinterpret_cast<cpx<T>*>(smem) + (size_t)(wave * L + lane / P) * fft_line_stride(M);
  const GTab<T> tw = gptr<cpx<T>>(E == 16 ? d.wtw : (E == 8 ? d.wtw8 : d.wtw32));
  const int b = ti.b0 + l;

  // the Green's row of the line, folded: G[fold(k)] for k = j + P m (coalesced; the upper
  // half of a row reads the lower half again, from cache), loaded ahead of the transforms
  // (its latency hides behind them)
  const auto* G = gptr<T>(d.g.G);
  const int64_t grow = ((int64_t)fold_index(ti.c, d.g.fold_c) * d.g.F_b + fold_index(b, d.g.fold_b)) *
                       (int64_t)d.g.F_line;
  T g[E];
#pragma unroll
  for (int m = 0; m < E; ++m) g[m] = G[grow + fold_index(j + P * m, d.g.fold_line)];

  cpx<T> v[E];
  const auto* src = gptr<cpx<T>>(in) + (int64_t)ti.comp * d.in_s_comp + (int64_t)ti.c * d.in_s_c +
                    (int64_t)b * d.in_s_b;
#pragma unroll
  for (int m = 0; m < E; ++m) {
    const int n = j + P * m;
    v[m] = cpx<T>{T(0), T(0)};
    if (n < d.n_data) {
      const auto& z = src[n];
      v[m] = cpx<T>{z.x, z.y};
    }
  }
  wave_stages<T, M, E, 0, -1>(v, j, buf, tw);
#pragma unroll
  for (int m = 0; m < E; ++m) v[m] = {v[m].x * g[m], v[m].y * g[m]};
  wave_stages<T, M, E, 0, +1>(v, j, buf, tw);
  auto* dst = (__attribute__((address_space(1))) cpx<T>*)(out) + (int64_t)ti.comp * d.out_s_comp +
              (int64_t)ti.c * d.out_s_c + (int64_t)b * d.out_s_b;
#pragma unroll
  for (int m = 0; m < E; ++m) {
    const int n = j + P * m;
    if (n < d.out_n) {
      dst[n].x = v[m].x;
      dst[n].y = v[m].y;
    }
  }
}

// One tile of the three-component fused pass (u = G i w x f): three wavefronts, wavefront
// q transforms component q of L lines at a time and walks the tile's groups of L lines.
// Component q of the product needs only the two other components of f, so each wavefront
// leaves its spectrum in its LDS lines, and after a workgroup barrier reads the two others
// at its own points; a second barrier frees the lines for the inverse's exchanges.
// A wavefront thus holds one line's E values instead of three lines': 128 registers and
// four waves per SIMD in FP32 at 1024 points, where one wavefront per line with its three
// components took 304 and ran one.  It is bound by the latency of its phases (HBM loads,
// exchanges, two barriers): requesting the next group's input during the inverse took
// registers from the occupancy and ran 10 % slower in FP32 and 2.4 times in FP64.
// Measured, one component set of 512^3 (13.45 GB in FP32): 5.61 ms (2.40 TB/s) against
// 8.77 ms, FP64 10.84 ms against 18.2 ms; 256^3 FP64: 1.12 ms against 1.55 ms.
template <typename T, int M, int EV>
__device__ __forceinline__ void wave_curl_tile(const PassDesc& d, const void* in, void* out, char* smem,
                                               int tile) {
  using WS = WaveShape<T, M, EV>;
  constexpr int E = WS::E, P = WS::P, L = WS::L;
  constexpr int LS = fft_line_stride(M);
  const int q = (int)threadIdx.x >> 6, lane = (int)threadIdx.x & 63;
  const int qa = q == 2 ? 0 : q + 1, qb = q == 0 ? 2 : q - 1;  // (q + 1) mod 3, (q + 2) mod 3
  const int j0 = lane % P, sub = lane / P;
  const TileIdx ti = tile_index(d, tile);
  cpx<T>* lines = reinterpret_cast<cpx<T>*>(smem);
  cpx<T>* buf = lines + (size_t)(q * L + sub) * LS;
  const cpx<T>* bufa = lines + (size_t)(qa * L + sub) * LS;
  const cpx<T>* bufb = lines + (size_t)(qb * L + sub) * LS;
  const GTab<T> tw = gptr<cpx<T>>(E == 16 ? d.wtw : (E == 8 ? d.wtw8 : d.wtw32));
  const auto* G = gptr<T>(d.g.G);
  const auto* wline = gptr<T>(d.g.dtab_line);
  const int64_t growc = (int64_t)fold_index(ti.c, d.g.fold_c) * d.g.F_b;
  T wc, mc;
  curl_factor<T>(d.g.csym, curl_wave<T>(ti.c, d.g.dtab_c), wc, mc);
  for (int g0 = 0; g0 < ti.nl; g0 += L) {  // uniform over the workgroup
    const int j = unlinked_lane(j0);
    const int l = g0 + sub;
    const bool live = l < ti.nl;
    const int b = ti.b0 + (live ? l : ti.nl - 1);  // idle lanes read the tile's last line
    const auto* src = gptr<cpx<T>>(in) + (int64_t)q * d.in_s_comp + (int64_t)ti.c * d.in_s_c +
                      (int64_t)b * d.in_s_b;
    cpx<T> v[E];
#pragma unroll
    for (int m = 0; m < E; ++m) {
      const int n = j + P * m;
      v[m] = cpx<T>{T(0), T(0)};
      if (n < d.n_data) {
        const auto& z = src[n];
        v[m] = cpx<T>{z.x, z.y};
      }
    }
    wave_stages<T, M, E, 0, -1>(v, j, buf, unlinked(tw));
    wave_lds_sync();  // the last exchange's reads are done
#pragma unroll
    for (int m = 0; m < E; ++m) buf[pad16(j + P * m)] = v[m];
    // the Green's row and the factors of the two directions a, b of the product, on their
    // way while the wavefronts meet: direction axis_line's factor varies along the line,
    // the two others are the same for the whole line
    const int64_t grow = (growc + fold_index(b, d.g.fold_b)) * (int64_t)d.g.F_line;
    T wb, mb;
    curl_factor<T>(d.g.csym_b, curl_wave<T>(b, d.g.dtab_b), wb, mb);
    auto fixed = [&](int a, T& re, T& im) {
      re = a == d.g.axis_b ? wb : (a == d.g.axis_c ? wc : T(0));
      im = a == d.g.axis_b ? mb : (a == d.g.axis_c ? mc : T(0));
    };
    T are, aim, bre, bim;
    fixed(qa, are, aim);
    fixed(qb, bre, bim);
    const bool la = qa == d.g.axis_line, lb = qb == d.g.axis_line;  // uniform over the wavefront
    const bool imag = d.g.csym != 0 || d.g.csym_b != 0;             // uniform over the grid
    T g[E], wl[E];
#pragma unroll
    for (int m = 0; m < E; ++m) {
      g[m] = G[grow + wave_fold<M, E>(j, m)];
      wl[m] = wline[j + P * m];
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < E; ++m) {
      if (m % 4 == 0) sched_fence();  // four points' values in registers at a time
      const int k = j + P * m;
      const T xa = la ? wl[m] : are, xb = lb ? wl[m] : bre;
      // i g (w_a f_b - w_b f_a)
      const cpx<T> fa = bufa[pad16(k)], fb = bufb[pad16(k)];
      cpx<T> z = {xa * fb.x - xb * fa.x, xa * fb.y - xb * fa.y};
      if (imag) {
        z.x += bim * fa.y - aim * fb.y;
        z.y += aim * fb.x - bim * fa.x;
      }
      v[m] = {-g[m] * z.y, g[m] * z.x};
    }
    sched_fence();
    __syncthreads();  // every wavefront has read the spectra
    wave_stages<T, M, E, 0, +1>(v, unlinked_lane(j), buf, unlinked(tw));
    if (live) {
      auto* dst = (__attribute__((address_space(1))) cpx<T>*)(out) + (int64_t)q * d.out_s_comp +
                  (int64_t)ti.c * d.out_s_c + (int64_t)b * d.out_s_b;
#pragma unroll
      for (int m = 0; m < E; ++m) {
        const int n = j + P * m;
        if (n < d.out_n) {
          dst[n].x = v[m].x;
          dst[n].y = v[m].y;
        }
      }
    }
    wave_lds_sync();  // the inverse's exchange reads are done before the next group's writes
  }
}

// Tiles in the XCD-aware order of the other pass kernels; a grid of one workgroup per
// tile gives each workgroup one tile.
// Occupancy targets (waves per SIMD) that the curl kernels fit: FP32 four with 16 values per
// lane (at most 5 dwords spilled at 1024 points) and six with 8, FP64 two and four.
template <typename T, int KIND, int E>
constexpr int wave_min_waves() {
  return KIND != K_F_CURL ? 1 : (sizeof(T) == 4 ? (E == 16 ? 4 : 6) : (E == 16 ? 2 : 4));
}

template <typename T, int M, int KIND, int E>
__global__ __launch_bounds__(KIND == K_F_CURL ? kCurlThreads : kThreads)
__attribute__((amdgpu_waves_per_eu(wave_min_waves<T, KIND, E>())))
void wave_pass_kernel(const PassDesc* __restrict__ dp, const void* in, void* out) {
  extern __shared__ __align__(16) char smem[];
  const PassDesc& d = *dp;
  for (int k = 0;; ++k) {
    const int tile = xcd_tile(blockIdx.x, gridDim.x, k, d.tiles);
    if (tile < 0) return;
    if constexpr (KIND == K_F_CURL) {
      if (k > 0) __syncthreads();
      wave_curl_tile<T, M, E>(d, in, out, smem, tile);
    } else {
      wave_tile<T, M, E>(d, in, out, smem, tile);
    }
  }
}

// ---------------------------------------------------------------------------------
// Per-wavefront form of the plain passes (one axis, forward or inverse, any gather and
// scatter).  The tile is staged in LDS as in the LDS-tile kernel, so strided lines are
// still loaded and stored in coalesced rows, but each wavefront then transforms its own
// FFT lines in registers with the schedule above: three workgroup barriers per tile
// instead of one per radix stage.  Four wavefronts of L = 64 / P FFT lines each; a
// packed kind (two real lines per FFT) holds 2 L tile lines per wavefront, so a tile is
// B = 4 L (or 8 L) lines, a power of two.  The raw lines of wavefront w sit inside the
// LDS region of its own FFT lines: all its raw values are read before its first exchange
// write, and no other wavefront touches the region until the next workgroup barrier.
//
// A persistent grid: each workgroup loops over its tiles, and the input of its next
// tile is loaded into registers while the current one is transformed and stored.  The
// stage twiddles (and the real-to-real post-twiddles) are copied to LDS once, so the
// transform issues no global load that would wait for that prefetch (vector-memory
// loads complete in order).  Every per-thread address that does not depend on the tile
// is formed once: in the strided (across-lines) walk a thread owns tile line tid mod B
// and rows tid / B + u kThreads / B.
// ---------------------------------------------------------------------------------
//
// HALF: the real-to-real types II and III with M points instead of the 2 M of their
// symmetric extension (Makhoul's orderings, as in the runtime-length kernel): half the
// butterflies, gather reads and slots for two more LDS reads per output.  With the same
// values per lane the tile has twice the lines, whose prefetched input and reads in flight
// cost registers (FP64, 8 values: 202 against 122), so 4 values per lane where the length
// allows it.  256^3 FP32, 512-point extensions 69.6 us, half 60.4 with 8 values, 55.5 with
// 4; 256 x 256 x 128 FP64 65.5, 50.1 and 43.0 us (3.1 TB/s); semi-unbounded lines of
// 1024-point extensions 150 and (8 values) 84 us.
template <typename T, int M, int KIND, int E_, bool HALF>
struct WavePlain {
  static constexpr int E = E_;
  static constexpr int P = M / E;                         // lanes per FFT line
  static constexpr int L = 64 / P;                        // FFT lines per wavefront
  static constexpr int PK = gather_of(KIND) == G_CPLX ? 1 : 2;  // tile lines per FFT line
  static constexpr int RW = L * PK;                       // tile lines per wavefront
  static constexpr int B = 4 * RW;                        // tile lines
  static constexpr int STEP = kThreads / B;               // rows per value, strided walk
  static constexpr int LS = fft_line_stride(M);
  static constexpr bool CIN = in_cplx_of(KIND);
  using In = typename std::conditional<CIN, cpx<T>, T>::type;
  static constexpr int REGION = L * LS * (CIN ? 1 : 2);   // a wavefront's LDS, in In units
  static constexpr int U = wave_plain_values(KIND == K_R2C || HALF, E);  // input values per thread
  static constexpr int NTW = wave_tw_size(M, E);          // stage twiddles
  static constexpr int NPOST = KIND == K_R2R ? wave_post(M, HALF) : 0;  // real-to-real post-twiddles
  static constexpr int NSLOT = KIND == K_R2R ? M : 0;     // real-to-real gather slots
};

// Input values of one tile into registers (strided walk: only rows below in_n).
template <class WP, class Stage>
__device__ __forceinline__ void wp_fetch(Stage& r, const PassDesc& d,
                                         const void* in, const TileIdx& ti, bool lc) {
  using In = typename WP::In;
  const char* base = reinterpret_cast<const char*>(in) +
                     ((int64_t)ti.comp * d.in_s_comp + (int64_t)ti.c * d.in_s_c +
                      (int64_t)ti.b0 * d.in_s_b) * (int64_t)sizeof(In);
  const int tid = (int)threadIdx.x;
  if (lc) {
    const int total = ti.nl * d.in_n;
#pragma unroll
    for (int u = 0; u < WP::U; ++u) {
      const int e = tid + u * kThreads;
      if (e < total) {
        const uint32_t l = fdiv((uint32_t)e, d.mag_in);
        const uint32_t i = (uint32_t)e - l * (uint32_t)d.in_n;
        r.set(u, *reinterpret_cast<const In*>(base + (l * (uint32_t)d.in_s_b + i) * (uint32_t)sizeof(In)));
      }
    }
  } else {
    const int l = tid % WP::B, i0 = tid / WP::B;
    if (l < ti.nl) {
      const uint32_t o0 = ((uint32_t)l * (uint32_t)d.in_s_b + (uint32_t)i0 * (uint32_t)d.in_s_line) *
                          (uint32_t)sizeof(In);
      const uint32_t ds = (uint32_t)WP::STEP * (uint32_t)d.in_s_line * (uint32_t)sizeof(In);
#pragma unroll
      for (int u = 0; u < WP::U; ++u)
        if (i0 + u * WP::STEP < d.in_n) r.set(u, *reinterpret_cast<const In*>(base + o0 + (uint32_t)u * ds));
    }
  }
}

// Registers -> raw tile: tile line l at (l / RW) REGION + (l mod RW) rs.
template <class WP, class Stage>
__device__ __forceinline__ void wp_commit(const Stage& r, const PassDesc& d,
                                          const TileIdx& ti, char* smem, bool lc) {
  using In = typename WP::In;
  In* raw = reinterpret_cast<In*>(smem);
  const int rs = d.wave_rs, tid = (int)threadIdx.x;
  if (lc) {
    const int total = ti.nl * d.in_n;
#pragma unroll
    for (int u = 0; u < WP::U; ++u) {
      const int e = tid + u * kThreads;
      if (e < total) {
        const int l = (int)fdiv((uint32_t)e, d.mag_in);
        const int i = e - l * d.in_n;
        raw[(l / WP::RW) * WP::REGION + (l % WP::RW) * rs + i] = r.get(u);
      }
    }
  } else {
    const int l = tid % WP::B, i0 = tid / WP::B;
    if (l < ti.nl) {
      In* row = raw + (l / WP::RW) * WP::REGION + (l % WP::RW) * rs + i0;
#pragma unroll
      for (int u = 0; u < WP::U; ++u)
        if (i0 + u * WP::STEP < d.in_n) row[u * WP::STEP] = r.get(u);
    }
  }
}

// Real-to-real gather: slot m of the symmetric extension of line pair (2f, 2f + 1) is
// W_m (x_{2f}[s_m] + i x_{2f+1}[s_m]), with the source index s_m and the complex weight
// W_m (end-point weight, mirror sign, pre-twiddle) the same for every line and tile:
// a table of M entries built in LDS once per workgroup.  The half form's slot is
// W_m (X_{idx} - i X_{pair}) of the samples X = x_{2f} + i x_{2f+1}, an index of -1 standing
// for a sample that is 0 (type II: always without a pair).
template <typename T>
struct R2RSlot {
  T wx, wy;
  int idx, pair;
};

// Slot m of the half form.
template <typename T>
__device__ __forceinline__ R2RSlot<T> half_slot(const PassDesc& d, GTab<T> tw, int m) {
  const R2R& r = d.r2r;
  const int nh = r.nh;
  auto index = [&](int p) {
    const int j = r.in_rev ? r.in_base - p : p - r.in_base;
    return p >= r.plo && p <= r.phi && j >= 0 && j < d.in_n ? j : -1;
  };
  if (r.half == R2R_II) {
    const bool odd = 2 * m >= nh;  // the odd samples, backwards, follow the even ones
    return {odd && r.sin ? T(-1) : T(1), T(0), index(odd ? 2 * (nh - m) - 1 : 2 * m), -1};
  }
  const int p = r.sin ? nh - m : m;
  const cpx<T> w = twid<T>(tw, m);
  return {w.x, -w.y, index(p), index(nh - p)};
}

template <typename T, int M, int KIND, int E, bool HALF>
__device__ __forceinline__ void wp_transform(const PassDesc& d, const TileIdx& ti, char* smem,
                                             const cpx<T>* ltw, const R2RSlot<T>* slots) {
  using WP = WavePlain<T, M, KIND, E, HALF>;
  using In = typename WP::In;
  constexpr int P = WP::P, L = WP::L, PK = WP::PK;
  constexpr int S = (KIND == K_C2C_I || KIND == K_C2R) ? +1 : -1;
  const int wave = (int)threadIdx.x >> 6, lane = (int)threadIdx.x & 63;
  const int j = lane % P, lf = lane / P;  // lane of the line, line of the wavefront
  const int f = wave * L + lf;            // FFT line of the tile
  if (f >= (ti.nl + PK - 1) / PK) return;
  cpx<T>* line = reinterpret_cast<cpx<T>*>(smem) + (size_t)f * WP::LS;
  const In* raw = reinterpret_cast<const In*>(smem) + wave * WP::REGION;
  const int nlw = ti.nl - wave * WP::RW;  // tile lines from the wavefront's first
  const int rs = d.wave_rs;
  cpx<T> v[E];
  if constexpr (gather_of(KIND) == G_CPLX) {
    const GatherCplx<T> g{raw, rs, d.n_data};
#pragma unroll
    for (int k = 0; k < E; ++k) v[k] = g(lf, j + P * k);
  } else if constexpr (gather_of(KIND) == G_REAL2) {
    const GatherReal2<T> g{raw, rs, d.n_data, nlw};
#pragma unroll
    for (int k = 0; k < E; ++k) v[k] = g(lf, j + P * k);
  } else if constexpr (gather_of(KIND) == G_HERM2) {
    const GatherHerm2<T> g{raw, rs, M, nlw};
#pragma unroll
    for (int k = 0; k < E; ++k) v[k] = g(lf, j + P * k);
  } else {
    const T* r0 = raw + (2 * lf) * rs;
    const T* r1 = (2 * lf + 1 < nlw) ? r0 + rs : nullptr;
    if constexpr (HALF) {
      auto at = [&](int i) {
        const cpx<T> x = {r0[i < 0 ? 0 : i], r1 ? r1[i < 0 ? 0 : i] : T(0)};
        return i < 0 ? cpx<T>{T(0), T(0)} : x;
      };
      if (d.r2r.half == R2R_II) {
#pragma unroll
        for (int k = 0; k < E; ++k) {
          const R2RSlot<T> sl = slots[j + P * k];
          const cpx<T> a = at(sl.idx);
          v[k] = cpx<T>{sl.wx * a.x, sl.wx * a.y};
        }
      } else {
#pragma unroll
        for (int k = 0; k < E; ++k) {
          const R2RSlot<T> sl = slots[j + P * k];
          const cpx<T> a = at(sl.idx), b = at(sl.pair);
          v[k] = cmul(cpx<T>{a.x + b.y, a.y - b.x}, cpx<T>{sl.wx, sl.wy});
        }
      }
    } else {
#pragma unroll
    for (int k = 0; k < E; ++k) {
      const R2RSlot<T> sl = slots[j + P * k];
      const T a = r0[sl.idx];
      const T b = r1 ? r1[sl.idx] : T(0);
      v[k] = cpx<T>{a * sl.wx - b * sl.wy, a * sl.wy + b * sl.wx};
    }
    }
  }
  wave_stages<T, M, E, 0, S>(v, j, line, ltw);
  wave_lds_sync();  // the last exchange's reads are done
#pragma unroll
  for (int k = 0; k < E; ++k) line[pad16(j + P * k)] = v[k];
}

// One output element (line l, index j) with the last pass's fix-ups.
template <bool FIX, typename O>
__device__ __forceinline__ void wp_put(O* o, const PassDesc& d, const TileIdx& ti, int l, uint32_t off,
                                       O w, bool czero, bool cdup) {
  if constexpr (FIX) {
    const Fixup& fx = d.fix;
    const int b = ti.b0 + l;
    if (czero || (fx.b_zero_lo && b == 0) || (fx.b_zero_hi && b == fx.b_last)) w = O{};
    o[off] = w;
    const bool bdup = fx.b_dup && b == 0;
    if (bdup) o[off + (int64_t)fx.b_last * d.out_s_b] = w;
    if (cdup) {
      o[off + (int64_t)fx.c_last * d.out_s_c] = w;
      if (bdup) o[off + (int64_t)fx.b_last * d.out_s_b + (int64_t)fx.c_last * d.out_s_c] = w;
    }
  } else {
    (void)d; (void)ti; (void)l; (void)czero; (void)cdup;
    o[off] = w;
  }
}

template <typename T, int M, int KIND, int E, bool HALF, bool FIX>
__device__ __forceinline__ void wp_store(const PassDesc& d, void* out, const TileIdx& ti,
                                         const char* smem, const cpx<T>* lpost, bool lc) {
  using WP = WavePlain<T, M, KIND, E, HALF>;
  constexpr int SC = scatter_of(KIND);
  using O = typename std::conditional<SC == S_CPLX || SC == S_R2C2, cpx<T>, T>::type;
  constexpr int LS = WP::LS;
  const cpx<T>* buf = reinterpret_cast<const cpx<T>*>(smem);
  O* o = reinterpret_cast<O*>(out) + (int64_t)ti.comp * d.out_s_comp + (int64_t)ti.c * d.out_s_c +
         (int64_t)ti.b0 * d.out_s_b;
  auto val = [&](int l, int j) -> O {
    if constexpr (SC == S_CPLX) {
      return buf[l * LS + pad16(j < M ? j : j - M)];
    } else if constexpr (SC == S_R2C2) {
      const cpx<T>* z = buf + (l >> 1) * LS;
      const cpx<T> zk = z[pad16(j)], zm = z[pad16(j == 0 ? 0 : M - j)];
      if (l & 1) return cpx<T>{T(0.5) * (zk.y + zm.y), T(-0.5) * (zk.x - zm.x)};
      return cpx<T>{T(0.5) * (zk.x + zm.x), T(0.5) * (zk.y - zm.y)};
    } else if constexpr (SC == S_REAL2) {
      const cpx<T> z = buf[(l >> 1) * LS + pad16(j < M ? j : j - M)];
      return (l & 1) ? z.y : z.x;
    } else if constexpr (HALF) {
      const R2R& r = d.r2r;
      const int q = r.out_rev ? r.out_base - j : j + r.out_base;
      const bool ok = q >= r.qlo && q <= r.qhi;  // outside: the coefficient is 0
      const int qc = ok ? q : r.qlo;
      const cpx<T>* z = buf + (l >> 1) * LS;
      T v;
      if (r.half == R2R_II) {
        // the two lines' spectra V1 = (Z_k + conj Z_{-k}) / 2, V2 = (Z_k - conj Z_{-k}) / 2i
        const int k = r.sin ? M - qc : qc;
        const cpx<T> a = z[pad16(k == M ? 0 : k)], b = z[pad16(k == 0 ? 0 : M - k)], w = lpost[k];
        v = (l & 1) ? w.x * (a.y + b.y) + w.y * (a.x - b.x) : w.x * (a.x + b.x) - w.y * (a.y - b.y);
      } else {
        // sample n = q / 2 or M - (q + 1) / 2 of the inverse DFT, slot -n of the forward one
        const int n = (qc & 1) ? M - ((qc + 1) >> 1) : qc >> 1;
        const cpx<T> y = z[pad16(n ? M - n : 0)];
        v = (l & 1) ? y.y : y.x;
        if (r.sin && (qc & 1)) v = -v;
      }
      return ok ? v : T(0);
    } else {
      return scatter_r2r<T>(buf, LS, d.r2r, lpost, l, j);
    }
  };
  bool czero = false, cdup = false;
  if constexpr (FIX) {
    czero = (d.fix.c_zero_lo && ti.c == 0) || (d.fix.c_zero_hi && ti.c == d.fix.c_last);
    cdup = d.fix.c_dup && ti.c == 0;
  }
  const int tid = (int)threadIdx.x;
  if (lc) {
    const int total = ti.nl * d.out_n;
    for (int e0 = tid; e0 < total; e0 += 4 * kThreads) {
      O w[4];
      int ll[4];
      uint32_t off[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int e = e0 + q * kThreads;
        ll[q] = -1;
        if (e < total) {
          const int l = (int)fdiv((uint32_t)e, d.mag_out);
          const int j = e - l * d.out_n;
          ll[q] = l;
          off[q] = (uint32_t)l * (uint32_t)d.out_s_b + (uint32_t)j;
          w[q] = val(l, j);
        }
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (ll[q] >= 0) wp_put<FIX>(o, d, ti, ll[q], off[q], w[q], czero, cdup);
    }
  } else {
    const int l = tid % WP::B, j0 = tid / WP::B;
    if (l >= ti.nl) return;
    const uint32_t ob = (uint32_t)l * (uint32_t)d.out_s_b;
    const uint32_t sl = (uint32_t)d.out_s_line;
    for (int jb = j0; jb < d.out_n; jb += 4 * WP::STEP) {
      O w[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int j = jb + q * WP::STEP;
        if (j < d.out_n) w[q] = val(l, j);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int j = jb + q * WP::STEP;
        if (j < d.out_n) wp_put<FIX>(o, d, ti, l, ob + (uint32_t)j * sl, w[q], czero, cdup);
      }
    }
  }
}

// Occupancy targets of the plain per-wavefront kernels that fit them without spilling:
// FP32 with 4 or 8 values per lane four waves per SIMD (128 VGPRs), with 16 three (168); FP64
// keeps the compiler's choice.
template <typename T, int E>
constexpr int wave_plain_min_waves() {
  return sizeof(T) == 4 ? (E <= 8 ? 4 : 3) : 1;
}

template <typename T, int M, int KIND, int E, bool HALF>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(wave_plain_min_waves<T, E>())))
void wave_plain_kernel(const PassDesc* __restrict__ dp, const void* in, void* out) {
  using WP = WavePlain<T, M, KIND, E, HALF>;
  using In = typename WP::In;
  extern __shared__ __align__(16) char smem[];
  const PassDesc& d = component<T, KIND>(dp, in, out);
  int k = 0;
  int tile = xcd_tile(blockIdx.x, gridDim.x, k, d.tiles);
  if (tile < 0) return;
  const bool lc_in = d.in_s_line == 1, lc_out = d.out_s_line == 1;
  // the first tile's input is requested before the tables are copied, so that its HBM
  // latency and the tables' overlap (the copy waits for both: loads complete in order)
  TileIdx ti = tile_index(d, tile);
  RegStage<T, In, WP::U> r;
  wp_fetch<WP>(r, d, in, ti, lc_in);
  // tables into LDS, per-thread real-to-real gather weights
  cpx<T>* ltw = reinterpret_cast<cpx<T>*>(smem + d.tab_off);
  cpx<T>* lpost = ltw + WP::NTW;
  {
    const GTab<T> gtw = gptr<cpx<T>>(E == 16 ? d.wtw : d.wtw8);
    for (int i = (int)threadIdx.x; i < WP::NTW; i += kThreads) ltw[i] = cpx<T>{gtw[i].x, gtw[i].y};
    if constexpr (WP::NPOST > 0) {
      const GTab<T> g4 = gptr<cpx<T>>(d.tw);
      for (int i = (int)threadIdx.x; i < WP::NPOST; i += kThreads) lpost[i] = cpx<T>{g4[i].x, g4[i].y};
    }
  }
  R2RSlot<T>* slots = reinterpret_cast<R2RSlot<T>*>(lpost + WP::NPOST);
  if constexpr (HALF) {
    for (int m = (int)threadIdx.x; m < M; m += kThreads) slots[m] = half_slot<T>(d, gptr<cpx<T>>(d.tw), m);
  } else if constexpr (KIND == K_R2R) {
    const GatherR2R<T, GTab<T>> g{nullptr, 0, d.in_n, 2, d.r2r, gptr<cpx<T>>(d.tw)};
    for (int m = (int)threadIdx.x; m < M; m += kThreads) {
      R2RSlot<T> sl;
      const cpx<T> w = g.weight(m, sl.idx);
      sl.wx = w.x;
      sl.wy = w.y;
      sl.pair = -1;
      slots[m] = sl;
    }
  }
  for (;;) {
    wp_commit<WP>(r, d, ti, smem, lc_in);
    __syncthreads();
    const int next = xcd_tile(blockIdx.x, gridDim.x, ++k, d.tiles);
    const TileIdx tn = next >= 0 ? tile_index(d, next) : ti;
    if (next >= 0) wp_fetch<WP>(r, d, in, tn, lc_in);  // in flight during the transform
    wp_transform<T, M, KIND, E, HALF>(d, ti, smem, ltw, slots);
    __syncthreads();
    if (d.has_fix) wp_store<T, M, KIND, E, HALF, true>(d, out, ti, smem, lpost, lc_out);
    else wp_store<T, M, KIND, E, HALF, false>(d, out, ti, smem, lpost, lc_out);
    if (next < 0) return;
    __syncthreads();  // the stores' LDS reads are done before the next commit
    ti = tn;
  }
}

}  // namespace fm
