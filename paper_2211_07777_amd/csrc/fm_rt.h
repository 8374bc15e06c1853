// Line passes of any length with factors 2, 3, 5 and 7 (the lengths without a
// compile-time kernel).
//
// A tile of B lines lives in two LDS buffers: every radix stage reads one and writes the
// other, so a thread holds one butterfly at a time (not its whole share of the tile in
// registers) and a stage ends in one barrier.  The index arithmetic divides by
// host-made multipliers only, tile elements are walked by adding constant steps, and a
// stage's twiddles lie in its own table, consecutive along k: with integer divisions and
// strided twiddle reads these lengths ran at 120-700 GB/s, bound by address arithmetic.  The
// three components of a curl share one buffer (rt_radix_in_place).  All kinds share the radix stages (sign -1); an inverse
// transform is taken as the conjugate of the forward transform of the conjugate.
#pragma once
#include "fm_device.h"

namespace fm {

// cos and sin of 2 pi num / den, for tables of constants (Taylor series on an eighth of
// the circle)
constexpr double ct_poly(double x2, int first) {  // sum (-x2)^j / ((2 j + first)!) * first!
  double s = 0.0, t = 1.0;
  for (int j = 0; j < 14; ++j) {
    s += t;
    t *= -x2 / ((2 * j + 1 + first) * (2 * j + 2 + first));
  }
  return s;
}
constexpr double ct_cos(int num, int den);
constexpr double ct_sin(int num, int den) {
  num %= den;
  if (2 * num > den) return -ct_sin(den - num, den);
  if (4 * num > den) return ct_sin(den - 2 * num, 2 * den);  // sin(pi - x), x = 2 pi num / den
  if (8 * num > den) return ct_cos(den - 4 * num, 4 * den);  // cos(pi / 2 - x)
  const double x = 6.28318530717958647693 * num / den;
  return x * ct_poly(x * x, 1);
}
constexpr double ct_cos(int num, int den) {
  num %= den;
  if (2 * num > den) num = den - num;
  if (4 * num > den) return -ct_cos(den - 2 * num, 2 * den);
  if (8 * num > den) return ct_sin(den - 4 * num, 4 * den);
  const double x = 6.28318530717958647693 * num / den;
  return ct_poly(x * x, 0);
}

// radix A B: DFTs of length A over the samples B n1 + n2, twiddles W^(n2 k1), DFTs of
// length B
template <int A, int B, int S, typename T>
struct CompositeDft {
  template <int NUM>
  __device__ __forceinline__ static cpx<T> turn(cpx<T> v) {
    if constexpr (NUM == 0) {
      return v;
    } else {
      constexpr double c = ct_cos(NUM, A * B), s = ct_sin(NUM, A * B);
      return cmul(v, cpx<T>{T(c), T(S * s)});
    }
  }
  template <int N2, int K1>
  __device__ __forceinline__ static void column(const cpx<T>* col, cpx<T> (&a)[B][A]) {
    if constexpr (K1 < A) {
      a[N2][K1] = turn<N2 * K1>(col[K1]);
      column<N2, K1 + 1>(col, a);
    }
  }
  template <int N2>
  __device__ __forceinline__ static void columns(const cpx<T>* v, cpx<T> (&a)[B][A]) {
    if constexpr (N2 < B) {
      cpx<T> col[A];
#pragma unroll
      for (int n1 = 0; n1 < A; ++n1) col[n1] = v[B * n1 + N2];
      SmallDft<A, S, T>::run(col);
      column<N2, 0>(col, a);
      columns<N2 + 1>(v, a);
    }
  }
  __device__ __forceinline__ static void run(cpx<T>* v) {
    cpx<T> a[B][A];
    columns<0>(v, a);
#pragma unroll
    for (int k1 = 0; k1 < A; ++k1) {
      cpx<T> row[B];
#pragma unroll
      for (int n2 = 0; n2 < B; ++n2) row[n2] = a[n2][k1];
      SmallDft<B, S, T>::run(row);
#pragma unroll
      for (int k2 = 0; k2 < B; ++k2) v[k1 + A * k2] = row[k2];
    }
  }
};
template <int S, typename T>
struct SmallDft<6, S, T> : CompositeDft<3, 2, S, T> {};
template <int S, typename T>
struct SmallDft<9, S, T> : CompositeDft<3, 3, S, T> {};
template <int S, typename T>
struct SmallDft<10, S, T> : CompositeDft<5, 2, S, T> {};
template <int S, typename T>
struct SmallDft<12, S, T> : CompositeDft<4, 3, S, T> {};
template <int S, typename T>
struct SmallDft<15, S, T> : CompositeDft<5, 3, S, T> {};

// n / d by the multiplier of rt_magic (0: d = 1)
__device__ __forceinline__ int rt_div(int n, uint32_t mag) {
  return mag ? (int)(((uint64_t)(uint32_t)n * mag) >> 32) : n;
}

// One radix-R stage of F lines, src -> dst (natural Stockham order, see fft_stage).
template <typename T, int R>
__device__ __forceinline__ void rt_radix(const cpx<T>* __restrict__ src, cpx<T>* __restrict__ dst, int ls, int F,
                                         int MR, uint32_t mMR, int Ns, uint32_t mNs, GTab<T> tw) {
  const int total = F * MR;
  for (int u = (int)threadIdx.x; u < total; u += (int)blockDim.x) {
    const int line = rt_div(u, mMR);
    const int t = u - line * MR;
    const int tk = rt_div(t, mNs) * Ns, k = t - tk;
    const cpx<T>* s = src + line * ls;
    cpx<T> v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = s[pad16(t + r * MR)];
    if (Ns > 1) {  // uniform
#pragma unroll
      for (int r = 1; r < R; ++r) v[r] = cmul(v[r], twid<T>(tw, (r - 1) * Ns + k));
    }
    SmallDft<R, -1, T>::run(v);
    cpx<T>* d = dst + line * ls;
    const int base = tk * R + k;
#pragma unroll
    for (int q = 0; q < R; ++q) d[pad16(base + q * Ns)] = v[q];
  }
}

// The same stage in place, for the three components of a curl: a thread reads its
// butterflies and writes them after a barrier.  At most 8 points per thread (the workgroup's
// size sees to it).  A second barrier per stage, for half the LDS: FP64 lines of 840 points
// ran one workgroup of five wavefronts per CU, now two of eight.  4704 lines of three
// components, two buffers / in place, us: FP64 450 points 173 / 116, 840 395 / 195, 1200 440
// / 276; FP32 450 points 98 / 89, 840 238 / 159, 1280 208 / 186.
template <typename T, int R>
__device__ __forceinline__ void rt_radix_in_place(cpx<T>* __restrict__ buf, int ls, int F, int MR, uint32_t mMR, int Ns,
                                                  uint32_t mNs, GTab<T> tw) {
  constexpr int NB = (8 + R - 1) / R;
  const int total = F * MR;
  cpx<T> v[NB][R];
  int at[NB], base[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int u = (int)threadIdx.x + i * (int)blockDim.x;
    at[i] = -1;
    base[i] = 0;
    if (u >= total) continue;
    const int line = rt_div(u, mMR);
    const int t = u - line * MR;
    const int tk = rt_div(t, mNs) * Ns, k = t - tk;
    at[i] = line * ls;
    base[i] = tk * R + k;
    const cpx<T>* s = buf + at[i];
#pragma unroll
    for (int r = 0; r < R; ++r) v[i][r] = s[pad16(t + r * MR)];
    if (Ns > 1) {  // uniform
#pragma unroll
      for (int r = 1; r < R; ++r) v[i][r] = cmul(v[i][r], twid<T>(tw, (r - 1) * Ns + k));
    }
    SmallDft<R, -1, T>::run(v[i]);
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    if (at[i] < 0) continue;
#pragma unroll
    for (int q = 0; q < R; ++q) buf[at[i] + pad16(base[i] + q * Ns)] = v[i][q];
  }
}

// Forward FFTs of the F lines in a, with b as the other buffer; returns the buffer that
// holds the result (natural order).  Begins and ends with a barrier.  IN_PLACE: b is not
// used.
template <typename T, bool IN_PLACE = false>
__device__ __forceinline__ cpx<T>* rt_fft(const PassDesc& d, cpx<T>* a, cpx<T>* b, int ls, int F) {
  GTab<T> tw = gptr<cpx<T>>(d.tw) + 4 * d.M;
  int Ns = 1;
  __syncthreads();
  for (int s = 0; s < d.rt_n; ++s) {
    const int R = d.rt_radix[s];
    const int MR = d.M / R;
    const uint32_t mMR = d.rt_mr[s], mNs = d.rt_ns[s];
#define FM_RT_CASE(RR) \
  case RR:                                                                        \
    if constexpr (IN_PLACE) rt_radix_in_place<T, RR>(a, ls, F, MR, mMR, Ns, mNs, tw); \
    else rt_radix<T, RR>(a, b, ls, F, MR, mMR, Ns, mNs, tw);                      \
    break;
    switch (R) {
      FM_RT_CASE(2)
      FM_RT_CASE(3)
      FM_RT_CASE(4)
      FM_RT_CASE(5)
      FM_RT_CASE(6)
      FM_RT_CASE(7)
      FM_RT_CASE(8)
      FM_RT_CASE(9)
      FM_RT_CASE(10)
      FM_RT_CASE(12)
      FM_RT_CASE(15)
      FM_RT_CASE(16)
      default: break;
    }
#undef FM_RT_CASE
    tw += (R - 1) * Ns;
    Ns *= R;
    if constexpr (!IN_PLACE) {
      cpx<T>* const x = a;
      a = b;
      b = x;
    }
    __syncthreads();
  }
  return a;
}

// The elements of a tile of nl lines x n values, spread over the workgroup: line l, index
// i, memory offset; lines contiguous in memory are walked along the line, others across
// the B lines of the tile.  Every step adds constants (at most one carry).
struct RtWalk {
  int l, i;
  int64_t off;
  int f, fext, df;           // fast index, its extent, its step
  int ds;                    // step of the slow index
  int64_t doff, coff;        // offset step, offset change of a carry
  bool lc;
  __device__ __forceinline__ RtWalk(bool lc_, int n, uint64_t mag_n, int B, uint64_t mag_B, int64_t s_line,
                                    int64_t s_b)
      : lc(lc_) {
    const int tid = (int)threadIdx.x, step = (int)blockDim.x;
    fext = lc ? n : B;
    const uint64_t mag = lc ? mag_n : mag_B;
    const int64_t sf = lc ? s_line : s_b, ss = lc ? s_b : s_line;
    const int s0 = (int)fdiv((uint32_t)tid, mag);
    f = tid - s0 * fext;
    ds = (int)fdiv((uint32_t)step, mag);
    df = step - ds * fext;
    l = lc ? s0 : f;
    i = lc ? f : s0;
    off = (int64_t)f * sf + (int64_t)s0 * ss;
    doff = (int64_t)df * sf + (int64_t)ds * ss;
    coff = ss - (int64_t)fext * sf;
  }
  __device__ __forceinline__ void next() {
    f += df;
    off += doff;
    int s = (lc ? l : i) + ds;
    if (f >= fext) {
      f -= fext;
      off += coff;
      ++s;
    }
    l = lc ? s : f;
    i = lc ? f : s;
  }
};

template <typename T>
__device__ __forceinline__ T rt_get(const __attribute__((address_space(1))) T* p, int64_t i) {
  return p[i];
}
template <typename T>
__device__ __forceinline__ cpx<T> rt_get(const __attribute__((address_space(1))) cpx<T>* p, int64_t i) {
  return cpx<T>{p[i].x, p[i].y};
}
template <typename T>
__device__ __forceinline__ void rt_set(__attribute__((address_space(1))) T* p, int64_t i, T v) {
  p[i] = v;
}
template <typename T>
__device__ __forceinline__ void rt_set(__attribute__((address_space(1))) cpx<T>* p, int64_t i, cpx<T> v) {
  p[i].x = v.x;
  p[i].y = v.y;
}

// Input of the tile's lines (one component): put(l, i, value) for every element, UN loads
// of a thread in flight.
template <int UN, typename E, class Put>
__device__ __forceinline__ void rt_load_n(const PassDesc& d, const void* in, int comp, const TileIdx& ti,
                                          const Put& put) {
  const auto* p = gptr<E>(in) + ((int64_t)comp * d.in_s_comp + (int64_t)ti.c * d.in_s_c + (int64_t)ti.b0 * d.in_s_b);
  RtWalk w(d.in_s_line == 1, d.in_n, d.mag_in, d.B, d.mag_B, d.in_s_line, d.in_s_b);
  const int n = d.in_n, nl = ti.nl;
  while (w.lc ? w.l < nl : w.i < n) {
    E v[UN];
    int ll[UN], ii[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      ll[u] = w.l < nl && w.i < n ? w.l : -1;
      ii[u] = w.i;
      v[u] = E{};
      if (ll[u] >= 0) v[u] = rt_get(p, w.off);
      w.next();
    }
#pragma unroll
    for (int u = 0; u < UN; ++u)
      if (ll[u] >= 0) put(ll[u], ii[u], v[u]);
  }
}

// Straight-line code runs about as fast as the instruction cache fills from L2 the first
// time (some 100 ns per 64 bytes), and every launch starts with it empty: a tile with at
// most one element per thread takes the short loop.
template <typename E, class Put>
__device__ __forceinline__ void rt_load(const PassDesc& d, const void* in, int comp, const TileIdx& ti, const Put& put) {
  if (d.B * d.in_n <= (int)blockDim.x) rt_load_n<1, E>(d, in, comp, ti, put);
  else rt_load_n<8, E>(d, in, comp, ti, put);
}

// Output of the tile's lines (one component): get(l, j) of every element, with the output
// conventions of the batch axes if FIX (see store_tile).
template <int UN, bool FIX, typename E, class Get>
__device__ __forceinline__ void rt_store_n(const PassDesc& d, void* out, int comp, const TileIdx& ti, const Get& get) {
  auto* p = (__attribute__((address_space(1))) E*)(out) +
            ((int64_t)comp * d.out_s_comp + (int64_t)ti.c * d.out_s_c + (int64_t)ti.b0 * d.out_s_b);
  RtWalk w(d.out_s_line == 1, d.out_n, d.mag_out, d.B, d.mag_B, d.out_s_line, d.out_s_b);
  const int n = d.out_n, nl = ti.nl;
  const Fixup& fx = d.fix;
  bool czero = false, cdup = false;
  if (FIX) {
    czero = (fx.c_zero_lo && ti.c == 0) || (fx.c_zero_hi && ti.c == fx.c_last);
    cdup = fx.c_dup && ti.c == 0;
  }
  while (w.lc ? w.l < nl : w.i < n) {
    E v[UN];
    int ll[UN];
    int64_t oo[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      ll[u] = w.l < nl && w.i < n ? w.l : -1;
      oo[u] = w.off;
      v[u] = E{};
      if (ll[u] >= 0) v[u] = get(w.l, w.i);
      w.next();
    }
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      if (ll[u] < 0) continue;
      if (FIX) {
        const int b = ti.b0 + ll[u];
        if (czero || (fx.b_zero_lo && b == 0) || (fx.b_zero_hi && b == fx.b_last)) v[u] = E{};
        const bool bdup = fx.b_dup && b == 0;
        if (bdup) rt_set(p, oo[u] + (int64_t)fx.b_last * d.out_s_b, v[u]);
        if (cdup) {
          rt_set(p, oo[u] + (int64_t)fx.c_last * d.out_s_c, v[u]);
          if (bdup) rt_set(p, oo[u] + (int64_t)fx.b_last * d.out_s_b + (int64_t)fx.c_last * d.out_s_c, v[u]);
        }
      }
      rt_set(p, oo[u], v[u]);
    }
  }
}

template <bool FIX, typename E, class Get>
__device__ __forceinline__ void rt_store(const PassDesc& d, void* out, int comp, const TileIdx& ti, const Get& get) {
  if (d.B * d.out_n <= (int)blockDim.x) rt_store_n<1, FIX, E>(d, out, comp, ti, get);
  else rt_store_n<4, FIX, E>(d, out, comp, ti, get);
}

// f(line, slot) over the F x M slots of a tile (m = slot of the line).
template <class Fn>
__device__ __forceinline__ void rt_slots(int F, int M, uint32_t mM, const Fn& f) {
  const int total = F * M;
  for (int e = (int)threadIdx.x; e < total; e += (int)blockDim.x) {
    const int line = rt_div(e, mM);
    f(line, e - line * M);
  }
}

// Real-to-real line pairs: the FFT input of a pair from its samples x_i = (line 2f, line
// 2f + 1) at x[f xs + i], by the form (R2RForm).
struct R2RLine {
  R2R r;
  int n;  // samples of a line
  // sample index of input p; -1 outside the line
  __device__ __forceinline__ int index(int p) const {
    const int j = r.in_rev ? r.in_base - p : p - r.in_base;
    return p >= r.plo && p <= r.phi && j >= 0 && j < n ? j : -1;
  }
};
template <typename T>
__device__ __forceinline__ cpx<T> rt_at(const cpx<T>* x, int j) {
  return j >= 0 ? x[j] : cpx<T>{T(0), T(0)};
}
template <typename T>
__device__ __forceinline__ cpx<T> rt_r2r_slot(const R2RLine& g, GTab<T> tw, const cpx<T>* x, int m) {
  const R2R& r = g.r;
  const int nh = r.nh;
  if (r.half == R2R_II) {
    const bool odd = 2 * m >= nh;  // the odd samples, backwards, follow the even ones
    const cpx<T> a = rt_at(x, g.index(odd ? 2 * (nh - m) - 1 : 2 * m));
    const T c = odd && r.sin ? T(-1) : T(1);
    return {c * a.x, c * a.y};
  }
  if (r.half == R2R_III) {
    const int p = r.sin ? nh - m : m;
    const cpx<T> a = rt_at(x, g.index(p)), b = rt_at(x, g.index(nh - p));
    const cpx<T> w = twid<T>(tw, m);
    return cmul(cpx<T>{a.x + b.y, a.y - b.x}, cpx<T>{w.x, -w.y});
  }
  // symmetric extension of period 2 nh: mirrored sample, weight, pre-twiddle
  const T eps = r.b2 ? T(-1) : T(1);          // wrap factor of a full period
  const T sigma = r.sin ? -eps : eps;          // sign of the mirrored sample
  const bool hi = r.a2 ? m >= nh : m > nh;
  const int p = hi ? 2 * nh - r.a2 - m : m;
  T c = hi ? sigma : T(1);
  if (!r.a2) {
    if (m == 0) c = T(1) + sigma * eps;
    if (m == nh) c = T(1) + sigma;
  }
  c *= T(p == r.plo ? r.wlo : (p == r.phi ? r.whi : 2)) * T(0.5);
  const cpx<T> a = rt_at(x, g.index(p));
  cpx<T> z = {c * a.x, c * a.y};
  if (r.b2) z = cmul(z, twid<T>(tw, 2 * m));
  return z;
}

// Output j of tile line l from the FFT lines of a real-to-real tile.
template <typename T>
__device__ __forceinline__ T rt_r2r_out(const cpx<T>* buf, int ls, const R2R& r, GTab<T> tw, int l, int j) {
  const int q = r.out_rev ? r.out_base - j : j + r.out_base;
  if (q < r.qlo || q > r.qhi) return T(0);  // outside: the coefficient is 0
  const cpx<T>* Z = buf + (l >> 1) * ls;
  const bool odd = l & 1;
  if (r.half == R2R_II) {
    // the two lines' spectra V1 = (Z_k + conj Z_{-k}) / 2, V2 = (Z_k - conj Z_{-k}) / 2i
    const int k = r.sin ? r.nh - q : q;
    const cpx<T> a = Z[pad16(k)], b = Z[pad16(k ? r.nh - k : 0)];
    const cpx<T> w = twid<T>(tw, k);
    return odd ? w.x * (a.y + b.y) + w.y * (a.x - b.x) : w.x * (a.x + b.x) - w.y * (a.y - b.y);
  }
  if (r.half == R2R_III) {
    // sample n = q / 2 or nh - (q + 1) / 2 of the inverse DFT, slot -n of the forward one
    const int n = (q & 1) ? r.nh - ((q + 1) >> 1) : q >> 1;
    const cpx<T> y = Z[pad16(n ? r.nh - n : 0)];
    const T v = odd ? y.y : y.x;
    return r.sin && (q & 1) ? -v : v;
  }
  cpx<T> y = Z[pad16(q)];
  if (r.a2) y = cmul(y, twid<T>(tw, 2 * q + r.b2));  // exp(-i pi a (q + b) / nh), a = 1/2
  return r.sin ? (odd ? y.x : -y.y) : (odd ? y.y : y.x);
}

// One tile.  KIND K_ANY reads the kind from the descriptor.  LDS: buffer a at 0, buffer b
// (which first holds the raw lines of the kinds that gather) at raw_off; raw_off = 0: buffer
// a alone (three components, rt_radix_in_place).
template <typename T, int KIND>
__device__ __forceinline__ void rt_tile(const PassDesc& d, const void* in, void* out, int tile, char* smem) {
  const int kind = KIND == K_ANY ? d.kind : KIND;
  const TileIdx ti = tile_index(d, tile);
  const int nl = ti.nl, M = d.M, ls = fft_line_stride(M);
  const int n = d.in_n, rsp = n | 1;  // raw line stride
  cpx<T>* a = reinterpret_cast<cpx<T>*>(smem);
  cpx<T>* b = reinterpret_cast<cpx<T>*>(smem + d.raw_off);
  const GTab<T> tw = gptr<cpx<T>>(d.tw);
  const int gather = gather_of(kind);
  const bool curl = kind == K_F_CURL;
  const int pairs = gather == G_CPLX ? (curl ? 3 * nl : nl) : (nl + 1) / 2;  // FFT lines
  const cpx<T> zero = {T(0), T(0)};
  T* ar = reinterpret_cast<T*>(a);
  T* br = reinterpret_cast<T*>(b);
  // conjugated on the way in and out: the inverse transforms
  const bool inv = kind == K_C2C_I;

  // ---- FFT input into a
  if (gather == G_CPLX || gather == G_REAL2) {
    if (d.n_data < M) {  // zero padding
      const int z = M - d.n_data;
      rt_slots(pairs, z, d.rt_mz, [&](int f, int m) { a[f * ls + pad16(d.n_data + m)] = zero; });
    }
    if (gather == G_CPLX) {
      const int q0 = curl ? 0 : ti.comp, nq = curl ? 3 : 1;
      for (int q = 0; q < nq; ++q)
        rt_load<cpx<T>>(d, in, q0 + q, ti, [&](int l, int i, cpx<T> v) {
          if (i < d.n_data) a[(q * nl + l) * ls + pad16(i)] = cpx<T>{v.x, inv ? -v.y : v.y};
        });
    } else {
      rt_load<T>(d, in, ti.comp, ti, [&](int l, int i, T v) {
        if (i >= d.n_data) return;
        const int at = 2 * ((l >> 1) * ls + pad16(i)) + (l & 1);
        ar[at] = v;
        if (l + 1 == nl && !(l & 1)) ar[at + 1] = T(0);  // no second line
      });
    }
  } else if (gather == G_HERM2) {
    rt_load<cpx<T>>(d, in, ti.comp, ti, [&](int l, int i, cpx<T> v) { b[l * rsp + i] = v; });
    __syncthreads();
    // conj(X1 + i X2) of the pair's Hermitian spectra
    rt_slots(pairs, M, d.rt_mM, [&](int f, int m) {
      const bool hi = 2 * m > M;
      const int mm = hi ? M - m : m;
      cpx<T> x1 = b[2 * f * rsp + mm], x2 = 2 * f + 1 < nl ? b[(2 * f + 1) * rsp + mm] : zero;
      if (mm == 0 || 2 * mm == M) {  // modes that are real for real data
        x1.y = T(0);
        x2.y = T(0);
      }
      a[f * ls + pad16(m)] = hi ? cpx<T>{x1.x + x2.y, x1.y - x2.x} : cpx<T>{x1.x - x2.y, -x1.y - x2.x};
    });
  } else {
    rt_load<T>(d, in, ti.comp, ti, [&](int l, int i, T v) {
      const int at = 2 * ((l >> 1) * rsp + i) + (l & 1);
      br[at] = v;
      if (l + 1 == nl && !(l & 1)) br[at + 1] = T(0);
    });
    __syncthreads();
    const R2RLine g{d.r2r, n};
    rt_slots(pairs, M, d.rt_mM, [&](int f, int m) { a[f * ls + pad16(m)] = rt_r2r_slot<T>(g, tw, b + f * rsp, m); });
  }
  const bool one = KIND == K_F_CURL && d.raw_off == 0;  // in place (uniform)
  cpx<T>* z = one ? rt_fft<T, KIND == K_F_CURL>(d, a, b, ls, pairs) : rt_fft<T>(d, a, b, ls, pairs);

  // ---- fused: times the Green's spectrum (and the curl), inverse transform
  const bool fused = fused_of(kind);
  if (fused) {
    cpx<T>* y = z == a ? b : a;  // the free buffer
    const auto* G = gptr<T>(d.g.G);
    const int64_t gc = (int64_t)fold_index(ti.c, d.g.fold_c) * d.g.F_b;
    auto row = [&](int l) { return (gc + fold_index(ti.b0 + l, d.g.fold_b)) * d.g.F_line; };
    if (kind == K_F_C2C) {
      rt_slots(nl, M, d.rt_mM, [&](int l, int k) {
        const T g = G[row(l) + fold_index(k, d.g.fold_line)];
        const cpx<T> v = z[l * ls + pad16(k)];
        z[l * ls + pad16(k)] = cpx<T>{g * v.x, -g * v.y};
      });
    } else if (kind == K_F_R2C) {
      // the two packed lines have their own rows: with X1, X2 the lines' spectra, the
      // conjugate of g0 X1 + i g1 X2
      rt_slots(pairs, M, d.rt_mM, [&](int f, int k) {
        const int l1 = min(2 * f + 1, nl - 1), kk = fold_index(k, d.g.fold_line);
        const T g0 = G[row(2 * f) + kk], g1 = G[row(l1) + kk];
        const cpx<T> zk = z[f * ls + pad16(k)], zm = z[f * ls + pad16(k ? M - k : 0)];
        const cpx<T> x1 = {T(0.5) * (zk.x + zm.x), T(0.5) * (zk.y - zm.y)};
        const cpx<T> x2 = {T(0.5) * (zk.y + zm.y), T(-0.5) * (zk.x - zm.x)};
        y[f * ls + pad16(k)] = cpx<T>{g0 * x1.x - g1 * x2.y, -(g0 * x1.y + g1 * x2.x)};
      });
      z = y;
    } else if (curl) {
      T wc, mc;
      curl_factor<T>(d.g.csym, curl_wave<T>(ti.c, d.g.dtab_c), wc, mc);
      rt_slots(nl, M, d.rt_mM, [&](int l, int k) {
        const T g = G[row(l) + fold_index(k, d.g.fold_line)];
        const T wl = curl_wave<T>(k, d.g.dtab_line);
        T wb, mb;
        curl_factor<T>(d.g.csym_b, curl_wave<T>(ti.b0 + l, d.g.dtab_b), wb, mb);
        const T wx = d.g.axis_line == 0 ? wl : (d.g.axis_b == 0 ? wb : wc);
        const T wy = d.g.axis_line == 1 ? wl : (d.g.axis_b == 1 ? wb : wc);
        const T wz = d.g.axis_line == 2 ? wl : (d.g.axis_b == 2 ? wb : wc);
        const int o = l * ls + pad16(k), s = nl * ls;
        cpx<T> fx = z[o], fy = z[o + s], fz = z[o + 2 * s];
        curl_point<T>(g, wx, wy, wz, d.g.axis_c, mc, d.g.axis_b, mb, fx, fy, fz);
        z[o] = cpx<T>{fx.x, -fx.y};
        z[o + s] = cpx<T>{fy.x, -fy.y};
        z[o + 2 * s] = cpx<T>{fz.x, -fz.y};
      });
    } else {  // K_F_R2R: the spectrum as sample pairs, then the inverse's FFT input over z
      const int ns = d.spec_n, ssp = ns | 1;
      T* yr = reinterpret_cast<T*>(y);
      const int lines = 2 * pairs;
      rt_slots(lines, ns, d.rt_msp, [&](int l, int j) {
        T v = T(0);
        if (l < nl) v = G[row(l) + fold_index(j, d.g.fold_line)] * rt_r2r_out<T>(z, ls, d.r2r, tw, l, j);
        yr[2 * ((l >> 1) * ssp + j) + (l & 1)] = v;
      });
      __syncthreads();
      const R2RLine g{d.r2r2, ns};
      rt_slots(pairs, M, d.rt_mM, [&](int f, int m) { z[f * ls + pad16(m)] = rt_r2r_slot<T>(g, tw, y + f * ssp, m); });
    }
    z = one ? rt_fft<T, KIND == K_F_CURL>(d, z, z, ls, pairs) : rt_fft<T>(d, z, z == a ? b : a, ls, pairs);
  }

  // ---- output
  if (curl) {
    for (int q = 0; q < 3; ++q)
      rt_store<false, cpx<T>>(d, out, q, ti, [&](int l, int j) {
        const cpx<T> v = z[(q * nl + l) * ls + pad16(j < M ? j : j - M)];
        return cpx<T>{v.x, -v.y};
      });
  } else if (kind == K_C2C_F || kind == K_C2C_I || kind == K_F_C2C) {
    const bool conj = kind != K_C2C_F;
    rt_store<false, cpx<T>>(d, out, ti.comp, ti, [&](int l, int j) {
      const cpx<T> v = z[l * ls + pad16(j < M ? j : j - M)];
      return cpx<T>{v.x, conj ? -v.y : v.y};
    });
  } else if (kind == K_R2C) {
    rt_store<false, cpx<T>>(d, out, ti.comp, ti, [&](int l, int k) {
      const cpx<T>* x = z + (l >> 1) * ls;
      const cpx<T> zk = x[pad16(k)], zm = x[pad16(k ? M - k : 0)];
      if (l & 1) return cpx<T>{T(0.5) * (zk.y + zm.y), T(-0.5) * (zk.x - zm.x)};
      return cpx<T>{T(0.5) * (zk.x + zm.x), T(0.5) * (zk.y - zm.y)};
    });
  } else {
    auto val = [&](int l, int j) {
      if (kind == K_R2R || kind == K_F_R2R) return rt_r2r_out<T>(z, ls, fused ? d.r2r2 : d.r2r, tw, l, j);
      const cpx<T> v = z[(l >> 1) * ls + pad16(j < M ? j : j - M)];
      return (l & 1) ? -v.y : v.x;  // conjugated: C2R and the fused R2C
    };
    if (d.out_cplx) {
      // a real-to-real spectrum handed on as complex values with a zero imaginary part
      rt_store<false, cpx<T>>(d, out, ti.comp, ti, [&](int l, int j) { return cpx<T>{val(l, j), T(0)}; });
    } else if (d.has_fix) {
      rt_store<true, T>(d, out, ti.comp, ti, val);
    } else {
      rt_store<false, T>(d, out, ti.comp, ti, val);
    }
  }
}

// One tile per workgroup (of rt_threads threads), in the XCD-aware order.
template <typename T, int KIND>
__global__ __launch_bounds__(kRtThreads) void rt_kernel(const PassDesc* __restrict__ dp, const void* in, void* out) {
  extern __shared__ __align__(16) char smem[];
  const PassDesc& d = component<T, KIND>(dp, in, out);
  for (int k = 0;; ++k) {
    const int tile = xcd_tile(blockIdx.x, gridDim.x, k, d.tiles);
    if (tile < 0) return;
    if (k > 0) __syncthreads();  // the previous tile's LDS reads are finished
    rt_tile<T, KIND>(d, in, out, tile, smem);
  }
}

// Batched form: tiles of many descriptors of one length class in one launch;
// prefix[i] = first tile of descriptor i, prefix[n] = total.
template <typename T, int MC>
__global__ __launch_bounds__(kThreads) void pass_kernel_batched(const PassDesc* __restrict__ ds,
                                                                const int* __restrict__ prefix,
                                                                int n) {
  extern __shared__ __align__(16) char smem[];
  const int tile = blockIdx.x;
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (prefix[mid] <= tile) lo = mid;
    else hi = mid - 1;
  }
  const PassDesc& d = ds[lo];
  if constexpr (MC > 1) run_tile<T, MC>(d, d.in, d.out, tile - prefix[lo], smem);
  else rt_tile<T, K_ANY>(d, d.in, d.out, tile - prefix[lo], smem);
}

}  // namespace fm
