// Transform passes of the split-operator step (templates; instantiated per N).
//
// One step of an FFT kinetic term (Sec. 2, eqs. HK1-HK3, with the symmetric
// split h F^-1[e^{-dt T} F[h psi]]) is carried out as passes over HBM, each
// reading and writing the state once:
//
//   plane pass  (x2-x3 plane in LDS): inverse x2,x3 -> x h^2 -> forward x3,x2
//   row pass    (x3 rows in LDS):     inverse x3 -> x h^2 -> forward x3
//   column pass (TC contiguous x3 columns along x1 or x2 in LDS):
//               forward -> x e^{-dt T(k)}/N^3 -> inverse
//
// Mode bits (common.h) select which of these pieces a launch performs, so
// the same kernels also start and end a chunk (x h instead of x h^2) and run
// plain forward/inverse transforms.
#pragma once

#include "fft_core.h"

namespace qf {

template <int N> __host__ __device__ constexpr int plane_threads() {
  int t = (N * N / 16 + 63) / 64 * 64;
  return t < 64 ? 64 : (t > 1024 ? 1024 : t);
}
// Row pitch of the plane in LDS (elements).  LDS serves a wave's 64 accesses
// in 128-byte passes (16 lanes of 8-byte or 8 lanes of 16-byte elements);
// distinct elements of one pass that share (index mod 128/element size)
// serialise.  The pitches below minimise those repeats over every access of
// the steady plane pass (both row-stage lane maps, the stride-R Stockham
// writes) for the sizes where the padded length alone leaves them; found with
// a model of that access pattern and checked against the LDS bank-conflict
// counter at N = 128 (7x fewer conflict cycles).
template <typename T, int N> __host__ __device__ constexpr int plane_pitch() {
  if constexpr (sizeof(T) == 4) {
    switch (N) {
      case 18: return 25; case 24: return 35; case 32: return 36; case 40: return 44; case 48: return 51;
      case 50: return 56; case 64: return 72; case 80: return 85; case 96: return 108; case 128: return 136;
      default: return padded_len(N);
    }
  } else {
    switch (N) {
      case 12: return 19; case 24: return 27; case 32: return 36; case 40: return 45; case 48: return 51;
      case 80: return 85;
      default: return padded_len(N);
    }
  }
}
template <typename T, int N> __host__ __device__ constexpr size_t plane_lds_t() {
  return (size_t)(N * plane_pitch<T, N>() + tw_total<PKT<T>, N>()) * sizeof(C<T>);
}
template <typename T, int N> __host__ __device__ constexpr bool plane_fits() {
  return plane_lds_t<T, N>() <= 160 * 1024 && N * N <= 16 * 1024;
}
template <typename T, int N> __host__ __device__ constexpr int row_block_t() { return row_block(N, sizeof(T) == 8); }
template <typename T, int N> __host__ __device__ constexpr size_t row_lds_t() {
  return (size_t)(row_block_t<T, N>() * padded_len(N) + tw_total<PKT<T>, N>()) * sizeof(C<T>);
}
template <typename T> __host__ __device__ constexpr int col_tile_t() { return col_tile(sizeof(T) == 8); }
template <typename T, int N> __host__ __device__ constexpr size_t col_lds_t() {
  return (size_t)(N * (col_tile_t<T>() + 1) + tw_total<PKT<T>, N>()) * sizeof(C<T>);
}

// psi * f where f is real (T) or complex (C<T>) at site `off`.
template <typename T>
__device__ __forceinline__ C<T> vmul_t(C<T> v, const void *f, int vcomplex, size_t off) {
  if (vcomplex) return cmul(v, ((const C<T> *)f)[off]);
  return cscale(v, ((const T *)f)[off]);
}

// k-space factor at FFT indices (i1, i2, i3): e^{-dt T(k)} / N^3 for the split
// step, dt T(k) / N^3 for the A/B update (the column pass then yields dt H_K psi).
template <typename T>
__device__ __forceinline__ T kin_factor_t(const PassDesc &d, int i1, int i2, int i3) {
  const T *kt = (const T *)d.ktab;
  if (d.kin == KIN_REL) {
    const T p2 = kt[i1] + kt[i2] + kt[i3];
    const T m = (T)d.m;
    if constexpr (sizeof(T) == 4) {
      // single-instruction sqrt, reciprocal and 2^x (about 1 ulp each).  The A/B factor is
      // dt T itself, so T = p^2 / (sqrt(p^2 + m^2) + m) avoids the cancellation; in the split
      // factor T only enters the exponent, where sqrt(p^2 + m^2) - m is off by at most
      // dt sqrt(p^2 + m^2) 2^-24 in absolute terms, and the reciprocal is saved
      const float r = __builtin_amdgcn_sqrtf(p2 + m * m);
      if (d.scheme == SCHEME_AB) return p2 * __builtin_amdgcn_rcpf(r + m) * (float)(d.dt * d.inv_n3);
      return __builtin_amdgcn_exp2f(-(float)d.dt * 1.4426950408889634f * (r - m)) * (float)d.inv_n3;
    } else {
      const T tk = p2 / (sqrt(p2 + m * m) + m);   // sqrt(p^2 + m^2) - m without cancellation
      if (d.scheme == SCHEME_AB) return tk * (T)(d.dt * d.inv_n3);
      return exp(-(T)d.dt * tk) * (T)d.inv_n3;
    }
  }
  // separable terms: the table holds t(k_j) (A/B) or e^{-dt t(k_j)} (split)
  if (d.scheme == SCHEME_AB) return (kt[i1] + kt[i2] + kt[i3]) * (T)(d.dt * d.inv_n3);
  return kt[i1] * kt[i2] * kt[i3] * (T)d.inv_n3;
}

// A/B update at one site: psi' = A psi - B x with x = dt H_K psi,
// A = (1 - dt V/2)/(1 + dt V/2), B = 1/(1 + dt V/2) (complex when V is).
template <typename T>
__device__ __forceinline__ C<T> ab_combine(C<T> p, C<T> x, const PassDesc &d, size_t off) {
  const T hdt = (T)(0.5 * d.dt);
  if (d.vcomplex) {
    const C<T> V = ((const C<T> *)d.vtab)[off];
    const T dr = fmaT(hdt, V.x, (T)1), di = hdt * V.y;
    const T den = (T)1 / fmaT(dr, dr, di * di);
    const C<T> B = mkc<T>(dr * den, -di * den);
    const C<T> A = cmul(mkc<T>(fmaT(-hdt, V.x, (T)1), -hdt * V.y), B);
    return csub(cmul(A, p), cmul(B, x));
  }
  const T V = ((const T *)d.vtab)[off];
  const T B = (T)1 / fmaT(hdt, V, (T)1);
  const T A = fmaT(-hdt, V, (T)1) * B;
  return mkc<T>(fmaT(A, p.x, -(B * x.x)), fmaT(A, p.y, -(B * x.y)));
}

template <typename T, int N, int NT>
__device__ __forceinline__ void load_tw(C<T> *tw, const PassDesc &d) {
  fill_twiddles<T, PKT<T>, N, NT>(tw, (const C<T> *)d.tw);
}

// ------------------------------------------------------------- plane pass

// Steady-state plane pass (inverse x2,x3 -> x h^2 -> forward x3,x2) with the
// first stage read from HBM, the last stage written to HBM, and the inverse-x3
// last stage, the potential factor and the forward-x3 first stage fused in
// registers.  The inverse uses the radix plan, the forward its reverse.
template <typename T, bool VC> struct FacT { using type = T; };
template <typename T> struct FacT<T, true> { using type = C<T>; };

//
// AB: the steady pass of the A/B update instead: g is alt (holding the
// transformed dt H_K psi), and the fused middle stage replaces the h^2
// multiply by psi' = A psi - B (dt H_K psi), reading psi and writing psi' at
// gp; the forward transform of psi' goes back to alt.
template <typename T, int N, int NT, int P, bool VC, bool AB = false>
__device__ __forceinline__ void plane_steady(C<T> *pl, const C<T> *tw, C<T> *g, const PassDesc &d, size_t voff,
                                             C<T> *gp = nullptr) {
  using Rows = RowsGeo<N, P>;
  using Cols = ColsGeo<N, P>;
  constexpr RPlan PL = plan_of<PKT<T>, N, false>();
  constexpr int M = PL.n - 1;
  // potential factors of the fused middle stage, fetched before any transform
  // work so their latency overlaps the inverse transforms
  constexpr int RMID = PL.r[M];
  using SMID = SG<Rows, N, RMID, NT>;
  using F = typename FacT<T, VC>::type;
  F hq[AB ? 1 : SMID::CAPQ][AB ? 1 : RMID];
  if constexpr (!AB) {
#pragma unroll
    for (int q = 0; q < SMID::CAPQ; ++q) {
      if (SMID::active(q)) {
        int j, b;
        SMID::jb(q, j, b);
#pragma unroll
        for (int r = 0; r < RMID; ++r) hq[q][r] = ((const F *)d.h2fac)[voff + (size_t)b * N + j + r * SMID::NR];
      }
    }
  }
  {
    constexpr int R = PL.r[0];
    C<T> v[SG<Cols, N, R, NT>::CAPQ][R];
    st_read<T, N, R, 1, true, Cols, NT, 0>(v, tw, [&](int b, int n) { return g[n * N + b]; });
    st_write<T, N, R, 1, Cols, NT>(v, [&](int b, int n, C<T> x) { pl[Cols::at(b, n)] = x; });
    __syncthreads();
  }
  lds_stages<T, PKT<T>, N, false, true, Cols, NT, 1, PL.n>(pl, tw);
  lds_stages<T, PKT<T>, N, false, true, Rows, NT, 0, M>(pl, tw);
  {
    constexpr int R = PL.r[M];
    constexpr int NSL = ns_before<PKT<T>, N, false, M>();
    using S = SG<Rows, N, R, NT>;
    C<T> v[S::CAPQ][R];
    st_read<T, N, R, NSL, true, Rows, NT, tw_off<PKT<T>, N, false, M>()>(v, tw, [&](int b, int n) { return pl[Rows::at(b, n)]; });
    __syncthreads();
#pragma unroll
    for (int q = 0; q < S::CAPQ; ++q) {
      if (S::active(q)) {
        int j, b;
        S::jb(q, j, b);
#pragma unroll
        for (int r = 0; r < R; ++r) {
          if constexpr (AB) {
            // the last inverse stage leaves element n = j + r N/R of line b in v[q][r]
            const size_t o = (size_t)b * N + j + r * S::NR;
            const C<T> y = ab_combine<T>(gp[o], v[q][r], d, voff + o);
            gp[o] = y;
            v[q][r] = y;
          } else if constexpr (VC) {
            v[q][r] = cmul(v[q][r], hq[q][r]);
          } else {
            v[q][r] = cscale(v[q][r], hq[q][r]);
          }
        }
        Dft<R, false, C<T>>::run(v[q]);
      }
    }
    st_write<T, N, R, 1, Rows, NT>(v, [&](int b, int n, C<T> x) { pl[Rows::at(b, n)] = x; });
    __syncthreads();
  }
  lds_stages<T, PKT<T>, N, true, false, Rows, NT, 1, PL.n>(pl, tw);
  lds_stages<T, PKT<T>, N, true, false, Cols, NT, 0, M>(pl, tw);
  {
    constexpr int R = plan_of<PKT<T>, N, true>().r[M];
    constexpr int NSL = ns_before<PKT<T>, N, true, M>();
    C<T> v[SG<Cols, N, R, NT>::CAPQ][R];
    st_read<T, N, R, NSL, false, Cols, NT, tw_off<PKT<T>, N, true, M>()>(v, tw, [&](int b, int n) { return pl[Cols::at(b, n)]; });
    st_write<T, N, R, NSL, Cols, NT>(v, [&](int b, int n, C<T> x) { g[n * N + b] = x; });
  }
}

// Memory row of row r of a transformed plane: r itself, or (M_SPLIT) its place in the split order of
// x2 = N1 N2 with N2, N1 the plan's radices (the inverse takes N2 first and N1 second, the forward of
// the steady passes, on the reversed plan, N1 first: the split-x2 passes with these factors do the
// operations of the plane pass).
template <typename T, int N>
__device__ __forceinline__ int split_row(int r, uint32_t mode) {
  constexpr RPlan PL = plan_of<PKT<T>, N, false>();
  if constexpr (PL.n == 2) {
    constexpr int N2 = PL.r[0], N1 = PL.r[1];
    if (mode & M_SPLIT) return N2 * (r % N1) + r / N1;
  }
  return r;
}

// A/B update on one plane.  Chunk start (M_FWD | M_ALT): psi -> F3 F2 -> alt.
// Steady (M_INV | M_COMB | M_FWD | M_ALT): alt -> F2^-1 F3^-1 gives dt H_K psi,
// combined with psi into psi' (written to psi), then F3 F2 psi' -> alt.
// Chunk end (M_INV | M_COMB): the same without the forward transform.
template <typename T, int N, int NT, int P>
__device__ __forceinline__ void plane_ab(C<T> *pl, const C<T> *tw, const PassDesc &d, uint32_t mode, int s, int i1) {
  constexpr size_t N2 = (size_t)N * N;
  const size_t base = ((size_t)s * N + i1) * N2;
  C<T> *gp = (C<T> *)d.psi + base;
  C<T> *ga = (C<T> *)d.alt + base;
  const size_t voff = (size_t)i1 * N2;
  const bool comb = (mode & M_COMB) != 0;
  const C<T> *src = comb ? ga : gp;
  for (int idx = threadIdx.x; idx < N * N; idx += NT) {
    const int r = idx / N, c = idx - r * N;
    pl[r * P + padn(c)] = src[(comb ? split_row<T, N>(r, mode) : r) * N + c];
  }
  __syncthreads();
  using Rows = RowsGeo<N, P>;
  using Cols = ColsGeo<N, P>;
  if (mode & M_INV) {
    fft_lines_t<T, PKT<T>, N, true, Cols, NT>(pl, tw);
    fft_lines_t<T, PKT<T>, N, true, Rows, NT>(pl, tw);
  }
  if (comb) {
    for (int idx = threadIdx.x; idx < N * N; idx += NT) {
      const int r = idx / N, c = idx - r * N;
      const int a = r * P + padn(c);
      const C<T> o = ab_combine<T>(gp[idx], pl[a], d, voff + idx);
      gp[idx] = o;
      pl[a] = o;
    }
    __syncthreads();
  }
  if (mode & M_FWD) {
    fft_lines_t<T, PKT<T>, N, false, Rows, NT>(pl, tw);
    fft_lines_t<T, PKT<T>, N, false, Cols, NT>(pl, tw);
    C<T> *dst = (mode & M_ALT) ? ga : gp;
    for (int idx = threadIdx.x; idx < N * N; idx += NT) {
      const int r = idx / N, c = idx - r * N;
      dst[split_row<T, N>(r, mode) * N + c] = pl[r * P + padn(c)];
    }
  }
}

// Tile = one x2-x3 plane (state s, i1).  NT = threads of the block (the
// plane kernel of a single size uses plane_threads<N>(); a multi-size kernel
// runs every size with its own, larger, block).
template <typename T, int N, int NT>
__device__ __forceinline__ void plane_body(const LaunchList &L, int e, int t, unsigned char *smem) {
  constexpr int P = plane_pitch<T, N>();
  const PassDesc &d = *(const PassDesc *)L.descp[e];
  const uint32_t mode = L.mode[e];
  const int s = t / N, i1 = t - s * N;
  C<T> *pl = (C<T> *)smem;
  C<T> *tw = pl + N * P;
  load_tw<T, N, NT>(tw, d);
  constexpr size_t N2 = (size_t)N * N;
  C<T> *g = (C<T> *)d.psi + ((size_t)s * N + i1) * N2;
  const size_t voff = (size_t)i1 * N2;
  if (mode & (M_COMB | M_ALT)) {
    if constexpr (plan_of<PKT<T>, N, false>().n >= 2) {
      if (mode == (M_INV | M_COMB | M_FWD | M_ALT)) {
        __syncthreads();
        C<T> *ga = (C<T> *)d.alt + ((size_t)s * N + i1) * N2;
        plane_steady<T, N, NT, P, false, true>(pl, tw, ga, d, voff, g);
        return;
      }
    }
    plane_ab<T, N, NT, P>(pl, tw, d, mode, s, i1);
    return;
  }
  if constexpr (plan_of<PKT<T>, N, false>().n >= 2) {
    if (mode == (M_INV | M_MID | M_FWD)) {
      __syncthreads();
      if (d.vcomplex) plane_steady<T, N, NT, P, true>(pl, tw, g, d, voff);
      else plane_steady<T, N, NT, P, false>(pl, tw, g, d, voff);
      return;
    }
  }
  for (int idx = threadIdx.x; idx < N * N; idx += NT) {
    const int r = idx / N, c = idx - r * N;
    C<T> v = g[((mode & M_INV) ? split_row<T, N>(r, mode) : r) * N + c];
    if (mode & M_PRE) v = vmul_t<T>(v, d.hfac, d.vcomplex, voff + idx);
    pl[r * P + padn(c)] = v;
  }
  __syncthreads();
  using Rows = RowsGeo<N, P>;
  using Cols = ColsGeo<N, P>;
  if (mode & M_INV) {
    fft_lines_t<T, PKT<T>, N, true, Cols, NT>(pl, tw);
    fft_lines_t<T, PKT<T>, N, true, Rows, NT>(pl, tw);
  }
  if (mode & M_MID) {
    for (int idx = threadIdx.x; idx < N * N; idx += NT) {
      const int r = idx / N, c = idx - r * N;
      const int a = r * P + padn(c);
      pl[a] = vmul_t<T>(pl[a], d.h2fac, d.vcomplex, voff + idx);
    }
    __syncthreads();
  }
  if (mode & M_FWD) {
    fft_lines_t<T, PKT<T>, N, false, Rows, NT>(pl, tw);
    fft_lines_t<T, PKT<T>, N, false, Cols, NT>(pl, tw);
  }
  for (int idx = threadIdx.x; idx < N * N; idx += NT) {
    const int r = idx / N, c = idx - r * N;
    C<T> v = pl[r * P + padn(c)];
    if (mode & M_POST) v = vmul_t<T>(v, d.hfac, d.vcomplex, voff + idx);
    g[((mode & M_FWD) ? split_row<T, N>(r, mode) : r) * N + c] = v;
  }
}

template <typename T, int N>
__global__ void __launch_bounds__(plane_threads<N>()) k_plane_t(const LaunchList L) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int e = find_entry(L, blockIdx.x);
  plane_body<T, N, plane_threads<N>()>(L, e, blockIdx.x - L.tile_start[e], smem);
}

// --------------------------------------------------------------- row pass

// Site offset within its state of element x (< RB N) of a row tile whose first row starts at
// offset voff0 (< N^3) of its state.  Where a tile spans at most two states (RB N <= N^3, all
// N >= 16) the offset wraps at most once and one compare replaces a 64-bit remainder per
// element.
template <typename T, int N>
__device__ __forceinline__ size_t row_site(size_t voff0, size_t x) {
  constexpr size_t N3 = (size_t)N * N * N;
  const size_t o = voff0 + x;
  if constexpr ((size_t)row_block_t<T, N>() * N <= N3) return o >= N3 ? o - N3 : o;
  else return o % N3;
}

// Steady-state row pass (inverse x3 -> x h^2 -> forward x3): first stage from
// HBM, last stage to HBM, middle stages fused around the potential factor.
template <typename T, int N, int NT, int RB, int P, bool AB = false>
__device__ __forceinline__ void row_steady(C<T> *buf, const C<T> *tw, C<T> *g, const PassDesc &d, size_t voff0,
                                           int nrows, C<T> *gp = nullptr) {
  using Rows = RowsGeo<RB, P>;
  constexpr RPlan PL = plan_of<PKT<T>, N, false>();
  constexpr int M = PL.n - 1;
  constexpr size_t N3 = (size_t)N * N * N;
  const C<T> zero = mkc<T>(0, 0);
  // complex64: the potential factors of the fused middle stage are fetched before the first
  // stage, so that their latency overlaps the inverse transform (at most one largest-radix
  // butterfly's worth of values per lane; complex128 keeps its registers for the transform)
  constexpr bool PRE = !AB && sizeof(T) == 4;
  using SMID = SG<Rows, N, PL.r[M], NT>;
  C<T> hq[PRE ? SMID::CAPQ : 1][PRE ? PL.r[M] : 1];
  if constexpr (PRE) {
    const bool vc = d.vcomplex != 0;
#pragma unroll
    for (int q = 0; q < SMID::CAPQ; ++q) {
      if (SMID::active(q)) {
        int j, b;
        SMID::jb(q, j, b);
#pragma unroll
        for (int r = 0; r < PL.r[M]; ++r) {
          hq[q][r] = zero;
          if (b < nrows) {
            const size_t s = row_site<T, N>(voff0, (size_t)b * N + j + r * SMID::NR);
            hq[q][r] = vc ? ((const C<T> *)d.h2fac)[s] : mkc<T>(((const T *)d.h2fac)[s], 0);
          }
        }
      }
    }
  }
  {
    constexpr int R = PL.r[0];
    C<T> v[SG<Rows, N, R, NT>::CAPQ][R];
    st_read<T, N, R, 1, true, Rows, NT, 0>(v, tw, [&](int b, int n) { return b < nrows ? g[b * N + n] : zero; });
    st_write<T, N, R, 1, Rows, NT>(v, [&](int b, int n, C<T> x) { buf[Rows::at(b, n)] = x; });
    __syncthreads();
  }
  lds_stages<T, PKT<T>, N, false, true, Rows, NT, 1, M>(buf, tw);
  {
    constexpr int R = PL.r[M];
    constexpr int NSL = ns_before<PKT<T>, N, false, M>();
    using SS = SG<Rows, N, R, NT>;
    C<T> v[SS::CAPQ][R];
    st_read<T, N, R, NSL, true, Rows, NT, tw_off<PKT<T>, N, false, M>()>(v, tw, [&](int b, int n) { return buf[Rows::at(b, n)]; });
    __syncthreads();
#pragma unroll
    for (int q = 0; q < SS::CAPQ; ++q) {
      if (SS::active(q)) {
        int j, b;
        SS::jb(q, j, b);
        if (b < nrows) {
#pragma unroll
          for (int r = 0; r < R; ++r) {
            if constexpr (AB) {
              // A/B update (g is alt): psi' = A psi - B (dt H_K psi), psi read and written at gp
              const size_t o = (size_t)b * N + j + r * SS::NR;
              const C<T> y = ab_combine<T>(gp[o], v[q][r], d, row_site<T, N>(voff0, o));
              gp[o] = y;
              v[q][r] = y;
            } else if constexpr (PRE) {
              v[q][r] = d.vcomplex ? cmul(v[q][r], hq[q][r]) : cscale(v[q][r], hq[q][r].x);
            } else {
              v[q][r] = vmul_t<T>(v[q][r], d.h2fac, d.vcomplex, row_site<T, N>(voff0, (size_t)b * N + j + r * SS::NR));
            }
          }
        }
        Dft<R, false, C<T>>::run(v[q]);
      }
    }
    st_write<T, N, R, 1, Rows, NT>(v, [&](int b, int n, C<T> x) { buf[Rows::at(b, n)] = x; });
    __syncthreads();
  }
  lds_stages<T, PKT<T>, N, true, false, Rows, NT, 1, M>(buf, tw);
  {
    constexpr int R = plan_of<PKT<T>, N, true>().r[M];
    constexpr int NSL = ns_before<PKT<T>, N, true, M>();
    C<T> v[SG<Rows, N, R, NT>::CAPQ][R];
    st_read<T, N, R, NSL, false, Rows, NT, tw_off<PKT<T>, N, true, M>()>(v, tw, [&](int b, int n) { return buf[Rows::at(b, n)]; });
    st_write<T, N, R, NSL, Rows, NT>(v, [&](int b, int n, C<T> x) {
      if (b < nrows) g[b * N + n] = x;
    });
  }
}

// A/B update on a row tile (modes as for plane_ab, transforms along x3 only).
template <typename T, int N, int NT, int RB, int P>
__device__ __forceinline__ void row_ab(C<T> *buf, const C<T> *tw, const PassDesc &d, uint32_t mode, long long row0,
                                       int nrows, size_t voff0) {
  constexpr size_t N3 = (size_t)N * N * N;
  C<T> *gp = (C<T> *)d.psi + (size_t)row0 * N;
  C<T> *ga = (C<T> *)d.alt + (size_t)row0 * N;
  const bool comb = (mode & M_COMB) != 0;
  const C<T> *src = comb ? ga : gp;
  for (int idx = threadIdx.x; idx < RB * N; idx += NT) {
    const int r = idx / N, c = idx - r * N;
    buf[r * P + padn(c)] = r < nrows ? src[idx] : mkc<T>(0, 0);
  }
  __syncthreads();
  using Rows = RowsGeo<RB, P>;
  if (mode & M_INV) fft_lines_t<T, PKT<T>, N, true, Rows, NT>(buf, tw);
  if (comb) {
    for (int idx = threadIdx.x; idx < nrows * N; idx += NT) {
      const int r = idx / N, c = idx - r * N;
      const int a = r * P + padn(c);
      const C<T> o = ab_combine<T>(gp[idx], buf[a], d, row_site<T, N>(voff0, idx));
      gp[idx] = o;
      buf[a] = o;
    }
    __syncthreads();
  }
  if (mode & M_FWD) {
    fft_lines_t<T, PKT<T>, N, false, Rows, NT>(buf, tw);
    C<T> *dst = (mode & M_ALT) ? ga : gp;
    for (int idx = threadIdx.x; idx < nrows * N; idx += NT) {
      const int r = idx / N, c = idx - r * N;
      dst[idx] = buf[r * P + padn(c)];
    }
  }
}

// Tile = RB consecutive x3 rows over all states (the last tile may be short).
template <typename T, int N, int NT>
__device__ __forceinline__ void row_body(const LaunchList &L, int e, int t, unsigned char *smem) {
  constexpr int P = padded_len(N);
  constexpr int RB = row_block_t<T, N>();
  const PassDesc &d = *(const PassDesc *)L.descp[e];
  const uint32_t mode = L.mode[e];
  const long long rows_total = (long long)d.k * N * N;
  // Where whole tiles tile each state, consecutive blocks take the same rows of successive
  // states: the k reads of the potential factor for those rows then fall close together in
  // time and all but the first are served by the shared last-level cache instead of HBM.
  // A bijection on [0, k N^2 / RB); the arithmetic of every tile is unchanged.
  long long tile = t;
  if constexpr (((long long)N * N) % RB == 0) {
    if (d.k > 1) tile = (long long)(t % d.k) * ((long long)N * N / RB) + t / d.k;
  }
  const long long row0 = tile * RB;
  const int nrows = (int)((rows_total - row0) < RB ? (rows_total - row0) : RB);
  C<T> *buf = (C<T> *)smem;
  C<T> *tw = buf + RB * P;
  load_tw<T, N, NT>(tw, d);
  constexpr size_t N3 = (size_t)N * N * N;
  C<T> *g = (C<T> *)d.psi + (size_t)row0 * N;
  // site offset of the tile's first row within its state; (voff0 + idx) % N^3 wraps at state boundaries
  const size_t voff0 = (size_t)(row0 % (long long)(N * N)) * N;
  if (mode & (M_COMB | M_ALT)) {
    if constexpr (plan_of<PKT<T>, N, false>().n >= 2) {
      if (mode == (M_INV | M_COMB | M_FWD | M_ALT)) {
        __syncthreads();
        row_steady<T, N, NT, RB, P, true>(buf, tw, (C<T> *)d.alt + (size_t)row0 * N, d, voff0, nrows, g);
        return;
      }
    }
    row_ab<T, N, NT, RB, P>(buf, tw, d, mode, row0, nrows, voff0);
    return;
  }
  if constexpr (plan_of<PKT<T>, N, false>().n >= 2) {
    if (mode == (M_INV | M_MID | M_FWD)) {
      __syncthreads();
      row_steady<T, N, NT, RB, P>(buf, tw, g, d, voff0, nrows);
      return;
    }
  }
  for (int idx = threadIdx.x; idx < RB * N; idx += NT) {
    const int r = idx / N, c = idx - r * N;
    C<T> v = mkc<T>(0, 0);
    if (r < nrows) {
      v = g[idx];
      if (mode & M_PRE) v = vmul_t<T>(v, d.hfac, d.vcomplex, row_site<T, N>(voff0, idx));
    }
    buf[r * P + padn(c)] = v;
  }
  __syncthreads();
  using Rows = RowsGeo<RB, P>;
  if (mode & M_INV) fft_lines_t<T, PKT<T>, N, true, Rows, NT>(buf, tw);
  if (mode & M_MID) {
    for (int idx = threadIdx.x; idx < nrows * N; idx += NT) {
      const int r = idx / N, c = idx - r * N;
      const int a = r * P + padn(c);
      buf[a] = vmul_t<T>(buf[a], d.h2fac, d.vcomplex, row_site<T, N>(voff0, idx));
    }
    __syncthreads();
  }
  if (mode & M_FWD) fft_lines_t<T, PKT<T>, N, false, Rows, NT>(buf, tw);
  for (int idx = threadIdx.x; idx < nrows * N; idx += NT) {
    const int r = idx / N, c = idx - r * N;
    C<T> v = buf[r * P + padn(c)];
    if (mode & M_POST) v = vmul_t<T>(v, d.hfac, d.vcomplex, row_site<T, N>(voff0, idx));
    g[idx] = v;
  }
}

template <typename T, int N>
__global__ void __launch_bounds__(LINE_THREADS) k_row_t(const LaunchList L) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int e = find_entry(L, blockIdx.x);
  row_body<T, N, LINE_THREADS>(L, e, blockIdx.x - L.tile_start[e], smem);
}

// ------------------------------------------------------------ column pass

template <int NL, int PC> struct TileGeo {
  static constexpr int nlines = NL;
  static constexpr bool linefast = true;
  static __device__ __forceinline__ int at(int b, int n) { return n * PC + b; }
};

// Steady-state column pass (forward -> x e^{-dt T}/N^3 -> inverse) with the
// first stage read from HBM, the last written to HBM, and the forward last
// stage, the kinetic factor and the inverse first stage fused in registers.
template <typename T, int N, int NT, class Geo>
__device__ __forceinline__ void col_steady(C<T> *buf, const C<T> *tw, C<T> *g, size_t S, const PassDesc &d, bool ax1,
                                           int o, int c0, int nc) {
  constexpr RPlan PL = plan_of<PKT<T>, N, false>();
  constexpr int M = PL.n - 1;
  constexpr int TC = Geo::nlines;
  const C<T> zero = mkc<T>(0, 0);
  {
    constexpr int R = PL.r[0];
    C<T> v[SG<Geo, N, R, NT>::CAPQ][R];
    st_read<T, N, R, 1, false, Geo, NT, 0>(
        v, tw, [&](int b, int n) { return (N % TC == 0 || b < nc) ? g[(size_t)n * S + b] : zero; });
    st_write<T, N, R, 1, Geo, NT>(v, [&](int b, int n, C<T> x) { buf[Geo::at(b, n)] = x; });
    __syncthreads();
  }
  lds_stages<T, PKT<T>, N, false, false, Geo, NT, 1, M>(buf, tw);
  {
    constexpr int R = PL.r[M];
    constexpr int NSL = ns_before<PKT<T>, N, false, M>();
    using SS = SG<Geo, N, R, NT>;
    C<T> v[SS::CAPQ][R];
    st_read<T, N, R, NSL, false, Geo, NT, tw_off<PKT<T>, N, false, M>()>(v, tw, [&](int b, int n) { return buf[Geo::at(b, n)]; });
    __syncthreads();
#pragma unroll
    for (int q = 0; q < SS::CAPQ; ++q) {
      if (SS::active(q)) {
        int j, b;
        SS::jb(q, j, b);
        const int i3 = (N % TC == 0 || b < nc) ? c0 + b : c0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const int n = j + r * SS::NR;
          v[q][r] = cscale(v[q][r], kin_factor_t<T>(d, ax1 ? n : o, ax1 ? o : n, i3));
        }
        Dft<R, true, C<T>>::run(v[q]);
      }
    }
    st_write<T, N, R, 1, Geo, NT>(v, [&](int b, int n, C<T> x) { buf[Geo::at(b, n)] = x; });
    __syncthreads();
  }
  lds_stages<T, PKT<T>, N, true, true, Geo, NT, 1, M>(buf, tw);
  {
    constexpr int R = plan_of<PKT<T>, N, true>().r[M];
    constexpr int NSL = ns_before<PKT<T>, N, true, M>();
    C<T> v[SG<Geo, N, R, NT>::CAPQ][R];
    st_read<T, N, R, NSL, true, Geo, NT, tw_off<PKT<T>, N, true, M>()>(v, tw, [&](int b, int n) { return buf[Geo::at(b, n)]; });
    st_write<T, N, R, NSL, Geo, NT>(v, [&](int b, int n, C<T> x) {
      if (N % TC == 0 || b < nc) g[(size_t)n * S + b] = x;
    });
  }
}

// Column pass in one direction only (forward, or inverse with optional 1/N^3):
// first stage from HBM, last stage to HBM.
template <typename T, int N, int NT, class Geo, bool INV>
__device__ __forceinline__ void col_single(C<T> *buf, const C<T> *tw, C<T> *g, size_t S, int nc, T post) {
  constexpr RPlan PL = plan_of<PKT<T>, N, false>();
  constexpr int M = PL.n - 1;
  constexpr int TC = Geo::nlines;
  const C<T> zero = mkc<T>(0, 0);
  {
    constexpr int R = PL.r[0];
    C<T> v[SG<Geo, N, R, NT>::CAPQ][R];
    st_read<T, N, R, 1, INV, Geo, NT, 0>(
        v, tw, [&](int b, int n) { return (N % TC == 0 || b < nc) ? g[(size_t)n * S + b] : zero; });
    st_write<T, N, R, 1, Geo, NT>(v, [&](int b, int n, C<T> x) { buf[Geo::at(b, n)] = x; });
    __syncthreads();
  }
  lds_stages<T, PKT<T>, N, false, INV, Geo, NT, 1, M>(buf, tw);
  {
    constexpr int R = PL.r[M];
    constexpr int NSL = ns_before<PKT<T>, N, false, M>();
    C<T> v[SG<Geo, N, R, NT>::CAPQ][R];
    st_read<T, N, R, NSL, INV, Geo, NT, tw_off<PKT<T>, N, false, M>()>(v, tw, [&](int b, int n) { return buf[Geo::at(b, n)]; });
    st_write<T, N, R, NSL, Geo, NT>(v, [&](int b, int n, C<T> x) {
      if (N % TC == 0 || b < nc) g[(size_t)n * S + b] = cscale(x, post);
    });
  }
}

// Tile = TC contiguous x3 columns at one position of the other transverse
// axis; all N elements along the transform axis (x1 if M_AXIS1, else x2).
template <typename T, int N, int NT>
__device__ __forceinline__ void col_body(const LaunchList &L, int e, int t, unsigned char *smem) {
  constexpr int TC = col_tile_t<T>();
  constexpr int PC = TC + 1;
  constexpr int NCB = (N + TC - 1) / TC;
  const PassDesc &d = *(const PassDesc *)L.descp[e];
  const uint32_t mode = L.mode[e];
  constexpr int per_state = N * NCB;
  const int s = t / per_state;
  const int rem = t - s * per_state;
  const int o = rem / NCB, cb = rem - o * NCB;
  const bool ax1 = (mode & M_AXIS1) != 0;
  const size_t S = ax1 ? (size_t)N * N : (size_t)N;
  const size_t OS = ax1 ? (size_t)N : (size_t)N * N;
  const int c0 = cb * TC;
  C<T> *buf = (C<T> *)smem;
  C<T> *tw = buf + N * PC;
  load_tw<T, N, NT>(tw, d);
  C<T> *g = (C<T> *)((mode & M_ALT) ? d.alt : d.psi) + (size_t)s * N * N * N + (size_t)o * OS + c0;
  using Geo = TileGeo<TC, PC>;
  if constexpr (plan_of<PKT<T>, N, false>().n >= 2) {
    const int nc = (N - c0) < TC ? (N - c0) : TC;
    const uint32_t m3 = mode & (M_FWD | M_KIN | M_INV);
    if (m3 == (M_FWD | M_KIN | M_INV) && !(mode & M_SCALE)) {
      col_steady<T, N, NT, Geo>(buf, tw, g, S, d, ax1, o, c0, nc);
      return;
    }
    if (m3 == M_FWD || m3 == M_INV) {
      const T post = (mode & M_SCALE) ? (T)d.inv_n3 : (T)1;
      if (m3 == M_FWD) col_single<T, N, NT, Geo, false>(buf, tw, g, S, nc, post);
      else col_single<T, N, NT, Geo, true>(buf, tw, g, S, nc, post);
      return;
    }
  }
  for (int idx = threadIdx.x; idx < N * TC; idx += NT) {
    const int n = idx / TC, c = idx - n * TC;
    C<T> v = mkc<T>(0, 0);
    if (N % TC == 0 || c0 + c < N) v = g[(size_t)n * S + c];
    buf[n * PC + c] = v;
  }
  __syncthreads();
  if (mode & M_FWD) fft_lines_t<T, PKT<T>, N, false, Geo, NT>(buf, tw);
  if (mode & M_KIN) {
    for (int idx = threadIdx.x; idx < N * TC; idx += NT) {
      const int n = idx / TC, c = idx - n * TC;
      const int i1 = ax1 ? n : o, i2 = ax1 ? o : n;
      const int i3 = (N % TC == 0 || c0 + c < N) ? c0 + c : c0;
      const int a = n * PC + c;
      buf[a] = cscale(buf[a], kin_factor_t<T>(d, i1, i2, i3));
    }
    __syncthreads();
  }
  if (mode & M_INV) fft_lines_t<T, PKT<T>, N, true, Geo, NT>(buf, tw);
  const T post = (mode & M_SCALE) ? (T)d.inv_n3 : (T)1;
  for (int idx = threadIdx.x; idx < N * TC; idx += NT) {
    const int n = idx / TC, c = idx - n * TC;
    if (N % TC == 0 || c0 + c < N) g[(size_t)n * S + c] = cscale(buf[n * PC + c], post);
  }
}

// Block order of the column passes.  From N = 192 up the states no longer fit the 256 MB
// on-package cache, and runs of 64 consecutive tiles per XCD (the x3 tiles of neighbouring x2
// rows) turn a row's scattered 128-byte segments into longer runs per XCD: 153 against 168 us
// per launch at 256^3 x 3 states.  Below that size the plain order is as fast or faster.
constexpr int COL_XCD_MIN_N = 192, COL_XCD_RUN = 64;
__device__ __forceinline__ int col_block(int N) {
  return N >= COL_XCD_MIN_N ? xcd_block_chunked(blockIdx.x, gridDim.x, COL_XCD_RUN) : (int)blockIdx.x;
}

template <typename T, int N>
__global__ void __launch_bounds__(LINE_THREADS) k_col_t(const LaunchList L) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int blk = col_block(N);
  const int e = find_entry(L, blk);
  col_body<T, N, LINE_THREADS>(L, e, blk - L.tile_start[e], smem);
}

// ------------------------------------------------------------ dispatch table


template <int N> void register_size(FftKernels *tab) {
  static_assert(N > 128 || plane_fits<float, N>(), "complex64 planes up to N = 128 must fit LDS");
  static_assert(N > 96 || plane_fits<double, N>(), "complex128 planes up to N = 96 must fit LDS");
  FftKernels &k = tab[N];
  if constexpr (plane_fits<float, N>()) {
    k.plane[0] = (const void *)k_plane_t<float, N>;
    k.plane_lds[0] = plane_lds_t<float, N>();
  }
  if constexpr (plane_fits<double, N>()) {
    k.plane[1] = (const void *)k_plane_t<double, N>;
    k.plane_lds[1] = plane_lds_t<double, N>();
  }
  k.plane_nt = plane_threads<N>();
  k.row[0] = (const void *)k_row_t<float, N>;
  k.row[1] = (const void *)k_row_t<double, N>;
  k.row_lds[0] = row_lds_t<float, N>();
  k.row_lds[1] = row_lds_t<double, N>();
  k.col[0] = (const void *)k_col_t<float, N>;
  k.col[1] = (const void *)k_col_t<double, N>;
  k.col_lds[0] = col_lds_t<float, N>();
  k.col_lds[1] = col_lds_t<double, N>();
}

}  // namespace qf
