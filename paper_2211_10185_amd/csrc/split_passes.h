// Transform passes of the split-x2 schedule (templates; instantiated per size, precision and
// variant by split_inst.hip).
#pragma once

#include "fft_passes.h"

namespace qf {

// ------------------------------------------------- slab and pencil passes (split x2)
//
// For large N the x2 transform is split four-step style, N = N1 N2 with i2 = N2 a + b
// (a < N1, b < N2):
//   forward  A (slab pass):   Y[k1][b] = W_N^{b k1} sum_a x[N2 a + b] W_N1^{a k1}, stored at row N2 k1 + b;
//            B (pencil pass): X[k1 + N1 k2] = sum_b Y[k1][b] W_N2^{b k2},        stored at row N2 k1 + k2;
//   inverse  B^-1 then A^-1 with conjugate roots, on the same rows.
// The slab pass holds the N1 rows {N2 a + b} of one x1 plane (b fixed): A^-1, the x3
// transforms around the potential factor, A.  The pencil pass holds the N2 consecutive rows
// N2 k1 .. N2 k1 + N2 - 1 of TT consecutive x3 columns over all x1: B, the x1 transforms
// around the kinetic factor (x2 frequency k1 + N1 k2 at row N2 k1 + k2), B^-1.  One step is
// then two passes over the state (a pencil pass and a slab pass) instead of a row pass and
// three column passes.  Between the passes of a chunk the state is held in this split x2
// order; the chunk's first and last slab passes take it from and return it to real space
// in natural order.
//
// Plane groups.  Between the passes the XI x1 planes XI p .. XI p + XI - 1 of a group are also
// interleaved: the memory of row r of plane XI p + j (its "row slot" j) holds columns
// j N/XI .. (j + 1) N/XI - 1 of all XI planes of the group, column j N/XI + w / XI of plane
// XI p + w mod XI at element w.  A pencil tile's (x1, row) piece then spans XI times the bytes of
// its TT columns, and a slab tile, which holds the N1 rows of all planes of a group, reads and
// writes exactly the memory of those rows in either order (the in-place chunk-edge passes that
// convert from and to natural order touch no other tile's memory).

template <typename T, int N, int N1, int XI, int PK> __host__ __device__ constexpr size_t slab_lds_t() {
  return (size_t)(XI * N1 * padded_len(N) + 8 * (XI - 1) + tw_total<PK, N>()) * sizeof(C<T>);
}
// Lines of a slab tile: row a of the group's plane j is line j N1 + a, and the lines of plane j start
// 8 j elements further, so that the A stages' lanes, which alternate between the planes of one
// column, fall on distinct LDS banks (N1 P elements is a multiple of 128 bytes at N1 = 16).
template <int NL, int P, int N1, int XI> struct SlabGeo {
  static constexpr int nlines = NL;
  static constexpr bool linefast = false;
  static __device__ __forceinline__ int at(int b, int n) {
    if constexpr (XI == 1) return b * P + padn(n);
    else return b * P + (b / N1) * 8 + padn(n);
  }
};
// Pencil tile in LDS: element n (x1) of line l = k2 TT + c at n PC + l.  PC = lines + 4 (+ 4 more
// where that is a multiple of 32) puts the 16 lanes of one 128-byte LDS pass (4 x1 positions x 4
// columns, or 8 x 2) on distinct banks when the B stage writes its outputs.
template <int N2, int TT> __host__ __device__ constexpr int pencil_pitch() {
  return N2 * TT + 4 + ((N2 * TT + 4) % 32 == 0 ? 4 : 0);
}
template <typename T, int N, int N2, int TT, int PK, bool HX> __host__ __device__ constexpr size_t pencil_lds_t() {
  return (size_t)N * pencil_pitch<N2, TT>() * sizeof(T) * (HX ? 1 : 2) + tw_total<PK, N>() * sizeof(C<T>) + N * sizeof(T);
}

// Loads and stores of one state with a block-uniform base and a 32-bit per-lane byte offset.
// The base goes through readfirstlane, so the compiler holds it (plus any uniform offset) in
// scalar registers and each access needs one 32-bit offset register instead of a 64-bit address:
// a lane keeps one access per x2 row of a split-x2 stage in flight.
// With G the pointer is taken in the global address space and each row's uniform offset is kept in a
// scalar register (the empty asm stops the compiler from folding it into a 64-bit vector address),
// so the accesses can use the global forms; without G they are flat accesses.  The slab pass
// measured faster with the global forms, the pencil pass with flat ones.
template <typename T, bool G = false> struct StateBuf {
  typedef __attribute__((address_space(1))) char gchar;
  typedef T pair_t __attribute__((ext_vector_type(2)));
  typedef __attribute__((address_space(1))) pair_t gelem;
  const char *base;
  __device__ __forceinline__ explicit StateBuf(const void *p) {
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    base = (const char *)(((uint64_t)hi << 32) | lo);
  }
  __device__ __forceinline__ gchar *grow(uint32_t soff) const {
    asm volatile("" : "+s"(soff));
    return (gchar *)base + soff;
  }
  __device__ __forceinline__ C<T> load(uint32_t voff, uint32_t soff) const {
    if constexpr (G) {
      const pair_t v = *(const gelem *)(grow(soff) + voff);
      return mkc<T>(v.x, v.y);
    } else {
      return *(const C<T> *)(base + soff + voff);
    }
  }
  __device__ __forceinline__ void store(C<T> x, uint32_t voff, uint32_t soff) const {
    if constexpr (G) {
      pair_t v;
      v.x = x.x;
      v.y = x.y;
      *(gelem *)(grow(soff) + voff) = v;
    } else {
      *(C<T> *)(const_cast<char *>(base) + soff + voff) = x;
    }
  }
};

// x with its two parts in scalar registers (x must be the same in every lane of the wave)
__device__ __forceinline__ float uniform(float x) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x))); }
__device__ __forceinline__ double uniform(double x) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_readfirstlane((int)(b & 0xffffffffLL));
  const int hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
template <typename V> __device__ __forceinline__ V uniform(V x) { V r; r.x = uniform(x.x); r.y = uniform(x.y); return r; }

// Slab pass on tile (plane group p, fast x2 digit b), for each state of the member in turn, so that
// the potential factor rows of the tile are read from HBM once for all k states (or, with the
// entry's aux = 1, for one state per tile: k times the tiles, each reading the factor rows).  The
// tile's LDS holds row a of the group's plane j as line j N1 + a.  M_INV reads the split order, M_FWD
// writes it; otherwise the state is read or written in natural order.  KIND:
//   SLAB_REAL, SLAB_COMPLEX: the steady mode (M_INV | M_MID | M_FWD) for a real or complex factor:
//     A^-1 from HBM, inverse x3, x h^2 (fused with the last inverse and first forward stages), forward
//     x3, A to HBM;
//   SLAB_AB: the steady mode of the A/B update (M_INV | M_COMB | M_FWD | M_ALT): the same on alt, with
//     psi' = A psi - B (dt H_K psi) as the fused middle stage (psi in natural order);
//   SLAB_EDGE: the chunk's start (M_PRE | M_FWD: x h, forward x3, A; A/B: M_FWD | M_ALT from psi to
//     alt) and end (M_INV | M_POST: A^-1, inverse x3, x h; A/B: M_INV | M_COMB).
// Kernels of their own, so that the registers of one kind do not weigh on another.
template <typename T, int N, int N1, int NT, int XI, int PK, int KIND>
__device__ __forceinline__ void slab_body(const LaunchList &L, int e, int t, unsigned char *smem) {
  constexpr int N2 = N / N1;
  constexpr int P = padded_len(N);
  constexpr int NR = XI * N1;               // LDS lines of a tile
  constexpr int NH = N / XI;                // columns of each plane in one row slot
  constexpr int NP = XI * N;                // (row slot, element) positions of one row
  constexpr int CQ = (NP + NT - 1) / NT;    // positions per thread in the A stages
  constexpr int TPS = (N / XI) * N2;        // tiles per state
  using Rows = SlabGeo<NR, P, N1, XI>;
  constexpr int NST = stages_of<PK, N, false>().n, M = NST - 1;
  static_assert(N % N1 == 0 && N % XI == 0 && NST >= 2, "slab pass needs N1 | N, XI | N and a plan of two or more stages");
  static_assert((size_t)N * N * N * sizeof(C<T>) < (1ull << 31), "states below 2 GiB");
  const PassDesc &d = *(const PassDesc *)L.descp[e];
  const uint32_t mode = L.mode[e];
  // aux 1: one state per tile (tiles of state s follow those of state s - 1), else all k states
  int s0 = 0, s1 = d.k;
  if (L.aux[e] == 1) {
    s0 = t / TPS;
    s1 = s0 + 1;
    t -= s0 * TPS;
  }
  const int p = t / N2, b = t - (t / N2) * N2;
  // the twiddle tables first, so that their addresses fit the LDS instructions' offset field
  C<T> *tw = (C<T> *)smem;
  C<T> *buf = tw + tw_total<PK, N>();
  constexpr size_t N3 = (size_t)N * N * N;
  const size_t voff = (size_t)XI * p * N * N;    // the group's first plane
  const C<T> *gtw = (const C<T> *)d.tw;
  // offset from the group's first plane of row N2 a + b of plane (or row slot) j, element n
  auto site = [&](int j, int a, int n) -> size_t { return ((size_t)j * N + N2 * a + b) * N + n; };
  // W_N^{b k1}, the twiddles of A: b is the same for the whole block, so they stay in scalar
  // registers
  C<T> wab[N1];
#pragma unroll
  for (int k1 = 1; k1 < N1; ++k1) wab[k1] = uniform(gtw[(b * k1) % N]);
  // A^-1: the N1 values of each (row slot, element) position are loaded (a_load), then conj twiddles,
  // inverse DFT over k1, to the LDS lines of the position's plane and column (a_inverse)
  auto a_load = [&](C<T> (&v)[N1], const StateBuf<T, true> &sb, int q) {
    const int pos = (int)threadIdx.x + q * NT;
    if (NP % NT == 0 || pos < NP) {
      const int j = pos / N, w = pos - (pos / N) * N;
      const uint32_t vo = (uint32_t)(site(j, 0, w) * sizeof(C<T>));
#pragma unroll
      for (int k1 = 0; k1 < N1; ++k1) v[k1] = sb.load(vo, (uint32_t)(k1 * N2 * N * sizeof(C<T>)));
    }
  };
  auto a_inverse = [&](C<T> (&v)[N1], int q) {
    const int pos = (int)threadIdx.x + q * NT;
    if (NP % NT == 0 || pos < NP) {
      const int j = pos / N, w = pos - (pos / N) * N;
      const int pl = w % XI, col = j * NH + w / XI;
#pragma unroll
      for (int k1 = 1; k1 < N1; ++k1) {
        C<T> w1 = wab[k1];
        w1.y = -w1.y;
        v[k1] = cmul(v[k1], w1);
      }
      Dft<N1, true, C<T>>::run(v);
#pragma unroll
      for (int a = 0; a < N1; ++a) buf[Rows::at(pl * N1 + a, col)] = v[a];
    }
  };
  // the state's split-order rows to the LDS lines.  The loads are issued before the block waits
  // for the twiddle tables and for the previous state's last reads of the LDS lines.
  auto a_inverse_to_lds = [&](const C<T> *g) {
    const StateBuf<T, true> sb(g);
    if constexpr (CQ == 1) {
      C<T> v[N1];
      a_load(v, sb, 0);
      __syncthreads();
      a_inverse(v, 0);
    } else {
      __syncthreads();
#pragma unroll
      for (int q = 0; q < CQ; ++q) {
        C<T> v[N1];
        a_load(v, sb, q);
        a_inverse(v, q);
      }
    }
    __syncthreads();
  };
  // A: columns from the LDS lines, DFT over a, twiddles, to HBM at rows N2 k1 + b
  auto a_forward_from_lds = [&](C<T> *g) {
    const StateBuf<T, true> sb(g);
#pragma unroll
    for (int q = 0; q < CQ; ++q) {
      const int pos = (int)threadIdx.x + q * NT;
      if (NP % NT == 0 || pos < NP) {
        const int j = pos / N, w = pos - (pos / N) * N;
        const int pl = w % XI, col = j * NH + w / XI;
        C<T> v[N1];
#pragma unroll
        for (int a = 0; a < N1; ++a) v[a] = buf[Rows::at(pl * N1 + a, col)];
        Dft<N1, false, C<T>>::run(v);
#pragma unroll
        for (int k1 = 1; k1 < N1; ++k1) v[k1] = cmul(v[k1], wab[k1]);
        const uint32_t vo = (uint32_t)(site(j, 0, w) * sizeof(C<T>));
#pragma unroll
        for (int k1 = 0; k1 < N1; ++k1) sb.store(v[k1], vo, (uint32_t)(k1 * N2 * N * sizeof(C<T>)));
      }
    }
  };
  if constexpr (KIND != SLAB_EDGE) {
    constexpr bool AB = KIND == SLAB_AB;
    constexpr int RM = StageOf<PK, N, false, M>::R;
    using SS = SG<Rows, N, RM, NT>;
    using F = typename FacT<T, KIND == SLAB_COMPLEX>::type;
    // potential factors of the fused middle stage, held in registers for all k states (one
    // fetch per tile)
    F hq[AB ? 1 : SS::CAPQ][AB ? 1 : RM];
    if constexpr (!AB) {
#pragma unroll
      for (int q = 0; q < SS::CAPQ; ++q) {
        if (SS::active(q)) {
          int j, bl;
          SS::jb(q, j, bl);
          const int pl = bl / N1, a = bl - (bl / N1) * N1;
#pragma unroll
          for (int r = 0; r < RM; ++r) hq[q][r] = ((const F *)d.h2fac)[voff + site(pl, a, j + r * SS::NR)];
        }
      }
    }
    fill_twiddles<T, PK, N, NT>(tw, gtw);
    // psi' or the factor, and the first forward stage, on the outputs of the last inverse one
    auto middle = [&](auto &v, int s) {
#pragma unroll
      for (int q = 0; q < SS::CAPQ; ++q) {
        if (SS::active(q)) {
          if constexpr (AB) {
            C<T> *gp = (C<T> *)d.psi + (size_t)s * N3 + voff;
            int j, bl;
            SS::jb(q, j, bl);
            const int pl = bl / N1, a = bl - (bl / N1) * N1;
#pragma unroll
            for (int r = 0; r < RM; ++r) {
              const size_t o = site(pl, a, j + r * SS::NR);
              v[q][r] = ab_combine<T>(gp[o], v[q][r], d, voff + o);
              gp[o] = v[q][r];
            }
          } else {
#pragma unroll
            for (int r = 0; r < RM; ++r) {
              if constexpr (KIND == SLAB_COMPLEX) v[q][r] = cmul(v[q][r], hq[q][r]);
              else v[q][r] = cscale(v[q][r], hq[q][r]);
            }
          }
          stage_first<T, PK, N, true, false>(v[q], tw);
        }
      }
    };
    for (int s = s0; s < s1; ++s) {
      C<T> *g = (C<T> *)(AB ? d.alt : d.psi) + (size_t)s * N3 + voff;
      a_inverse_to_lds(g);
      lds_stages<T, PK, N, false, true, Rows, NT, 0, M>(buf, tw);
      {
        C<T> v[SS::CAPQ][RM];
        stage_read<T, PK, N, false, M, true, Rows, NT>(v, tw, [&](int bl, int n) { return buf[Rows::at(bl, n)]; });
        __syncthreads();
        middle(v, s);
        stage_write<T, PK, N, true, 0, Rows, NT>(v, [&](int bl, int n, C<T> x) { buf[Rows::at(bl, n)] = x; });
        __syncthreads();
      }
      lds_stages<T, PK, N, true, false, Rows, NT, 1, NST>(buf, tw);
      a_forward_from_lds(g);
    }
    return;
  }
  // Natural-order tile accesses of the chunk's edges: each thread takes elements
  // threadIdx.x + it NT, UB at a time, with all UB global loads issued before they are used.
  constexpr int NE = NR * N;
  constexpr int EPT = (NE + NT - 1) / NT;
  constexpr int UB = EPT < 8 ? EPT : 8;
  const bool vc = d.vcomplex != 0;
  auto fac = [&](const void *f, size_t o) -> C<T> {
    return vc ? ((const C<T> *)f)[voff + o] : mkc<T>(((const T *)f)[voff + o], 0);
  };
  fill_twiddles<T, PK, N, NT>(tw, gtw);
  // state rows (times the factor f if given) to the LDS lines
  auto natural_to_lds = [&](const C<T> *g, const void *f) {
    const StateBuf<T, true> sb(g);
    __syncthreads();       // the twiddle tables; the previous state's reads of the LDS lines
#pragma unroll 1
    for (int it0 = 0; it0 < EPT; it0 += UB) {
      C<T> v[UB], h[UB];
#pragma unroll
      for (int u = 0; u < UB; ++u) {
        const int idx = (int)threadIdx.x + (it0 + u) * NT;
        if (it0 + u < EPT && (NE % NT == 0 || idx < NE)) {
          const int bl = idx / N, n = idx - bl * N, pl = bl / N1, a = bl - pl * N1;
          v[u] = sb.load((uint32_t)(site(pl, a, n) * sizeof(C<T>)), 0);
          if (f) h[u] = fac(f, site(pl, a, n));
        }
      }
#pragma unroll
      for (int u = 0; u < UB; ++u) {
        const int idx = (int)threadIdx.x + (it0 + u) * NT;
        if (it0 + u < EPT && (NE % NT == 0 || idx < NE)) {
          const int bl = idx / N, n = idx - bl * N;
          C<T> x = v[u];
          if (f) x = vc ? cmul(x, h[u]) : cscale(x, h[u].x);
          buf[Rows::at(bl, n)] = x;
        }
      }
    }
    __syncthreads();
  };
  // LDS lines times the factor f to the state rows
  auto lds_to_natural = [&](C<T> *g, const void *f) {
    const StateBuf<T, true> sb(g);
#pragma unroll 1
    for (int it0 = 0; it0 < EPT; it0 += UB) {
      C<T> h[UB];
#pragma unroll
      for (int u = 0; u < UB; ++u) {
        const int idx = (int)threadIdx.x + (it0 + u) * NT;
        if (it0 + u < EPT && (NE % NT == 0 || idx < NE)) {
          const int bl = idx / N, n = idx - bl * N, pl = bl / N1, a = bl - pl * N1;
          h[u] = fac(f, site(pl, a, n));
        }
      }
#pragma unroll
      for (int u = 0; u < UB; ++u) {
        const int idx = (int)threadIdx.x + (it0 + u) * NT;
        if (it0 + u < EPT && (NE % NT == 0 || idx < NE)) {
          const int bl = idx / N, n = idx - bl * N, pl = bl / N1, a = bl - pl * N1;
          C<T> x = buf[Rows::at(bl, n)];
          x = vc ? cmul(x, h[u]) : cscale(x, h[u].x);
          sb.store(x, (uint32_t)(site(pl, a, n) * sizeof(C<T>)), 0);
        }
      }
    }
  };
  const bool comb = (mode & M_COMB) != 0;
  for (int s = s0; s < s1; ++s) {
    const size_t so = (size_t)s * N3 + voff;
    C<T> *gp = (C<T> *)d.psi + so;
    // split order is read from and written to alt in the A/B update, psi otherwise
    C<T> *gs = (mode & (M_COMB | M_ALT)) ? (C<T> *)d.alt + so : gp;
    if (mode & M_INV) a_inverse_to_lds(gs);
    else natural_to_lds(gp, (mode & M_PRE) ? d.hfac : nullptr);
    if (mode & M_INV) fft_lines_t<T, PK, N, true, Rows, NT>(buf, tw);
    if (comb) {
      for (int idx = threadIdx.x; idx < NE; idx += NT) {
        const int bl = idx / N, n = idx - bl * N, pl = bl / N1, a = bl - pl * N1;
        const size_t o = site(pl, a, n);
        gp[o] = ab_combine<T>(gp[o], buf[Rows::at(bl, n)], d, voff + o);
      }
      continue;            // the chunk's last combine: no forward transform follows
    }
    if (mode & M_FWD) {
      fft_lines_t<T, PK, N, false, Rows, NT>(buf, tw);
      a_forward_from_lds(gs);
    } else {
      lds_to_natural(gp, d.hfac);     // the factor of the chunk's end is applied on the way out
    }
  }
}

// Pencil pass on tile (state s, slow x2 frequency k1, x3 columns c0 .. c0 + TT - 1): B, forward x1,
// x e^{-dt T(k)}/N^3, inverse x1, B^-1.  The state (alt in the A/B update) is in split order with
// plane groups of XI.  Next to a plane pass at the chunk's edges x2 is transformed as a whole there
// and B (M_PRE) or B^-1 (M_POST) is left out.  HX: the values stay in registers between the stages, and
// LDS holds one part of them at a time (the real parts are exchanged, then the imaginary parts): half the
// LDS and twice the barriers.  It pays where a whole tile leaves one or two blocks per compute unit and
// the registers allow more (us per step, relativistic, one / three states on one stream: complex64 192^3
// 88 / 215 -> 77 / 172, 240^3 144 / 452 -> 129 / 403; complex128 216^3 245 / 735 -> 210 / 580), and costs
// elsewhere (complex64 160^3 49 / 113 -> 51 / 115, 180^3 90 / 199 -> 95 / 210; complex128 256^3 330 / 925 -> 346 /
// 961, whose 200 registers allow no more blocks).
template <typename T, int N, int N2, int TT, int NT, int XI, int PK, bool HX>
__device__ __forceinline__ void pencil_body(const LaunchList &L, int e, int t, unsigned char *smem) {
  constexpr int N1 = N / N2;
  constexpr int NH = N / XI;
  constexpr int NL = N2 * TT;
  constexpr int PC = pencil_pitch<N2, TT>();
  constexpr int NCB = N / TT;
  constexpr int PPT = (N * TT + NT - 1) / NT;    // (x1, column) positions per thread in the B stages
  using Geo = TileGeo<NL, PC>;
  constexpr int NST = stages_of<PK, N, false>().n, M = NST - 1;
  static_assert(N % N2 == 0 && N % TT == 0 && N % XI == 0 && N % 2 == 0 && NST >= 2, "pencil tile must divide the lattice");
  static_assert((size_t)N * N * N * sizeof(C<T>) < (1ull << 31), "states below 2 GiB");
  const PassDesc &d = *(const PassDesc *)L.descp[e];
  const int cb = t % NCB;
  const int u = t / NCB;
  const int k1 = u % N1, s = u / N1;
  const int c0 = cb * TT;
  // the twiddle and kinetic tables first, so that their addresses fit the LDS instructions'
  // offset field
  C<T> *tw = (C<T> *)smem;
  T *ktl = (T *)(tw + tw_total<PK, N>());      // the per-axis kinetic table
  C<T> *buf = (C<T> *)(ktl + N);
  constexpr size_t N3 = (size_t)N * N * N;
  const uint32_t mode = L.mode[e];
  const StateBuf<T> sb((C<T> *)((mode & M_ALT) ? d.alt : d.psi) + (size_t)s * N3);
  // the k-space factor of kin_factor_t, with the table read from LDS
  const bool rel = d.kin == KIN_REL, ab = d.scheme == SCHEME_AB;
  const T mm = (T)d.m, dtT = (T)d.dt, in3 = (T)d.inv_n3, dtn = (T)(d.dt * d.inv_n3);
  auto kfac = [&](int i1, int i2, int i3) -> T {
    if (rel) {
      const T p2 = ktl[i1] + ktl[i2] + ktl[i3];
      if constexpr (sizeof(T) == 4) {
        const float r = __builtin_amdgcn_sqrtf(p2 + mm * mm);
        if (ab) return p2 * __builtin_amdgcn_rcpf(r + mm) * dtn;
        return __builtin_amdgcn_exp2f(-dtT * 1.4426950408889634f * (r - mm)) * in3;
      } else {
        const T tk = p2 / (sqrt(p2 + mm * mm) + mm);
        if (ab) return tk * dtn;
        return exp(-dtT * tk) * in3;
      }
    }
    if (ab) return (ktl[i1] + ktl[i2] + ktl[i3]) * dtn;
    return ktl[i1] * ktl[i2] * ktl[i3] * in3;
  };
  // byte offset of (x1 plane i1, row N2 k1, column c0 + c): row slot (c0 + c) / NH of the plane
  // group, element XI ((c0 + c) mod NH) + i1 mod XI; rows b apart by b N elements
  auto at = [&](int i1, int c) -> uint32_t {
    const int col = c0 + c, j = col / NH, w = XI * (col - j * NH) + i1 % XI;
    return (uint32_t)((((size_t)(i1 - i1 % XI + j) * N + (size_t)(N2 * k1)) * N + w) * sizeof(C<T>));
  };
  auto b_load = [&](C<T> (&v)[N2], int q) {
    const int pos = (int)threadIdx.x + q * NT;
    if ((N * TT) % NT == 0 || pos < N * TT) {
      const int i1 = pos / TT, c = pos - (pos / TT) * TT;
#pragma unroll
      for (int bb = 0; bb < N2; ++bb) v[bb] = sb.load(at(i1, c), (uint32_t)(bb * N * sizeof(C<T>)));
    }
  };
  // B: DFT over the N2 rows of each (x1, column) position, outputs to the x1 lines (k2, c)
  auto b_forward = [&](C<T> (&v)[N2], int q) {
    const int pos = (int)threadIdx.x + q * NT;
    if ((N * TT) % NT == 0 || pos < N * TT) {
      const int i1 = pos / TT, c = pos - (pos / TT) * TT;
      if (!(mode & M_PRE)) Dft<N2, false, C<T>>::run(v);
#pragma unroll
      for (int k2 = 0; k2 < N2; ++k2) buf[Geo::at(k2 * TT + c, i1)] = v[k2];
    }
  };
  if constexpr (HX) {
    static_assert(PPT == 1, "one position per thread");
    constexpr int R0 = StageOf<PK, N, false, 0>::R, R1 = StageOf<PK, N, true, 1>::R;
    T *hb = (T *)buf;
    C<T> v[N2];
    b_load(v, 0);
    fill_twiddles<T, PK, N, NT>(tw, (const C<T> *)d.tw);
    for (int i = threadIdx.x; i < N; i += NT) ktl[i] = ((const T *)d.ktab)[i];
    const int pos = (int)threadIdx.x, i1 = pos / TT, c = pos - (pos / TT) * TT;
    const bool act = (N * TT) % NT == 0 || pos < N * TT;
    if (act && !(mode & M_PRE)) Dft<N2, false, C<T>>::run(v);
    C<T> w[SG<Geo, N, R0, NT>::CAPQ][R0];
    exchange_parts(
        [&](auto p) {
          if (act) {
#pragma unroll
            for (int k2 = 0; k2 < N2; ++k2) hb[Geo::at(k2 * TT + c, i1)] = part_of<decltype(p)::value, T>(v[k2]);
          }
        },
        [&](auto p) { part_read<decltype(p)::value, T, PK, N, false, 0, Geo, NT>(w, hb); });
    part_stages<T, PK, N, false, false, Geo, NT, 0, NST>(hb, tw, w, [&](auto &x) {
      constexpr int R = StageOf<PK, N, false, M>::R;
      using SS = SG<Geo, N, R, NT>;
#pragma unroll
      for (int q = 0; q < SS::CAPQ; ++q) {
        if (SS::active(q)) {
          int j, l;
          SS::jb(q, j, l);
          const int k2 = l / TT, cc = l - (l / TT) * TT;
#pragma unroll
          for (int r = 0; r < R; ++r) x[q][r] = cscale(x[q][r], kfac(j + r * SS::NR, k1 + N1 * k2, c0 + cc));
          stage_first<T, PK, N, true, true>(x[q], tw);
        }
      }
      C<T> y[SG<Geo, N, R1, NT>::CAPQ][R1];
      exchange_parts([&](auto p) { part_write<decltype(p)::value, T, PK, N, true, 0, Geo, NT>(x, hb); },
                     [&](auto p) { part_read<decltype(p)::value, T, PK, N, true, 1, Geo, NT>(y, hb); });
      part_stages<T, PK, N, true, true, Geo, NT, 1, NST>(hb, tw, y, [&](auto &z) {
        exchange_parts([&](auto p) { part_write<decltype(p)::value, T, PK, N, true, M, Geo, NT>(z, hb); },
                       [&](auto p) {
                         if (act) {
#pragma unroll
                           for (int k2 = 0; k2 < N2; ++k2)
                             part_of<decltype(p)::value, T>(v[k2]) = hb[Geo::at(k2 * TT + c, i1)];
                         }
                       });
      });
    });
    if (act) {
      if (!(mode & M_POST)) Dft<N2, true, C<T>>::run(v);
#pragma unroll
      for (int bb = 0; bb < N2; ++bb) sb.store(v[bb], at(i1, c), (uint32_t)(bb * N * sizeof(C<T>)));
    }
    return;
  }
  {
    // the first position's loads are in flight while the tables are filled
    C<T> v[N2];
    b_load(v, 0);
    fill_twiddles<T, PK, N, NT>(tw, (const C<T> *)d.tw);
    for (int i = threadIdx.x; i < N; i += NT) ktl[i] = ((const T *)d.ktab)[i];
    b_forward(v, 0);
  }
#pragma unroll
  for (int q = 1; q < PPT; ++q) {
    C<T> v[N2];
    b_load(v, q);
    b_forward(v, q);
  }
  __syncthreads();
  lds_stages<T, PK, N, false, false, Geo, NT, 0, M>(buf, tw);
  {
    constexpr int R = StageOf<PK, N, false, M>::R;
    using SS = SG<Geo, N, R, NT>;
    C<T> v[SS::CAPQ][R];
    stage_read<T, PK, N, false, M, false, Geo, NT>(v, tw, [&](int l, int n) { return buf[Geo::at(l, n)]; });
    __syncthreads();
#pragma unroll
    for (int q = 0; q < SS::CAPQ; ++q) {
      if (SS::active(q)) {
        int j, l;
        SS::jb(q, j, l);
        const int k2 = l / TT, c = l - (l / TT) * TT;
#pragma unroll
        for (int r = 0; r < R; ++r) v[q][r] = cscale(v[q][r], kfac(j + r * SS::NR, k1 + N1 * k2, c0 + c));
        stage_first<T, PK, N, true, true>(v[q], tw);
      }
    }
    stage_write<T, PK, N, true, 0, Geo, NT>(v, [&](int l, int n, C<T> x) { buf[Geo::at(l, n)] = x; });
    __syncthreads();
  }
  lds_stages<T, PK, N, true, true, Geo, NT, 1, NST>(buf, tw);
  // B^-1: inverse DFT over k2 of each position, to the N2 rows in HBM
#pragma unroll
  for (int q = 0; q < PPT; ++q) {
    const int pos = (int)threadIdx.x + q * NT;
    if ((N * TT) % NT == 0 || pos < N * TT) {
      const int i1 = pos / TT, c = pos - (pos / TT) * TT;
      C<T> v[N2];
#pragma unroll
      for (int k2 = 0; k2 < N2; ++k2) v[k2] = buf[Geo::at(k2 * TT + c, i1)];
      if (!(mode & M_POST)) Dft<N2, true, C<T>>::run(v);
#pragma unroll
      for (int bb = 0; bb < N2; ++bb) sb.store(v[bb], at(i1, c), (uint32_t)(bb * N * sizeof(C<T>)));
    }
  }
}

// FP64 energy measurement in two passes over the states.  The kinetic energy is sum_k T(k) |psi^(k)|^2 / N^3,
// so the transform's last stage feeds the sum and its output is never written; the slab pass reads the
// state as it is stored (complex64 or complex128), adds up |psi|^2 and V |psi|^2 on the way, and leaves
// x3 and the slab part of x2 transformed in scratch64.  40 B per site and state (complex64) instead of
// the 152 B of a copy, three transform passes and two sums.  128^3 x 3 states: slab pass 45 us, pencil
// pass 25 us, with the final sums 75 us for a readout that took 203; 256^3 x 3 states with complex V: 432
// and 358 us of 1.68 ms before.  Bound by the slab pass's natural-order loads and by HBM; its tiles are taken
// state by state, so V is read once per state.

// Fixed-order block sums of NV values per thread: wave shuffles, then the waves in order.  Thread 0
// returns with the sums in acc.
template <int NV, int NT> __host__ __device__ constexpr size_t block_sums_lds() { return (NT + 63) / 64 * NV * sizeof(double); }
template <int NV, int NT> __device__ __forceinline__ void block_sums(double (&acc)[NV]) {
  constexpr int NW = (NT + 63) / 64;
  __shared__ double red[NW][NV];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q < NV; ++q) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc[q] += __shfl_xor(acc[q], off, 64);
    if (lane == 0) red[w][q] = acc[q];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      double v = 0.0;
      for (int ww = 0; ww < NW; ++ww) v += red[ww][q];
      acc[q] = v;
    }
  }
}

// Slab pass of the measurement on tile (state s, plane group p, fast x2 digit b): the state's natural rows
// to LDS in FP64 with the sums over the tile's sites, forward x3, A to scratch64 in split order.
template <typename TI, int N, int N1, int NT, int XI, int PK>
__device__ __forceinline__ void slab_meas_body(const PassDesc &d, int t, unsigned char *smem) {
  using V2 = C<double>;
  constexpr int N2 = N / N1, P = padded_len(N), NR = XI * N1, NH = N / XI, NP = XI * N;
  constexpr int CQ = (NP + NT - 1) / NT, TPS = (N / XI) * N2;
  using Rows = SlabGeo<NR, P, N1, XI>;
  static_assert(NT % 64 == 0, "whole waves");
  const int s = t / TPS, tile = t - s * TPS;
  const int p = tile / N2, b = tile - p * N2;
  V2 *tw = (V2 *)smem;
  V2 *buf = tw + tw_total<PK, N>();
  constexpr size_t N3 = (size_t)N * N * N;
  const size_t voff = (size_t)XI * p * N * N;
  auto site = [&](int j, int a, int n) -> size_t { return ((size_t)j * N + N2 * a + b) * N + n; };
  const C<TI> *g = (const C<TI> *)d.psi + (size_t)s * N3 + voff;
  const bool vc = d.vcomplex != 0;
  double acc[3] = {0.0, 0.0, 0.0};
  constexpr int NE = NR * N, EPT = (NE + NT - 1) / NT, UB = EPT < 8 ? EPT : 8;
#pragma unroll 1
  for (int it0 = 0; it0 < EPT; it0 += UB) {
    C<TI> v[UB];
    double vr[UB], vi[UB];
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      const int idx = (int)threadIdx.x + (it0 + u) * NT;
      vr[u] = vi[u] = 0.0;
      if (it0 + u < EPT && (NE % NT == 0 || idx < NE)) {
        const int bl = idx / N, n = idx - bl * N, pl = bl / N1, a = bl - pl * N1;
        const size_t o = site(pl, a, n);
        v[u] = g[o];
        if (vc) { const V2 w = ((const V2 *)d.v64)[voff + o]; vr[u] = w.x; vi[u] = w.y; }
        else vr[u] = d.v64[voff + o];
      }
    }
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      const int idx = (int)threadIdx.x + (it0 + u) * NT;
      if (it0 + u < EPT && (NE % NT == 0 || idx < NE)) {
        const int bl = idx / N, n = idx - bl * N;
        const double ur = v[u].x, ui = v[u].y;
        const double n2 = ur * ur + ui * ui;
        acc[0] += n2;
        acc[1] += vr[u] * n2;
        acc[2] += vi[u] * n2;
        buf[Rows::at(bl, n)] = mkc<double>(ur, ui);
      }
    }
  }
  fill_twiddles<double, PK, N, NT>(tw, (const V2 *)d.tw64);
  block_sums<3, NT>(acc);
  if (threadIdx.x == 0)
    for (int q = 0; q < 3; ++q) d.partials[(size_t)(s * 3 + q) * TPS + tile] = acc[q];
  __syncthreads();
  fft_lines_t<double, PK, N, false, Rows, NT>(buf, tw);
  const StateBuf<double, true> sb((V2 *)d.scratch64 + (size_t)s * N3 + voff);
#pragma unroll
  for (int q = 0; q < CQ; ++q) {
    const int pos = (int)threadIdx.x + q * NT;
    if (NP % NT == 0 || pos < NP) {
      const int j = pos / N, w = pos - (pos / N) * N;
      const int pl = w % XI, col = j * NH + w / XI;
      V2 v[N1];
#pragma unroll
      for (int a = 0; a < N1; ++a) v[a] = buf[Rows::at(pl * N1 + a, col)];
      Dft<N1, false, V2>::run(v);
#pragma unroll
      for (int k1 = 1; k1 < N1; ++k1) v[k1] = cmul(v[k1], uniform(((const V2 *)d.tw64)[(b * k1) % N]));
      const uint32_t vo = (uint32_t)(site(j, 0, w) * sizeof(V2));
#pragma unroll
      for (int k1 = 0; k1 < N1; ++k1) sb.store(v[k1], vo, (uint32_t)(k1 * N2 * N * sizeof(V2)));
    }
  }
}

// Pencil pass of the measurement on tile (state s, slow x2 frequency k1, TT x3 columns): B and forward x1 of
// scratch64; the last stage's outputs are weighted with T(k) and summed.
template <int N, int N2, int TT, int NT, int XI, int PK>
__device__ __forceinline__ void pencil_meas_body(const PassDesc &d, int t, unsigned char *smem) {
  using V2 = C<double>;
  constexpr int N1 = N / N2, NH = N / XI, NL = N2 * TT, PC = pencil_pitch<N2, TT>(), NCB = N / TT;
  constexpr int PPT = (N * TT + NT - 1) / NT, PPS = N1 * NCB;
  constexpr int M = stages_of<PK, N, false>().n - 1;
  using Geo = TileGeo<NL, PC>;
  const int s = t / PPS, tile = t - s * PPS;
  const int k1 = tile / NCB, c0 = (tile - k1 * NCB) * TT;
  V2 *tw = (V2 *)smem;
  double *ktl = (double *)(tw + tw_total<PK, N>());
  V2 *buf = (V2 *)(ktl + N);
  const StateBuf<double> sb((V2 *)d.scratch64 + (size_t)s * N * N * N);
  auto at = [&](int i1, int c) -> uint32_t {
    const int col = c0 + c, j = col / NH, w = XI * (col - j * NH) + i1 % XI;
    return (uint32_t)((((size_t)(i1 - i1 % XI + j) * N + (size_t)(N2 * k1)) * N + w) * sizeof(V2));
  };
#pragma unroll
  for (int q = 0; q < PPT; ++q) {
    const int pos = (int)threadIdx.x + q * NT;
    const int i1 = pos / TT, c = pos - (pos / TT) * TT;
    const bool in = (N * TT) % NT == 0 || pos < N * TT;
    V2 v[N2];
    if (in) {
#pragma unroll
      for (int bb = 0; bb < N2; ++bb) v[bb] = sb.load(at(i1, c), (uint32_t)(bb * N * sizeof(V2)));
    }
    if (q == 0) {
      // the first position's loads are in flight while the tables are filled
      fill_twiddles<double, PK, N, NT>(tw, (const V2 *)d.tw64);
      for (int i = threadIdx.x; i < N; i += NT) ktl[i] = d.ksym64[i];
    }
    if (in) {
      Dft<N2, false, V2>::run(v);
#pragma unroll
      for (int k2 = 0; k2 < N2; ++k2) buf[Geo::at(k2 * TT + c, i1)] = v[k2];
    }
  }
  __syncthreads();
  lds_stages<double, PK, N, false, false, Geo, NT, 0, M>(buf, tw);
  constexpr int R = StageOf<PK, N, false, M>::R;
  using SS = SG<Geo, N, R, NT>;
  V2 v[SS::CAPQ][R];
  stage_read<double, PK, N, false, M, false, Geo, NT>(v, tw, [&](int l, int n) { return buf[Geo::at(l, n)]; });
  double acc[1] = {0.0};
  const bool rel = d.kin == KIN_REL;
  const double mm = d.m;
#pragma unroll
  for (int q = 0; q < SS::CAPQ; ++q) {
    if (SS::active(q)) {
      int j, l;
      SS::jb(q, j, l);
      const int k2 = l / TT, c = l - (l / TT) * TT;
      const double k23 = ktl[k1 + N1 * k2] + ktl[c0 + c];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const double ks = ktl[j + r * SS::NR] + k23;
        const double tk = rel ? ks / (sqrt(ks + mm * mm) + mm) : ks;
        acc[0] += tk * (v[q][r].x * v[q][r].x + v[q][r].y * v[q][r].y);
      }
    }
  }
  block_sums<1, NT>(acc);
  if (threadIdx.x == 0) d.partials[(size_t)d.k * 3 * d.en_nb + (size_t)s * PPS + tile] = acc[0];
}

// Tile shapes of the split-x2 passes per size, precision and variant: x2 = N1 x N2 (N1 stride rows
// per slab tile, N2 consecutive rows per pencil tile; both have register butterflies), plane groups
// of XI, TT x3 columns per pencil tile, and per pass its threads and the radix plan of its line
// transforms.  A pencil tile's (x1, row) pieces are XI TT elements.
//
// Complex64 factors and plans are fixed by results: the x2 factors and the radix sequence of a size
// decide every rounding, and energies of complex64 solves keep their digits only as long as both stay
// (other two-stage plans moved them by 1e-6).  So the plans are make_rplan's, with adjacent stages
// fused in registers where that is faster, and up to N = 90 the factors are those of the plane pass
// (see split_row).  The rest, and all of a complex128 shape, was found by timing: plane groups,
// columns, threads, fused stages (complex128: factors up to 25, line plans of two stages and, at 162, 200
// and 250, of three), each slab kernel in turn with the pencil kernels of the same factors, with one and
// three states on an MI355X.  (In
// turn, because at small N a pass run by itself finds in its XCD's L2 what it has just written there:
// 128^3, one state, 21 us for the two passes by themselves and 30 us in turn.)  What decides:
//   - an LDS exchange less per direction: 240^3, one complex64 state, 16 x (3 x 5) against 16 x 3 x 5:
//     slab pass 86 -> 62 us, pencil pass 89 -> 77 us;
//   - the passes are bound by latency, so registers decide: at most 128 leave four waves per SIMD;
//   - pencil pieces of 32 bytes and more (XI TT >= 4 in complex64, >= 2 in complex128): the L1 is
//     bound by requests below that; 64 bytes where the LDS holds the tile (256^3, complex128, one / three
//     states: 420 / 1169 -> 330 / 925 us per step; one pencil tile of 157 KB per CU).  The complex64
//     defaults at 40, 48, 50, 54, 90, 150, 162 and 250 have pieces of 16 bytes all the same: of 1, 2, 4 and 8
//     columns only 1 and 2 divide 50, 54, 90, 150, 162 and 250, and there plane pairs were slower (150^3,
//     one state, 58.1 -> 61.6 us per step);
//   - at small N more, smaller tiles: one per (plane, row digit) with 64 to 256 threads;
//   - a complex factor takes twice the registers of a real one in the slab pass's middle stage.  Where that
//     goes past the 256 of a lane or costs a wave per SIMD the kernel has threads (and fused stages) of its
//     own, found by timing them at every size (us per step with a complex V, one / three states, the
//     threads of the real factor -> its own): complex64 150^3 59 / 124 -> 57 / 121, 180^3 131 / 275 -> 92 /
//     194, 192^3 94 / 211 -> 85 / 187, 216^3 three states 460 -> 383, complex128 216^3 315 / 816 -> 284 / 729.
// Variants:
//   0: the fastest for three states with a real potential when the shapes were searched (at 162 in
//   complex128 the second one is, in the solver: 250.7 against 254.3 us per step);  1: complex64 from 96
//   up: the fastest other shape of the same factors and line plans; complex128: the fastest for one state
//   or for the A/B update where that is another shape, with factors or plans of its own at most sizes;
//   2: 8 consecutive rows per pencil tile and 8 columns;  3: the factors swapped;  4 (not selectable by
//   flags): the A/B update of complex64 up to N = 128, with the factors of the plane pass.
struct SplitDef {
  int N, dbl, v, N1, XI, TT, slab_nt, slab_plan, pencil_nt, pencil_plan;
  bool pencil_hx = false;
  int slab_c_nt = 0, slab_c_plan = 0;      // of the slab pass with a complex factor, where they are its own
};
constexpr SplitDef SPLIT_DEFS[] = {
    {32, 0, 0, 4, 1, 4, 64, rp(8, 4), 128, rp(8, 4)},
    {32, 0, 4, 4, 1, 4, 64, rp(8, 4), 128, rp(8, 4)},
    {36, 0, 0, 9, 1, 4, 64, rp(4, 9), 192, rp(4, 9)},
    {36, 0, 4, 9, 1, 4, 64, rp(4, 9), 192, rp(4, 9)},
    {40, 0, 0, 5, 1, 2, 64, rp(8, 5), 128, rp(8, 5)},
    {40, 0, 4, 5, 1, 2, 64, rp(8, 5), 128, rp(8, 5)},
    {48, 0, 0, 3, 1, 2, 64, rp(16, 3), 128, rp(16, 3)},
    {48, 0, 4, 3, 1, 2, 64, rp(16, 3), 128, rp(16, 3)},
    {50, 0, 0, 5, 1, 2, 64, rp(10, 5), 128, rp(10, 5)},
    {50, 0, 4, 5, 1, 2, 64, rp(10, 5), 128, rp(10, 5)},
    {54, 0, 0, 9, 1, 2, 64, rp(6, 9), 128, rp(6, 9)},
    {54, 0, 4, 9, 1, 2, 64, rp(6, 9), 128, rp(6, 9)},
    {60, 0, 0, 10, 1, 4, 64, rp(6, 10), 256, rp(6, 10)},
    {60, 0, 4, 10, 1, 4, 64, rp(6, 10), 256, rp(6, 10)},
    {64, 0, 0, 8, 1, 8, 64, rp(8, 8), 512, rp(8, 8)},
    {64, 0, 4, 8, 1, 8, 64, rp(8, 8), 512, rp(8, 8)},
    {72, 0, 0, 9, 1, 8, 128, rp(8, 9), 576, rp(8, 9)},
    {72, 0, 4, 9, 1, 8, 128, rp(8, 9), 576, rp(8, 9)},
    {80, 0, 0, 5, 1, 4, 128, rp(16, 5), 320, rp(16, 5)},
    {80, 0, 4, 5, 1, 4, 128, rp(16, 5), 320, rp(16, 5)},
    {90, 0, 0, 9, 1, 2, 128, rp(10, 9), 192, rp(10, 9)},
    {90, 0, 4, 9, 1, 2, 128, rp(10, 9), 192, rp(10, 9)},
    {96, 0, 0, 16, 1, 4, 128, rp(16, 6), 384, rp(16, 6)},
    {96, 0, 1, 16, 1, 8, 128, rp(16, 6), 768, rp(16, 6)},
    {96, 0, 3, 6, 2, 4, 192, rp(16, 6), 384, rp(16, 6)},
    {96, 0, 4, 6, 1, 4, 128, rp(16, 6), 384, rp(16, 6)},
    {100, 0, 0, 10, 1, 4, 128, rp(10, 10), 448, rp(10, 10)},
    {100, 0, 1, 10, 2, 4, 256, rp(10, 10), 448, rp(10, 10)},
    {100, 0, 4, 10, 1, 4, 128, rp(10, 10), 448, rp(10, 10)},
    {108, 0, 0, 12, 1, 4, 192, rp(12, 9), 448, rp(12, 9)},
    {108, 0, 1, 12, 2, 2, 320, rp(12, 9), 256, rp(12, 9)},
    {108, 0, 3, 9, 2, 4, 256, rp(12, 9), 448, rp(12, 9)},
    {108, 0, 4, 9, 1, 4, 128, rp(12, 9), 448, rp(12, 9)},
    {120, 0, 0, 12, 1, 4, 128, rp(8, 15), 512, rp(8, 15)},
    {120, 0, 1, 12, 2, 4, 256, rp(8, 15), 512, rp(8, 15)},
    {120, 0, 3, 10, 2, 4, 256, rp(8, 15), 512, rp(8, 15)},
    {120, 0, 4, 15, 1, 4, 128, rp(8, 15), 512, rp(8, 15)},
    {128, 0, 0, 16, 2, 4, 256, rp(16, 8), 512, rp(16, 8)},
    {128, 0, 1, 16, 1, 4, 128, rp(16, 8), 512, rp(16, 8)},
    {128, 0, 2, 16, 2, 8, 256, rp(16, 8), 1024, rp(16, 8)},
    {128, 0, 3, 8, 2, 4, 256, rp(16, 8), 512, rp(16, 8)},
    {128, 0, 4, 8, 1, 4, 128, rp(16, 8), 512, rp(16, 8)},
    {144, 0, 0, 16, 1, 4, 256, rp(16, 9), 576, rp(16, 9)},
    {144, 0, 1, 16, 2, 2, 512, rp(16, 9), 320, rp(16, 9)},
    {144, 0, 3, 9, 2, 2, 192, rp(16, 9), 320, rp(16, 9)},
    {150, 0, 0, 15, 1, 2, 128, rp(6, st(5, 5)), 320, rp(6, 5, 5), false, 256, rp(6, 5, 5)},
    {150, 0, 1, 15, 2, 2, 320, rp(6, st(5, 5)), 320, rp(6, 5, 5)},
    {150, 0, 3, 10, 1, 2, 256, rp(6, 5, 5), 320, rp(6, 5, 5)},
    {160, 0, 0, 16, 1, 4, 256, rp(16, 10), 640, rp(16, 10)},
    {160, 0, 1, 16, 2, 2, 512, rp(16, 10), 320, rp(16, 10)},
    {160, 0, 3, 10, 2, 2, 256, rp(16, 10), 320, rp(16, 10)},
    {162, 0, 0, 18, 1, 2, 192, rp(18, 9), 384, rp(18, 9)},
    {162, 0, 1, 18, 2, 2, 384, rp(18, 9), 384, rp(18, 9)},
    {162, 0, 3, 9, 1, 2, 192, rp(18, 9), 384, rp(18, 9)},
    {180, 0, 0, 18, 1, 4, 192, rp(4, 9, 5), 768, rp(4, 9, 5), false, 256},
    {180, 0, 1, 18, 1, 2, 192, rp(4, 9, 5), 384, rp(4, 9, 5), false, 256},
    {180, 0, 3, 10, 1, 4, 256, rp(4, 9, 5), 768, rp(4, 9, 5)},
    {192, 0, 0, 16, 1, 4, 192, rp(8, st(8, 3)), 768, rp(8, 8, 3), true, 256, rp(8, 8, 3)},
    {192, 0, 1, 16, 2, 2, 256, rp(8, st(8, 3)), 384, rp(8, 8, 3)},
    {192, 0, 3, 12, 1, 4, 192, rp(8, 8, 3), 768, rp(8, st(8, 3))},
    {200, 0, 0, 20, 1, 4, 256, rp(8, st(5, 5)), 832, rp(8, 5, 5)},
    {200, 0, 1, 20, 1, 2, 256, rp(8, st(5, 5)), 448, rp(8, 5, 5)},
    {200, 0, 3, 10, 1, 4, 256, rp(8, 5, 5), 832, rp(8, st(5, 5))},
    {216, 0, 0, 18, 2, 2, 448, rp(8, st(9, 3)), 448, rp(8, 9, 3), false, 512},
    {216, 0, 1, 18, 1, 2, 256, rp(8, st(9, 3)), 448, rp(8, 9, 3)},
    {216, 0, 3, 12, 1, 4, 128, rp(8, st(9, 3)), 896, rp(8, st(9, 3))},
    {240, 0, 0, 16, 2, 2, 512, rp(16, st(3, 5)), 512, rp(16, st(3, 5)), true},
    {240, 0, 1, 16, 1, 4, 256, rp(16, st(3, 5)), 960, rp(16, st(3, 5))},
    {240, 0, 3, 15, 1, 2, 256, rp(16, st(3, 5)), 512, rp(16, st(3, 5))},
    {250, 0, 0, 25, 1, 2, 256, rp(10, st(5, 5)), 512, rp(10, 5, 5)},
    {250, 0, 1, 25, 1, 2, 256, rp(10, st(5, 5)), 512, rp(10, st(5, 5))},
    {250, 0, 3, 10, 2, 2, 256, rp(10, st(5, 5)), 512, rp(10, st(5, 5))},
    {256, 0, 0, 16, 2, 2, 512, rp(16, 16), 512, rp(16, 16)},
    {256, 0, 1, 16, 2, 4, 512, rp(16, 16), 1024, rp(16, 16)},
    {256, 0, 2, 32, 2, 8, 512, rp(16, 16), 1024, rp(16, 16)},
    {32, 1, 0, 8, 2, 4, 128, rp(8, 4), 128, rp(8, 4)},
    {36, 1, 0, 9, 1, 4, 64, rp(6, 6), 192, rp(6, 6)},
    {40, 1, 0, 8, 1, 4, 64, rp(8, 5), 192, rp(8, 5)},
    {40, 1, 1, 8, 1, 2, 64, rp(8, 5), 128, rp(8, 5)},
    {48, 1, 0, 8, 1, 4, 64, rp(8, 6), 192, rp(6, 8)},
    {48, 1, 1, 6, 1, 2, 64, rp(6, 8), 128, rp(6, 8)},
    {50, 1, 0, 10, 1, 2, 128, rp(10, 5), 128, rp(10, 5)},
    {54, 1, 0, 9, 2, 1, 192, rp(9, 6), 64, rp(9, 6)},
    {60, 1, 0, 10, 1, 4, 128, rp(6, 10), 256, rp(10, 6)},
    {64, 1, 0, 8, 2, 2, 128, rp(8, 8), 128, rp(8, 8)},
    {72, 1, 0, 8, 2, 2, 192, rp(9, 8), 192, rp(8, 9)},
    {72, 1, 1, 9, 1, 4, 128, rp(8, 9), 320, rp(9, 8)},
    {80, 1, 0, 8, 2, 4, 192, rp(8, 10), 320, rp(8, 10)},
    {80, 1, 1, 10, 1, 4, 128, rp(10, 8), 320, rp(10, 8)},
    {90, 1, 0, 10, 2, 2, 256, rp(10, 9), 192, rp(9, 10)},
    {96, 1, 0, 8, 2, 2, 192, rp(12, 8), 192, rp(12, 8)},
    {96, 1, 1, 8, 1, 4, 128, rp(8, 12), 384, rp(8, 12)},
    {100, 1, 0, 10, 2, 4, 256, rp(10, 10), 448, rp(10, 10)},
    {108, 1, 0, 9, 1, 2, 128, rp(9, 12), 256, rp(9, 12)},
    {108, 1, 1, 9, 1, 4, 128, rp(9, 12), 448, rp(9, 12)},
    {120, 1, 0, 12, 1, 2, 128, rp(12, 10), 256, rp(12, 10)},
    {120, 1, 1, 8, 1, 4, 128, rp(12, 10), 512, rp(10, 12)},
    {128, 1, 0, 16, 2, 4, 512, rp(16, 8), 512, rp(16, 8)},
    {144, 1, 0, 12, 1, 2, 192, rp(16, 9), 320, rp(12, 12)},
    {150, 1, 0, 15, 1, 2, 256, rp(15, 10), 320, rp(15, 10)},
    {150, 1, 1, 15, 1, 2, 256, rp(10, 15), 320, rp(15, 10)},
    {160, 1, 0, 16, 1, 2, 256, rp(16, 10), 320, rp(16, 10)},
    {160, 1, 1, 16, 1, 4, 256, rp(16, 10), 640, rp(10, 16)},
    {162, 1, 0, 9, 2, 1, 384, rp(18, 9), 192, rp(9, 18)},
    {162, 1, 1, 9, 1, 2, 192, rp(2, 9, 9), 384, rp(9, 18)},
    {180, 1, 0, 10, 2, 1, 384, rp(18, 10), 192, rp(10, 18)},
    {192, 1, 0, 12, 2, 1, 384, rp(12, 16), 192, rp(12, 16)},
    {192, 1, 1, 12, 1, 2, 192, rp(16, 12), 384, rp(12, 16)},
    {200, 1, 0, 10, 1, 2, 256, rp(5, 8, 5), 448, rp(10, 20)},
    {216, 1, 0, 12, 2, 1, 448, rp(12, 18), 256, rp(12, 18), true, 256},
    {216, 1, 1, 12, 1, 2, 256, rp(12, 18), 448, rp(12, 18)},
    {240, 1, 0, 15, 1, 2, 256, rp(15, 16), 512, rp(15, 16)},
    {250, 1, 0, 25, 1, 2, 256, rp(25, 10), 512, rp(25, 10)},
    {250, 1, 1, 10, 2, 1, 512, rp(5, 10, 5), 256, rp(5, 10, 5)},
    {256, 1, 0, 16, 2, 2, 512, rp(16, 16), 512, rp(16, 16)},
};
__host__ __device__ constexpr int slab_threads(const SplitDef &s, int kind) {
  return kind == SLAB_COMPLEX && s.slab_c_nt ? s.slab_c_nt : s.slab_nt;
}
__host__ __device__ constexpr int slab_plan_of(const SplitDef &s, int kind) {
  return kind == SLAB_COMPLEX && s.slab_c_plan ? s.slab_c_plan : s.slab_plan;
}
__host__ __device__ constexpr SplitDef split_def(int N, int dbl, int v) {
  for (const SplitDef &s : SPLIT_DEFS)
    if (s.N == N && s.dbl == dbl && s.v == v) return s;
  return {N, dbl, v, 0, 1, 1, 64, 0, 64, 0};
}
// The first variant of the size with the shape of variant v (variants that coincide share kernels).
__host__ __device__ constexpr int split_same(int N, int dbl, int v) {
  const SplitDef a = split_def(N, dbl, v);
  for (int u = 0; u < v; ++u) {
    const SplitDef b = split_def(N, dbl, u);
    if (a.N1 == b.N1 && a.XI == b.XI && a.TT == b.TT && a.slab_nt == b.slab_nt && a.slab_plan == b.slab_plan &&
        a.pencil_nt == b.pencil_nt && a.pencil_plan == b.pencil_plan && a.pencil_hx == b.pencil_hx && a.slab_c_nt == b.slab_c_nt &&
        a.slab_c_plan == b.slab_c_plan)
      return u;
  }
  return v;
}

// Pencil block order: runs of consecutive x3 tiles per XCD, so that the pieces of one 128-byte
// row segment are fetched by blocks that share an L2.
constexpr int PENCIL_XCD_RUN = 128;

template <typename T, int N, int V, int KIND>
__global__ void __launch_bounds__((slab_threads(split_def(N, PKT<T>, V), KIND))) k_slab_t(const LaunchList L) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr SplitDef D = split_def(N, PKT<T>, V);
  const int e = find_entry(L, blockIdx.x);
  slab_body<T, N, D.N1, slab_threads(D, KIND), D.XI, slab_plan_of(D, KIND), KIND>(L, e, blockIdx.x - L.tile_start[e], smem);
}

template <typename T, int N, int V>
__global__ void __launch_bounds__((split_def(N, PKT<T>, V).pencil_nt)) k_pencil_t(const LaunchList L) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr SplitDef D = split_def(N, PKT<T>, V);
  const int blk = xcd_block_chunked(blockIdx.x, gridDim.x, PENCIL_XCD_RUN);
  const int e = find_entry(L, blk);
  pencil_body<T, N, N / D.N1, D.TT, D.pencil_nt, D.XI, D.pencil_plan, D.pencil_hx>(L, e, blk - L.tile_start[e], smem);
}

template <typename T, int N, int V> void register_split_variant(FftKernels *tab) {
  constexpr SplitDef D = split_def(N, PKT<T>, V);
  if constexpr (D.N1 > 0) {
    constexpr int U = split_same(N, PKT<T>, V);
    constexpr bool F = sizeof(T) == 4;
    static_assert(slab_lds_t<T, N, D.N1, D.XI, D.slab_plan>() <= 160 * 1024, "slab tile fits LDS");
    static_assert(pencil_lds_t<T, N, N / D.N1, D.TT, D.pencil_plan, D.pencil_hx>() <= 160 * 1024, "pencil tile fits LDS");
    SplitKernels &k = tab[N].split[PKT<T>][V];
    k.plane_edges = F && (N < 96 || V == 4);
    static_assert(!(F && (N < 96 || V == 4)) || (D.XI == 1 && plan_of<0, N, false>().n == 2 &&
                                                  D.N1 == plan_of<0, N, false>().r[1]),
                  "plane passes at the chunk's edges: the factors of split_row, one plane per group");
    if constexpr (V != 4) {
      k.slab[SLAB_REAL] = (const void *)k_slab_t<T, N, U, SLAB_REAL>;
      k.slab[SLAB_COMPLEX] = (const void *)k_slab_t<T, N, U, SLAB_COMPLEX>;
    }
    if constexpr (!F || (N >= 96 && V != 4)) k.slab[SLAB_EDGE] = (const void *)k_slab_t<T, N, U, SLAB_EDGE>;
    if constexpr (!F || V == 4) k.slab[SLAB_AB] = (const void *)k_slab_t<T, N, U, SLAB_AB>;
    for (int kind = 0; kind < SLAB_KINDS; ++kind) k.slab_nt[kind] = slab_threads(D, kind);
    k.slab_lds = slab_lds_t<T, N, D.N1, D.XI, D.slab_plan>();
    k.n1 = D.N1;
    k.xi = D.XI;
    k.pencil = (const void *)k_pencil_t<T, N, U>;
    k.pencil_nt = D.pencil_nt;
    k.pencil_lds = pencil_lds_t<T, N, N / D.N1, D.TT, D.pencil_plan, D.pencil_hx>();
    k.pencil_tt = D.TT;
  }
}
template <typename T, int N> void register_split(FftKernels *tab) {
  register_split_variant<T, N, 0>(tab);
  register_split_variant<T, N, 1>(tab);
  register_split_variant<T, N, 2>(tab);
  register_split_variant<T, N, 3>(tab);
  register_split_variant<T, N, 4>(tab);
}

// Measurement kernels: the shapes of complex128 variant 0.
template <typename TI, int N>
__global__ void __launch_bounds__((split_def(N, 1, 0).slab_nt)) k_slab_meas_t(const LaunchList L) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr SplitDef D = split_def(N, 1, 0);
  const int e = find_entry(L, blockIdx.x);
  slab_meas_body<TI, N, D.N1, D.slab_nt, D.XI, D.slab_plan>(*(const PassDesc *)L.descp[e],
                                                            blockIdx.x - L.tile_start[e], smem);
}
template <int N>
__global__ void __launch_bounds__((split_def(N, 1, 0).pencil_nt)) k_pencil_meas_t(const LaunchList L) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr SplitDef D = split_def(N, 1, 0);
  const int blk = xcd_block_chunked(blockIdx.x, gridDim.x, PENCIL_XCD_RUN);
  const int e = find_entry(L, blk);
  pencil_meas_body<N, N / D.N1, D.TT, D.pencil_nt, D.XI, D.pencil_plan>(*(const PassDesc *)L.descp[e],
                                                                        blk - L.tile_start[e], smem);
}
template <int N> void register_meas(FftKernels *tab) {
  constexpr SplitDef D = split_def(N, 1, 0);
  static_assert(slab_lds_t<double, N, D.N1, D.XI, D.slab_plan>() + block_sums_lds<3, D.slab_nt>() <= 160 * 1024,
                "slab tile and block sums fit LDS");
  static_assert(pencil_lds_t<double, N, N / D.N1, D.TT, D.pencil_plan, false>() + block_sums_lds<1, D.pencil_nt>() <= 160 * 1024,
                "pencil tile and block sums fit LDS");
  MeasKernels &k = tab[N].meas;
  k.slab[0] = (const void *)k_slab_meas_t<float, N>;
  k.slab[1] = (const void *)k_slab_meas_t<double, N>;
  k.pencil = (const void *)k_pencil_meas_t<N>;
  k.slab_lds = slab_lds_t<double, N, D.N1, D.XI, D.slab_plan>();
  k.pencil_lds = pencil_lds_t<double, N, N / D.N1, D.TT, D.pencil_plan, false>();
  k.slab_nt = D.slab_nt;
  k.pencil_nt = D.pencil_nt;
  k.tps = N / D.XI * (N / D.N1);
  k.pps = D.N1 * (N / D.TT);
}

}  // namespace qf
