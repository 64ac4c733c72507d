// FFT pass kernels of the Green's-function convolution (Sec. IV-A), shared by
// the complex64 and complex128 translation units. Each pass exists in three
// tile variants (points per workgroup for row passes, columns per workgroup for
// strided passes); the variant is picked per (pass, length, precision) from
// the tuning table that the on-device autotuner fills.
#pragma once

#include <algorithm>

#include "bufview.hpp"
#include "fft.hpp"
#include "fft_tiles.hpp"
#include "internal.hpp"

namespace fwi {

constexpr long kNarrowMax = 0x7fffffffL;  // bytes a 32-bit buffer view can cover

// Column tile of a strided-pass workgroup. Workgroups are dealt to the 8
// XCDs in turn (linear id modulo 8); when a tile's row segment is narrower
// than a 128-byte cache line, each XCD takes a contiguous range of tiles in
// launch order, so neighbouring tiles (halves of one line) are fetched into
// the same L2 at about the same time.
template <int NL, int ES>
__device__ __forceinline__ int col_tile() {
  const int x = blockIdx.x, n = gridDim.x;
  if constexpr (NL * ES >= 128) {
    return x;
  } else {
    if (n % 8 != 0) return x;
    return (x % 8) * (n / 8) + x / 8;
  }
}

// A value that is the same in every lane, moved to scalar registers (values
// read from LDS are otherwise treated as per-lane).
__device__ __forceinline__ long uniform_long(long v) {
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)(unsigned long)v);
  const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)((unsigned long)v >> 32));
  return (long)(((unsigned long)hi << 32) | lo);
}

// true if any row of the workgroup is to be processed (uniform: LDS flags)
__device__ __forceinline__ bool any_row(const int* s_ok, int nl) {
  int any = 0;
  for (int l = 0; l < nl; ++l) any |= s_ok[l];
  return any != 0;
}

// ------------------------------------------------------------- row pass 1 ---
// Input of the first pass: the rows of x as they are, or a combination with
// basis vectors formed first (see k_row_fwd).
enum RowInKind {
  RI_PLAIN = 0,
  RI_UPD32 = 1,
  RI_UPD64 = 2,
  RI_ORTH = 3,
  RI_ORTH_ONLY = 4,
  RI_START = 5,
  RI_ORTH_SUM = 6,       // RI_ORTH and RI_ORTH_ONLY that sum the inner-product
  RI_ORTH_ONLY_SUM = 7,  // parts themselves
};
__host__ __device__ constexpr bool row_in_sums(int k) { return k == RI_ORTH_SUM || k == RI_ORTH_ONLY_SUM; }
__host__ __device__ constexpr bool row_in_orth_only(int k) { return k == RI_ORTH_ONLY || k == RI_ORTH_ONLY_SUM; }
__host__ __device__ constexpr bool row_in_orth(int k) { return k == RI_ORTH || row_in_orth_only(k) || row_in_sums(k); }

template <typename T>
struct RowFwdArgs {
  const cplx<T>* x;      // rows of length nin, row stride in_stride
  const cplx<T>* m;      // [rows_per_rhs][nin] or null
  const int* active;     // [B] or null
  cplx<T>* out;          // rows of length L
  const cplx<T>* tw;
  long nrows;
  int rows_per_rhs, nin;
  long in_stride;
  // combined input (kind != RI_PLAIN)
  int kind;
  const void* lc_basis;  // V_0; vector i at lc_basis + i * lc_vs elements
  long lc_vs;
  const int* lc_ncol;    // update: [B] vectors per RHS
  int lc_nvec;           // orthogonalisation: vectors of every RHS
  const c128* lc_coef;   // [B][lc_cstride]
  int lc_cstride, lc_first;
  cplx<T>* lc_out;       // = x, written
  double* lc_rowpart;    // orthogonalisation / start: |v|^2 per row
  const c128* lc_src;    // start: the right-hand sides
  // orthogonalisation with the sum of the inner-product parts (see OrthIn)
  int per_rhs;           // workgroups per RHS
  int ndot, nB;
  const c128* dotp;
  const cplx<T>* vscale;
  c128* H;
};

template <typename T, int K>
using lc_basis_t = std::conditional_t<K == RI_UPD32, float, std::conditional_t<K == RI_UPD64, double, T>>;

// Rows of x (times m) zero-padded to L and transformed. HIN: nin <= L/2, so
// the upper half of every padded row is skipped.
// K != RI_PLAIN: the input is first formed, in FP64 registers for the points
// the first stage will ask this thread for, and stored back to x:
//   RI_UPD32 / RI_UPD64 (complex128 x, complex64 / complex128 basis): the
//     solution update x = (first ? 0 : x) + sum_{i < ncol_b} coef[b][i] V_i;
//   RI_ORTH (x the new Arnoldi vector w, basis of type T): classical
//     Gram-Schmidt v = w + sum_{i < nvec} coef[b][i] V_i (coef = -h_i times
//     the vector's scale, accumulated in T like every vector update of the
//     solver), stored, and |v|^2 summed per row in FP64 into rowpart;
//     RI_ORTH_ONLY stops there (no transform);
//   RI_ORTH_SUM / RI_ORTH_ONLY_SUM: the same with the coefficients summed from
//     their parts first, a workgroup's rows all of one RHS. Kinds of their own:
//     the coefficient's place chosen at run time inside the basis loop keeps
//     fewer loads in flight (complex64 pass at 256^2 / 384^2 / 512^2, full
//     batches: 275 / 544 / 611 us against 271 / 537 / 605);
//   RI_START (first cycle, x_0 = 0): x = src rounded to T (src complex128),
//     with |src|^2 summed per row in FP64 into rowpart.
template <typename T, int L, int NLV, bool HIN, int K = RI_PLAIN>
__global__ void __launch_bounds__(NT) k_row_fwd(RowFwdArgs<T> a) {
  using C = LineCfg<T, L, NLV, NT, false>;
  constexpr bool ORTH = row_in_orth(K), SUM = row_in_sums(K);
  constexpr bool START = K == RI_START;
  constexpr bool NORM = ORTH || START;  // per-row sums of |v|^2
  __shared__ cplx<T> sh[C::LDS_ELEMS];
  __shared__ long s_x[C::NL];
  __shared__ int s_m[C::NL];
  __shared__ int s_ok[C::NL];
  __shared__ int s_k[K != RI_PLAIN ? C::NL : 1];
  __shared__ int s_b[K != RI_PLAIN ? C::NL : 1];
  __shared__ c128 s_coef[SUM ? kMaxDotVec : 1];
  long g0 = (long)blockIdx.x * C::NL, gend = a.nrows;  // the workgroup's first row, end of its rows
  if constexpr (SUM) {
    const unsigned b = blockIdx.x / (unsigned)a.per_rhs, part = blockIdx.x % (unsigned)a.per_rhs;
    g0 = (long)b * a.rows_per_rhs + (long)part * C::NL;
    gend = (long)(b + 1) * a.rows_per_rhs;
  }
  for (int l = threadIdx.x; l < C::NL; l += NT) {
    const long g = g0 + l;
    int ok = g < gend;
    const long gc = ok ? g : gend - 1;  // rows past the end read the last row (not stored)
    const long b = gc / a.rows_per_rhs;
    if (ok && a.active && !a.active[b]) ok = 0;
    const long z = gc - b * a.rows_per_rhs;
    s_ok[l] = ok;
    s_x[l] = gc * a.in_stride;
    s_m[l] = (int)z * a.nin;
    if constexpr (K != RI_PLAIN) {
      s_k[l] = ORTH ? a.lc_nvec : START ? 0 : a.lc_ncol[b];
      s_b[l] = (int)b;
    }
  }
  __syncthreads();
  if (!any_row(s_ok, C::NL)) return;  // converged right-hand sides: no traffic
  // branch-free loads (clamped index, masked value), so every leg's loads can
  // be in flight before the first product; without a contrast the x row
  // stands in for m and the blend below makes the factor exactly 1
  const T km = a.m ? (T)1 : (T)0;
  const cplx<T>* mp = a.m ? a.m : a.x;
  auto snk = [&](int line, int pb, int ro, cplx<T> v) {
    if (s_ok[line]) a.out[(g0 + line) * L + pb + ro] = v;
  };
  if constexpr (K == RI_PLAIN) {
    auto src = [&](int line, int pb, int ro) -> cplx<T> {
      const int p = pb + ro;
      const int pc = p < a.nin ? p : a.nin - 1;
      const cplx<T> xv = a.x[s_x[line] + pc];
      const cplx<T> mv = mp[s_m[line] + pc];
      const cplx<T> mf = mk(km * mv.x + ((T)1 - km), km * mv.y);
      const cplx<T> v = xv * mf;
      return p < a.nin ? v : mk((T)0, (T)0);
    };
    fft_line_transform<C, 0, HIN, false>(a.tw, sh, src, snk);
  } else {
    static_assert(HIN, "combined inputs are rows of zero-padded operators");
    static_assert(ORTH || START || sizeof(T) == 8, "the solution update is complex128");
    using TB = lc_basis_t<T, K>;
    using TA = std::conditional_t<ORTH, T, double>;  // accumulation type
    if constexpr (SUM) {
      // column of H and the coefficients from the parts (one RHS): wave w
      // sums vectors w, w + 4, ..., each lane a fixed subset of the parts
      const int lane = threadIdx.x & 63, b = s_b[0];
      for (int i = threadIdx.x >> 6; i < a.lc_nvec; i += NT / 64) {
        double r = 0.0, m = 0.0;
        for (int k = lane; k < a.ndot; k += 64) {
          const c128 d = a.dotp[((long)b * a.ndot + k) * a.lc_cstride + i];
          r += d.x;
          m += d.y;
        }
        r = wave_sum(r);
        m = wave_sum(m);
        if (lane == 0) {
          const double sc = (double)a.vscale[(long)i * a.nB + b].x;
          s_coef[i] = mk(-(r * sc), -(m * sc));
          if (g0 == (long)b * a.rows_per_rhs)
            a.H[((long)b * a.lc_cstride + i) * (a.lc_cstride - 1) + a.lc_nvec - 1] = mk(r, m);
        }
      }
      __syncthreads();
    }
    // the points the first stage will ask this thread for: slot t, leg r
    constexpr int R0 = stage_radix(L, 0, 0, C::BIG);
    constexpr int NJ = L / R0, NB0 = C::NL * NJ, TT0 = (NB0 + NT - 1) / NT, RIN0 = R0 / 2;
    int kmax = 0;
    for (int l = 0; l < C::NL; ++l) kmax = max(kmax, s_k[l]);
    // addresses: a uniform base at the workgroup's first row (made scalar
    // explicitly, it comes from LDS) plus small per-lane element offsets, the
    // same for every basis vector
    const long x0 = uniform_long(s_x[0]);
    unsigned off[TT0][RIN0];
    cplx<TA> acc[TT0][RIN0];
#pragma unroll
    for (int t = 0; t < TT0; ++t) {
      int line, j;
      C::template split<R0>(t, line, j);
      if (line >= C::NL) line = C::NL - 1;  // idle slot of a partial tile: any valid line
#pragma unroll
      for (int r = 0; r < RIN0; ++r) {
        const int p = j + r * NJ;
        const int pc = p < a.nin ? p : a.nin - 1;
        off[t][r] = (unsigned)(s_x[line] - x0 + pc);
        if constexpr (START) {
          acc[t][r] = a.lc_src[x0 + off[t][r]];
        } else {
          const cplx<T> w = a.x[x0 + off[t][r]];
          acc[t][r] = (!ORTH && a.lc_first) ? mk((TA)0, (TA)0) : mk((TA)w.x, (TA)w.y);
        }
      }
    }
    const cplx<TB>* V0 = START ? nullptr : static_cast<const cplx<TB>*>(a.lc_basis) + x0;
#pragma unroll 4
    for (int i = 0; i < kmax; ++i) {
      const cplx<TB>* Vi = V0 + (long)i * a.lc_vs;  // uniform
#pragma unroll
      for (int t = 0; t < TT0; ++t) {
        int line, j;
        C::template split<R0>(t, line, j);
        if (line >= C::NL) line = C::NL - 1;
        const bool use = ORTH || i < s_k[line];  // every RHS of an orthogonalisation has nvec vectors
        const c128 c64 = SUM ? s_coef[i] : a.lc_coef[(long)s_b[line] * a.lc_cstride + i];
        const cplx<TA> c = mk((TA)c64.x, (TA)c64.y);
#pragma unroll
        for (int r = 0; r < RIN0; ++r) {
          // 32-bit byte offset from a uniform base: a scalar-base load
          const unsigned bo = off[t][r] * (unsigned)sizeof(cplx<TB>);
          const cplx<TB> v = *reinterpret_cast<const cplx<TB>*>(reinterpret_cast<const char*>(Vi) + bo);
          const cplx<TA> u = cfma(c, mk((TA)v.x, (TA)v.y), acc[t][r]);
          // select per component (unused vectors may hold anything)
          acc[t][r].x = use ? u.x : acc[t][r].x;
          acc[t][r].y = use ? u.y : acc[t][r].y;
        }
      }
    }
    cplx<T> xin[TT0][RIN0];
    double nrm[TT0];
#pragma unroll
    for (int t = 0; t < TT0; ++t) {
      nrm[t] = 0.0;
      int line, j;
      C::template split<R0>(t, line, j);
      const bool slot = (NB0 % NT == 0 || (int)threadIdx.x + t * NT < NB0);
      if (line >= C::NL) line = C::NL - 1;
#pragma unroll
      for (int r = 0; r < RIN0; ++r) {
        const int p = j + r * NJ;
        xin[t][r] = mk((T)acc[t][r].x, (T)acc[t][r].y);
        if (slot && s_ok[line] && p < a.nin) {
          a.lc_out[x0 + off[t][r]] = xin[t][r];
          if constexpr (ORTH)
            nrm[t] += (double)xin[t][r].x * (double)xin[t][r].x + (double)xin[t][r].y * (double)xin[t][r].y;
          if constexpr (START) nrm[t] += norm2(acc[t][r]);  // of the complex128 value
        }
      }
    }
    if constexpr (!row_in_orth_only(K)) {
      auto src = [&](int line, int pb, int ro, int t, int r) -> cplx<T> {
        const int p = pb + ro;
        const int pc = p < a.nin ? p : a.nin - 1;
        const cplx<T> mv = mp[s_m[line] + pc];
        const cplx<T> mf = mk(km * mv.x + ((T)1 - km), km * mv.y);
        const cplx<T> v = xin[t][r] * mf;
        return p < a.nin ? v : mk((T)0, (T)0);
      };
      fft_line_transform<C, 0, HIN, false>(a.tw, sh, src, snk);
    }
    if constexpr (NORM) {
      // per-row sums in a fixed order: first-stage slot (line, j) belongs to
      // one thread; the LDS tile is free once the transform is done
      double* part = reinterpret_cast<double*>(sh);
      __syncthreads();
#pragma unroll
      for (int t = 0; t < TT0; ++t) {
        if (NB0 % NT == 0 || (int)threadIdx.x + t * NT < NB0) {
          int line, j;
          C::template split<R0>(t, line, j);
          part[line * NJ + j] = nrm[t];
        }
      }
      __syncthreads();
      // one wave per row: lanes over the slots, then a fixed-order wave sum
      const int lane = threadIdx.x & 63;
      for (int l = threadIdx.x >> 6; l < C::NL; l += NT / 64) {
        double s = 0.0;
        for (int q = lane; q < NJ; q += 64) s += part[l * NJ + q];
        s = wave_sum(s);
        if (lane == 0 && s_ok[l]) a.lc_rowpart[g0 + l] = s;
      }
    }
  }
}

// ------------------------------------------------------------- row pass 3 ---
template <typename T>
struct RowInvArgs {
  const cplx<T>* in;     // rows of length L
  const cplx<T>* x;      // [rows][nout] operand (its result is scaled by s_b) or null for EPI_COPY
  const cplx<T>* rhs;    // [rows][nout] (EPI_RESID)
  const cplx<T>* scale;
  const int* active;
  cplx<T>* y;            // [rows][nout]
  const cplx<T>* tw;
  long nrows;
  int rows_per_rhs, nout;  // nout <= L/2 (cropped output)
  c64* y32;              // EPI_RESID32 output [rows][nout]
  double* rowpart;       // EPI_RESID / EPI_RESID32: [rows] sum of |residual|^2
  // EPI_VIE_DOT: Arnoldi inner products of y against the basis (see VieDots)
  const cplx<T>* basis;
  long vs;
  int nvec;
  const cplx<T>* vscale;
  int B;
  c128* dotp;
  int nparts, dstride;
};

template <typename T, int L, int NLV, int EPI>
__global__ void __launch_bounds__(NT) k_row_inv(RowInvArgs<T> a) {
  using C = LineCfg<T, L, NLV, NT, false>;
  constexpr bool RESID = EPI == EPI_RESID || EPI == EPI_RESID32;
  // last stage: butterfly j < NsL of a line stores points j + r NsL, so
  // (line, p mod NsL) names one thread: per-row sums need no atomics
  constexpr int NsL = L / stage_radix(L, 1, plan_stages(L, C::BIG) - 1, C::BIG);
  __shared__ cplx<T> sh[C::LDS_ELEMS];
  __shared__ cplx<T> s_s[C::NL];
  __shared__ int s_ok[C::NL];
  __shared__ double s_part[RESID ? C::NL * NsL : 1];
  if constexpr (RESID)
    for (int i = threadIdx.x; i < C::NL * NsL; i += NT) s_part[i] = 0.0;
  // with inner products a workgroup's rows belong to one RHS (nparts per RHS,
  // the last one ragged); else rows are packed across RHS
  constexpr bool DOT = EPI == EPI_VIE_DOT;
  long g0 = (long)blockIdx.x * C::NL, gend = a.nrows;
  unsigned dot_b = 0, dot_part = 0;
  if constexpr (DOT) {
    dot_b = blockIdx.x / (unsigned)a.nparts;
    dot_part = blockIdx.x - dot_b * (unsigned)a.nparts;
    g0 = (long)dot_b * a.rows_per_rhs + (long)dot_part * C::NL;
    gend = (long)(dot_b + 1) * a.rows_per_rhs;
  }
  for (int l = threadIdx.x; l < C::NL; l += NT) {
    const long g = g0 + l;
    int ok = g < gend;
    const long b = DOT ? (long)dot_b : ok ? g / a.rows_per_rhs : 0;
    if (ok && a.active && !a.active[b]) ok = 0;
    s_ok[l] = ok;
    s_s[l] = a.scale ? a.scale[b] : mk((T)1, (T)0);
  }
  __syncthreads();
  if (!any_row(s_ok, C::NL)) return;  // converged right-hand sides: no traffic
  // rows past the end read the last row and are not stored; epilogue loads
  // use clamped indices so they are not behind the store predicate
  auto row = [&](int line) { return g0 + line < gend ? g0 + line : gend - 1; };
  auto src = [&](int line, int pb, int ro) -> cplx<T> { return a.in[row(line) * L + pb + ro]; };
  auto snk = [&](int line, int pb, int ro, cplx<T> v) {
    const int p = pb + ro;
    const bool st = s_ok[line] && p < a.nout;
    const long o = row(line) * a.nout + (p < a.nout ? p : a.nout - 1);
    if constexpr (EPI == EPI_VIE || DOT) {
      const cplx<T> y = (a.x[o] - v) * s_s[line];  // the operator is linear: s (x - conv(m x))
      if (st) a.y[o] = y;
    } else if constexpr (RESID) {
      const cplx<T> r = a.rhs[o] - (a.x[o] - v);
      if (st) {
        if constexpr (EPI == EPI_RESID) a.y[o] = r;
        else a.y32[o] = mk((float)r.x, (float)r.y);
        s_part[line * NsL + p % NsL] += (double)r.x * (double)r.x + (double)r.y * (double)r.y;
      }
    } else {
      if (st) a.y[o] = v;
    }
  };
  fft_line_transform<C, 1, false, true>(a.tw, sh, src, snk);
  if constexpr (RESID) {
    __syncthreads();
    if (threadIdx.x < C::NL && s_ok[threadIdx.x]) {
      double s = 0.0;
      for (int i = 0; i < NsL; ++i) s += s_part[threadIdx.x * NsL + i];
      a.rowpart[g0 + threadIdx.x] = s;
    }
  }
  if constexpr (DOT) {
    // The workgroup's rows (one RHS, contiguous in y and in every basis
    // vector) were just stored; after the barrier each thread reads back EPD
    // elements of them and streams the basis vectors over the same elements
    // (two or four vectors at a time cost registers: 1.5% of a 256^2 gradient).
    __syncthreads();
    constexpr int EPD = (C::NL * (L / 2) + NT - 1) / NT;
    const long base = g0 * a.nout;
    const int cnt = (int)(gend - g0 < C::NL ? gend - g0 : C::NL) * a.nout;
    const int t = threadIdx.x;
    double yx[EPD], yy[EPD];
#pragma unroll
    for (int q = 0; q < EPD; ++q) {
      const int e = t + q * NT;
      const cplx<T> y = a.y[base + (e < cnt ? e : cnt - 1)];
      yx[q] = e < cnt ? (double)y.x : 0.0;
      yy[q] = e < cnt ? (double)y.y : 0.0;
    }
    __shared__ double red[2][kMaxDotVec][NT / 64];
    const int lane = t & 63, wv = t >> 6;
    for (int i = 0; i < a.nvec; ++i) {
      const cplx<T>* Vi = a.basis + i * a.vs + base;
      cplx<T> vv[EPD];
#pragma unroll
      for (int q = 0; q < EPD; ++q) {
        const int e = t + q * NT;
        vv[q] = Vi[e < cnt ? e : cnt - 1];
      }
      double r = 0.0, m = 0.0;
#pragma unroll
      for (int q = 0; q < EPD; ++q) {
        const double vx = vv[q].x, vy = vv[q].y;
        r = fma(vx, yx[q], r);
        r = fma(vy, yy[q], r);
        m = fma(vx, yy[q], m);
        m = fma(-vy, yx[q], m);
      }
      r = wave_sum(r);
      m = wave_sum(m);
      if (lane == 0) {
        red[0][i][wv] = r;
        red[1][i][wv] = m;
      }
    }
    __syncthreads();
    if (t < a.nvec) {
      double r = 0.0, m = 0.0;
#pragma unroll
      for (int w = 0; w < NT / 64; ++w) {
        r += red[0][t][w];
        m += red[1][t][w];
      }
      const double sc = (double)a.vscale[(long)t * a.B + dot_b].x;  // stored V_i = basis vector / sc
      a.dotp[(long)blockIdx.x * a.dstride + t] = mk(sc * r, sc * m);
    }
  }
}

// --------------------------------------------------------- strided passes ---
template <typename T>
struct StridedArgs {
  const cplx<T>* in;
  cplx<T>* out;
  const cplx<T>* tw;
  const cplx<T>* ghat;    // conv only: [nf][...] same layout as a data plane
  const int* rhs_freq;    // conv only
  const int* active;
  long in_ps, out_ps;     // plane strides
  long pstride;           // elements between consecutive points of a line
  long gstride;           // Ghat stride between frequencies
  int nlines;             // lines per plane
  int planes_per_rhs;
  int lin, lout;          // nonzero input points, output points kept
  long nplanes;           // planes in the launch
  long gpstride;          // Ghat stride between points of a line (conv)
  int tile_major;         // conv: one-dimensional grid ordered tile by tile (see conv_item)
};

// Work item of a convolution workgroup in the tile-major order: item j is
// column tile j / nplanes of plane j % nplanes, so the planes (right-hand
// sides) that share a tile of the kernel spectrum run back to back, and the
// items are dealt so that each XCD takes a contiguous range of them
// (workgroups go to the 8 XCDs in turn): a spectrum tile is then fetched into
// one L2 and reused by every plane, instead of the whole spectrum being
// streamed from HBM once per plane when it does not fit the caches (3D).
__device__ __forceinline__ void conv_item(unsigned nplanes, int& tile, long& plane) {
  // 32-bit arithmetic: a 64-bit division is a hundred instructions of every
  // wave, and the launch has fewer than 2^31 items. complex64 at 384 x 384 and
  // 384 right-hand sides: 704 -> 690 us, 512 x 512 and 192: 616 -> 596 us.
  const unsigned x = blockIdx.x, n = gridDim.x;
  const unsigned j = n % 8 == 0 ? (x % 8) * (n / 8) + x / 8 : x;
  const unsigned t = j / nplanes;
  tile = (int)t;
  plane = (long)(j - t * nplanes);
}

constexpr int CONV_RPW = 1;  // right-hand sides per workgroup in the convolution pass

// The complex64 convolution keeps its twiddle powers in an LDS table (the pass
// is bound by vector issue; the table replaces the product trees, about a
// sixth of its instructions) when the plan's radices are at most 16 and the
// table costs no workgroup per compute unit, or one where five or more remain
// (160 KB of LDS, 32 wave slots per compute unit; measured on the length-192
// tile: five workgroups with the table beat six without it).
template <class C>
constexpr bool conv_pow_table() {
  if constexpr (sizeof(typename C::T) != 4 || plan_max_radix<C::L, C::BIG>() > 16) {
    return false;
  } else {
    constexpr long kLds = 160 * 1024, es = sizeof(cplx<typename C::T>);
    constexpr long slots = 32 / (C::NT / 64);
    constexpr long base = C::LDS_ELEMS * es, with = base + pow_table_size<C>() * es;
    constexpr long wg0 = kLds / base < slots ? kLds / base : slots;
    constexpr long wg1 = kLds / with < slots ? kLds / with : slots;
    return wg1 == wg0 || (wg1 >= 5 && wg1 == wg0 - 1);
  }
}

// MODE 0 forward, 1 inverse, 2 convolution. HALF: the input occupies at most
// the first half of a line (mode 0), only the first half of the output is kept
// (mode 1); the convolution always has both. WIDE: 64-bit addressing for
// planes of 2 GiB or more; otherwise every plane is a 32-bit buffer view whose
// bounds do the zero padding and cropping.
template <typename T, int L, int NLV, int NTV, int MODE, bool HALF, bool WIDE>
__global__ void __launch_bounds__(NTV) k_strided(StridedArgs<T> a) {
  using C = LineCfg<T, L, NLV, NTV, true>;
  constexpr bool PT = MODE == 2 && conv_pow_table<C>();
  __shared__ cplx<T> sh[C::LDS_ELEMS + (PT ? pow_table_size<C>() : 0)];  // lines, then the power table
  constexpr unsigned ES = sizeof(cplx<T>);
  int tile = 0;
  long plane_tm = 0;  // tile-major convolution: the workgroup's plane
  if (MODE == 2 && a.tile_major) conv_item((unsigned)a.nplanes, tile, plane_tm);
  else tile = col_tile<C::NL, (int)ES>();
  const int line0 = tile * C::NL;
  const int nl = a.nlines - line0;
  // line-fastest mapping: the thread's line is fixed; a line past the plane
  // gets an offset past every view (its loads read zero, its stores drop)
  const int myline = (int)threadIdx.x % C::NL;
  const unsigned loff = myline < nl ? (unsigned)(line0 + myline) * ES : kBufferOut;
  const unsigned ps8 = (unsigned)a.pstride * ES;
  if constexpr (MODE == 2) {
    // CONV_RPW consecutive planes (right-hand sides) per workgroup share the
    // kernel-spectrum tile, which is prefetched into registers once per
    // frequency; the loads complete while the forward stages run
    using Map = ConvMidMap<C>;
    cplx<T> gpre[Map::TT][Map::R];
    int fcur = -1;
    for (int q = 0; q < CONV_RPW; ++q) {
      const long plane = a.tile_major ? plane_tm + q : (long)blockIdx.y * CONV_RPW + q;
      if (plane >= a.nplanes) break;
      const int b = (int)plane;  // one plane per right-hand side
      if (a.active && !a.active[b]) continue;  // uniform per workgroup
      const int f = a.rhs_freq[b];
      // the spectrum tile is loaded after the first stage's data (hook of
      // fft_line_convolve), only when the frequency changes
      auto prefetch = [&] {
        if (q > 0 && f == fcur) return;  // the first plane always loads (no branch around its loads)
        if constexpr (WIDE) {
          const cplx<T>* gp = a.ghat + (long)f * a.gstride + line0;
#pragma unroll
          for (int t = 0; t < Map::TT; ++t)
#pragma unroll
            for (int r = 0; r < Map::R; ++r) {
              int line, p;
              gpre[t][r] = (Map::at(t, r, line, p) && line < nl) ? gp[p * a.gpstride + line] : mk((T)0, (T)0);
            }
        } else {
          const unsigned gps8 = (unsigned)a.gpstride * ES;
          const BufView gv(a.ghat + (long)f * a.gstride, (unsigned)L * gps8);
#pragma unroll
          for (int t = 0; t < Map::TT; ++t)
#pragma unroll
            for (int r = 0; r < Map::R; ++r) {
              int line, p;
              if (Map::at(t, r, line, p)) gpre[t][r] = gv.ld<T>(loff + (unsigned)p * gps8);
            }
        }
      };
      auto gh = [&](int t, int r, int, int) -> cplx<T> { return gpre[t][r]; };
      if constexpr (WIDE) {
        const cplx<T>* ip = a.in + plane * a.in_ps + line0;
        cplx<T>* op = a.out + plane * a.out_ps + line0;
        auto src = [&](int line, int pb, int ro) -> cplx<T> {
          const int p = pb + ro;
          if (p >= a.lin || line >= nl) return mk((T)0, (T)0);
          return ip[p * a.pstride + line];
        };
        auto snk = [&](int line, int pb, int ro, cplx<T> v) {
          const int p = pb + ro;
          if (p < a.lout && line < nl) op[p * a.pstride + line] = v;
        };
        fft_line_convolve<C, PT>(a.tw, sh, src, gh, snk, PT ? sh + C::LDS_ELEMS : nullptr, prefetch);
      } else {
        const BufView iv(a.in + plane * a.in_ps, (unsigned)a.lin * ps8);
        const BufView ov(a.out + plane * a.out_ps, (unsigned)a.lout * ps8);
        auto src = [&](int, int pb, int ro) { return iv.ld<T>(loff + (unsigned)(pb + ro) * ps8); };
        auto snk = [&](int, int pb, int ro, cplx<T> v) { ov.st<T>(loff + (unsigned)(pb + ro) * ps8, v); };
        fft_line_convolve<C, PT>(a.tw, sh, src, gh, snk, PT ? sh + C::LDS_ELEMS : nullptr, prefetch);
      }
      fcur = f;
      __syncthreads();  // LDS is reused by the next plane
    }
  } else {
    const long plane = blockIdx.y;
    const int b = (int)(plane / a.planes_per_rhs);
    if (a.active && !a.active[b]) return;  // uniform per workgroup
    constexpr bool HIN = MODE == 0 && HALF, HOUT = MODE == 1 && HALF;
    if constexpr (WIDE) {
      const cplx<T>* ip = a.in + plane * a.in_ps + line0;
      cplx<T>* op = a.out + plane * a.out_ps + line0;
      auto src = [&](int line, int pb, int ro) -> cplx<T> {
        const int p = pb + ro;
        if (p >= a.lin || line >= nl) return mk((T)0, (T)0);
        return ip[p * a.pstride + line];
      };
      auto snk = [&](int line, int pb, int ro, cplx<T> v) {
        const int p = pb + ro;
        if (p < a.lout && line < nl) op[p * a.pstride + line] = v;
      };
      fft_line_transform<C, MODE, HIN, HOUT>(a.tw, sh, src, snk);
    } else {
      const BufView iv(a.in + plane * a.in_ps, (unsigned)a.lin * ps8);
      const BufView ov(a.out + plane * a.out_ps, (unsigned)a.lout * ps8);
      auto src = [&](int, int pb, int ro) { return iv.ld<T>(loff + (unsigned)(pb + ro) * ps8); };
      auto snk = [&](int, int pb, int ro, cplx<T> v) { ov.st<T>(loff + (unsigned)(pb + ro) * ps8, v); };
      fft_line_transform<C, MODE, HIN, HOUT>(a.tw, sh, src, snk);
    }
  }
}

// ---------------------------------------------------------------- dispatch ---
template <typename T, int L, int V>
void launch_row_fwd_v(const RowFwdArgs<T>& a, hipStream_t st) {
  constexpr int NL = row_nl<T, L, V>();
  const unsigned grid = (unsigned)((a.nrows + NL - 1) / NL);
  if (grid == 0) return;
  if (a.kind != RI_PLAIN) {
    if (2 * a.nin > L) throw Error(-6, "combined row inputs need zero-padded rows");
    if (row_in_sums(a.kind)) {
      // the built-in tile only, as the caller decided; the coefficients are formed
      // per workgroup, so each takes rows of one RHS
      if constexpr (V == 0) {
        RowFwdArgs<T> b = a;
        b.per_rhs = (a.rows_per_rhs + NL - 1) / NL;
        const unsigned wg = (unsigned)(a.nrows / a.rows_per_rhs) * (unsigned)b.per_rhs;
        if (a.kind == RI_ORTH_SUM) FWI_TIMED_LAUNCH((k_row_fwd<T, L, NL, true, RI_ORTH_SUM>), dim3(wg), dim3(NT), 0, st, b);
        else FWI_TIMED_LAUNCH((k_row_fwd<T, L, NL, true, RI_ORTH_ONLY_SUM>), dim3(wg), dim3(NT), 0, st, b);
      } else {
        throw Error(-6, "the fused coefficient sum takes the built-in row tile");
      }
    } else if (a.kind == RI_ORTH) {
      FWI_TIMED_LAUNCH((k_row_fwd<T, L, NL, true, RI_ORTH>), dim3(grid), dim3(NT), 0, st, a);
    } else if (a.kind == RI_ORTH_ONLY) {
      FWI_TIMED_LAUNCH((k_row_fwd<T, L, NL, true, RI_ORTH_ONLY>), dim3(grid), dim3(NT), 0, st, a);
    } else if (a.kind == RI_START) {
      FWI_TIMED_LAUNCH((k_row_fwd<T, L, NL, true, RI_START>), dim3(grid), dim3(NT), 0, st, a);
    } else if constexpr (sizeof(T) == 8) {
      if (a.kind == RI_UPD32) FWI_TIMED_LAUNCH((k_row_fwd<T, L, NL, true, RI_UPD32>), dim3(grid), dim3(NT), 0, st, a);
      else FWI_TIMED_LAUNCH((k_row_fwd<T, L, NL, true, RI_UPD64>), dim3(grid), dim3(NT), 0, st, a);
    } else {
      throw Error(-6, "the fused solution update is for complex128 residuals");
    }
  } else if (2 * a.nin <= L) {
    FWI_TIMED_LAUNCH((k_row_fwd<T, L, NL, true>), dim3(grid), dim3(NT), 0, st, a);
  } else if constexpr (sizeof(T) == 8) {
    FWI_TIMED_LAUNCH((k_row_fwd<T, L, NL, false>), dim3(grid), dim3(NT), 0, st, a);
  } else {
    throw Error(-6, "complex64 row transforms need zero-padded rows");
  }
  FWI_LAUNCH_CHECK();
}
template <typename T, int L, int V>
void launch_row_inv_v(const RowInvArgs<T>& a, int epi, hipStream_t st) {
  constexpr int NL = row_nl<T, L, V>();
  const unsigned grid = (unsigned)((a.nrows + NL - 1) / NL);
  if (grid == 0) return;
  if (2 * a.nout > L) throw Error(-6, "inverse row transform must crop to half a padded row");
  if (epi == EPI_VIE_DOT) {
    RowInvArgs<T> b = a;
    b.nparts = (a.rows_per_rhs + NL - 1) / NL;
    if (b.nparts > kMaxDotParts || a.nvec > kMaxDotVec) throw Error(-6, "fused inner products not applicable");
    const unsigned parts = (unsigned)(a.nrows / a.rows_per_rhs) * (unsigned)b.nparts;
    FWI_TIMED_LAUNCH((k_row_inv<T, L, NL, EPI_VIE_DOT>), dim3(parts), dim3(NT), 0, st, b);
  } else if (epi == EPI_VIE) {
    FWI_TIMED_LAUNCH((k_row_inv<T, L, NL, EPI_VIE>), dim3(grid), dim3(NT), 0, st, a);
  } else if (epi == EPI_COPY) {
    FWI_TIMED_LAUNCH((k_row_inv<T, L, NL, EPI_COPY>), dim3(grid), dim3(NT), 0, st, a);
  } else if constexpr (sizeof(T) == 8) {
    if (epi == EPI_RESID) FWI_TIMED_LAUNCH((k_row_inv<T, L, NL, EPI_RESID>), dim3(grid), dim3(NT), 0, st, a);
    else FWI_TIMED_LAUNCH((k_row_inv<T, L, NL, EPI_RESID32>), dim3(grid), dim3(NT), 0, st, a);
  } else {
    throw Error(-6, "residual epilogue needs the complex128 operator");
  }
  FWI_LAUNCH_CHECK();
}
template <typename T, int L, int V, int MODE, bool HALF, bool WIDE>
void launch_strided_k(const StridedArgs<T>& a, dim3 grid, hipStream_t st) {
  constexpr int NL = col_nl<T, L, V>();
  constexpr int NTV = col_nt<V>();
  FWI_TIMED_LAUNCH((k_strided<T, L, NL, NTV, MODE, HALF, WIDE>), grid, dim3(NTV), 0, st, a);
}
// CONV: 1 the convolution only, 0 the transforms only, -1 both (keeps the tiles of
// the lengths with one tile per pass from being built for the other pass).
template <typename T, int L, int V, int CONV = -1>
void launch_strided_v(const StridedArgs<T>& a, long planes, int mode, hipStream_t st) {
  constexpr int NL = col_nl<T, L, V>();
  if (planes == 0) return;
  StridedArgs<T> args = a;
  args.nplanes = planes;
  const long gy = mode == 2 ? (planes + CONV_RPW - 1) / CONV_RPW : planes;
  if (gy > 65535) throw Error(-6, "too many planes for one strided pass");
  dim3 grid((a.nlines + NL - 1) / NL, (unsigned)gy);
  // 32-bit views need every offset of a line point (p < L) below 2^31, so that
  // an out-of-plane line (offset kBufferOut + ...) cannot wrap into range
  const long es = sizeof(cplx<T>);
  const long span = (long)L * std::max(a.pstride, mode == 2 ? a.gpstride : 0L) * es + (long)a.nlines * es;
  const bool wide = span > kNarrowMax || tl_force_wide;
  const bool hin = 2 * a.lin <= L, hout = 2 * a.lout <= L;
  if (mode == 2) {
    if constexpr (CONV != 0) {
      if (a.planes_per_rhs != 1) throw Error(-6, "the convolution takes one plane per right-hand side");
      if (!hin || !hout) throw Error(-6, "convolution lines must be zero-padded to twice their length");
      // 64-bit path: one tile variant, planes along y
      if (wide) {
        args.tile_major = 0;
        const dim3 g0((a.nlines + col_nl<T, L, 0>() - 1) / col_nl<T, L, 0>(), grid.y);
        launch_strided_k<T, L, 0, 2, true, true>(args, g0, st);
      } else if (args.tile_major) {
        if (CONV_RPW != 1) throw Error(-6, "tile-major convolution takes one plane per workgroup");
        const long items = (long)grid.x * planes;
        if (items > 0x7fffffffL) throw Error(-6, "too many convolution work items for one launch");
        launch_strided_k<T, L, V, 2, true, false>(args, dim3((unsigned)items), st);
      } else {
        launch_strided_k<T, L, V, 2, true, false>(args, grid, st);
      }
    }
  } else if constexpr (CONV != 1) {
    const dim3 g0((a.nlines + col_nl<T, L, 0>() - 1) / col_nl<T, L, 0>(), grid.y);
    if (mode == 0) {
      if (wide) {
        if (hin) {
          launch_strided_k<T, L, 0, 0, true, true>(args, g0, st);
        } else if constexpr (sizeof(T) == 8) {
          launch_strided_k<T, L, 0, 0, false, true>(args, g0, st);
        } else {
          throw Error(-6, "complex64 strided transforms need zero-padded lines");
        }
      } else if (hin) {
        launch_strided_k<T, L, V, 0, true, false>(args, grid, st);
      } else if constexpr (sizeof(T) == 8) {
        launch_strided_k<T, L, V, 0, false, false>(args, grid, st);
      } else {
        throw Error(-6, "complex64 strided transforms need zero-padded lines");
      }
    } else {
      if (!hout) throw Error(-6, "inverse strided transform must crop to half a line");
      if (wide) launch_strided_k<T, L, 0, 1, true, true>(args, g0, st);
      else launch_strided_k<T, L, V, 1, true, false>(args, grid, st);
    }
  }
  FWI_LAUNCH_CHECK();
}

#define FWI_VARIANTS(FN, L, v, ...)           \
  do {                                        \
    if (v == 0) FN<T, L, 0>(__VA_ARGS__);     \
    else if (v == 1) FN<T, L, 1>(__VA_ARGS__); \
    else FN<T, L, 2>(__VA_ARGS__);            \
  } while (0)

#define FWI_LENGTHS(FN, L, v, ...)                                           \
  switch (L) {                                                               \
    case 32: FWI_VARIANTS(FN, 32, v, __VA_ARGS__); break;                    \
    case 48: FWI_VARIANTS(FN, 48, v, __VA_ARGS__); break;                    \
    case 64: FWI_VARIANTS(FN, 64, v, __VA_ARGS__); break;                    \
    case 96: FWI_VARIANTS(FN, 96, v, __VA_ARGS__); break;                    \
    case 128: FWI_VARIANTS(FN, 128, v, __VA_ARGS__); break;                  \
    case 192: FWI_VARIANTS(FN, 192, v, __VA_ARGS__); break;                  \
    case 256: FWI_VARIANTS(FN, 256, v, __VA_ARGS__); break;                  \
    case 384: FWI_VARIANTS(FN, 384, v, __VA_ARGS__); break;                  \
    case 512: FWI_VARIANTS(FN, 512, v, __VA_ARGS__); break;                  \
    case 768: FWI_VARIANTS(FN, 768, v, __VA_ARGS__); break;                  \
    case 1024: FWI_VARIANTS(FN, 1024, v, __VA_ARGS__); break;                \
    default: throw Error(-6, "unsupported FFT length " + std::to_string(L)); \
  }

// sz: the launch within the operator; without one (spectra, diagnostics) the
// pass's own input and output
template <typename T>
void strided_call(int L, const StridedArgs<T>& a, long planes, int mode, hipStream_t st, const LaunchSize* sz = nullptr) {
#define FWI_X(LL)                                                                              \
  case LL:                                                                                     \
    if (mode == 2) launch_strided_v<T, LL, op_conv_variant<T>(LL), 1>(a, planes, mode, st);    \
    else launch_strided_v<T, LL, op_strided_variant<T>(LL), 0>(a, planes, mode, st);           \
    return;
  switch (L) { FWI_OP_LENGTHS(FWI_X) }
#undef FWI_X
  LaunchSize own;
  if (!sz) {
    own.tiles = (long)(a.nlines + 15) / 16 * planes;
    own.planes = planes;
    own.bytes = (double)sizeof(cplx<T>) * a.nlines * (a.lin + a.lout) * planes;
  }
  const int v = tune_variant(mode == 2 ? PK_CONV : PK_STRIDED, sizeof(T) == 8, L, sz ? *sz : own);
  FWI_LENGTHS(launch_strided_v, L, v, a, planes, mode, st);
}
template <typename T>
void row_fwd_call(int L, const RowFwdArgs<T>& a, hipStream_t st) {
#define FWI_X(LL) \
  case LL: launch_row_fwd_v<T, LL, 0>(a, st); return;
  switch (L) { FWI_OP_LENGTHS(FWI_X) }
#undef FWI_X
  const int v = tune_variant(PK_ROW_FWD, sizeof(T) == 8, L);
  FWI_LENGTHS(launch_row_fwd_v, L, v, a, st);
}
template <typename T>
void row_inv_call(int L, const RowInvArgs<T>& a, int epi, hipStream_t st) {
#define FWI_X(LL) \
  case LL: launch_row_inv_v<T, LL, 0>(a, epi, st); return;
  switch (L) { FWI_OP_LENGTHS(FWI_X) }
#undef FWI_X
  const int v = tune_variant(PK_ROW_INV, sizeof(T) == 8, L);
  FWI_LENGTHS(launch_row_inv_v, L, v, a, epi, st);
}
// rows per workgroup of the inverse row pass that row_inv_call will launch
template <typename T, int L, int V>
void row_inv_nl_v(int& nl) {
  nl = row_nl<T, L, V>();
}
template <typename T>
int row_inv_nl(int L) {
#define FWI_X(LL) \
  case LL: return row_nl<T, LL, 0>();
  switch (L) { FWI_OP_LENGTHS(FWI_X) }
#undef FWI_X
  const int v = tune_variant(PK_ROW_INV, sizeof(T) == 8, L);
  int nl = 0;
  FWI_LENGTHS(row_inv_nl_v, L, v, nl);
  return nl;
}

// The convolution pass runs tile-major (conv_item) when one frequency's
// spectrum exceeds an XCD's 4 MiB L2: swept plane by plane, it would be
// streamed from HBM once per right-hand side.
inline int conv_tile_major(const Geo& g, size_t es) { return g.npad() * (long)es > (4L << 20) ? 1 : 0; }

}  // namespace fwi
#include "xy_passes.hpp"
namespace fwi {

// Arguments of the fused lateral-elevation passes of geometry g.
template <typename T>
XyArgs<T> xy_args(const Geo& g, const Twiddles& tw, int B, const int* active, cplx<T>* U2) {
  XyArgs<T> a{};
  a.nx = g.nx;
  a.ny = g.ny;
  a.nz = g.nz;
  a.Lx = g.Lx;
  a.Ly = g.Ly;
  a.B = B;
  a.active = active;
  a.twx = tw.get<T>(g.Lx);
  a.twy = tw.get<T>(g.Ly);
  a.twm = tw.get<T>(g.Lx / 4);
  a.twh = tw.get<T>(g.Ly / 2);
  a.U2 = U2;
  return a;
}

template <typename T>
void launch_vie_rows(const Geo& g, const Twiddles& tw, int B, const cplx<T>* x, const int* active, const cplx<T>* m,
                     cplx<T>* U1, hipStream_t st, const XUpdate* xu, const OrthIn* orth, const StartIn* start,
                     cplx<T>* U2) {
  const long rows_per_rhs = (long)g.nz * g.ny;
  const double es = sizeof(cplx<T>);
  const bool masked = active != nullptr;  // converged RHS skipped (profiled bytes)
  const double n = (double)g.n();
  const int po = sizeof(T) == 8 ? KC_COUNT : 0;  // FP64 launches are separate classes
  RowFwdArgs<T> f{};
  f.x = x;
  f.m = m;
  f.active = active;
  f.out = U1;
  f.tw = tw.get<T>(g.Lx);
  f.nrows = rows_per_rhs * B;
  f.rows_per_rhs = (int)rows_per_rhs;
  f.nin = g.nx;
  f.in_stride = g.nx;
  // per RHS: x read, the x-pass intermediate written (m once)
  double per_rhs = (n + g.u1()) * es;
  if ((xu != nullptr) + (orth != nullptr) + (start != nullptr) > 1) throw Error(-6, "one combined input per pass");
  if (xu) {
    if (sizeof(T) != 8 || active) throw Error(-6, "the fused solution update is for complex128 residuals");
    f.kind = xu->fp32 ? RI_UPD32 : RI_UPD64;
    f.lc_basis = xu->basis;
    f.lc_vs = xu->vs;
    f.lc_ncol = xu->ncol;
    f.lc_coef = xu->coef;
    f.lc_cstride = xu->cstride;
    f.lc_first = xu->first;
    f.lc_out = const_cast<cplx<T>*>(x);
    // x read (unless first) and written, up to kmax basis vectors read
    per_rhs = g.u1() * es + n * es * (xu->first ? 1.0 : 2.0) + (double)xu->kmax * n * (xu->fp32 ? 8.0 : 16.0);
  } else if (orth) {
    f.kind = orth->transform ? RI_ORTH : RI_ORTH_ONLY;
    f.lc_basis = orth->basis;
    f.lc_vs = orth->vs;
    f.lc_nvec = orth->nvec;
    f.lc_coef = orth->coef;
    f.lc_cstride = orth->cstride;
    f.lc_out = const_cast<cplx<T>*>(x);
    f.lc_rowpart = orth->rowpart;
    if (orth->ndot) {
      if (orth->nvec > kMaxDotVec) throw Error(-6, "too many vectors for the fused coefficient sum");
      f.kind = orth->transform ? RI_ORTH_SUM : RI_ORTH_ONLY_SUM;
      f.ndot = orth->ndot;
      f.nB = B;
      f.dotp = orth->dotp;
      f.vscale = static_cast<const cplx<T>*>(orth->vscale);
      f.H = orth->H;
    }
    // w read, nvec basis vectors read, v written, per-row norms (and the x-pass intermediate)
    per_rhs = (2.0 + orth->nvec) * n * es + 8.0 * rows_per_rhs + (orth->transform ? g.u1() * es : 0.0);
  } else if (start) {
    if (!m || active) throw Error(-6, "the start pass needs the contrast and every RHS");
    f.kind = RI_START;
    f.lc_src = start->b;
    f.lc_out = const_cast<cplx<T>*>(x);
    f.lc_rowpart = start->rowpart;
    // b read (complex128), V_0 written, per-row norms, the x-pass intermediate
    per_rhs = n * (16.0 + es) + 8.0 * rows_per_rhs + g.u1() * es;
  }
  // the orthogonalising first pass and the orthogonalisation alone are classes of their own
  const int cls = orth ? (orth->transform ? KC_ORTH_FWD : KC_ORTH) : KC_ROW_FWD;
  if constexpr (sizeof(T) == 4) {
    if (g.xy && f.ndot) throw Error(-6, "the fused lateral-elevation pass takes the coefficients");
    if (g.xy && !row_in_orth_only(f.kind)) {
      // fused lateral-elevation pass: the operand straight to the padded
      // spectrum U2 (class-major), no x-pass intermediate
      if (!U2) throw Error(-6, "the fused lateral-elevation pass needs the y-pass buffer");
      XyArgs<T> xa = xy_args<T>(g, tw, B, active, U2);
      xa.x = x;
      xa.m = m;
      xa.basis = static_cast<const cplx<T>*>(f.lc_basis);
      xa.vs = f.lc_vs;
      xa.nvec = f.lc_nvec;
      xa.coef = f.lc_coef;
      xa.cstride = f.lc_cstride;
      xa.xout = f.lc_out;
      xa.rowpart = f.lc_rowpart;
      xa.src = f.lc_src;
      prof_begin(cls + po, st);
      FWI_XY_SHAPES(launch_xy_fwd_s, T, g.Lx / 4, g.Ly / 2, xa, f.kind, st);
      prof_end(cls + po, st, per_rhs + (double)(g.u2() - g.u1()) * es, n * es, masked, B);
      return;
    }
  }
  prof_begin(cls + po, st);
  row_fwd_call<T>(g.Lx, f, st);
  prof_end(cls + po, st, per_rhs, n * es, masked, B);
}

template <typename T>
void launch_vie_tail(const Geo& g, const Twiddles& tw, int B, const cplx<T>* x, const cplx<T>* scale,
                     const int* active, const cplx<T>* ghat, const int* rhs_freq, cplx<T>* U1, cplx<T>* U2,
                     cplx<T>* y, const cplx<T>* rhs, int epi, hipStream_t st, c64* y32, double* rowpart,
                     VieDots* dots) {
  const long rows_per_rhs = (long)g.nz * g.ny;
  const double es = sizeof(cplx<T>);
  const bool masked = active != nullptr;  // converged RHS skipped (profiled bytes)
  const double gbytes = (double)(tl_nfreq > 0 ? tl_nfreq : 1) * g.npad() * es;
  const double n = (double)g.n();
  const int po = sizeof(T) == 8 ? KC_COUNT : 0;  // FP64 launches are separate classes
  if constexpr (sizeof(T) == 4) {
    if (g.xy) {
      // U2 holds the class-major padded spectrum (launch_vie_rows): the
      // convolution along z, then the fused inverse lateral-elevation pass
      StridedArgs<T> c{};
      c.in = U2;
      c.out = U2;
      c.tw = tw.get<T>(g.Lz);
      c.ghat = ghat;
      c.rhs_freq = rhs_freq;
      c.active = active;
      c.in_ps = c.out_ps = (long)g.nz * g.Ly * g.Lx;
      c.pstride = (long)g.Ly * g.Lx;
      c.gstride = g.npad();
      c.gpstride = (long)g.Ly * g.Lx;
      c.nlines = g.Ly * g.Lx;
      c.planes_per_rhs = 1;
      c.lin = c.lout = g.nz;
      c.tile_major = conv_tile_major(g, sizeof(cplx<T>));
      prof_begin(KC_CONV + po, st);
      strided_call<T>(g.Lz, c, B, 2, st);
      prof_end(KC_CONV + po, st, 2.0 * g.u2() * es, gbytes, masked, B);
      if (epi != EPI_VIE && epi != EPI_COPY) throw Error(-6, "the fused lateral-elevation pass has no residual epilogue");
      XyArgs<T> xa = xy_args<T>(g, tw, B, active, U2);
      xa.x = x;
      xa.scale = scale;
      xa.y = y;
      if (dots) {
        dots->nparts = 0;
        if (epi == EPI_VIE && fused_dot_parts(g.nz, 1, dots->nvec)) {
          epi = EPI_VIE_DOT;
          xa.dbasis = static_cast<const cplx<T>*>(dots->basis);
          xa.dvs = dots->vs;
          xa.dnvec = dots->nvec;
          xa.vscale = static_cast<const cplx<T>*>(dots->vscale);
          xa.dotp = dots->dotp;
          xa.dstride = dots->dstride;
          dots->nparts = g.nz;
        }
      }
      const double epi_bytes = epi == EPI_VIE_DOT ? (2.0 + (dots ? dots->nvec : 0)) * n * es
                               : epi == EPI_VIE   ? 2.0 * n * es
                                                  : n * es;
      prof_begin(KC_ROW_INV + po, st);
      FWI_XY_SHAPES(launch_xy_inv_s, T, g.Lx / 4, g.Ly / 2, xa, epi, st);
      prof_end(KC_ROW_INV + po, st, (double)g.u2() * es + epi_bytes, 0.0, masked, B);
      return;
    }
  }
  const LaunchSize conv_size = strided_size(g, B, PK_CONV, sizeof(cplx<T>));
  const LaunchSize y_size = strided_size(g, B, PK_STRIDED, sizeof(cplx<T>));
  if (g.dim == 2) {
    // pass 2: columns along z, convolution, in place
    StridedArgs<T> s{};
    s.in = U1;
    s.out = U1;
    s.tw = tw.get<T>(g.Lz);
    s.ghat = ghat;
    s.rhs_freq = rhs_freq;
    s.active = active;
    s.in_ps = s.out_ps = (long)g.nz * g.Lx;
    s.pstride = g.Lx;
    s.gstride = g.npad();
    s.gpstride = g.Lx;
    s.nlines = g.Lx;
    s.planes_per_rhs = 1;
    s.lin = s.lout = g.nz;
    s.tile_major = conv_tile_major(g, sizeof(cplx<T>));
    prof_begin(KC_CONV + po, st);
    strided_call<T>(g.Lz, s, B, 2, st, &conv_size);
    prof_end(KC_CONV + po, st, 2.0 * g.u1() * es, gbytes, masked, B);
  } else {
    // forward along y: U1 [b][z][ny][Lx] -> U2 [b][z][Ly][Lx]
    StridedArgs<T> s{};
    s.in = U1;
    s.out = U2;
    s.tw = tw.get<T>(g.Ly);
    s.active = active;
    s.in_ps = (long)g.ny * g.Lx;
    s.out_ps = (long)g.Ly * g.Lx;
    s.pstride = g.Lx;
    s.nlines = g.Lx;
    s.planes_per_rhs = g.nz;
    s.lin = g.ny;
    s.lout = g.Ly;
    prof_begin(KC_Y_FWD + po, st);
    strided_call<T>(g.Ly, s, (long)B * g.nz, 0, st, &y_size);
    prof_end(KC_Y_FWD + po, st, (double)(g.u1() + g.u2()) * es, 0.0, masked, B);
    // convolution along z, in place on U2
    StridedArgs<T> c{};
    c.in = U2;
    c.out = U2;
    c.tw = tw.get<T>(g.Lz);
    c.ghat = ghat;
    c.rhs_freq = rhs_freq;
    c.active = active;
    c.in_ps = c.out_ps = (long)g.nz * g.Ly * g.Lx;
    c.pstride = (long)g.Ly * g.Lx;
    c.gstride = g.npad();
    c.gpstride = (long)g.Ly * g.Lx;
    c.nlines = g.Ly * g.Lx;
    c.planes_per_rhs = 1;
    c.lin = c.lout = g.nz;
    c.tile_major = conv_tile_major(g, sizeof(cplx<T>));
    prof_begin(KC_CONV + po, st);
    strided_call<T>(g.Lz, c, B, 2, st, &conv_size);
    prof_end(KC_CONV + po, st, 2.0 * g.u2() * es, gbytes, masked, B);
    // inverse along y with crop: U2 -> U1
    StridedArgs<T> v{};
    v.in = U2;
    v.out = U1;
    v.tw = tw.get<T>(g.Ly);
    v.active = active;
    v.in_ps = (long)g.Ly * g.Lx;
    v.out_ps = (long)g.ny * g.Lx;
    v.pstride = g.Lx;
    v.nlines = g.Lx;
    v.planes_per_rhs = g.nz;
    v.lin = g.Ly;
    v.lout = g.ny;
    prof_begin(KC_Y_INV + po, st);
    strided_call<T>(g.Ly, v, (long)B * g.nz, 1, st, &y_size);
    prof_end(KC_Y_INV + po, st, (double)(g.u1() + g.u2()) * es, 0.0, masked, B);
  }
  // last pass: rows along x, inverse, crop, epilogue
  RowInvArgs<T> r{};
  r.in = U1;
  r.x = x;
  r.rhs = rhs;
  r.scale = scale;
  r.active = active;
  r.y = y;
  r.tw = tw.get<T>(g.Lx);
  r.nrows = rows_per_rhs * B;
  r.rows_per_rhs = (int)rows_per_rhs;
  r.nout = g.nx;
  r.y32 = y32;
  r.rowpart = rowpart;
  if (dots) {
    dots->nparts = 0;
    const int nl = row_inv_nl<T>(g.Lx);
    const int parts = fused_dot_parts(rows_per_rhs, nl, dots->nvec);
    if (epi == EPI_VIE && parts) {
      epi = EPI_VIE_DOT;
      r.basis = static_cast<const cplx<T>*>(dots->basis);
      r.vs = dots->vs;
      r.nvec = dots->nvec;
      r.vscale = static_cast<const cplx<T>*>(dots->vscale);
      r.B = B;
      r.dotp = dots->dotp;
      r.dstride = dots->dstride;
      dots->nparts = parts;
    }
  }
  // per RHS: the x-pass intermediate, then x and y (VIE), or x, rhs, the
  // residual (complex128 or complex64) and one norm partial per row
  const double rows = (double)g.nz * g.ny;
  const double epi_bytes = epi == EPI_RESID     ? 3.0 * n * es + 8.0 * rows
                           : epi == EPI_RESID32 ? (2.0 * es + 8.0) * n + 8.0 * rows
                           : epi == EPI_VIE_DOT ? (2.0 + (dots ? dots->nvec : 0)) * n * es
                                                : 2.0 * n * es;
  prof_begin(KC_ROW_INV + po, st);
  row_inv_call<T>(g.Lx, r, epi, st);
  prof_end(KC_ROW_INV + po, st, (double)g.u1() * es + epi_bytes, 0.0, masked, B);
}

template <typename T>
void launch_vie(const Geo& g, const Twiddles& tw, int B, const cplx<T>* x, const cplx<T>* scale, const int* active,
                const cplx<T>* m, const cplx<T>* ghat, const int* rhs_freq, cplx<T>* U1, cplx<T>* U2, cplx<T>* y,
                const cplx<T>* rhs, int epi, hipStream_t st, c64* y32, double* rowpart, VieDots* dots,
                const XUpdate* xu) {
  launch_vie_rows<T>(g, tw, B, x, active, m, U1, st, xu, nullptr, nullptr, U2);
  launch_vie_tail<T>(g, tw, B, x, scale, active, ghat, rhs_freq, U1, U2, y, rhs, epi, st, y32, rowpart, dots);
}

#ifdef FWI_FFT_WITH_FULL
void launch_fft_full(const Geo& g, const Twiddles& tw, c128* u, hipStream_t st) {
  // every pass in place: a workgroup reads all its lines before it stores any
  RowFwdArgs<double> f{};
  f.x = u;
  f.out = u;
  f.tw = tw.get<double>(g.Lx);
  f.nrows = (long)g.Lz * g.Ly;
  f.rows_per_rhs = (int)f.nrows;
  f.nin = g.Lx;
  f.in_stride = g.Lx;
  row_fwd_call<double>(g.Lx, f, st);
  if (g.dim == 3) {
    StridedArgs<double> s{};
    s.in = u;
    s.out = u;
    s.tw = tw.get<double>(g.Ly);
    s.in_ps = s.out_ps = (long)g.Ly * g.Lx;
    s.pstride = g.Lx;
    s.nlines = g.Lx;
    s.planes_per_rhs = g.Lz;
    s.lin = s.lout = g.Ly;
    strided_call<double>(g.Ly, s, g.Lz, 0, st);
  }
  StridedArgs<double> z{};
  z.in = u;
  z.out = u;
  z.tw = tw.get<double>(g.Lz);
  z.in_ps = z.out_ps = 0;
  z.pstride = (long)g.Ly * g.Lx;
  z.nlines = g.Ly * g.Lx;
  z.planes_per_rhs = 1;
  z.lin = z.lout = g.Lz;
  strided_call<double>(g.Lz, z, 1, 0, st);
}

#endif

template <typename T>
void launch_fft_padded(const Geo& g, const Twiddles& tw, const cplx<T>* in, cplx<T>* U1, cplx<T>* out,
                       hipStream_t st) {
  RowFwdArgs<T> f{};
  f.x = in;
  f.out = U1;
  f.tw = tw.get<T>(g.Lx);
  f.nrows = (long)g.nz * g.ny;
  f.rows_per_rhs = (int)f.nrows;
  f.nin = g.nx;
  f.in_stride = g.nx;
  row_fwd_call<T>(g.Lx, f, st);
  const cplx<T>* cur = U1;
  long cur_ny = g.ny;
  if (g.dim == 3) {
    // y pass: U1 [nz][ny][Lx] -> out [nz][Ly][Lx] (rows z < nz), then z pass in place
    StridedArgs<T> s{};
    s.in = U1;
    s.out = out;
    s.tw = tw.get<T>(g.Ly);
    s.in_ps = (long)g.ny * g.Lx;
    s.out_ps = (long)g.Ly * g.Lx;
    s.pstride = g.Lx;
    s.nlines = g.Lx;
    s.planes_per_rhs = g.nz;
    s.lin = g.ny;
    s.lout = g.Ly;
    strided_call<T>(g.Ly, s, g.nz, 0, st);
    cur = out;
    cur_ny = g.Ly;
  }
  StridedArgs<T> z{};
  z.in = cur;
  z.out = out;
  z.tw = tw.get<T>(g.Lz);
  z.in_ps = z.out_ps = 0;
  z.pstride = (long)cur_ny * g.Lx;
  z.nlines = (int)(cur_ny * g.Lx);
  z.planes_per_rhs = 1;
  z.lin = g.nz;
  z.lout = g.Lz;
  strided_call<T>(g.Lz, z, 1, 0, st);
}

}  // namespace fwi
