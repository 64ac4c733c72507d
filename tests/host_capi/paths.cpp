// Single calls of the C ABI on the host stand-in (see driver.cpp), each a
// condition that the call sequences there do not set up. Prints "ok <name>" per
// check; run under the sanitizers.
#include <algorithm>
#include <complex>
#include <cstdio>
#include <cstdlib>
#include <string>
#include <vector>

#include "data.hpp"
#include "emu.hpp"
#include "fwi.h"
#include "internal.hpp"

namespace {

using cd = std::complex<double>;
int g_fail = 0;
void expect(bool ok, const char* what) {
  std::printf("%s %s\n", ok ? "ok" : "FAILED", what);
  if (!ok) g_fail = 1;
}

struct Prob {
  fwi_problem p{};
  std::vector<double> f, e;
  long n = 0, npad = 0;
  Prob(int nx, int ny, int nz, int ne, int nf) {
    p.dim = ny > 1 ? 3 : 2;
    p.nx = nx;
    p.ny = ny;
    p.nz = nz;
    p.dx = 0.154e-3;
    p.c0 = 1540.0;
    p.nf = nf;
    p.ne = ne;
    for (int l = 0; l < nf; ++l) f.push_back(0.3e6 + 0.1e6 * l);
    for (int k = 0; k < ne; ++k) {
      e.push_back((k + 0.5) / ne * nx * p.dx);
      e.push_back(p.dim == 3 ? ny * p.dx / 2 : 0.0);
      e.push_back(0.0);
    }
    p.freq_hz = f.data();
    p.elem_xyz = e.data();
    n = (long)nx * ny * nz;
    npad = (long)fwi_padded_length(nx) * (ny > 1 ? fwi_padded_length(ny) : 1) * fwi_padded_length(nz);
  }
};

// The spectrum call takes no memory on any grid, also where the operator pads
// to other lengths than the call's, and leaves a caller's workspace alone.
void spectrum(fwi_ctx* ctx) {
  for (int k = 0; k < 4; ++k) {
    Prob q = k == 0 ? Prob(37, 1, 70, 3, 2) : k == 1 ? Prob(40, 36, 30, 2, 1) : k == 2 ? Prob(64, 1, 64, 2, 1) : Prob(33, 20, 40, 2, 1);
    std::vector<cd> p0((size_t)q.p.ne * q.n), out((size_t)q.npad);
    bool ok = fwi_incident(ctx, &q.p, 0, p0.data()) == FWI_OK;  // the problem's cache
    std::vector<char> ws(256, 7);
    for (int own = 0; own < 2; ++own) {
      if (own) fwi_set_workspace(ctx, ws.data(), ws.size());
      emu::malloc_left = 0;
      const long before = emu::malloc_calls;
      ok = ok && fwi_green_spectrum(ctx, &q.p, q.p.nf - 1, out.data()) == FWI_OK && emu::malloc_calls == before;
      emu::malloc_left = -1;
      fwi_set_workspace(ctx, nullptr, 0);
    }
    for (char v : ws) ok = ok && v == 7;
    expect(ok, "spectrum without memory");
  }
}

// Element-wise launches over any count: contiguous pieces, each well below the
// 2^32 work items that a launch holds.
void launches(fwi_ctx*) {
  for (long count : {0L, 1L, 1L << 30, (1L << 30) + 1, 1L << 32, (5L << 32) + 3}) {
    long next = 0;
    bool ok = true;
    fwi::in_launches(count, [&](long o, long c) {
      ok = ok && o == next && c > 0 && (c + 255) / 256 * 256 < (1L << 32);
      next = o + c;
    });
    expect(ok && next == count, "launch pieces");
  }
}

// The tile of a strided pass: by the launch's size where no table entry is, the
// entry's at every size, and the tuner compares with the former.
void tiles(fwi_ctx* ctx) {
  using namespace fwi;
  Geo g2{}, g3{};
  g2.dim = 2, g2.nx = g2.nz = 64, g2.Lx = g2.Lz = 128, g2.ny = g2.Ly = 1;
  g3.dim = 3, g3.nx = g3.ny = 128, g3.nz = 96, g3.Lx = g3.Ly = 256, g3.Lz = 192;
  const size_t es = sizeof(c128);
  auto conv = [&](int B) { return default_variant(PK_CONV, true, 128, strided_size(g2, B, PK_CONV, es)); };
  auto elev = [&](int B) { return default_variant(PK_STRIDED, true, 256, strided_size(g3, B, PK_STRIDED, es)); };
  expect(conv(4) == 0 && conv(16) == 0 && conv(64) == 0 && conv(1024) == 0 && conv(2048) == 1, "convolution");
  expect(elev(1) == 0 && elev(2) == 1 + 1 && elev(32) == 2, "elevation");
  FftTuning table;
  tl_tune = &table;
  table.v[PK_CONV][1][length_index(128)] = 1;
  bool ok = true;
  for (int B : {1, 16, 4096}) ok = ok && tune_variant(PK_CONV, true, 128, strided_size(g2, B, PK_CONV, es)) == 1;
  tl_tune = nullptr;
  expect(ok, "table entry at every size");
  Prob small(64, 1, 64, 4, 1);
  fwi_tune_report r{};
  ok = fwi_autotune(ctx, &small.p, FWI_FP64, 4, 1, &r) == FWI_OK && r.default_variant[1] == 0;
  expect(ok, "tuner's default on a short launch");
}

// Splits of the sampling product: the matrix units' work of the fullest compute
// unit (workgroups in rounds of 256, each a split's points) may not exceed that of
// the coarsest count, one split per 1024 points, by more than 3%; a chunk
// of the transmits has the splits of the whole problem.
void splits(fwi_ctx* ctx) {
  const int cases[][5] = {{256, 256, 3, 33, 33}, {64, 64, 4, 128, 128}, {96, 80, 8, 64, 64}, {150, 100, 5, 48, 21},
                          {128, 64, 4, 128, 100}, {40, 30, 1, 7, 3}, {3, 2, 1, 1, 1}};
  for (auto& k : cases) {
    Prob q(k[0], 1, k[1], k[3], k[2]);
    const int nf = k[2], ne = k[3], nt = k[4];
    std::vector<cd> tx((size_t)nf * nt * q.n), rx((size_t)nf * ne * q.n), a(q.n), out((size_t)nf * nt * ne);
    bool ok = fwi_jacobian_apply_tx(ctx, &q.p, nt, tx.data(), rx.data(), a.data(), out.data()) == FWI_OK;
    auto rounds = [&](int s) {
      const long chunk = fwi::gemm_chunk(q.n, s), r = (q.n + chunk - 1) / chunk;
      return (double)chunk * (double)((r * nf * ((nt + 63) / 64) * ((ne + 63) / 64) + 255) / 256);
    };
    ok = ok && emu::gemm_splits >= 1 && rounds(emu::gemm_splits) <= 1.03 * rounds((int)((q.n + 1023) / 1024));
    expect(ok, "splits fill their rounds");
  }
  Prob q(48, 1, 40, 20, 3);
  std::vector<double> c(q.n, 1540.0);
  std::vector<cd> data((size_t)3 * 20 * 20);
  fwi_solve_opts o;
  fwi_default_opts(&o);
  int seen[3];
  for (int k = 0; k < 3; ++k) {
    o.max_rhs = k == 1 ? 20 : 0;
    o.tx_chunk = k == 2 ? 7 : 0;
    fwi_forward(ctx, &q.p, c.data(), nullptr, &o, data.data(), nullptr, nullptr);
    seen[k] = emu::gemm_splits;
  }
  expect(seen[0] == seen[1] && seen[0] == seen[2], "one count for every chunk");
}

// A batch in a caller's workspace: the splits of the call without one where they
// fit, one per 1024 points in a smaller one, and NOMEM below that.
void batch_workspace(fwi_ctx* ctx) {
  Prob q(64, 1, 64, 64, 1);
  std::vector<double> c(q.n, 1540.0);
  std::vector<cd> d0(64 * 64), d1(64 * 64);
  const fwi_problem probs[2] = {q.p, q.p};
  const double* cs[2] = {c.data(), c.data()};
  void* outs[2] = {d0.data(), d1.data()};
  fwi_solve_opts o;
  fwi_default_opts(&o);
  o.restart = 8;
  fwi_batch_stats st{};
  auto run = [&](size_t bytes) {
    std::vector<char> ws(bytes);
    fwi_set_workspace(ctx, bytes ? ws.data() : nullptr, bytes);
    const int rc = fwi_forward_batch(ctx, 2, probs, cs, nullptr, &o, outs, &st);
    fwi_set_workspace(ctx, nullptr, 0);
    return rc;
  };
  bool ok = run(0) == FWI_OK;
  const int full = emu::gemm_splits;
  size_t lo = 0, hi = size_t(256) << 20;  // the least workspace that is accepted
  ok = ok && full > 4 && run(hi) == FWI_OK && emu::gemm_splits == full;
  expect(ok, "ample workspace: the splits of the call without one");
  while (hi - lo > 4096) {
    const size_t mid = (lo + hi) / 2;
    (run(mid) == FWI_OK ? hi : lo) = mid;
  }
  ok = run(hi) == FWI_OK && emu::gemm_splits < full;
  expect(ok, "least workspace: fewer splits");
  expect(run(lo) == FWI_E_NOMEM, "below it: refused");
}

// Where the coefficients of an Arnoldi step are summed: in the orthogonalising
// pass on short launches with the built-in row tile, else in a kernel of its own,
// one launch per step; and where the inner products are a kernel of their own.
void sums(fwi_ctx* ctx) {
  signed char none[88], wide[88];
  std::fill(none, none + 88, (signed char)-1);
  std::copy(none, none + 88, wide);
  for (int d = 0; d < 2; ++d)
    for (int l = 0; l < 11; ++l) wide[(fwi::PK_ROW_FWD * 2 + d) * 11 + l] = 1;
  struct {
    Prob q;
    const signed char* table;
    bool own_sum, own_dots;
  } cases[] = {{Prob(37, 1, 70, 5, 2), none, false, false},    // ragged last part
               {Prob(37, 1, 37, 5, 2), wide, false, false},    // length 80 has no tuned tile
               {Prob(64, 1, 50, 5, 2), wide, true, false},     // tuned row tile
               {Prob(16, 20, 210, 2, 1), none, true, false},   // 66 parts
               {Prob(120, 1, 130, 61, 4), none, true, false},  // 17 parts, 244 right-hand sides
               {Prob(20, 1, 13, 3, 1), none, false, true}};    // fewer rows than a workgroup's
  for (auto& k : cases) {
    fwi_set_tuning(ctx, k.table, 88);
    std::vector<double> c(k.q.n, 1540.0);
    std::vector<cd> data((size_t)k.q.p.nf * k.q.p.ne * k.q.p.ne);
    bool ok = true;
    for (int prec = 0; prec < 2; ++prec) {
      fwi_solve_opts o;
      fwi_default_opts(&o);
      o.restart = 8;
      o.precision = prec;
      const long s0 = emu::launches("hsum"), d0 = emu::launches("dots"), g0 = emu::launches("givens");
      ok = ok && fwi_forward(ctx, &k.q.p, c.data(), nullptr, &o, data.data(), nullptr, nullptr) == FWI_OK;
      const long steps = emu::launches("givens") - g0;
      ok = ok && steps > 0;
      // (a step enqueued after the last right-hand side stopped may lack its rotations)
      const long s = emu::launches("hsum") - s0, d = emu::launches("dots") - d0;
      ok = ok && (k.own_sum ? s >= steps : s == 0) && (k.own_dots ? d >= steps : d == 0);
    }
    expect(ok, "sums");
  }
  fwi_set_tuning(ctx, nullptr, 0);
}

}  // namespace

int main(int argc, char** argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  fwi_ctx* ctx = nullptr;
  if (fwi_create(&ctx, 0, nullptr) != FWI_OK) return 1;
  if (what == "spectrum") spectrum(ctx);
  if (what == "launches") launches(ctx);
  if (what == "tiles") tiles(ctx);
  if (what == "splits") splits(ctx);
  if (what == "sums") sums(ctx);
  if (what == "batch") batch_workspace(ctx);
  fwi_destroy(ctx);
  if (emu::counts().violations) g_fail = 1;
  return g_fail;
}
