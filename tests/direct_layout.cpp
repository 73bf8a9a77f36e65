// LDS layout of the direct family, checked on the host: for every valid schedule with LDS
// of the ops listed in the input file (one per line, the 16 numbers of ct_op), the words
// that the kernel's copies write and its windows read lie inside the block's LDS, wide
// reads are aligned, and a chunk goes the way the instance's registers allow. Prints one
// line per op and "done"; any fault ends the run with status 1. With a second argument
// also how each schedule's chunks go, in the words of direct_paths.py.
#include <cstdint>
#include <cstdio>
#include <vector>

#include "ct_internal.h"

using namespace ct;
namespace ct {
void set_error(const std::string&) {}
}  // namespace ct

static int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

#define CHECK(cond)                                                                          \
  do {                                                                                       \
    if (!(cond)) {                                                                           \
      std::printf("FAIL %s: toh %d tow %d tk %d mk %d mw %d ct %d split %d spec %d alt %d\n", #cond, \
                  s.knob[TOH], s.knob[TOW], s.knob[TK], mk, mw, ct, s.knob[SPLIT], (int)g.spec, g.d_alt); \
      return 1;                                                                              \
    }                                                                                        \
  } while (0)

static int check(const OpX& x, const ct_schedule& s, const Geom& g, int* ways) {
  using namespace direct_knob;
  const ct_op& o = x.op;
  const int mk = s.knob[MK], mw = s.knob[MW], ct = s.knob[CT], groups = s.knob[TK] / mk;
  const int64_t threads = g.threads, words = g.lds_bytes / 4;
  const int64_t w0 = (int64_t)groups * g.d_ks, wt = g.d_wt, halo = cdiv(wt, 4) * 4;
  const int64_t plane = (int64_t)g.ih_t * g.d_pitch, xt = ct * plane;
  const int64_t nst = cdiv(wt, threads) + cdiv(xt, threads);
  const bool padded = g.spec != SPEC_GENERIC, deep = padded && g.d_alt;
  const int sc = direct_spec_s(g.spec), stc = direct_spec_stride(g.spec);
  CHECK(g.d_wpc == ct * o.r * o.s && g.d_ks >= g.d_wpc * mk && wt >= w0 && g.d_pitch >= g.iw_t);
  CHECK(halo + xt <= words && words <= kMaxLdsBytes / 4);
  const DirectRegs held = direct_regs(mk, mw, g.spec);
  const bool quads = padded && g.d_wpc % 4 == 0 && x.kred % 4 == 0;
  if (deep) {
    CHECK(quads && g.d_ks % 4 == 0);
    CHECK(cdiv(w0, 4 * threads) * 4 * threads <= halo);   // 16 bytes per lane, whole rows
    CHECK(halo + cdiv(xt, threads) * threads <= words);   // a word per lane, whole rows
    ++ways[2];
  } else if (nst <= held.staged) {
    CHECK(cdiv(wt, threads) * threads <= halo && halo + cdiv(xt, threads) * threads <= words);
    ++ways[0];
  } else {
    // a chunk that neither goes through registers nor has a plan: only where the filter
    // rows are no whole quads, in the generic path, or where whole rows exceed the LDS
    CHECK(!quads || 4 * (cdiv(w0, 4 * threads) * 4 * threads + cdiv(xt, threads) * threads) > kMaxLdsBytes);
    ++ways[1];
  }
  if (padded) {
    // the last window of the last thread, and the widest read its start allows
    const int64_t row = (int64_t)(s.knob[TOH] - 1) * o.stride_h + (int64_t)(o.r - 1) * o.dil_h;
    const int64_t col = (int64_t)(s.knob[TOW] - mw) * o.stride_w;
    const int window = sc == 1 ? (mw - 1) * stc + 1 : held.x_words;
    CHECK((ct - 1) * plane + row * g.d_pitch + col + window <= xt);
    if (!(sc == 1 && stc == 2)) {
      const int step = mw * stc, align = step % 4 == 0 ? 4 : (step % 2 == 0 ? 2 : 1);
      CHECK(g.d_pitch % align == 0);
    } else {
      CHECK(g.d_pitch == g.iw_t);  // read word by word: padded rows would only share banks
    }
  }
  return 0;
}

static void list(const ct_schedule& s, const Geom& g) {
  using namespace direct_knob;
  const int mk = s.knob[MK], threads = g.threads, groups = s.knob[TK] / mk;
  const DirectRegs held = direct_regs(mk, s.knob[MW], g.spec);
  auto rows = [&](int64_t words) { return (int)cdiv(words, threads); };
  auto fills = [&](int words) { return 2 * words > rows(words) * threads; };
  const int plane = g.ih_t * g.d_pitch, quads = g.d_ks / 4;
  const int64_t xt = (int64_t)s.knob[CT] * plane;
  const int nst = rows(g.d_wt) + rows(xt);
  for (int i = 0; i < COUNT; ++i) std::printf("%d ", s.knob[i]);
  if (g.spec != SPEC_GENERIC && g.d_alt) {
    if (rows((int64_t)groups * quads) <= held.plan && rows(xt) <= held.plan)
      std::printf("plan\n");
    else
      std::printf("deep %d %d %d\n", fills(plane), fills(quads), fills(g.d_ks));
  } else if (nst <= held.staged) {
    std::printf("staged %d\n", nst);
  } else {
    std::printf("copied %d %d\n", fills(plane), fills(g.d_ks));
  }
}

int main(int argc, char** argv) {
  std::FILE* f = argc > 1 ? std::fopen(argv[1], "r") : nullptr;
  if (!f) return 2;
  ct_op op{};
  int ops = 0;
  while (std::fscanf(f, "%d %d %d %d %d %d %d %d %d %d %d %d %d %d %d %d", &op.n, &op.c, &op.h, &op.w, &op.k, &op.r,
                     &op.s, &op.stride_h, &op.stride_w, &op.pad_h, &op.pad_w, &op.dil_h, &op.dil_w, &op.groups,
                     &op.dtype, &op.layout) == 16) {
    OpX x;
    std::string why;
    if (!derive_op(op, &x, &why)) return 2;
    const FamilyDef& fam = *family_def(CT_FAM_DIRECT_F32);
    int ways[3] = {0, 0, 0}, n = 0;
    for (int64_t i = 0; i < family_grid_size(fam); ++i) {
      ct_schedule s;
      Geom g;
      ct_grid_decode(CT_FAM_DIRECT_F32, i, &s);
      if (!s.knob[direct_knob::LDS] || compute_geom(x, s, &g, nullptr) != CT_OK) continue;
      ++n;
      if (check(x, s, g, ways)) return 1;
      if (argc > 2) list(s, g);
    }
    std::printf("op %d: %d schedules, %d through registers, %d copied, %d with a plan\n", ops++, n, ways[0], ways[1],
                ways[2]);
  }
  std::printf("done: %d ops\n", ops);
  return 0;
}
