// Family 1, DIRECT_F32: launcher. The kernel and its description are in
// k_direct.inc.h; the instantiations live in one unit per MK value.
#include "k_direct.inc.h"

namespace ct {

DirectFn pick_direct_mk1(int mw, int lds, int spec, int unr, bool alt);
DirectFn pick_direct_mk2(int mw, int lds, int spec, int unr, bool alt);
DirectFn pick_direct_mk4(int mw, int lds, int spec, int unr, bool alt);
DirectFn pick_direct_mk8(int mw, int lds, int spec, int unr, bool alt);

static DirectFn pick_direct(int mk, int mw, int lds, int spec, int unr, bool alt) {
  switch (mk) {
    case 1: return pick_direct_mk1(mw, lds, spec, unr, alt);
    case 2: return pick_direct_mk2(mw, lds, spec, unr, alt);
    case 4: return pick_direct_mk4(mw, lds, spec, unr, alt);
    default: return pick_direct_mk8(mw, lds, spec, unr, alt);
  }
}

int launch_direct_f32(const OpX& x, const ct_schedule& s, const Geom& g, const void* xin,
                      const void* w, void* y, float* ws, void* stream) {
  using namespace direct_knob;
  const ct_op& o = x.op;
  DirectArgs a;
  a.N = o.n; a.C = o.c; a.H = o.h; a.W = o.w; a.K = o.k; a.R = o.r; a.S = o.s;
  a.sh = o.stride_h; a.sw = o.stride_w; a.ph = o.pad_h; a.pw = o.pad_w; a.dh = o.dil_h; a.dw = o.dil_w;
  a.OH = (int)x.oh; a.OW = (int)x.ow;
  a.toh = s.knob[TOH]; a.tow = s.knob[TOW]; a.tk = s.knob[TK]; a.ct = s.knob[CT];
  a.tiles_w = (int)g.tiles_w;
  a.split = g.split; a.cps = g.chunks_per_split;
  a.ih_t = g.ih_t; a.iw_t = g.iw_t;
  a.threads = g.threads;
  a.cols = a.tow / s.knob[MW];
  a.tp = a.toh * a.cols;
  a.pitch = g.d_pitch; a.wpc = g.d_wpc; a.ks = g.d_ks; a.wt = g.d_wt;
  a.inv_tp = 1.0f / (float)a.tp;
  a.inv_cols = 1.0f / (float)a.cols;
  a.deep_x = a.deep_w = a.vec_w = 0;
  a.inv_plane = a.inv_pitch = a.inv_ks = a.inv_wpc = a.inv_wq = 0.f;
  if (s.knob[LDS]) {
    a.inv_plane = 1.0f / (float)(a.ih_t * a.pitch);
    a.inv_pitch = 1.0f / (float)a.pitch;
    a.inv_ks = 1.0f / (float)a.ks;
    a.inv_wpc = 1.0f / (float)a.wpc;
    // deep chunks: 16-byte copies where the filter rows are whole quads (d_alt)
    // and w is aligned; plane by plane (slice by slice) where a plane
    // fills at least half of the rows of threads it takes
    auto fills = [&](int words) { return 2 * words > ((words + a.threads - 1) / a.threads) * a.threads; };
    a.vec_w = g.d_alt && (uintptr_t)w % 16 == 0;
    if (a.vec_w) a.inv_wq = 4.0f / (float)a.wpc;
    a.deep_x = fills(a.ih_t * a.pitch);
    a.deep_w = fills(a.vec_w ? a.ks / 4 : a.ks);
  }
  a.ny = x.ny;
  DirectFn fn = pick_direct(s.knob[MK], s.knob[MW], s.knob[LDS], g.spec, s.knob[UNR], g.d_alt);
  dim3 grid((unsigned)(g.tiles_h * g.tiles_w), (unsigned)g.tiles_k, (unsigned)g.tiles_n);
  float* out = g.split > 1 ? ws : (float*)y;
  hipLaunchKernelGGL(fn, grid, dim3(g.threads), g.lds_bytes, (hipStream_t)stream, (const float*)xin,
                     (const float*)w, out, a);
  if (hipGetLastError() != hipSuccess) return -1;
  if (g.split > 1) return launch_split_reduce(ws, (float*)y, x.ny, g.split, stream);
  return 0;
}

}  // namespace ct
