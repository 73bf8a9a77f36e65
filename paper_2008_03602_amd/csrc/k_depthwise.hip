// Family 2, DEPTHWISE_F32: depthwise convolution (groups = C = K, one filter
// per channel) on the vector ALU, NCHW fp32. The operator does one
// multiply-add per filter tap and output, so its floor is memory traffic:
// the knobs trade parallelism against halo re-reads.
//
// A block computes TOH x TOW outputs for TC channels of NB images. A thread
// owns VEC output columns (TOW/VEC apart) in each of RPT consecutive output
// rows, so the lanes of a wave sweep consecutive columns.
// LDS = 1 stages the input halo tile of the block once; LDS = 0 reads taps
// straight from global memory (L1/L2 absorb the overlap). ORDER picks the
// block numbering: tiles fastest (0) or channel groups fastest (1).
// Q4 = 1 (3x3 filters with pad 1 only) switches to depthwise_q4_kernel: a
// thread owns 4 consecutive output columns of RPT consecutive rows, reads
// each input row it needs once with 16-byte loads (plus the edge words) and
// keeps the taps in registers, so a wave reads and writes whole 16-byte
// words and an output costs well under one load instruction instead of nine.
// Every global access is bounds-checked.
#include <hip/hip_runtime.h>

#include "ct_internal.h"
#include "k_util.h"

namespace ct {

struct DwArgs {
  int N, C, H, W, R, S, sh, sw, ph, pw, dh, dw;
  int OH, OW;
  int tc, toh, tow, nb, order;
  int ih_t, iw_t;
  int threads, rows, cols;
  FastDiv f_tw, f_th, f_tc;                              // block index over the tile counts
  float inv_cols, inv_rows, inv_tc, inv_plane, inv_iwt;  // see qdiv
  int st_n, st_c, st_h, st_w, st_p;  // a staging step of `threads` elements, as indices and as a plane offset
  int vec_ld, vec_st;  // depthwise_q4_kernel: 16-byte input loads / output stores allowed
};

// Threads per block of the strided kernel that leave registers for its
// outputs per thread (16 outputs need 256 VGPRs: at most 512 threads).
__host__ __device__ constexpr int dw_max_threads(int outs) { return outs >= 16 ? 512 : 1024; }
__host__ __device__ constexpr int dw_spec_r(int spec) { return spec == 3 || spec == 4 ? 3 : 0; }
__host__ __device__ constexpr int dw_spec_stride(int spec) { return spec == 3 ? 1 : (spec == 4 ? 2 : 0); }

// Block -> first channel and image of its group, first output row and column.
struct DwBlock {
  int c0, n0, oh0, ow0;
};
__device__ __forceinline__ DwBlock dw_block(const DwArgs& a) {
  int b = blockIdx.x, tw, th, cg, ng;
  if (a.order == 0) {
    const int q0 = fdiv(b, a.f_tw), q1 = fdiv(q0, a.f_th), q2 = fdiv(q1, a.f_tc);
    tw = b - q0 * a.f_tw.d; th = q0 - q1 * a.f_th.d; cg = q1 - q2 * a.f_tc.d; ng = q2;
  } else {
    const int q0 = fdiv(b, a.f_tc), q1 = fdiv(q0, a.f_tw), q2 = fdiv(q1, a.f_th);
    cg = b - q0 * a.f_tc.d; tw = q0 - q1 * a.f_tw.d; th = q1 - q2 * a.f_th.d; ng = q2;
  }
  return {cg * a.tc, ng * a.nb, th * a.toh, tw * a.tow};
}
// Thread -> (image, channel, row group, column group) of the block, columns fastest.
struct DwThread {
  int ni, ci, rowg, colg;
};
__device__ __forceinline__ DwThread dw_thread(const DwArgs& a) {
  const int t = threadIdx.x;
  const int q0 = qdiv(t, a.inv_cols), q1 = qdiv(q0, a.inv_rows), q2 = qdiv(q1, a.inv_tc);
  return {q2, q1 - q2 * a.tc, q0 - q1 * a.rows, t - q0 * a.cols};
}

// What bounds this kernel is vector instructions, not bytes: a 3x3 output needs 9 loads
// and 9 multiply-adds, and everything else is address work. So block and thread indices
// come from reciprocals instead of divisions, every global access is a buffer access at
// plane + row + column (an offset part outside the image sends the sum past the buffer,
// which reads 0 and stores nothing: one addition per access, no 64-bit address, no
// select), the RPT rows of a thread are consecutive (an input row is read once for all of
// its output rows) and the halo is copied straight into LDS with carry counters for its
// indices. Measured on MobileNet-v2 b16's 10 layers and a ragged one, the mean over
// 160 sampled schedules each, against divisions, 64-bit addresses and strided rows: 30.5
// to 18.7 us on the whole GPU, 102 to 56 us on a quarter.
// WIDE: a block whose planes span more than 32-bit part offsets reach (geom_depthwise);
// with LDS only the generic filter path has that variant (3x3, planes of 538 MB, 40
// sampled schedules: 159 ms with that path alone, 127 with the fixed ones without LDS).
template <int VEC, int RPT, bool LDS, int SPEC, bool WIDE>
__global__ void __launch_bounds__(dw_max_threads(VEC * RPT))
depthwise_f32_kernel(const float* __restrict__ x, const float* __restrict__ w, float* __restrict__ y,
                     DwArgs a) {
  constexpr int RC = dw_spec_r(SPEC), STC = dw_spec_stride(SPEC);
  static_assert(!WIDE || !LDS || RC == 0, "the fixed filters have no wide variant with LDS");
  const int R = RC ? RC : a.R, S = RC ? RC : a.S;
  const int sh = STC ? STC : a.sh, sw = STC ? STC : a.sw;
  const int dh = RC ? 1 : a.dh, dw = RC ? 1 : a.dw;
  const int ph = RC ? 1 : a.ph, pw = RC ? 1 : a.pw;
  const int H = a.H, W = a.W, C = a.C;

  const DwBlock bk = dw_block(a);
  const DwThread td = dw_thread(a);
  const int c = bk.c0 + td.ci, n = bk.n0 + td.ni;
  const bool live = c < C && n < a.N;
  const int oh = bk.oh0 + td.rowg * RPT;  // first output row of the thread

  // buffers from the block's first plane (and filter) on
  const int HW = H * W, OHW = a.OH * a.OW;
  const int64_t plane0 = (int64_t)bk.n0 * C + bk.c0, planes = (int64_t)a.N * C - plane0;
  auto range = [](int64_t bytes) { return bytes < kPartOob ? bytes : (int64_t)kPartOob; };
  const float* xb = x + plane0 * HW;
  const __amdgpu_buffer_rsrc_t rx = make_rsrc(xb, range(planes * HW * 4));
  const __amdgpu_buffer_rsrc_t rwt = make_rsrc(w + (int64_t)bk.c0 * R * S, range((int64_t)(C - bk.c0) * R * S * 4));
  const int wofs = live ? td.ci * R * S * 4 : kPartOob;

  float wv[RC ? RC * RC : 1];
  if constexpr (WIDE && RC != 0) {
#pragma unroll
    for (int i = 0; i < RC * RC; ++i) wv[i] = load_or_zero(w, (int64_t)c * RC * RC + i, live);
  } else if constexpr (RC != 0) {
#pragma unroll
    for (int r = 0; r < RC; ++r) bload3(rwt, wofs + r * 12, wv + r * 3);
  }
  float acc[RPT][VEC];
#pragma unroll
  for (int u = 0; u < RPT; ++u)
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[u][v] = 0.f;

  const int ih_org = bk.oh0 * sh - ph, iw_org = bk.ow0 * sw - pw;
  const int plane = a.ih_t * a.iw_t;
  extern __shared__ float smem[];
  if constexpr (LDS) {
    const int total = a.nb * a.tc * plane;
    if constexpr (WIDE) {
      for (int e = threadIdx.x; e < total; e += a.threads) {
        const int p = e / plane;  // (image, channel) pair within the block
        const int rem = e - p * plane;
        const int hh = rem / a.iw_t, ww = rem - hh * a.iw_t;
        const int pn = bk.n0 + p / a.tc, pc = bk.c0 + p % a.tc;
        const int gh = ih_org + hh, gw = iw_org + ww;
        const bool ok = pn < a.N && pc < C && (unsigned)gh < (unsigned)H && (unsigned)gw < (unsigned)W;
        smem[e] = load_or_zero(x, (((int64_t)pn * C + pc) * H + gh) * W + gw, ok);
      }
    } else {
      // element e = i * threads + t of the tile, [image][channel][row][column], goes to
      // LDS word e; its indices advance by `threads` elements per step with carries
      const int t = threadIdx.x;
      const int p0 = qdiv(t, a.inv_plane), rem = t - p0 * plane;
      int hh = qdiv(rem, a.inv_iwt), ww = rem - hh * a.iw_t;
      int ni = qdiv(p0, a.inv_tc), ci = p0 - ni * a.tc;
      unsigned pofs = (unsigned)(ni * C + ci) * (unsigned)HW;  // (runs past the last plane)
      const int n_left = a.N - bk.n0, c_left = C - bk.c0;
      const int wbase = wave_id() * 64;
      for (int e0 = 0; e0 < total; e0 += a.threads) {
        const int gh = ih_org + hh, gw = iw_org + ww;
        const bool ok = ni < n_left && ci < c_left && (unsigned)gh < (unsigned)H && (unsigned)gw < (unsigned)W;
        if (e0 + t < total) copy_to_lds(rx, smem + e0 + wbase, ok ? (pofs + gh * W + gw) * 4 : (unsigned)kPartOob);
        ww += a.st_w;
        const bool k1 = ww >= a.iw_t;
        ww -= k1 ? a.iw_t : 0;
        hh += a.st_h + (k1 ? 1 : 0);
        const bool k2 = hh >= a.ih_t;
        hh -= k2 ? a.ih_t : 0;
        ci += a.st_c + (k2 ? 1 : 0);
        const bool k3 = ci >= a.tc;
        ci -= k3 ? a.tc : 0;
        ni += a.st_n + (k3 ? 1 : 0);
        pofs += (unsigned)a.st_p + (k2 ? (unsigned)HW : 0u) + (k3 ? (unsigned)(C - a.tc) * (unsigned)HW : 0u);
      }
      wait_copies();
    }
    __syncthreads();
  }

  // operand (input row `row` of the thread's window rows, column `col`) sources:
  // LDS at (row, column) of the staged tile, or global at row and column offsets
  const float* xs = smem + (td.ni * a.tc + td.ci) * plane + td.rowg * RPT * sh * a.iw_t + td.colg * sw;
  const int pofs = WIDE ? 0 : (live ? (td.ni * C + td.ci) * HW * 4 : kPartOob);
  const int ih0 = oh * sh - ph;
  if constexpr (WIDE && !LDS) {
    // one output row at a time: planes this large come from HBM, and the rows of a tap are
    // far apart
    const float* xc = x + ((int64_t)(live ? n : 0) * C + (live ? c : 0)) * HW;
#pragma unroll
    for (int u = 0; u < RPT; ++u) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int gh = ih0 + u * sh + r * dh;
        const bool hok = live && (unsigned)gh < (unsigned)H;
#pragma unroll
        for (int s = 0; s < S; ++s) {
          const float wt = RC ? wv[r * RC + s] : (live ? w[((int64_t)c * R + r) * S + s] : 0.f);
#pragma unroll
          for (int v = 0; v < VEC; ++v) {
            const int gw = (bk.ow0 + td.colg + v * a.cols) * sw - pw + s * dw;
            const float xv = load_or_zero(xc, (int64_t)gh * W + gw, hok && (unsigned)gw < (unsigned)W);
            acc[u][v] = fmaf(wt, xv, acc[u][v]);
          }
        }
      }
    }
  } else if constexpr (RC != 0) {
    constexpr int NIN = (RPT - 1) * STC + RC;  // input rows of the thread's outputs
    int cofs[VEC][RC];
    if constexpr (!LDS) {
#pragma unroll
      for (int v = 0; v < VEC; ++v)
#pragma unroll
        for (int s = 0; s < RC; ++s) {
          const int gw = (bk.ow0 + td.colg + v * a.cols) * STC - 1 + s;
          cofs[v][s] = (unsigned)gw < (unsigned)W ? gw * 4 : kPartOob;
        }
    }
#pragma unroll
    for (int i = 0; i < NIN; ++i) {
      float xv[VEC][RC];
      if constexpr (LDS) {
        const float* xr = xs + i * a.iw_t;
#pragma unroll
        for (int v = 0; v < VEC; ++v)
#pragma unroll
          for (int s = 0; s < RC; ++s) xv[v][s] = xr[v * a.cols * STC + s];
      } else {
        const int gh = ih0 + i;
        const int rofs = pofs + ((unsigned)gh < (unsigned)H ? gh * W * 4 : kPartOob);
#pragma unroll
        for (int v = 0; v < VEC; ++v)
#pragma unroll
          for (int s = 0; s < RC; ++s) xv[v][s] = bload1(rx, part_sum(rofs, cofs[v][s]));
      }
      // input row i feeds output row u through filter row i - u * STC; every output
      // adds its terms in (r, s) order
#pragma unroll
      for (int u = 0; u < RPT; ++u) {
        const int r = i - u * STC;
        if (r < 0 || r >= RC) continue;
#pragma unroll
        for (int v = 0; v < VEC; ++v)
#pragma unroll
          for (int s = 0; s < RC; ++s) acc[u][v] = fmaf(wv[r * RC + s], xv[v][s], acc[u][v]);
      }
    }
  } else {
    for (int r = 0; r < R; ++r) {
      for (int s = 0; s < S; ++s) {
        float wt;
        if constexpr (WIDE)
          wt = live ? w[((int64_t)c * R + r) * S + s] : 0.f;
        else
          wt = bload1(rwt, wofs + (r * S + s) * 4);
#pragma unroll
        for (int u = 0; u < RPT; ++u) {
          const int gh = ih0 + u * sh + r * dh;
          const bool hok = (unsigned)gh < (unsigned)H;
          const int rofs = pofs + (hok ? gh * W * 4 : kPartOob);
#pragma unroll
          for (int v = 0; v < VEC; ++v) {
            const int gw = (bk.ow0 + td.colg + v * a.cols) * sw - pw + s * dw;
            float xv;
            if constexpr (LDS)
              xv = xs[(u * sh + r * dh) * a.iw_t + v * a.cols * sw + s * dw];
            else
              xv = bload1(rx, part_sum(rofs, (unsigned)gw < (unsigned)W ? gw * 4 : kPartOob));
            acc[u][v] = fmaf(wt, xv, acc[u][v]);
          }
        }
      }
    }
  }

  if constexpr (WIDE) {
    if (!live) return;
    float* yc = y + ((int64_t)n * C + c) * OHW;
#pragma unroll
    for (int u = 0; u < RPT; ++u) {
      if (oh + u >= a.OH) continue;
#pragma unroll
      for (int v = 0; v < VEC; ++v) {
        const int ow = bk.ow0 + td.colg + v * a.cols;
        if (ow < a.OW) yc[(int64_t)(oh + u) * a.OW + ow] = acc[u][v];
      }
    }
  } else {
    const __amdgpu_buffer_rsrc_t ry = make_rsrc(y + plane0 * OHW, range(planes * OHW * 4));
    const int yofs = live ? (td.ni * C + td.ci) * OHW * 4 : kPartOob;
#pragma unroll
    for (int u = 0; u < RPT; ++u) {
      const int rofs = yofs + (oh + u < a.OH ? (oh + u) * a.OW * 4 : kPartOob);
#pragma unroll
      for (int v = 0; v < VEC; ++v) {
        const int ow = bk.ow0 + td.colg + v * a.cols;
        bstore1(ry, part_sum(rofs, ow < a.OW ? ow * 4 : kPartOob), acc[u][v]);
      }
    }
  }
}

typedef float dwf4 __attribute__((ext_vector_type(4)));

// 3x3, pad 1, stride STRIDE: a thread computes 4 consecutive output columns of
// RPT consecutive output rows of one (image, channel) plane. It reads the
// (RPT - 1) * STRIDE + 3 input rows those outputs need, each as the
// 3 * STRIDE + 3 columns from ow * STRIDE - 1 on: with vec_ld, the interior
// 4 (stride 1) or 8 (stride 2) columns as 16-byte loads and the edge columns
// as words (which the neighbouring lanes' 16-byte loads have brought into
// L1). vec_ld holds when W is a multiple of 4, W = STRIDE * OW, OW is a
// multiple of 4 and x is 16-byte aligned: every 16-byte load then lies inside
// its row. Columns and rows outside the image read as zero.
template <int STRIDE, int RPT>
__global__ void __launch_bounds__(1024)
depthwise_q4_kernel(const float* __restrict__ x, const float* __restrict__ w, float* __restrict__ y, DwArgs a) {
  constexpr int NIN = (RPT - 1) * STRIDE + 3;  // input rows read
  constexpr int NCOL = 3 * STRIDE + 3;         // input columns per row
  const int H = a.H, W = a.W, C = a.C, OH = a.OH, OW = a.OW;

  const DwBlock bk = dw_block(a);
  const DwThread td = dw_thread(a);
  const int c = bk.c0 + td.ci, n = bk.n0 + td.ni;
  const int ow = bk.ow0 + 4 * td.colg, oh = bk.oh0 + td.rowg * RPT;
  if (c >= C || n >= a.N || ow >= OW || oh >= OH) return;  // no barriers in this kernel

  float wv[9];
#pragma unroll
  for (int i = 0; i < 9; ++i) wv[i] = w[(int64_t)c * 9 + i];
  const float* xp = x + ((int64_t)n * C + c) * H * W;
  const int ih0 = oh * STRIDE - 1, iw0 = ow * STRIDE - 1;

  float acc[RPT][4];
#pragma unroll
  for (int u = 0; u < RPT; ++u)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[u][j] = 0.f;

#pragma unroll
  for (int i = 0; i < NIN; ++i) {
    const int ih = ih0 + i;
    float v[NCOL];
#pragma unroll
    for (int k = 0; k < NCOL; ++k) v[k] = 0.f;
    if ((unsigned)ih < (unsigned)H) {
      const float* row = xp + (int64_t)ih * W;
      if (a.vec_ld) {
        v[0] = iw0 >= 0 ? row[iw0] : 0.f;
        const dwf4 q0 = *(const dwf4*)(row + iw0 + 1);
        v[1] = q0.x; v[2] = q0.y; v[3] = q0.z; v[4] = q0.w;
        if constexpr (STRIDE == 1) {
          v[5] = iw0 + 5 < W ? row[iw0 + 5] : 0.f;
        } else {
          const dwf4 q1 = *(const dwf4*)(row + iw0 + 5);
          v[5] = q1.x; v[6] = q1.y; v[7] = q1.z; v[8] = q1.w;
        }
      } else {
#pragma unroll
        for (int k = 0; k < NCOL; ++k) v[k] = load_or_zero(row, iw0 + k, (unsigned)(iw0 + k) < (unsigned)W);
      }
    }
    // input row i feeds output row u through filter row r = i - u * STRIDE
#pragma unroll
    for (int u = 0; u < RPT; ++u) {
      const int r = i - u * STRIDE;
      if (r < 0 || r > 2) continue;
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int s = 0; s < 3; ++s) acc[u][j] = fmaf(wv[r * 3 + s], v[j * STRIDE + s], acc[u][j]);
    }
  }

  float* yp = y + ((int64_t)n * C + c) * OH * OW;
#pragma unroll
  for (int u = 0; u < RPT; ++u) {
    if (oh + u >= OH) break;
    float* o = yp + (int64_t)(oh + u) * OW + ow;
    if (a.vec_st) {
      dwf4 q;
      q.x = acc[u][0]; q.y = acc[u][1]; q.z = acc[u][2]; q.w = acc[u][3];
      *(dwf4*)o = q;
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (ow + j < OW) o[j] = acc[u][j];
    }
  }
}

using DwFn = void (*)(const float*, const float*, float*, DwArgs);

template <int STRIDE>
static DwFn dw_q4_pick(int rpt) {
  switch (rpt) {
    case 1: return depthwise_q4_kernel<STRIDE, 1>;
    case 2: return depthwise_q4_kernel<STRIDE, 2>;
    default: return depthwise_q4_kernel<STRIDE, 4>;
  }
}

template <int VEC, int RPT, bool LDS>
static DwFn dw_pick_spec(int spec, bool wide) {
  if (wide) {
    if (!LDS && spec == SPEC_3X3_S1) return depthwise_f32_kernel<VEC, RPT, LDS, LDS ? 0 : 3, true>;
    if (!LDS && spec == SPEC_3X3_S2) return depthwise_f32_kernel<VEC, RPT, LDS, LDS ? 0 : 4, true>;
    return depthwise_f32_kernel<VEC, RPT, LDS, 0, true>;
  }
  switch (spec) {
    case SPEC_3X3_S1: return depthwise_f32_kernel<VEC, RPT, LDS, 3, false>;
    case SPEC_3X3_S2: return depthwise_f32_kernel<VEC, RPT, LDS, 4, false>;
    default: return depthwise_f32_kernel<VEC, RPT, LDS, 0, false>;
  }
}
template <int VEC, int RPT>
static DwFn dw_pick_lds(int lds, int spec, bool wide) {
  return lds ? dw_pick_spec<VEC, RPT, true>(spec, wide) : dw_pick_spec<VEC, RPT, false>(spec, wide);
}
template <int VEC>
static DwFn dw_pick_rpt(int rpt, int lds, int spec, bool wide) {
  switch (rpt) {
    case 1: return dw_pick_lds<VEC, 1>(lds, spec, wide);
    case 2: return dw_pick_lds<VEC, 2>(lds, spec, wide);
    default: return dw_pick_lds<VEC, 4>(lds, spec, wide);
  }
}
static DwFn dw_pick(int vec, int rpt, int lds, int spec, bool wide) {
  switch (vec) {
    case 1: return dw_pick_rpt<1>(rpt, lds, spec, wide);
    case 2: return dw_pick_rpt<2>(rpt, lds, spec, wide);
    default: return dw_pick_rpt<4>(rpt, lds, spec, wide);
  }
}

int launch_depthwise_f32(const OpX& x, const ct_schedule& s, const Geom& g, const void* xin,
                         const void* w, void* y, float* /*ws*/, void* stream) {
  using namespace dw_knob;
  const ct_op& o = x.op;
  DwArgs a;
  a.N = o.n; a.C = o.c; a.H = o.h; a.W = o.w; a.R = o.r; a.S = o.s;
  a.sh = o.stride_h; a.sw = o.stride_w; a.ph = o.pad_h; a.pw = o.pad_w; a.dh = o.dil_h; a.dw = o.dil_w;
  a.OH = (int)x.oh; a.OW = (int)x.ow;
  a.tc = s.knob[TC]; a.toh = s.knob[TOH]; a.tow = s.knob[TOW]; a.nb = s.knob[NB]; a.order = s.knob[ORDER];
  a.f_tw = make_fastdiv(g.tiles_w); a.f_th = make_fastdiv(g.tiles_h); a.f_tc = make_fastdiv(g.tiles_c);
  a.ih_t = g.ih_t; a.iw_t = g.iw_t;
  a.threads = g.threads;
  a.rows = a.toh / s.knob[RPT];
  a.cols = a.tow / s.knob[VEC];
  const int plane = a.ih_t * a.iw_t;
  a.inv_cols = 1.0f / (float)a.cols;
  a.inv_rows = 1.0f / (float)a.rows;
  a.inv_tc = 1.0f / (float)a.tc;
  a.inv_plane = 1.0f / (float)plane;
  a.inv_iwt = 1.0f / (float)a.iw_t;
  a.st_w = a.threads % plane % a.iw_t;
  a.st_h = a.threads % plane / a.iw_t;
  a.st_c = a.threads / plane % a.tc;
  a.st_n = a.threads / plane / a.tc;
  // (a step of nb images or more ends the staging loop: its offset is not used)
  a.st_p = !s.knob[LDS] || g.dw_wide || a.st_n >= a.nb ? 0 : (a.st_n * a.C + a.st_c) * a.H * a.W;
  // the 3x3 specialisation needs pad 1 and dilation 1, which op_spec checks
  DwFn fn;
  if (s.knob[Q4]) {  // the validator admits it for 3x3 pad-1 ops (spec 3 or 4) with VEC = 4, LDS = 0
    const int st = g.spec == SPEC_3X3_S2 ? 2 : 1;
    a.vec_ld = a.W % 4 == 0 && a.W == st * a.OW && a.OW % 4 == 0 && ((uintptr_t)xin % 16) == 0;
    a.vec_st = a.OW % 4 == 0 && ((uintptr_t)y % 16) == 0;
    fn = st == 2 ? dw_q4_pick<2>(s.knob[RPT]) : dw_q4_pick<1>(s.knob[RPT]);
  } else {
    a.vec_ld = a.vec_st = 0;
    fn = dw_pick(s.knob[VEC], s.knob[RPT], s.knob[LDS], g.spec, g.dw_wide);
  }
  hipLaunchKernelGGL(fn, dim3((unsigned)g.blocks), dim3(g.threads), g.lds_bytes, (hipStream_t)stream,
                     (const float*)xin, (const float*)w, (float*)y, a);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace ct
