// Family 3, IGEMM_BF16: pointwise (1x1) convolution as a GEMM on the bf16
// matrix cores (v_mfma_f32_16x16x32_bf16 / v_mfma_f32_32x32x16_bf16), NHWC
// bf16 x, K x C bf16 w, NHWC fp32 y (fp32 accumulation).
//
// GEMM view: rows = output pixels (N*OH*OW), columns = output channels K,
// reduction = C. With NHWC x and K x C w both operands are row-major along
// the reduction, so every MFMA fragment is one 16-byte load of 8 bf16.
//
// A block owns a BM x BN tile (BM = WM*TM*MF pixels, BN = WN*TN*MF
// channels), one wave per WM x WN sub-tile. SPLIT > 1 spreads
// contiguous chunk ranges over grid.y (partials added in split order by a
// second kernel). SWZ = 1 renumbers blocks so that the tiles each XCD
// receives (blocks are dealt to the 8 XCDs in turn) are contiguous, which
// keeps a row band of x in one XCD's L2.
//
// What bounds it: a tile has few reduction steps (C = 16 to 960 is 1 to 30 of
// 32), so the loads' latency, once per step or chunk, and the instructions
// beside the loads and matrix products.
//   * LDS = 0 loads each wave's fragments straight from global memory through
//     a ring of D k-steps, each reloaded right after its products. D is the
//     smallest of 1, 2, 4, 8 that holds the wave's whole reduction: a longer
//     one loads steps that are not there and takes registers from other waves
//     (0.78 times as fast at one step on a quarter), up to
//     bf16_most_steps().
//   * LDS = 1 copies chunks of KC straight into LDS, 16 bytes per lane, as
//     many chunks as fit kBf16GroupBytes before the first wait, so that most
//     tiles wait once. Rows lie unpadded; the 16-byte groups of a row are
//     permuted by the low bits of its number, so that the 16 rows a fragment
//     reads at one k lie in distinct banks.
//     The copies take 16-byte addresses; a tensor off them goes through
//     registers, eight loads of a lane at a time (D = 1). Read without LDS
//     instead, every fragment row at its own misaligned addresses, a
//     1024-channel layer's schedules took up to 4 times as long.
//   * Reads are range-checked buffer loads from a base that advances with k:
//     no bounds branch, no select, no address arithmetic per load.
// Measured, 3076 sampled schedules of the MobileNet-v2 b16 pointwise layers and
// a ragged one, summed, against one chunk through registers (LDS = 1) and two
// chunks of fragments with clamped addresses (LDS = 0): 37.5 to 28.0 ms on the
// whole GPU, 65.9 to 44.5 ms on a quarter (LDS = 1: 22.6 to 15.2 and 40.7 to
// 23.7; LDS = 0: 14.9 to 12.9 and 25.3 to 20.9). Channels as the matrix
// instruction's rows, for 16-byte stores, lost: 30 % slower at K = 96 and up,
// where a store then touches 16 pixels instead of 4.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "ct_internal.h"
#include "k_util.h"

namespace ct {

struct IgBf16Args {
  int H, W, C, K, sh, sw;
  int npix;
  uint32_t xbytes, wbytes;
  int wn_shift, kc;
  int bm, bn, threads;
  int cps, chunks, group;  // chunks in LDS at once
  int tiles_m, tiles_n, swz;
  FastDiv dtn, dohw, dow;
  int64_t ny;
};

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

template <int MF>
struct MfmaBf16;
template <>
struct MfmaBf16<16> {
  static constexpr int ACC = 4, KSTEP = 32;
  typedef float V __attribute__((ext_vector_type(4)));
  __device__ static V op(bf16x8 a, bf16x8 b, V c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
  __device__ static int row(int e, int lane) { return 4 * (lane >> 4) + e; }
};
template <>
struct MfmaBf16<32> {
  static constexpr int ACC = 16, KSTEP = 16;
  typedef float V __attribute__((ext_vector_type(16)));
  __device__ static V op(bf16x8 a, bf16x8 b, V c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }
  __device__ static int row(int e, int lane) { return 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3); }
};

__host__ __device__ constexpr int bf16_max_threads(int acc_regs) { return acc_regs <= 64 ? 512 : 256; }
// Byte offset past every operand (fewer than 2^32 - 15 bytes): reads as 0.
constexpr unsigned kOobBytes = 0xFFFFFFF0u;

// Element offset of output pixel m's channels in x.
__device__ __forceinline__ int pixel_offset(int m, const IgBf16Args& a) {
  const int n = fdiv(m, a.dohw), rem = m - n * a.dohw.d;
  const int oh = fdiv(rem, a.dow), ow = rem - oh * a.dow.d;
  return ((n * a.H + oh * a.sh) * a.W + ow * a.sw) * a.C;
}
__device__ __forceinline__ bf16x8 load8(__amdgpu_buffer_rsrc_t r, unsigned off) {
  return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0));
}

template <int MF, int TM, int TN, int KC, int D>
__global__ void __launch_bounds__(bf16_max_threads(TM * TN * MfmaBf16<MF>::ACC))
igemm_bf16_kernel(const unsigned short* __restrict__ x, const unsigned short* __restrict__ w,
                  float* __restrict__ out, IgBf16Args a) {
  using M = MfmaBf16<MF>;
  using V = typename M::V;
  constexpr int ACC = M::ACC, KSTEP = M::KSTEP;

  // block -> tile (optionally renumbered so each XCD gets a contiguous range)
  const int T = a.tiles_m * a.tiles_n;
  int b = blockIdx.x;
  if (a.swz) b = xcd_band_tile(b, T);
  const int tmi = fdiv(b, a.dtn), tni = b - tmi * a.tiles_n;
  const int m0 = tmi * a.bm, n0 = tni * a.bn, sp = blockIdx.y;

  const int t = threadIdx.x, lane = t & 63, wave = wave_id();
  const int wmi = wave >> a.wn_shift, wni = wave - (wmi << a.wn_shift);
  const int m_off = wmi * TM * MF, n_off = wni * TN * MF;
  const int lrow = lane % MF, kg = lane / MF;  // fragment row and 8-value group of this lane

  const int ch_begin = sp * a.cps;
  const int ch_end = min(a.chunks, ch_begin + a.cps);

  V acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < ACC; ++e) acc[i][j][e] = 0.f;

  if constexpr (KC == 0) {
    unsigned aoff[TM], boff[TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int m = m0 + m_off + i * MF + lrow;
      aoff[i] = m < a.npix ? 2u * (unsigned)pixel_offset(m, a) + 16u * kg : kOobBytes;
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = n0 + n_off + j * MF + lrow;
      boff[j] = n < a.K ? 2u * (unsigned)(n * a.C) + 16u * kg : kOobBytes;
    }
    bf16x8 fa[D][TM], fb[D][TN];
    const int kb = ch_begin * a.kc, n = (min(a.C, ch_end * a.kc) - kb + KSTEP - 1) / KSTEP;
    auto load = [&](int u, int st) __attribute__((always_inline)) {
      const bool live = st < n;  // steps past the end read 0 and are not used
      const int k = live ? kb + st * KSTEP : 0;
      if (live && k + KSTEP > a.C) {  // the reduction's last step: what follows reads 0
        const bool ok = k + 8 * kg < a.C;
#pragma unroll
        for (int i = 0; i < TM; ++i) aoff[i] = ok ? aoff[i] : kOobBytes;
#pragma unroll
        for (int j = 0; j < TN; ++j) boff[j] = ok ? boff[j] : kOobBytes;
      }
      const __amdgpu_buffer_rsrc_t rx = make_rsrc(x + k, live ? (int64_t)(a.xbytes - 2u * (uint32_t)k) : 0);
      const __amdgpu_buffer_rsrc_t rw = make_rsrc(w + k, live ? (int64_t)(a.wbytes - 2u * (uint32_t)k) : 0);
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[u][i] = load8(rx, aoff[i]);
#pragma unroll
      for (int j = 0; j < TN; ++j) fb[u][j] = load8(rw, boff[j]);
      __builtin_amdgcn_sched_barrier(0);
    };
    auto mma = [&](int u) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = M::op(fa[u][i], fb[u][j], acc[i][j]);
      __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll
    for (int u = 0; u < D; ++u) load(u, u);
    int st = 0;
    for (; st + D < n; st += D)
#pragma unroll
      for (int u = 0; u < D; ++u) {
        mma(u);
        load(u, st + D + u);
      }
#pragma unroll
    for (int u = 0; u < D; ++u)
      if (st + u < n) mma(u);
  } else {
    extern __shared__ __align__(16) unsigned short lds16[];
    constexpr int VPR = KC / 8, RPC = 64 / VPR;  // 16-byte groups of a row, rows of a wave's copy
    constexpr int SW = VPR == 4 ? 2 : VPR == 8 ? 1 : 0;
    const int nw_shift = 31 - __builtin_clz(a.threads >> 6), qa = a.bm / RPC, q_end = (a.bm + a.bn) / RPC;
    // this wave's copies q = wave + i * waves: the first na of its nq are rows of x
    const int nq = (q_end - wave + (1 << nw_shift) - 1) >> nw_shift;
    const int na = max(0, (qa - wave + (1 << nw_shift) - 1) >> nw_shift);
    // group of this lane in copy q: rows 16 apart differ in the same way
    auto col = [&](int q) __attribute__((always_inline)) {
      return (lane % VPR) ^ (((q * RPC + lane / VPR) >> SW) & (VPR - 1));
    };
    unsigned off[2 * kMaxLoadsPerThread];
#pragma unroll
    for (int i = 0; i < 2 * kMaxLoadsPerThread; ++i) {
      const int q = wave + (i << nw_shift);
      if (i < nq) {
        const int r = q * RPC + lane / VPR, m = m0 + r, n = n0 + r - a.bm;
        if (i < na)
          off[i] = m < a.npix ? 2u * (unsigned)pixel_offset(m, a) + 16u * col(q) : kOobBytes;
        else
          off[i] = n < a.K ? 2u * (unsigned)(n * a.C) + 16u * col(q) : kOobBytes;
      }
    }
    auto copy_chunk = [&](int ch, unsigned short* dst) __attribute__((always_inline)) {
      const int k = ch * KC;
      const __amdgpu_buffer_rsrc_t rx = make_rsrc(x + k, (int64_t)(a.xbytes - 2u * (uint32_t)k));
      const __amdgpu_buffer_rsrc_t rw = make_rsrc(w + k, (int64_t)(a.wbytes - 2u * (uint32_t)k));
      // opaque here, so that the comparisons are made where they are used
      // rather than kept in scalar register pairs, which do not suffice
      int cq = nq, ca = na;
      asm volatile("" : "+s"(cq), "+s"(ca));
      auto copies = [&](auto tail) __attribute__((always_inline)) {
        constexpr int G = D ? 8 : 4;
#pragma unroll
        for (int i0 = 0; i0 < 2 * kMaxLoadsPerThread; i0 += G)
          if (i0 < cq) {
            bf16x8 v[D ? G : 1];
#pragma unroll
            for (int i = i0; i < i0 + G; ++i)
              if (i < cq) {
                const int q = wave + (i << nw_shift);
                unsigned o = off[i];
                if constexpr (tail.value) o = k + 8 * col(q) < a.C ? o : kOobBytes;
                if constexpr (D)
                  v[i - i0] = load8(i < ca ? rx : rw, o);
                else
                  copy16_to_lds(i < ca ? rx : rw, (float*)(dst + q * 512), o);
              }
            if constexpr (D) {
#pragma unroll
              for (int i = i0; i < i0 + G; ++i)
                if (i < cq) *(bf16x8*)(dst + (wave + (i << nw_shift)) * 512 + 8 * lane) = v[i - i0];
            }
          }
      };
      if (k + KC <= a.C)
        copies(std::false_type{});
      else
        copies(std::true_type{});
    };
    const int csw = (lrow >> SW) & (VPR - 1);
    auto mma_step = [&](const unsigned short* src, int st) __attribute__((always_inline)) {
      const int c = (st * (KSTEP / 8) + kg) ^ csw;
      bf16x8 fa[TM], fb[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i)
        fa[i] = __builtin_bit_cast(bf16x8, *(const u32x4*)(src + (m_off + i * MF + lrow) * KC + c * 8));
#pragma unroll
      for (int j = 0; j < TN; ++j)
        fb[j] = __builtin_bit_cast(bf16x8, *(const u32x4*)(src + (a.bm + n_off + j * MF + lrow) * KC + c * 8));
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = M::op(fa[i], fb[j], acc[i][j]);
    };
    const int stage = (a.bm + a.bn) * KC;
    for (int c0 = ch_begin; c0 < ch_end; c0 += a.group) {
      const int nc = min(a.group, ch_end - c0);
      if (c0 > ch_begin) __syncthreads();
      for (int c = 0; c < nc; ++c) copy_chunk(c0 + c, lds16 + c * stage);
      wait_copies();
      __syncthreads();
      for (int c = 0; c < nc; ++c) {
        const int left = a.C - (c0 + c) * KC;
        const unsigned short* src = lds16 + c * stage;
        mma_step(src, 0);
#pragma unroll
        for (int st = 1; st < KC / KSTEP; ++st)
          if (st * KSTEP < left) mma_step(src, st);
      }
    }
  }

  // Store. An accumulator's pixel row is a wave-uniform part (tile i,
  // element e) plus a lane part, so where every pixel row of the wave tile
  // exists each store is a buffer store whose scalar offset carries the
  // uniform row and whose one 32-bit lane offset (row group and channel) is
  // computed once per channel column; a ragged pixel tail checks every
  // element.
  const int mw = m0 + m_off;  // first pixel row of this wave's tile
  float* ob = out + (int64_t)sp * a.ny + (int64_t)mw * a.K;
  if (mw + TM * MF <= a.npix) {
    const __amdgpu_buffer_rsrc_t ro = make_rsrc(ob, (int64_t)TM * MF * a.K * 4);
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = n0 + n_off + j * MF + lrow;
      if (n >= a.K) continue;
      const int lo = (M::row(0, lane) * a.K + n) * 4;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int e = 0; e < ACC; ++e) {
          // through a scalar: a bit cast of a vector element read element 0
          const float v = acc[i][j][e];
          __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), ro, lo, (i * MF + M::row(e, 0)) * a.K * 4, 0);
        }
    }
  } else {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = n0 + n_off + j * MF + lrow;
      if (n >= a.K) continue;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int e = 0; e < ACC; ++e) {
          const int mr = i * MF + M::row(e, lane);
          if (mw + mr < a.npix) ob[(int64_t)mr * a.K + n] = acc[i][j][e];
        }
    }
  }
}

using IgBf16Fn = void (*)(const unsigned short*, const unsigned short*, float*, IgBf16Args);

template <int MF, int TM, int TN>
static IgBf16Fn bf_pick_kc(int kc, int ring) {
  if constexpr (TM * TN * MfmaBf16<MF>::ACC > 128) {
    return nullptr;  // accumulator tiles the validator rejects: not instantiated
  } else {
    switch (kc) {
      case 32: return ring ? igemm_bf16_kernel<MF, TM, TN, 32, 1> : igemm_bf16_kernel<MF, TM, TN, 32, 0>;
      case 64: return ring ? igemm_bf16_kernel<MF, TM, TN, 64, 1> : igemm_bf16_kernel<MF, TM, TN, 64, 0>;
      case 128: return ring ? igemm_bf16_kernel<MF, TM, TN, 128, 1> : igemm_bf16_kernel<MF, TM, TN, 128, 0>;
    }
    constexpr int most = bf16_most_steps(TM + TN);
    if (ring == 1) return igemm_bf16_kernel<MF, TM, TN, 0, 1>;
    if (ring == 2) return igemm_bf16_kernel<MF, TM, TN, 0, 2>;
    if (ring == 4) return igemm_bf16_kernel<MF, TM, TN, 0, most < 4 ? most : 4>;
    return igemm_bf16_kernel<MF, TM, TN, 0, most>;
  }
}
template <int MF, int TM>
static IgBf16Fn bf_pick_tn(int tn, int kc, int ring) {
  switch (tn) {
    case 1: return bf_pick_kc<MF, TM, 1>(kc, ring);
    case 2: return bf_pick_kc<MF, TM, 2>(kc, ring);
    default: return bf_pick_kc<MF, TM, 4>(kc, ring);
  }
}
template <int MF>
static IgBf16Fn bf_pick_tm(int tm, int tn, int kc, int ring) {
  switch (tm) {
    case 1: return bf_pick_tn<MF, 1>(tn, kc, ring);
    case 2: return bf_pick_tn<MF, 2>(tn, kc, ring);
    default: return bf_pick_tn<MF, 4>(tn, kc, ring);
  }
}

int launch_igemm_bf16(const OpX& x, const ct_schedule& s, const Geom& g, const void* xin,
                      const void* w, void* y, float* ws, void* stream) {
  using namespace bf16_knob;
  const ct_op& o = x.op;
  IgBf16Args a;
  a.H = o.h; a.W = o.w; a.C = o.c; a.K = o.k;
  a.sh = o.stride_h; a.sw = o.stride_w;
  a.npix = (int)x.npix;
  a.xbytes = (uint32_t)(2 * x.nx); a.wbytes = (uint32_t)(2 * x.nw);
  a.wn_shift = s.knob[WN] == 4 ? 2 : s.knob[WN] == 2 ? 1 : 0; a.kc = s.knob[KC];
  a.bm = g.bm; a.bn = g.bn; a.threads = g.threads;
  a.cps = g.chunks_per_split; a.chunks = g.chunks;
  a.group = g.bf_group;
  a.dtn = make_fastdiv(g.tiles_k); a.dohw = make_fastdiv(x.oh * x.ow); a.dow = make_fastdiv(x.ow);
  a.tiles_m = (int)g.tiles_h; a.tiles_n = (int)g.tiles_k; a.swz = s.knob[SWZ];
  a.ny = x.ny;
  // copies into LDS take 16 bytes at 16-byte addresses; tensors off them go
  // through registers
  const bool aligned = ((uintptr_t)xin | (uintptr_t)w) % 16 == 0;
  const int kc = s.knob[LDS] ? s.knob[KC] : 0;
  const int ring = s.knob[LDS] ? !aligned : g.bf_ring;
  IgBf16Fn fn = s.knob[MF] == 32 ? bf_pick_tm<32>(s.knob[TM], s.knob[TN], kc, ring)
                                 : bf_pick_tm<16>(s.knob[TM], s.knob[TN], kc, ring);
  if (!fn) {
    set_error("igemm_bf16: no kernel instance for this accumulator tile");
    return -2;
  }
  dim3 grid((unsigned)(g.tiles_h * g.tiles_k), (unsigned)g.split);
  float* out = g.split > 1 ? ws : (float*)y;
  hipLaunchKernelGGL(fn, grid, dim3(g.threads), g.lds_bytes, (hipStream_t)stream,
                     (const unsigned short*)xin, (const unsigned short*)w, out, a);
  if (hipGetLastError() != hipSuccess) return -1;
  if (g.split > 1) return launch_split_reduce(ws, (float*)y, x.ny, g.split, stream);
  return 0;
}

}  // namespace ct
