// VALU product path: one lane per output element, INT16 x INT16 products
// summed with 32-bit wrapping integer adds, one INT32 partial per chunk of L
// reduction indices, each converted to FP32 and added in chunk order, then
// scaled once by 2^(Ea+Eb) (Algorithm 2 and Sec. 4.3 of the paper).
//
// It walks the canonical reduction order of each direction
//   forward          t = (r*S + s)*C + c
//   backward-data    t = (r*S + s)*K + k
//   backward-weights t = (n*P + p)*Q + q   (segments of G chunks)
// and handles every shape, stride and chunk length.  It is the measured
// alternative to the MFMA path, the default only for small layers at P = 16,
// where it also stands behind the MFMA path for tensors that path cannot
// represent (see Gate).
#include <algorithm>

#include "dfp_internal.h"

namespace dfp {

namespace {

constexpr int kBlock = 256;

// P = 16 on the matrix cores.  The byte digits of the MFMA path hold integers
// up to 32639; P = 16 tensors reach 32767.  Only a tensor whose max falls in
// the top 1/256 of its binade holds larger ones (0.6% of tensors whose max is
// log-uniform), so the MFMA kernels run on the tensors as they are, between
// k_p16_scan, which notes whether any operand element lies beyond, and a gated
// launch of the VALU kernel, which recomputes the whole output if one does and
// returns at once otherwise (a step of ResNet-50's res4 3x3 layer, N = 32,
// L = 16: 5950 us with the VALU kernels alone, 303 us so; a tensor beyond the
// digits costs the MFMA kernels on top of the VALU ones).
constexpr int kScanWgs = 256;
struct Gate {
  const uint32_t* seen;   // per scan workgroup: any element beyond the digits (null: not gated)
  const dfp_scale* mfma;  // the output scale the MFMA kernels raised (null: none)
};

// True if the gated launch has nothing to compute; workgroup 0 then hands the
// MFMA kernels' output scale on (with its exponent for the DFP-32 outputs).
template <bool I32>
__device__ __forceinline__ bool gate_closed(const Gate& gt, dfp_scale* so) {
  if (!gt.seen) return false;
  static_assert(kScanWgs == kBlock, "one word per thread");
  if (__syncthreads_or((int)gt.seen[threadIdx.x])) return false;
  if (so && gt.mfma && blockIdx.x == 0 && threadIdx.x == 0) {
    so->amax_bits = gt.mfma->amax_bits;
    so->flags = gt.mfma->flags;
    if (I32) so->exp = gt.mfma->exp;
  }
  return true;
}

// Max of n INT16 elements: 16-byte loads when the tensor is 16-byte aligned.
__device__ __forceinline__ int32_t scan_max(const int16_t* __restrict__ a, int64_t n) {
  typedef short s2 __attribute__((ext_vector_type(2)));
  const int64_t id = (int64_t)blockIdx.x * kBlock + threadIdx.x, step = (int64_t)gridDim.x * kBlock;
  int32_t m = -32768;
  int64_t done = 0;
  if ((reinterpret_cast<uintptr_t>(a) & 15) == 0) {
    const uint4* a4 = reinterpret_cast<const uint4*>(a);
    const int64_t n8 = n >> 3;
    s2 mv[4] = {{-32768, -32768}, {-32768, -32768}, {-32768, -32768}, {-32768, -32768}};
    for (int64_t i = id; i < n8; i += 4 * step) {
      uint4 v[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = a4[min(i + k * step, n8 - 1)];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        mv[0] = __builtin_elementwise_max(mv[0], __builtin_bit_cast(s2, v[k].x));
        mv[1] = __builtin_elementwise_max(mv[1], __builtin_bit_cast(s2, v[k].y));
        mv[2] = __builtin_elementwise_max(mv[2], __builtin_bit_cast(s2, v[k].z));
        mv[3] = __builtin_elementwise_max(mv[3], __builtin_bit_cast(s2, v[k].w));
      }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) m = max(m, max((int32_t)mv[k].x, (int32_t)mv[k].y));
    done = n8 << 3;
  }
  for (int64_t i = done + id; i < n; i += step) m = max(m, (int32_t)a[i]);
  return m;
}

// seen[workgroup] = whether its share of either operand has an element above
// 32639; also clears the output scale, which the gated launch writes.
__global__ __launch_bounds__(kBlock) void k_p16_scan(const int16_t* __restrict__ a, int64_t na,
                                                     const int16_t* __restrict__ b, int64_t nb,
                                                     uint32_t* __restrict__ seen, dfp_scale* so) {
  if (so && blockIdx.x == 0 && threadIdx.x == 0) {
    so->amax_bits = 0u;
    so->flags = 0u;
  }
  const int any = __syncthreads_or(max(scan_max(a, na), scan_max(b, nb)) > 32639);
  if (threadIdx.x == 0) seen[blockIdx.x] = any ? 1u : 0u;
}

// Running state of one output's chunked reduction.
struct ChunkAcc {
  uint32_t acc = 0;   // INT32 partial of the current chunk (wraps mod 2^32)
  int32_t fill = 0;   // products in the current chunk so far
  int64_t j = 0;      // index of the current chunk
  float sum = 0.f;    // FP32 sum over finished chunks (or segments)
  float seg = 0.f;    // FP32 sum inside the current segment (backward-weights)
};

template <bool PARTIALS, bool SEGMENTED>
__device__ __forceinline__ void flush(ChunkAcc& st, int32_t G, int32_t* partials, int64_t O, int64_t o) {
  const float f = (float)(int32_t)st.acc;
  if (PARTIALS) partials[st.j * O + o] = (int32_t)st.acc;
  if (SEGMENTED) {
    const int64_t in_seg = st.j % G;
    st.seg = (in_seg == 0) ? f : st.seg + f;
    if (in_seg == G - 1) {
      st.sum = (st.j / G == 0) ? st.seg : st.sum + st.seg;
    }
  } else {
    st.sum = (st.j == 0) ? f : st.sum + f;
  }
  ++st.j;
  st.acc = 0;
  st.fill = 0;
}

template <bool PARTIALS, bool SEGMENTED>
__device__ __forceinline__ void push(ChunkAcc& st, int32_t prod, int32_t L, int32_t G, int32_t* partials,
                                     int64_t O, int64_t o) {
  st.acc += (uint32_t)prod;
  if (++st.fill == L) flush<PARTIALS, SEGMENTED>(st, G, partials, O, o);
}

template <bool SEGMENTED>
__device__ __forceinline__ void finish_tail(ChunkAcc& st, int32_t G) {
  if (SEGMENTED && (st.j % G) != 0) {  // close a partly filled last segment
    st.sum = (st.j / G == 0) ? st.seg : st.sum + st.seg;
  }
}

// Block max of per-lane |y| bit patterns into so->amax_bits, plus the OUTPUT_INF flag.
__device__ __forceinline__ void epilogue_amax(uint32_t m, dfp_scale* so) {
  __shared__ uint32_t red[kBlock / 64];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off, 64));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t b = red[0];
    for (int i = 1; i < kBlock / 64; ++i) b = max(b, red[i]);
    if (b > __atomic_load_n(&so->amax_bits, __ATOMIC_RELAXED)) atomicMax(&so->amax_bits, b);
    if (b == 0x7f800000u) atomicOr(&so->flags, DFP_FLAG_OUTPUT_INF);
  }
}

// Single-chunk DFP-32 output: the wrapped INT32 sum, its |.| into so->amax_bits
// (one relaxed-read-guarded atomic per lane; this path is the reference one)
// and the output exponent.
__device__ __forceinline__ void store_i32(float* out, int64_t o, uint32_t acc, dfp_scale* so, int32_t e) {
  const int32_t v = (int32_t)acc;
  reinterpret_cast<int32_t*>(out)[o] = v;
  if (so) {
    const uint32_t m = v < 0 ? 0u - (uint32_t)v : (uint32_t)v;
    if (m > __atomic_load_n(&so->amax_bits, __ATOMIC_RELAXED)) atomicMax(&so->amax_bits, m);
    if (o == 0) so->exp = e;
  }
}

template <bool PARTIALS, bool I32 = false>
__global__ __launch_bounds__(kBlock) void k_fwd_valu(Geom g, const int16_t* __restrict__ x,
                                                    const dfp_scale* __restrict__ sx,
                                                    const int16_t* __restrict__ w,
                                                    const dfp_scale* __restrict__ sw, float* __restrict__ y,
                                                    dfp_scale* so, int32_t* __restrict__ partials, Gate gt) {
  if (gate_closed<I32>(gt, so)) return;
  const int64_t O = (int64_t)g.n * g.k * g.p * g.q;
  uint32_t mx = 0u;
  for (int64_t o = (int64_t)blockIdx.x * kBlock + threadIdx.x; o < O; o += (int64_t)gridDim.x * kBlock) {
    const int32_t q = (int32_t)(o % g.q), p = (int32_t)((o / g.q) % g.p);
    const int32_t k = (int32_t)((o / ((int64_t)g.q * g.p)) % g.k);
    const int64_t n = o / ((int64_t)g.q * g.p * g.k);
    const int64_t hw = (int64_t)g.h * g.w, rs = (int64_t)g.r * g.s;
    ChunkAcc st;
    for (int32_t r = 0; r < g.r; ++r) {
      const int32_t ih = p * g.sh - g.ph + r;
      for (int32_t s = 0; s < g.s; ++s) {
        const int32_t iw = q * g.sw - g.pw + s;
        const bool valid = ih >= 0 && ih < g.h && iw >= 0 && iw < g.w;
        const int16_t* xp = x + (n * g.c) * hw + (valid ? (int64_t)ih * g.w + iw : 0);
        const int16_t* wp = w + ((int64_t)k * g.c) * rs + r * g.s + s;
        for (int32_t c = 0; c < g.c; ++c) {
          const int32_t prod = valid ? (int32_t)xp[c * hw] * (int32_t)wp[c * rs] : 0;
          if (I32) st.acc += (uint32_t)prod;
          else push<PARTIALS, false>(st, prod, g.L, g.G, partials, O, o);
        }
      }
    }
    if (I32) {
      store_i32(y, o, st.acc, so, sx->exp + sw->exp);
      continue;
    }
    if (st.fill) flush<PARTIALS, false>(st, g.G, partials, O, o);
    const float yv = ldexpf(st.sum, sx->exp + sw->exp);
    y[o] = yv;
    mx = max(mx, __float_as_uint(yv) & 0x7fffffffu);
  }
  if (so && !I32) epilogue_amax(mx, so);
}

template <bool PARTIALS, bool I32 = false>
__global__ __launch_bounds__(kBlock) void k_bwdd_valu(Geom g, const int16_t* __restrict__ dy,
                                                     const dfp_scale* __restrict__ sdy,
                                                     const int16_t* __restrict__ w,
                                                     const dfp_scale* __restrict__ sw, float* __restrict__ dx,
                                                     dfp_scale* so, int32_t* __restrict__ partials, Gate gt) {
  if (gate_closed<I32>(gt, so)) return;
  const int64_t O = (int64_t)g.n * g.c * g.h * g.w;
  uint32_t mx = 0u;
  for (int64_t o = (int64_t)blockIdx.x * kBlock + threadIdx.x; o < O; o += (int64_t)gridDim.x * kBlock) {
    const int32_t iw = (int32_t)(o % g.w), ih = (int32_t)((o / g.w) % g.h);
    const int32_t c = (int32_t)((o / ((int64_t)g.w * g.h)) % g.c);
    const int64_t n = o / ((int64_t)g.w * g.h * g.c);
    const int64_t pq = (int64_t)g.p * g.q, crs = (int64_t)g.c * g.r * g.s;
    ChunkAcc st;
    for (int32_t r = 0; r < g.r; ++r) {
      const int32_t nh = ih + g.ph - r;
      const bool vh = nh >= 0 && (nh % g.sh) == 0 && nh / g.sh < g.p;
      for (int32_t s = 0; s < g.s; ++s) {
        const int32_t nw = iw + g.pw - s;
        const bool valid = vh && nw >= 0 && (nw % g.sw) == 0 && nw / g.sw < g.q;
        const int16_t* dp = dy + (n * g.k) * pq + (valid ? (int64_t)(nh / g.sh) * g.q + nw / g.sw : 0);
        const int16_t* wp = w + ((int64_t)c * g.r + r) * g.s + s;
        for (int32_t k = 0; k < g.k; ++k) {
          const int32_t prod = valid ? (int32_t)dp[k * pq] * (int32_t)wp[k * crs] : 0;
          if (I32) st.acc += (uint32_t)prod;
          else push<PARTIALS, false>(st, prod, g.L, g.G, partials, O, o);
        }
      }
    }
    if (I32) {
      store_i32(dx, o, st.acc, so, sdy->exp + sw->exp);
      continue;
    }
    if (st.fill) flush<PARTIALS, false>(st, g.G, partials, O, o);
    const float yv = ldexpf(st.sum, sdy->exp + sw->exp);
    dx[o] = yv;
    mx = max(mx, __float_as_uint(yv) & 0x7fffffffu);
  }
  if (so && !I32) epilogue_amax(mx, so);
}

template <bool PARTIALS>
__global__ __launch_bounds__(kBlock) void k_bwdw_valu(Geom g, const int16_t* __restrict__ x,
                                                     const dfp_scale* __restrict__ sx,
                                                     const int16_t* __restrict__ dy,
                                                     const dfp_scale* __restrict__ sdy, float* __restrict__ dw,
                                                     int32_t* __restrict__ partials, Gate gt) {
  if (gate_closed<false>(gt, nullptr)) return;
  const int64_t O = (int64_t)g.k * g.c * g.r * g.s;
  for (int64_t o = (int64_t)blockIdx.x * kBlock + threadIdx.x; o < O; o += (int64_t)gridDim.x * kBlock) {
    const int32_t s = (int32_t)(o % g.s), r = (int32_t)((o / g.s) % g.r);
    const int32_t c = (int32_t)((o / ((int64_t)g.s * g.r)) % g.c);
    const int32_t k = (int32_t)(o / ((int64_t)g.s * g.r * g.c));
    const int64_t hw = (int64_t)g.h * g.w, pq = (int64_t)g.p * g.q;
    ChunkAcc st;
    for (int32_t n = 0; n < g.n; ++n) {
      const int16_t* xn = x + ((int64_t)n * g.c + c) * hw;
      const int16_t* dn = dy + ((int64_t)n * g.k + k) * pq;
      for (int32_t p = 0; p < g.p; ++p) {
        const int32_t ih = p * g.sh - g.ph + r;
        const bool vh = ih >= 0 && ih < g.h;
        for (int32_t q = 0; q < g.q; ++q) {
          const int32_t iw = q * g.sw - g.pw + s;
          const bool valid = vh && iw >= 0 && iw < g.w;
          const int32_t prod = valid ? (int32_t)xn[(int64_t)ih * g.w + iw] * (int32_t)dn[(int64_t)p * g.q + q] : 0;
          push<PARTIALS, true>(st, prod, g.L, g.G, partials, O, o);
        }
      }
    }
    if (st.fill) flush<PARTIALS, true>(st, g.G, partials, O, o);
    finish_tail<true>(st, g.G);
    dw[o] = ldexpf(st.sum, sx->exp + sdy->exp);
  }
}

}  // namespace

namespace {
dfp_status launch_valu(int32_t dir, const Geom& g, const int16_t* a, const dfp_scale* sa, const int16_t* b,
                       const dfp_scale* sb, float* out, dfp_scale* so, int32_t* partials, bool i32, int64_t max_wgs,
                       const Gate& gt, hipStream_t st) {
  int64_t O;
  if (dir == DFP_FWD) O = (int64_t)g.n * g.k * g.p * g.q;
  else if (dir == DFP_BWD_DATA) O = (int64_t)g.n * g.c * g.h * g.w;
  else O = (int64_t)g.k * g.c * g.r * g.s;
  const dim3 grid((unsigned)std::min<int64_t>((O + kBlock - 1) / kBlock, max_wgs)), block(kBlock);
#define DFP_VALU(ID, KERNEL) DFP_LAUNCH(ID, (KERNEL), grid, block, 0, st, g, a, sa, b, sb, out, so, partials, gt)
  if (i32) {  // forward or backward-data, one chunk
    if (dir == DFP_FWD) DFP_VALU(K_FWD_I32, (k_fwd_valu<false, true>));
    else DFP_VALU(K_BWDD_I32, (k_bwdd_valu<false, true>));
  } else if (dir == DFP_FWD) {
    if (partials) DFP_VALU(K_FWD_VALU, k_fwd_valu<true>);
    else DFP_VALU(K_FWD_VALU, k_fwd_valu<false>);
  } else if (dir == DFP_BWD_DATA) {
    if (partials) DFP_VALU(K_BWDD_VALU, k_bwdd_valu<true>);
    else DFP_VALU(K_BWDD_VALU, k_bwdd_valu<false>);
  } else {
    if (partials) DFP_LAUNCH(K_BWDW_VALU, k_bwdw_valu<true>, grid, block, 0, st, g, a, sa, b, sb, out, partials, gt);
    else DFP_LAUNCH(K_BWDW_VALU, k_bwdw_valu<false>, grid, block, 0, st, g, a, sa, b, sb, out, partials, gt);
  }
#undef DFP_VALU
  return DFP_OK;
}

struct P16Ws {
  uint32_t* seen;
  dfp_scale* mfma;
};
P16Ws p16_ws(void* gate_ws) {
  uint8_t* w = reinterpret_cast<uint8_t*>(gate_ws);
  return {reinterpret_cast<uint32_t*>(w), reinterpret_cast<dfp_scale*>(w + kScanWgs * 4)};
}
static_assert(kScanWgs * 4 + (int)sizeof(dfp_scale) <= kP16GateBytes, "gate workspace");
}  // namespace

dfp_status launch_conv_valu(int32_t dir, const Geom& g, const int16_t* a, const dfp_scale* sa, const int16_t* b,
                            const dfp_scale* sb, float* out, dfp_scale* so, int32_t* partials, hipStream_t st,
                            bool i32) {
  return launch_valu(dir, g, a, sa, b, sb, out, so, partials, i32, INT32_MAX, Gate{nullptr, nullptr}, st);
}

dfp_status launch_p16_scan(const int16_t* a, int64_t na, const int16_t* b, int64_t nb, dfp_scale* so, void* gate_ws,
                           hipStream_t st) {
  DFP_LAUNCH(K_SCALE_RESET, k_p16_scan, dim3(kScanWgs), dim3(kBlock), 0, st, a, na, b, nb, p16_ws(gate_ws).seen, so);
  return DFP_OK;
}

dfp_scale* p16_mfma_scale(void* gate_ws) { return p16_ws(gate_ws).mfma; }

dfp_status launch_conv_valu_gated(int32_t dir, const Geom& g, const int16_t* a, const dfp_scale* sa, const int16_t* b,
                                  const dfp_scale* sb, float* out, dfp_scale* so, void* gate_ws, hipStream_t st,
                                  bool i32) {
  // 2048 workgroups fill the chip and cost little when they return at once
  const P16Ws w = p16_ws(gate_ws);
  return launch_valu(dir, g, a, sa, b, sb, out, so, nullptr, i32, 2048, Gate{w.seen, so ? w.mfma : nullptr}, st);
}

}  // namespace dfp
