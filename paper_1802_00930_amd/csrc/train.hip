// The FP32 steps either side of a layer's convolutions in a DFP16 training
// step (Sec. 4.1, Fig. 2): batch normalisation with an optional residual add
// and ReLU on an up-converted DFP16 tensor, its backward pass, and FP32 SGD on
// master weights; each ends in the quantiser of its output (Q_a, Q_e, Q_w).
//
// Batch-norm statistics need no floating-point accumulation: a channel's
// values are i * 2^E with integer i, so sum i and sum i^2 (and in the backward
// pass the masked sums of dz and dz * y) are exact in 64-bit integers and
// independent of the reduction order.  Per-channel values are computed once
// in float64 and rounded to FP32; per-element work is FP32 with a fixed
// operation order, every step one IEEE rounding (no contraction in this
// file), so the rounding pass can recompute an element bit for bit instead of
// reading it back.
//
// Passes (all HBM-bound):
//   forward   k_bn_stats (y) -> k_bn_finalize -> [res: k_bn_amax + max reduce]
//             -> k_bn_convert (y [, res]) writing zq [and z]; with res and z
//             the max pass writes z and the tensor quantiser reads it
//   backward  k_bn_stats (y, dz [, res]; with res it leaves the ReLU mask, a
//             byte per four elements, so that res is read once) ->
//             k_bn_finalize -> k_bn_amax (writes dy / dres if asked) -> max
//             reduce -> k_bn_convert (or, with dy, the tensor quantiser)
// 64 x 256 x 56 x 56 with a residual, z and dres (26 B per element at least):
// forward stats 21, max pass + z 89, quantiser 62 us; backward stats 110, max
// pass 74, convert 67 us, the four small kernels 20 (746 -> 446 us a call; copies
// run at 5.1 TB/s, the passes at 3.9 to 5.9).
//   SGD       k_sgd (update + max) -> max reduce -> the tensor quantiser
// Without a residual the forward output is a monotone function of the input
// integer within a channel (ReLU of an affine map evaluated with monotone
// roundings), so its max is the larger of the values at the channel's
// smallest and largest integer and the max pass over z is skipped.
#pragma clang fp contract(off)

#include <algorithm>
#include <climits>
#include <type_traits>

#include "dfp_internal.h"
#include "dfp_round.h"

namespace dfp {

namespace {

constexpr int kBlock = 256;
constexpr int kMaxParts = 2048;

struct Chan {
  float mean, inv, gamma, beta;
};
__device__ __forceinline__ Chan load_chan(const float* mean, const float* inv, const float* gamma,
                                          const float* beta, int32_t c) {
  return {mean[c], inv[c], gamma[c], beta[c]};
}

// xhat = (i 2^E - mean) * inv_std; i 2^E is exact for |i| < 2^24.
__device__ __forceinline__ float bn_xhat(int32_t yi, int32_t ey, const Chan& p) {
  return __fmul_rn(__fsub_rn(ldexpf((float)yi, ey), p.mean), p.inv);
}
// gamma * xhat + beta (fused); the residual, if any, is added to it.
__device__ __forceinline__ float bn_affine(float xh, const Chan& p) { return __fmaf_rn(xh, p.gamma, p.beta); }
__device__ __forceinline__ float relu(float v) { return v > 0.0f ? v : 0.0f; }

__device__ __forceinline__ int32_t lo16(uint32_t w) { return (int32_t)(int16_t)(w & 0xffffu); }
__device__ __forceinline__ int32_t hi16(uint32_t w) { return (int32_t)w >> 16; }

// The backward ReLU mask is a byte per group of four elements (bit q: element q
// passes) in the INT16 output buffer, at the start of the 512 bytes that the
// 64 groups' own results fill.  The rounding pass therefore takes these 64
// groups with one wave at a time, all of whose lanes load before any stores
// (mask_barrier, and loops whose bounds are the same for the whole wave).
__device__ __forceinline__ int64_t mask_at(int32_t group) { return (int64_t)(group >> 6) * 512 + (group & 63); }
// Between a wave's mask loads and its first store (no instruction of its own):
// neither the compiler nor a lane moves a memory access across it.
__device__ __forceinline__ void mask_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// ------------------------------------------------------------ statistics
// Workgroup (s, c) reduces channel c over images [N s / S, N (s+1) / S).
// Forward: S1 = sum i, S2 = sum i^2, min i, max i.  Backward: D = sum g_i,
// Pd = sum g_i * y_i with g_i = dz_i where the recomputed pre-activation is
// positive, else 0.  Partials: part[(s*C + c)*3 + {0, 1, 2}], slot 2 holding
// (max << 32) | (uint32)min.  VEC: 8 elements per unit (hw % 8 == 0).
template <bool BWD, int V, bool RES>
__global__ __launch_bounds__(kBlock) void k_bn_stats(const int16_t* __restrict__ y, const int16_t* __restrict__ dz,
                                                     const float* __restrict__ res, const float* __restrict__ mean,
                                                     const float* __restrict__ inv, const float* __restrict__ gamma,
                                                     const float* __restrict__ beta, const dfp_scale* __restrict__ sy,
                                                     int32_t N, int32_t C, int32_t HW, int32_t S, FastDiv upr_div,
                                                     int64_t* __restrict__ part, uint8_t* __restrict__ mask,
                                                     dfp_scale* __restrict__ sz) {
  const int32_t s = blockIdx.x, c = blockIdx.y;
  if (sz && s == 0 && c == 0 && threadIdx.x == 0) {  // the finalize kernel max-reduces into it
    sz->amax_bits = 0u;
    sz->flags = 0u;
  }
  const int32_t n0 = (int32_t)((int64_t)N * s / S), n1 = (int32_t)((int64_t)N * (s + 1) / S);
  const int32_t upr = HW / V;
  const int32_t units = (n1 - n0) * upr;
  int64_t a = 0, b = 0;
  int32_t mn = INT_MAX, mx = INT_MIN;
  Chan p{};
  int32_t ey = 0;
  if (BWD) {
    p = load_chan(mean, inv, gamma, beta, c);
    ey = sy->exp;
  }
  // one unit's loads (V elements); the next unit's are in flight while one is summed
  struct Unit {
    int32_t off;
    uint32_t y[(V + 1) / 2], d[(V + 1) / 2];
    float r[V];
  };
  auto load = [&](int32_t j) {
    Unit u;
    const int32_t row = (int32_t)fdiv((uint32_t)j, upr_div);
    u.off = ((n0 + row) * C + c) * HW + (j - row * upr) * V;
    auto ints = [&](const int16_t* src, uint32_t(&w)[(V + 1) / 2]) {
      if constexpr (V == 8) {
        const uint4 q = *reinterpret_cast<const uint4*>(src + u.off);
        w[0] = q.x; w[1] = q.y; w[2] = q.z; w[3] = q.w;
      } else if constexpr (V == 4) {
        const uint2 q = *reinterpret_cast<const uint2*>(src + u.off);
        w[0] = q.x; w[1] = q.y;
      } else {
        w[0] = (uint16_t)src[u.off];
      }
    };
    ints(y, u.y);
    if (BWD) ints(dz, u.d);
    if (BWD && RES) {
      if constexpr (V >= 4) {
#pragma unroll
        for (int q = 0; q < V / 4; ++q) {
          const float4 f = *reinterpret_cast<const float4*>(res + u.off + 4 * q);
          u.r[4 * q] = f.x; u.r[4 * q + 1] = f.y; u.r[4 * q + 2] = f.z; u.r[4 * q + 3] = f.w;
        }
      } else {
        u.r[0] = res[u.off];
      }
    }
    return u;
  };
  auto add = [&](const Unit& u) {
    uint32_t bits = 0u;
#pragma unroll
    for (int q = 0; q < V; ++q) {
      const int32_t yv = (q & 1) ? hi16(u.y[q >> 1]) : lo16(u.y[q >> 1]);
      if (BWD) {
        const float zp = bn_affine(bn_xhat(yv, ey, p), p);
        const float pre = RES ? __fadd_rn(zp, u.r[q]) : zp;
        const int32_t dv = (q & 1) ? hi16(u.d[q >> 1]) : lo16(u.d[q >> 1]);
        const int32_t g = pre > 0.0f ? dv : 0;
        if (RES) bits |= (pre > 0.0f ? 1u : 0u) << q;
        a += g;
        b += g * yv;  // |g y| <= 2^30
      } else {
        a += yv;
        b += yv * yv;
        mn = min(mn, yv);
        mx = max(mx, yv);
      }
    }
    if (BWD && RES && V == 4) mask[mask_at(u.off >> 2)] = (uint8_t)bits;
  };
  int32_t j = threadIdx.x;
  if (j < units) {
    Unit u = load(j);
    for (; j + kBlock < units; j += kBlock) {
      const Unit nx = load(j + kBlock);
      add(u);
      u = nx;
    }
    add(u);
  }
  __shared__ int64_t ra[kBlock], rb[kBlock];
  __shared__ int32_t rmn[kBlock], rmx[kBlock];
  ra[threadIdx.x] = a;
  rb[threadIdx.x] = b;
  rmn[threadIdx.x] = mn;
  rmx[threadIdx.x] = mx;
  __syncthreads();
  for (int w = kBlock / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      ra[threadIdx.x] += ra[threadIdx.x + w];
      rb[threadIdx.x] += rb[threadIdx.x + w];
      rmn[threadIdx.x] = min(rmn[threadIdx.x], rmn[threadIdx.x + w]);
      rmx[threadIdx.x] = max(rmx[threadIdx.x], rmx[threadIdx.x + w]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    int64_t* o = part + ((int64_t)s * C + c) * 3;
    o[0] = ra[0];
    o[1] = rb[0];
    o[2] = (int64_t)(((uint64_t)(uint32_t)rmx[0] << 32) | (uint32_t)rmn[0]);
  }
}

// -------------------------------------------------------------- finalize
// One wave per channel: the lanes add the channel's S partials (exact
// integers), lane 0 derives the per-channel values.
// Forward: mean / inv_std from the exact sums (float64, rounded once), and
// without a residual the output max from the channel's extreme integers,
// max-reduced into the output scale (cleared by the statistics kernel).
// Per channel for the element passes: forward (mean, inv_std, gamma, beta),
// backward (k1, k2, k3, mean), with dbeta and dgamma.
template <bool BWD>
__global__ __launch_bounds__(kBlock) void k_bn_finalize(const int64_t* __restrict__ part, int32_t S, int32_t C,
                                                        int64_t cnt, const dfp_scale* __restrict__ sy,
                                                        const dfp_scale* __restrict__ sdz, float eps,
                                                        const float* __restrict__ gamma,
                                                        const float* __restrict__ beta, float* __restrict__ mean,
                                                        float* __restrict__ inv, int64_t* __restrict__ sums,
                                                        float* __restrict__ dgamma, float* __restrict__ dbeta,
                                                        float4* __restrict__ kco,
                                                        dfp_scale* __restrict__ sz, bool write_max) {
  const int lane = threadIdx.x & 63;
  const int32_t c = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
  if (c >= C) return;
  int64_t a = 0, b = 0;
  int32_t mn = INT_MAX, mx = INT_MIN;
  for (int32_t s = lane; s < S; s += 64) {
    const int64_t* o = part + ((int64_t)s * C + c) * 3;
    a += o[0];
    b += o[1];
    const uint64_t e = (uint64_t)o[2];
    mn = min(mn, (int32_t)(uint32_t)e);
    mx = max(mx, (int32_t)(uint32_t)(e >> 32));
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    a += __shfl_xor(a, off, 64);
    b += __shfl_xor(b, off, 64);
    mn = min(mn, __shfl_xor(mn, off, 64));
    mx = max(mx, __shfl_xor(mx, off, 64));
  }
  if (lane != 0) return;
  const int32_t ey = sy->exp;
  const double dcnt = (double)cnt;
  if (sums) {
    sums[2 * c] = a;
    sums[2 * c + 1] = b;
  }
  if (!BWD) {
    const double mu = __ddiv_rn(ldexp((double)a, ey), dcnt);
    double var = __dsub_rn(__ddiv_rn(ldexp((double)b, 2 * ey), dcnt), __dmul_rn(mu, mu));
    if (var < 0.0) var = 0.0;
    const float mf = (float)mu;
    const float t = __fadd_rn((float)var, eps);
    const float sq = (float)__dsqrt_rn((double)t);  // correctly rounded FP32 square root
    const float iv = __fdiv_rn(1.0f, sq);
    mean[c] = mf;
    inv[c] = iv;
    kco[c] = make_float4(mf, iv, gamma[c], beta[c]);
    if (write_max) {
      const Chan p{mf, iv, gamma[c], beta[c]};
      const float zlo = relu(bn_affine(bn_xhat(mn, ey, p), p));
      const float zhi = relu(bn_affine(bn_xhat(mx, ey, p), p));
      const uint32_t m = max(__float_as_uint(zlo), __float_as_uint(zhi)) & 0x7fffffffu;
      if (m) atomicMax(&sz->amax_bits, m);
    }
  } else {
    const int32_t edz = sdz->exp;
    const double mf = (double)mean[c], iv = (double)inv[c];
    const double db = ldexp((double)a, edz);
    const double dg = __dmul_rn(iv, ldexp(__dsub_rn(ldexp((double)b, ey), __dmul_rn(mf, (double)a)), edz));
    const float dbf = (float)db, dgf = (float)dg;
    dbeta[c] = dbf;
    dgamma[c] = dgf;
    const double al = __dmul_rn((double)gamma[c], iv);  // exact: two FP32 factors
    kco[c] = make_float4((float)al, (float)__ddiv_rn(__dmul_rn(-al, (double)dgf), dcnt),
                         (float)__ddiv_rn(__dmul_rn(-al, (double)dbf), dcnt), mean[c]);
  }
}

// ------------------------------------------------------ element groups
// Flat groups of four consecutive elements (the Philox block of stochastic
// rounding).  Channel of element idx: (idx / hw) mod C.
struct Elems {
  const int16_t* y;
  const int16_t* dz;
  const float* res;     // null where the mask replaces it
  const uint8_t* mask;  // backward with res and hw % 4 == 0 (mask_at)
  const float4* kco;    // forward mean, inv_std, gamma, beta; backward k1, k2, k3, mean
  const float *inv, *gamma, *beta;  // backward
  const dfp_scale* sy;
  const dfp_scale* sdz;
  int32_t total, C;
  FastDiv hw_div, c_div;
  bool hw4;  // hw % 4 == 0
};

__device__ __forceinline__ int32_t chan_of(const Elems& e, int32_t idx) {
  const uint32_t row = fdiv((uint32_t)idx, e.hw_div);
  return (int32_t)(row - fdiv(row, e.c_div) * (uint32_t)e.C);
}

// A group's operands, loaded ahead of their use (the last group may be short).
//   HW4: hw % 4 == 0, so a group lies in one channel.  SRC: where the ReLU's
//   sign comes from: kPlain the affine value, kRes that plus the residual,
//   kMask (backward, HW4, with a residual) the mask of the statistics pass.
enum Src { kPlain = 0, kRes = 1, kMask = 2 };
struct Group {
  uint2 y, d;
  float4 r;
  uint32_t mask;
  float4 k;     // channel values (HW4): kco, and backward inv_std, gamma, beta
  float inv, gamma, beta;
};
__device__ __forceinline__ int32_t group_int(const uint2& w, int q) {
  const uint32_t v = q < 2 ? w.x : w.y;
  return (q & 1) ? hi16(v) : lo16(v);
}
__device__ __forceinline__ uint2 short_group(const int16_t* src, int32_t left) {
  const uint32_t a = (uint16_t)src[0], b = left > 1 ? (uint16_t)src[1] : 0u, c = left > 2 ? (uint16_t)src[2] : 0u;
  return make_uint2(a | (b << 16), c);
}
template <bool BWD, int SRC>
__device__ __forceinline__ void load_channel(const Elems& e, int32_t c, Group& g) {
  g.k = e.kco[c];
  if (BWD) {
    g.inv = e.inv[c];
    if (SRC != kMask) {
      g.gamma = e.gamma[c];
      g.beta = e.beta[c];
    }
  }
}
template <bool BWD, bool HW4, int SRC>
__device__ __forceinline__ Group load_group(const Elems& e, int32_t gi) {
  Group g;
  const int32_t base = gi << 2;
  const float4 z4 = make_float4(0.f, 0.f, 0.f, 0.f);
  g.d = make_uint2(0u, 0u);
  g.r = g.k = z4;
  g.inv = g.gamma = g.beta = 0.f;
  if (base + 4 <= e.total) {
    g.y = *reinterpret_cast<const uint2*>(e.y + base);
    if (BWD) g.d = *reinterpret_cast<const uint2*>(e.dz + base);
    if (SRC == kRes) g.r = *reinterpret_cast<const float4*>(e.res + base);
  } else {
    const int32_t left = e.total - base;
    g.y = short_group(e.y + base, left);
    if (BWD) g.d = short_group(e.dz + base, left);
    if (SRC == kRes) g.r = make_float4(e.res[base], left > 1 ? e.res[base + 1] : 0.f, left > 2 ? e.res[base + 2] : 0.f, 0.f);
  }
  g.mask = SRC == kMask ? e.mask[mask_at(gi)] : 0u;
  if (HW4) load_channel<BWD, SRC>(e, chan_of(e, base), g);
  return g;
}

// Values of group gi (elements past the tensor's end: 0): the forward output
// z, or the backward gradient dy = fma(k1, g, fma(k2, xhat, k3)) with g =
// pre > 0 ? dz 2^Edz : 0, which is also the gradient at res.
template <bool BWD, bool HW4, int SRC>
__device__ __forceinline__ void group_values(const Elems& e, Group in, int32_t gi, int32_t ey, int32_t edz,
                                             float v[4], float g[4]) {
  const int32_t base = gi << 2;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    v[q] = 0.0f;
    g[q] = 0.0f;
    if (base + q >= e.total) continue;
    if (!HW4) load_channel<BWD, SRC>(e, chan_of(e, base + q), in);
    const float4 k = in.k;
    const Chan p = BWD ? Chan{k.w, in.inv, in.gamma, in.beta} : Chan{k.x, k.y, k.z, k.w};
    const int32_t yi = group_int(in.y, q);
    const float xh = bn_xhat(yi, ey, p);
    bool pass = false;
    float pre = 0.0f;
    if (SRC == kMask) {
      pass = (in.mask >> q) & 1u;
    } else {
      pre = bn_affine(xh, p);
      if (SRC == kRes) pre = __fadd_rn(pre, q == 0 ? in.r.x : q == 1 ? in.r.y : q == 2 ? in.r.z : in.r.w);
      pass = pre > 0.0f;
    }
    if (BWD) {
      const int32_t di = group_int(in.d, q);
      g[q] = pass ? ldexpf((float)di, edz) : 0.0f;
      v[q] = __fmaf_rn(k.x, g[q], __fmaf_rn(k.y, xh, k.z));
    } else {
      v[q] = pass ? pre : 0.0f;
    }
  }
}

// Stores the group's valid values.
__device__ __forceinline__ void store_group(float* dst, int32_t base, int32_t total, const float v[4]) {
  if (base + 4 <= total) {
    *reinterpret_cast<float4*>(dst + base) = make_float4(v[0], v[1], v[2], v[3]);
  } else {
#pragma unroll
    for (int q = 0; q < 3; ++q)
      if (base + q < total) dst[base + q] = v[q];
  }
}

// Max pass: part[workgroup] = max |v| bits over its groups (part == nullptr:
// a single workgroup writes the scale directly and clears its flags).  Also
// stores the values (forward z, backward dy) and the gradient at res where
// asked.  Two groups' loads are in flight per thread.
template <bool BWD, bool HW4, int SRC>
__global__ __launch_bounds__(kBlock) void k_bn_amax(Elems e, float* __restrict__ out, float* __restrict__ dres,
                                                    uint32_t* __restrict__ part, dfp_scale* __restrict__ s) {
  const int32_t ey = e.sy->exp;
  const int32_t edz = BWD ? e.sdz->exp : 0;
  const int32_t groups = (e.total + 3) >> 2;
  const int32_t stride = gridDim.x * kBlock;
  uint32_t m = 0u;
  auto use = [&](Group in, int32_t gi) {
    float v[4], g[4];
    group_values<BWD, HW4, SRC>(e, in, gi, ey, edz, v, g);
#pragma unroll
    for (int q = 0; q < 4; ++q) m = max(m, __float_as_uint(v[q]) & 0x7fffffffu);
    if (out) store_group(out, gi << 2, e.total, v);
    if (BWD && dres) store_group(dres, gi << 2, e.total, g);
  };
  int32_t gi = blockIdx.x * kBlock + threadIdx.x;
  for (; gi < groups - stride; gi += 2 * stride) {
    const Group a = load_group<BWD, HW4, SRC>(e, gi), b = load_group<BWD, HW4, SRC>(e, gi + stride);
    use(a, gi);
    use(b, gi + stride);
  }
  if (gi < groups) use(load_group<BWD, HW4, SRC>(e, gi), gi);
  __shared__ uint32_t red[kBlock / 64];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off, 64));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t r = red[0];
    for (int i = 1; i < kBlock / 64; ++i) r = max(r, red[i]);
    if (part) {
      part[blockIdx.x] = r;
    } else {
      s->amax_bits = r;
      s->flags = 0u;
    }
  }
}

// Rounding pass: recomputes each element's value, rounds it with the shared
// exponent of the tensor max (Eq. 2-3, the descriptor's mode), writes the
// INT16 result and, forward, the FP32 value when z != nullptr.
template <bool BWD, bool HW4, int SRC, int MODE, bool SAT>
__global__ __launch_bounds__(kBlock) void k_bn_convert(Elems e, float* __restrict__ z, int16_t* dst,
                                                       dfp_scale* __restrict__ s, int32_t bits, uint32_t key0,
                                                       uint32_t key1, uint32_t role) {
  const ScaleFromMax sc = scale_from_max(s->amax_bits, bits);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    s->exp = sc.es;
    if (sc.flags) atomicOr(&s->flags, sc.flags);
  }
  const int32_t ey = e.sy->exp;
  const int32_t edz = BWD ? e.sdz->exp : 0;
  const int32_t groups = (e.total + 3) >> 2;
  const int32_t stride = gridDim.x * kBlock;
  bool saturated = false;
  auto use = [&](Group in, int32_t gi) {
    const int32_t base = gi << 2;
    float v[4], g[4];
    group_values<BWD, HW4, SRC>(e, in, gi, ey, edz, v, g);
    uint32_t u[4] = {0u, 0u, 0u, 0u};
    if (MODE == DFP_ROUND_STOCHASTIC) {
      const uint4 r = philox4x32_10(make_uint4((uint32_t)gi, 0u, role, 0u), key0, key1);
      u[0] = r.x; u[1] = r.y; u[2] = r.z; u[3] = r.w;
    }
    int32_t iv[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      int32_t t = round_one<MODE>(__float_as_uint(v[q]), sc.es, u[q]);
      t = sc.all_zero ? 0 : t;
      if (SAT) {
        const int32_t cl = min(max(t, -32767), 32767);
        saturated |= cl != t;
        t = cl;
      }
      iv[q] = t;
    }
    if (base + 4 <= e.total) {
      uint2 packed;
      packed.x = ((uint32_t)iv[0] & 0xffffu) | ((uint32_t)iv[1] << 16);
      packed.y = ((uint32_t)iv[2] & 0xffffu) | ((uint32_t)iv[3] << 16);
      *reinterpret_cast<uint2*>(dst + base) = packed;
    } else {
#pragma unroll
      for (int q = 0; q < 3; ++q)
        if (base + q < e.total) dst[base + q] = (int16_t)iv[q];
    }
    if (!BWD && z) store_group(z, base, e.total, v);
  };
  // Bounds on the wave's first group: a bound per lane would split a wave where
  // the number of groups is not a multiple of 64, and its first lanes would store
  // over mask bytes that the others load afterwards.  (first < groups - stride:
  // every lane of the wave has a first group, since stride is a multiple of 64.)
  int32_t gi = blockIdx.x * kBlock + threadIdx.x;
  int32_t first = __builtin_amdgcn_readfirstlane(gi);
  for (; first < groups - stride; gi += 2 * stride, first += 2 * stride) {
    const bool two = gi + stride < groups;
    const Group a = load_group<BWD, HW4, SRC>(e, gi);
    Group b{};
    if (two) b = load_group<BWD, HW4, SRC>(e, gi + stride);
    if (SRC == kMask) mask_barrier();
    use(a, gi);
    if (two) use(b, gi + stride);
  }
  Group a{};
  if (gi < groups) a = load_group<BWD, HW4, SRC>(e, gi);
  if (SRC == kMask) mask_barrier();
  if (gi < groups) use(a, gi);
  if (SAT && saturated) atomicOr(&s->flags, DFP_FLAG_SATURATED);
}

// ------------------------------------------------------------------ SGD
// g = fma(wd, w, dw); v = fma(mu, v, g); w = fma(-lr, v, w), in place, and the
// max |w| per workgroup (as k_bn_amax).
__global__ __launch_bounds__(kBlock) void k_sgd(int64_t n, float lr, float mu, float wd, float* __restrict__ w,
                                                float* __restrict__ v, const float* __restrict__ dw,
                                                uint32_t* __restrict__ part, dfp_scale* __restrict__ s) {
  const int64_t groups = (n + 3) >> 2;
  uint32_t m = 0u;
  for (int64_t gi = (int64_t)blockIdx.x * kBlock + threadIdx.x; gi < groups; gi += (int64_t)gridDim.x * kBlock) {
    const int64_t base = gi << 2;
    if (base + 4 <= n) {
      float4 w4 = reinterpret_cast<const float4*>(w)[gi];
      float4 v4 = reinterpret_cast<const float4*>(v)[gi];
      const float4 d4 = reinterpret_cast<const float4*>(dw)[gi];
      float* wp = &w4.x;
      float* vp = &v4.x;
      const float* dp = &d4.x;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float g = __fmaf_rn(wd, wp[q], dp[q]);
        vp[q] = __fmaf_rn(mu, vp[q], g);
        wp[q] = __fmaf_rn(-lr, vp[q], wp[q]);
        m = max(m, __float_as_uint(wp[q]) & 0x7fffffffu);
      }
      reinterpret_cast<float4*>(w)[gi] = w4;
      reinterpret_cast<float4*>(v)[gi] = v4;
    } else {
      for (int64_t i = base; i < n; ++i) {
        const float g = __fmaf_rn(wd, w[i], dw[i]);
        const float vn = __fmaf_rn(mu, v[i], g);
        const float wn = __fmaf_rn(-lr, vn, w[i]);
        v[i] = vn;
        w[i] = wn;
        m = max(m, __float_as_uint(wn) & 0x7fffffffu);
      }
    }
  }
  __shared__ uint32_t red[kBlock / 64];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off, 64));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t r = red[0];
    for (int i = 1; i < kBlock / 64; ++i) r = max(r, red[i]);
    if (part) {
      part[blockIdx.x] = r;
    } else {
      s->amax_bits = r;
      s->flags = 0u;
    }
  }
}

// ------------------------------------------------------------ host side
int32_t bn_splits(const dfp_bn_desc& d) {
  const int32_t want = (2048 + d.c - 1) / d.c;
  return std::max(1, std::min(want, d.n));
}

// Workgroups of a max pass over `groups` groups of four whose per-workgroup
// maxima have room for `room`; <= 1 means one workgroup writing the scale
// directly.
int32_t max_parts(int64_t groups, int64_t room) {
  int64_t parts = (groups + kBlock - 1) / kBlock;
  parts = std::min<int64_t>(std::min<int64_t>(parts, kMaxParts), room);
  return (int32_t)std::max<int64_t>(parts, 1);
}

// Workspace: the statistics' partial sums, the per-channel values and, where the
// sums of few images and channels are too little room for them, the max pass's
// partial maxima; else these follow the sums in the same place once the finalize
// kernel has read them.  A workspace without that last part (bn_least_bytes) gets
// as many workgroups as the sums have room for (N = 1, C = 16, hw = 2^20, with a
// residual forward 190 and backward 497 us, with 128 workgroups 225 and 559).
struct BnWs {
  int64_t* part;
  float4* kco;
  uint32_t* maxima;
  int64_t room;  // words at maxima
};
int64_t align256(int64_t v) { return (v + 255) / 256 * 256; }
int64_t bn_part_bytes(const dfp_bn_desc& d) { return align256((int64_t)bn_splits(d) * d.c * 24); }
int64_t bn_least(const dfp_bn_desc& d) { return bn_part_bytes(d) + align256((int64_t)d.c * 16); }
int64_t bn_maxima_bytes(const dfp_bn_desc& d) {  // 0: in the sums' place
  const int64_t b = align256((int64_t)max_parts(((int64_t)d.n * d.c * d.hw + 3) / 4, kMaxParts) * 4);
  return b > bn_part_bytes(d) ? b : 0;
}
BnWs bn_ws(const dfp_bn_desc& d, void* ws, size_t ws_bytes) {
  const int64_t part = bn_part_bytes(d), least = bn_least(d), maxima = bn_maxima_bytes(d);
  uint8_t* w = reinterpret_cast<uint8_t*>(ws);
  const bool own = maxima > 0 && ws_bytes >= (size_t)(least + maxima);
  return {reinterpret_cast<int64_t*>(w), reinterpret_cast<float4*>(w + part),
          reinterpret_cast<uint32_t*>(own ? w + least : w), (own ? maxima : part) / 4};
}

template <bool BWD, bool RES>
dfp_status launch_stats(const dfp_bn_desc& d, const int16_t* y, const int16_t* dz, const float* res,
                        const float* mean, const float* inv, const float* gamma, const float* beta,
                        const dfp_scale* sy, const BnWs& w, uint8_t* mask, dfp_scale* sz, hipStream_t st) {
  const int32_t S = bn_splits(d);
  // elements per load (every tensor is 16-byte aligned); with a residual four,
  // so that a wave's loads of it are contiguous
  const int32_t V = !RES && d.hw % 8 == 0 ? 8 : d.hw % 4 == 0 ? 4 : 1;
  const FastDiv upr = make_fastdiv((uint32_t)(d.hw / V));
  const dim3 grid((unsigned)S, (unsigned)d.c);
  if (V == 8)
    DFP_LAUNCH(K_BN_STATS, (k_bn_stats<BWD, RES ? 4 : 8, RES>), grid, dim3(kBlock), 0, st, y, dz, res, mean, inv, gamma, beta,
               sy, d.n, d.c, d.hw, S, upr, w.part, mask, sz);
  else if (V == 4)
    DFP_LAUNCH(K_BN_STATS, (k_bn_stats<BWD, 4, RES>), grid, dim3(kBlock), 0, st, y, dz, res, mean, inv, gamma, beta,
               sy, d.n, d.c, d.hw, S, upr, w.part, mask, sz);
  else
    DFP_LAUNCH(K_BN_STATS, (k_bn_stats<BWD, 1, RES>), grid, dim3(kBlock), 0, st, y, dz, res, mean, inv, gamma, beta,
               sy, d.n, d.c, d.hw, S, upr, w.part, mask, sz);
  return DFP_OK;
}

Elems make_elems(const dfp_bn_desc& d, const int16_t* y, const float* res, const BnWs& w, const dfp_scale* sy) {
  Elems e{};
  e.y = y; e.res = res; e.kco = w.kco;
  e.sy = sy;
  e.total = d.n * d.c * d.hw;
  e.C = d.c;
  e.hw_div = make_fastdiv((uint32_t)d.hw);
  e.c_div = make_fastdiv((uint32_t)d.c);
  e.hw4 = (d.hw % 4) == 0;
  return e;
}

// Calls f(HW4, SRC) with the element kernels' template arguments.
template <bool BWD, typename F>
dfp_status with_src(const Elems& e, F f) {
  using std::false_type;
  using std::true_type;
  if (!e.hw4)
    return e.res ? f(false_type{}, std::integral_constant<int, kRes>{}) : f(false_type{}, std::integral_constant<int, kPlain>{});
  if constexpr (BWD)
    return e.mask ? f(true_type{}, std::integral_constant<int, kMask>{}) : f(true_type{}, std::integral_constant<int, kPlain>{});
  else
    return e.res ? f(true_type{}, std::integral_constant<int, kRes>{}) : f(true_type{}, std::integral_constant<int, kPlain>{});
}

// Max pass (k_bn_amax + the max reduce) into s.
template <bool BWD>
dfp_status launch_max(const Elems& e, float* out, float* dres, const BnWs& w, dfp_scale* s, hipStream_t st) {
  const int32_t parts = max_parts((e.total + 3) / 4, w.room);
  uint32_t* part = parts > 1 ? w.maxima : nullptr;
  dfp_status rc = with_src<BWD>(e, [&](auto hw4, auto src) -> dfp_status {
    DFP_LAUNCH(K_BN_AMAX, (k_bn_amax<BWD, decltype(hw4)::value, decltype(src)::value>), dim3((unsigned)parts),
               dim3(kBlock), 0, st, e, out, dres, part, s);
    return DFP_OK;
  });
  if (rc != DFP_OK || !part) return rc;
  return launch_amax_final(part, parts, s, st);
}

template <bool BWD, int MODE>
dfp_status launch_convert_mode(const Elems& e, float* z, int16_t* dst, dfp_scale* s, int32_t bits, uint64_t seed,
                               uint32_t role, hipStream_t st) {
  int64_t blocks = ((int64_t)(e.total + 3) / 4 + kBlock - 1) / kBlock;
  blocks = std::max<int64_t>(1, std::min<int64_t>(blocks, 8192));
  const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
  return with_src<BWD>(e, [&](auto hw4, auto src) -> dfp_status {
    constexpr bool H = decltype(hw4)::value;
    constexpr int S = decltype(src)::value;
    if (bits == 16)
      DFP_LAUNCH(K_BN_CONVERT, (k_bn_convert<BWD, H, S, MODE, true>), dim3((unsigned)blocks), dim3(kBlock), 0, st, e,
                 z, dst, s, bits, k0, k1, role);
    else
      DFP_LAUNCH(K_BN_CONVERT, (k_bn_convert<BWD, H, S, MODE, false>), dim3((unsigned)blocks), dim3(kBlock), 0, st, e,
                 z, dst, s, bits, k0, k1, role);
    return DFP_OK;
  });
}

template <bool BWD>
dfp_status launch_convert(const Elems& e, float* z, int16_t* dst, dfp_scale* s, int32_t bits, int32_t rounding,
                          uint64_t seed, uint32_t role, hipStream_t st) {
  switch (rounding) {
    case DFP_ROUND_NEAREST: return launch_convert_mode<BWD, DFP_ROUND_NEAREST>(e, z, dst, s, bits, seed, role, st);
    case DFP_ROUND_STOCHASTIC:
      return launch_convert_mode<BWD, DFP_ROUND_STOCHASTIC>(e, z, dst, s, bits, seed, role, st);
    case DFP_ROUND_BIASED: return launch_convert_mode<BWD, DFP_ROUND_BIASED>(e, z, dst, s, bits, seed, role, st);
    default: return launch_convert_mode<BWD, DFP_ROUND_DOWN>(e, z, dst, s, bits, seed, role, st);
  }
}

}  // namespace

size_t bn_workspace_bytes(const dfp_bn_desc& d) { return (size_t)(bn_least(d) + bn_maxima_bytes(d)); }
size_t bn_least_bytes(const dfp_bn_desc& d) { return (size_t)bn_least(d); }

dfp_status launch_bn_relu_fwd(const dfp_bn_desc& d, const int16_t* y, const dfp_scale* sy, const float* gamma,
                              const float* beta, const float* res, float* z, int16_t* zq, dfp_scale* sz, float* mean,
                              float* inv_std, int64_t* sums, void* ws, size_t ws_bytes, hipStream_t st) {
  const BnWs w = bn_ws(d, ws, ws_bytes);
  dfp_status rc;
  if ((rc = launch_stats<false, false>(d, y, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, sy, w, nullptr,
                                       res ? nullptr : sz, st)) != DFP_OK)
    return rc;
  const int64_t cnt = (int64_t)d.n * d.hw;
  DFP_LAUNCH(K_BN_FINAL, k_bn_finalize<false>, dim3((unsigned)((d.c + 3) / 4)), dim3(kBlock), 0, st, w.part, bn_splits(d), d.c, cnt, sy,
             (const dfp_scale*)nullptr, d.eps, gamma, beta, mean, inv_std, sums, (float*)nullptr, (float*)nullptr,
             w.kco, sz, res == nullptr);
  const Elems e = make_elems(d, y, res, w, sy);
  if (res) {
    if ((rc = launch_max<false>(e, z, nullptr, w, sz, st)) != DFP_OK) return rc;
    // z written: 4 bytes of it per element to read against 6 of y and res
    if (z) return launch_quant_convert(z, zq, e.total, sz, d.bits, d.rounding, d.seed, DFP_ROLE_X, st);
  }
  return launch_convert<false>(e, z, zq, sz, d.bits, d.rounding, d.seed, DFP_ROLE_X, st);
}

dfp_status launch_bn_relu_bwd(const dfp_bn_desc& d, const int16_t* dz, const dfp_scale* sdz, const int16_t* y,
                              const dfp_scale* sy, const float* gamma, const float* beta, const float* res,
                              const float* mean, const float* inv_std, float* dy, int16_t* dyq, dfp_scale* sdy,
                              float* dgamma, float* dbeta, float* dres, int64_t* sums, void* ws,
                              size_t ws_bytes, hipStream_t st) {
  const BnWs w = bn_ws(d, ws, ws_bytes);
  dfp_status rc;
  // with a residual the statistics pass leaves the ReLU mask in dyq
  uint8_t* mask = res && d.hw % 4 == 0 ? reinterpret_cast<uint8_t*>(dyq) : nullptr;
  rc = res ? launch_stats<true, true>(d, y, dz, res, mean, inv_std, gamma, beta, sy, w, mask, nullptr, st)
           : launch_stats<true, false>(d, y, dz, res, mean, inv_std, gamma, beta, sy, w, mask, nullptr, st);
  if (rc != DFP_OK) return rc;
  const int64_t cnt = (int64_t)d.n * d.hw;
  DFP_LAUNCH(K_BN_FINAL, k_bn_finalize<true>, dim3((unsigned)((d.c + 3) / 4)), dim3(kBlock), 0, st, w.part, bn_splits(d), d.c, cnt, sy, sdz,
             d.eps, gamma, beta, const_cast<float*>(mean), const_cast<float*>(inv_std), sums, dgamma, dbeta, w.kco,
             (dfp_scale*)nullptr, false);
  Elems e = make_elems(d, y, mask ? nullptr : res, w, sy);
  e.dz = dz; e.sdz = sdz; e.mask = mask;
  e.inv = inv_std; e.gamma = gamma; e.beta = beta;
  if ((rc = launch_max<true>(e, dy, dres, w, sdy, st)) != DFP_OK) return rc;
  if (dy) return launch_quant_convert(dy, dyq, e.total, sdy, d.bits, d.rounding, d.seed, DFP_ROLE_DY, st);
  return launch_convert<true>(e, nullptr, dyq, sdy, d.bits, d.rounding, d.seed, DFP_ROLE_DY, st);
}

dfp_status launch_sgd_quantize(int64_t n, float lr, float mu, float wd, int32_t bits, int32_t rounding,
                               uint64_t seed, float* w, float* v, const float* dw, int16_t* wq, dfp_scale* sw,
                               hipStream_t st) {
  const int32_t parts = max_parts((n + 3) / 4, n / 2);  // in wq
  if (parts <= 1) {
    DFP_LAUNCH(K_SGD, k_sgd, dim3(1), dim3(kBlock), 0, st, n, lr, mu, wd, w, v, dw, (uint32_t*)nullptr, sw);
  } else {
    uint32_t* part = reinterpret_cast<uint32_t*>(wq);
    DFP_LAUNCH(K_SGD, k_sgd, dim3((unsigned)parts), dim3(kBlock), 0, st, n, lr, mu, wd, w, v, dw, part, sw);
    dfp_status rc;
    if ((rc = launch_amax_final(part, parts, sw, st)) != DFP_OK) return rc;
  }
  return launch_quant_convert(w, wq, n, sw, bits, rounding, seed, DFP_ROLE_W, st);
}

}  // namespace dfp
