// DFP16 GEMM (the paper's INT16 kernels serve "convolutions and GEMM",
// Sec. 4): D[i][j] = sum over t of opA[i][t] * opB[t][j], with the forward
// convolution's numeric contract (Algorithm 2, Sec. 4.3): INT32 partials over
// chunks of L consecutive t (mod 2^32), each converted to FP32 and added in
// chunk order, one scale 2^(Ea+Eb) at the end.
//
// A GEMM is the 1x1 forward convolution whose pixels are the columns of D:
// the matrix-core path prepares opA as the filter digit planes and opB as the
// channels-last activation digit planes (reduction padded with zero digits to
// a multiple of 32) and runs the convolution's main kernels on them.  The
// VALU kernel below serves P = 16 and path = VALU.
#include <algorithm>
#include <cmath>

#include "dfp_internal.h"
#include "conv_mfma.h"

namespace dfp {

namespace {

constexpr int kBlock = 256;

__device__ __forceinline__ uint32_t hi_byte(int32_t a) { return (uint32_t)((a + 128) >> 8) & 0xffu; }
__device__ __forceinline__ uint32_t lo_byte(int32_t a) { return (uint32_t)a & 0xffu; }

// Digit planes of one operand view: element (row, t) = src[row * rs + t * ts]
// for row < rows and t < K, else 0.  Unit (row, g) covers t in [16g, 16g+16)
// and is stored as 16 hi bytes then 16 lo bytes at
//   A layout (a_layout = 1): ((g / 2) * rows_pad + row) * 64 + (g % 2) * 32
//   B layout (a_layout = 0): (row * G16 + g) * 32
// One thread per unit.  row_fast: consecutive threads take consecutive rows
// (coalesced when t is the strided index), else consecutive g.  One launch
// prepares the operands that need it (workgroups [0, na) the rows, the rest the
// columns), clears the output scale and writes the per-block B offset table.
struct DigitOp {
  const int16_t* src;
  int64_t rs, ts;
  uint8_t* dst;
  int32_t rows, rows_pad, a_layout, row_fast;
};
__global__ __launch_bounds__(kBlock) void k_gemm_digits(DigitOp opa, DigitOp opb, int32_t na, int32_t K, int32_t G16,
                                                        dfp_scale* so, int2* boff) {
  if (so && blockIdx.x == 0 && threadIdx.x == 0) {
    so->amax_bits = 0u;
    so->flags = 0u;
  }
  // block kb reads its two 16-index halves at byte offsets 32*(2kb), 32*(2kb+1)
  // of a column; halves at or past K read offset 0 (their A digits are zero)
  if (boff) {
    const int64_t kb = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (kb < G16 / 2) {
      const int32_t t0 = (int32_t)kb * 32;
      boff[kb] = make_int2(t0 < K ? (t0 >> 4) * 32 : 0, t0 + 16 < K ? ((t0 + 16) >> 4) * 32 : 0);
    }
  }
  const bool is_a = (int32_t)blockIdx.x < na;
  const int16_t* __restrict__ src = is_a ? opa.src : opb.src;
  uint8_t* dst = is_a ? opa.dst : opb.dst;
  const int64_t rs = is_a ? opa.rs : opb.rs, ts = is_a ? opa.ts : opb.ts;
  const int32_t rows = is_a ? opa.rows : opb.rows, rows_pad = is_a ? opa.rows_pad : opb.rows_pad;
  const int32_t a_layout = is_a ? opa.a_layout : opb.a_layout;
  const int64_t idx = (int64_t)(blockIdx.x - (is_a ? 0 : na)) * kBlock + threadIdx.x;
  const int64_t units = (int64_t)rows_pad * G16;
  if (idx >= units) return;
  int32_t row, g;
  if (is_a ? opa.row_fast : opb.row_fast) {
    row = (int32_t)(idx % rows_pad);
    g = (int32_t)(idx / rows_pad);
  } else {
    g = (int32_t)(idx % G16);
    row = (int32_t)(idx / G16);
  }
  uint32_t hi[4] = {0u, 0u, 0u, 0u}, lo[4] = {0u, 0u, 0u, 0u};
  if (row < rows) {
    const int16_t* p = src + (int64_t)row * rs;
    const int32_t t0 = g * 16;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int32_t t = t0 + i;
      const int32_t v = t < K ? (int32_t)p[(int64_t)t * ts] : 0;
      hi[i >> 2] |= hi_byte(v) << (8 * (i & 3));
      lo[i >> 2] |= lo_byte(v) << (8 * (i & 3));
    }
  }
  const int64_t off = a_layout ? (((int64_t)(g >> 1) * rows_pad + row) * 64 + (g & 1) * 32)
                               : (((int64_t)row * G16 + g) * 32);
  uint4* d = reinterpret_cast<uint4*>(dst + off);
  d[0] = make_uint4(hi[0], hi[1], hi[2], hi[3]);
  d[1] = make_uint4(lo[0], lo[1], lo[2], lo[3]);
}

// VALU GEMM: one lane per output, chunked INT32 partials, FP32 fold in chunk
// order, one scale; epilogue max |D| into so (cleared by the launcher).
template <bool PARTIALS>
__global__ __launch_bounds__(kBlock) void k_gemm_valu(const int16_t* __restrict__ a, int64_t ars, int64_t ats,
                                                      const int16_t* __restrict__ b, int64_t bts, int64_t bcs,
                                                      int32_t m, int32_t n, int32_t K, int32_t L,
                                                      const dfp_scale* __restrict__ sa,
                                                      const dfp_scale* __restrict__ sb, float* __restrict__ d,
                                                      dfp_scale* so, int32_t* __restrict__ partials) {
  const int64_t O = (int64_t)m * n;
  const int64_t o = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  const bool active = o < O;
  float y = 0.f;
  if (active) {
    const int64_t i = o / n, j = o % n;
    const int16_t* pa = a + i * ars;
    const int16_t* pb = b + j * bcs;
    float sum = 0.f;
    int64_t chunk = 0;
    for (int32_t t0 = 0; t0 < K; t0 += L, ++chunk) {
      const int32_t t1 = min(K, t0 + L);
      uint32_t acc = 0u;
      for (int32_t t = t0; t < t1; ++t) acc += (uint32_t)((int32_t)pa[t * ats] * (int32_t)pb[t * bts]);
      if (PARTIALS) partials[chunk * O + o] = (int32_t)acc;
      const float f = (float)(int32_t)acc;
      sum = chunk == 0 ? f : sum + f;
    }
    y = ldexpf(sum, sa->exp + sb->exp);
    d[o] = y;
  }
  if (so) {
    __shared__ uint32_t red[kBlock / 64];
    uint32_t mx = active ? (__float_as_uint(y) & 0x7fffffffu) : 0u;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mx = max(mx, (uint32_t)__shfl_xor((int)mx, off, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
      uint32_t bm = red[0];
      for (int w = 1; w < kBlock / 64; ++w) bm = max(bm, red[w]);
      if (bm > __atomic_load_n(&so->amax_bits, __ATOMIC_RELAXED)) atomicMax(&so->amax_bits, bm);
      if (bm == 0x7f800000u) atomicOr(&so->flags, DFP_FLAG_OUTPUT_INF);
    }
  }
}

// VALU Blocked-DFP GEMM (t contiguous in both operands): every chunk partial is
// scaled by 2^(ea[blk][i] + eb[blk][j]) before it joins the FP32 sum.
template <bool PARTIALS>
__global__ __launch_bounds__(kBlock) void k_gemm_blocked_valu(const int16_t* __restrict__ a,
                                                              const int8_t* __restrict__ ea,
                                                              const int16_t* __restrict__ b,
                                                              const int8_t* __restrict__ eb, int32_t m, int32_t n,
                                                              int32_t K, int32_t L, int32_t bk,
                                                              float* __restrict__ d, dfp_scale* so,
                                                              int32_t* __restrict__ partials) {
  const int64_t O = (int64_t)m * n;
  const int64_t o = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  const bool active = o < O;
  float y = 0.f;
  if (active) {
    const int64_t i = o / n, j = o % n;
    const int16_t* pa = a + i * K;
    const int16_t* pb = b + j * K;
    float sum = 0.f;
    int64_t chunk = 0;
    for (int32_t t0 = 0; t0 < K; t0 += L, ++chunk) {
      const int32_t t1 = min(K, t0 + L);
      uint32_t acc = 0u;
      for (int32_t t = t0; t < t1; ++t) acc += (uint32_t)((int32_t)pa[t] * (int32_t)pb[t]);
      if (PARTIALS) partials[chunk * O + o] = (int32_t)acc;
      const int32_t blk = t0 / bk;
      const float term = ldexpf((float)(int32_t)acc, (int32_t)ea[(int64_t)blk * m + i] + (int32_t)eb[(int64_t)blk * n + j]);
      sum = chunk == 0 ? term : sum + term;
    }
    y = sum;
    d[o] = y;
  }
  if (so) {
    __shared__ uint32_t red[kBlock / 64];
    uint32_t mx = active ? (__float_as_uint(y) & 0x7fffffffu) : 0u;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mx = max(mx, (uint32_t)__shfl_xor((int)mx, off, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
      uint32_t bm = red[0];
      for (int w = 1; w < kBlock / 64; ++w) bm = max(bm, red[w]);
      if (bm > __atomic_load_n(&so->amax_bits, __ATOMIC_RELAXED)) atomicMax(&so->amax_bits, bm);
      if (bm == 0x7f800000u) atomicOr(&so->flags, DFP_FLAG_OUTPUT_INF);
    }
  }
}

// ---------------------------------------------------------------------------
// Split-chunk GEMM for outputs too small to fill the chip with 64 x 128 tiles
// (a fully connected layer's 64 x 1000 output is 8 of them, each a serial
// chain of k / 32 blocks).  Only the FP32 fold over the chunks is ordered; the
// chunks' INT32 partials are independent.  A workgroup of 16 waves takes a
// tile of 16 RT rows x 16 columns; wave w computes the partials of chunks w,
// w + 16, ... (v_mfma_i32_16x16x64_i8), converts them (Blocked-DFP: and scales
// them) and leaves them in LDS, and after each round of 16 chunks one thread
// per output adds them in chunk order.  An operand whose reduction is
// contiguous is read as INT16 and split into digits in registers (16 indices
// are 32 bytes of a lane); the other kind comes from the digit preparation.
// Chunks of a multiple of 64 indices, or of 32 (half of the lanes' row digits
// are then zeroed).
// 64 x 1000 x 2048 at L = 64: 55 us on the tiled kernel with its preparation,
// 12 us here (Blocked-DFP 61 and 12).
constexpr int kSplitWaves = 16;
typedef int gv4i __attribute__((ext_vector_type(4)));

struct SplitArgs {
  const int16_t* a;    // raw: [m][k]
  const int16_t* b;    // raw: [n][k]
  const uint8_t* ad;   // digits [KB][Mp][2][32 B]
  const uint8_t* bd;   // digits [n][G16][32 B]
  const dfp_scale *sa, *sb;
  const int8_t *exa, *exb;  // Blocked-DFP exponents [nb][m], [nb][n]
  float* d;
  dfp_scale* so;
  int32_t m, n, k, L, J, Mp, G16, bk;
};

struct Digits {
  gv4i hi, lo;
};
// Digits of 16 INT16 values in eight dwords: the high bytes of v + 128 (as
// 16-bit lanes) and the low bytes of v.
__device__ __forceinline__ Digits split16(const uint4& p, const uint4& q) {
  typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
  const uint32_t w[8] = {p.x, p.y, p.z, p.w, q.x, q.y, q.z, q.w};
  const u16x2 r = {128, 128};
  Digits o;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t h0 = __builtin_bit_cast(uint32_t, (u16x2)(__builtin_bit_cast(u16x2, w[2 * i]) + r));
    const uint32_t h1 = __builtin_bit_cast(uint32_t, (u16x2)(__builtin_bit_cast(u16x2, w[2 * i + 1]) + r));
    o.hi[i] = (int)__builtin_amdgcn_perm(h1, h0, 0x07050301u);
    o.lo[i] = (int)__builtin_amdgcn_perm(w[2 * i + 1], w[2 * i], 0x06040200u);
  }
  return o;
}

// An operand's 16 indices t0 .. t0 + 15 of one row (row < rows, else the last
// row: its products are not stored), zero at and past k.
struct Piece {
  uint4 p, q;
};
template <bool RAW>
__device__ __forceinline__ Piece load_piece(const int16_t* __restrict__ src, const uint8_t* __restrict__ dig,
                                            int64_t dig_off, int32_t row, int32_t k, int32_t t0) {
  Piece r;
  if (!RAW) {  // hi digits, lo digits
    const uint4* d = reinterpret_cast<const uint4*>(dig + dig_off);
    r.p = d[0];
    r.q = d[1];
    return r;
  }
  const int16_t* x = src + (int64_t)row * k;
  if (t0 + 16 <= k) {
    struct __attribute__((packed, aligned(2))) Raw32 { uint32_t w[8]; };
    const Raw32 v = *reinterpret_cast<const Raw32*>(x + t0);
    r.p = make_uint4(v.w[0], v.w[1], v.w[2], v.w[3]);
    r.q = make_uint4(v.w[4], v.w[5], v.w[6], v.w[7]);
  } else {
    uint32_t w[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int32_t t = t0 + 2 * i;
      const uint32_t lo = t < k ? (uint16_t)x[t] : 0u, hi = t + 1 < k ? (uint16_t)x[t + 1] : 0u;
      w[i] = lo | (hi << 16);
    }
    r.p = make_uint4(w[0], w[1], w[2], w[3]);
    r.q = make_uint4(w[4], w[5], w[6], w[7]);
  }
  return r;
}
template <bool RAW>
__device__ __forceinline__ Digits digits_of(const Piece& r) {
  if (RAW) return split16(r.p, r.q);
  return {(gv4i){(int)r.p.x, (int)r.p.y, (int)r.p.z, (int)r.p.w}, (gv4i){(int)r.q.x, (int)r.q.y, (int)r.q.z, (int)r.q.w}};
}

template <int RT, bool ARAW, bool BRAW, bool BLOCKED>
__global__ __launch_bounds__(64 * kSplitWaves) void k_gemm_split(SplitArgs a) {
  __shared__ float part[2][kSplitWaves][RT * 256];  // [round parity][chunk of the round][subtile, value, lane]
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lc = lane & 15, kg = lane >> 4;
  const int32_t m0 = blockIdx.y * 16 * RT, n0 = blockIdx.x * 16;
  const int32_t jb = min(n0 + lc, a.n - 1);  // this lane's column
  const bool half = a.L == 32;               // two chunks per 64 indices
  const int32_t ngrp = half ? 1 : a.L / 64;  // groups of 64 indices per chunk
  const int32_t rounds = (a.J + kSplitWaves - 1) / kSplitWaves;
  const int32_t e = BLOCKED ? 0 : a.sa->exp + a.sb->exp;

  auto load_b = [&](int32_t t0) { return load_piece<BRAW>(a.b, a.bd, ((int64_t)jb * a.G16 + (t0 >> 4)) * 32, jb, a.k, t0); };
  auto load_a = [&](int32_t t0, int sb) {
    const int32_t i = m0 + sb * 16 + lc;
    return load_piece<ARAW>(a.a, a.ad, ((int64_t)(t0 >> 5) * a.Mp + i) * 64 + ((t0 >> 4) & 1) * 32, min(i, a.m - 1),
                            a.k, t0);
  };
  // indices of this lane in the chunk's first group; digit planes end at the padded k
  auto first_t = [&](int32_t j) { return (half ? (j >> 1) * 64 : j * a.L) + kg * 16; };
  const int32_t t_end = a.G16 * 16;
  const gv4i z = {0, 0, 0, 0};

  // output of this thread in the fold: (subtile, value, lane) as in part
  const int32_t fs = (int32_t)threadIdx.x >> 8, fv = ((int32_t)threadIdx.x >> 6) & 3;
  float sum = 0.f;
  for (int32_t r = 0; r < rounds; ++r) {
    const int32_t j = r * kSplitWaves + wave;
    if (j < a.J) {
      gv4i hh[RT], xx[RT], ll[RT];
#pragma unroll
      for (int sb = 0; sb < RT; ++sb) hh[sb] = xx[sb] = ll[sb] = z;
      const bool mine = !half || (kg >> 1) == (j & 1);
      for (int32_t g = 0; g < ngrp; ++g) {
        const int32_t t0 = first_t(j) + g * 64;
        const bool in = (ARAW && BRAW) || t0 < t_end;
        Piece pb, pa[RT];
        const int32_t tt = in ? t0 : 0;  // (digit planes: a piece past the end is read nowhere; its row digits are zeroed)
        pb = load_b(tt);
#pragma unroll
        for (int sb = 0; sb < RT; ++sb) pa[sb] = load_a(tt, sb);
        const Digits db = digits_of<BRAW>(pb);
#pragma unroll
        for (int sb = 0; sb < RT; ++sb) {
          Digits da = digits_of<ARAW>(pa[sb]);
          if (!mine || !in) da.hi = da.lo = z;
          hh[sb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(da.hi, db.hi, hh[sb], 0, 0, 0);
          ll[sb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(da.lo, db.lo, ll[sb], 0, 0, 0);
          xx[sb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(da.hi, db.lo, xx[sb], 0, 0, 0);
          xx[sb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(da.lo, db.hi, xx[sb], 0, 0, 0);
        }
      }
      int32_t eb = 0, blk = 0;
      if (BLOCKED) {
        blk = (int32_t)((int64_t)j * a.L / a.bk);
        eb = a.exb[(int64_t)blk * a.n + jb];
      }
#pragma unroll
      for (int sb = 0; sb < RT; ++sb)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const uint32_t p = ((((uint32_t)hh[sb][v] << 8) + (uint32_t)xx[sb][v]) << 8) + (uint32_t)ll[sb][v];
          float f = (float)(int32_t)p;
          if (BLOCKED) {
            const int32_t i = min(m0 + sb * 16 + 4 * kg + v, a.m - 1);
            f = ldexpf(f, (int32_t)a.exa[(int64_t)blk * a.m + i] + eb);
          }
          part[r & 1][wave][(sb * 4 + v) * 64 + lane] = f;
        }
    }
    __syncthreads();  // one barrier a round: the next round writes the other half
    if (threadIdx.x < 256 * RT) {
      const int32_t nj = min(kSplitWaves, a.J - r * kSplitWaves);
      for (int32_t i = 0; i < nj; ++i) sum += part[r & 1][i][threadIdx.x];
    }
  }
  uint32_t amax = 0;
  const int32_t i = m0 + fs * 16 + 4 * kg + fv, jo = n0 + lc;
  if (threadIdx.x < 256 * RT && i < a.m && jo < a.n) {
    const float y = BLOCKED ? sum : ldexpf(sum, e);
    a.d[(int64_t)i * a.n + jo] = y;
    amax = __float_as_uint(y) & 0x7fffffffu;
  }
  if (a.so) {
    __shared__ uint32_t red[kSplitWaves];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) amax = max(amax, (uint32_t)__shfl_xor((int)amax, off, 64));
    if (lane == 0) red[wave] = amax;
    __syncthreads();
    if (threadIdx.x == 0) {
      uint32_t bm = red[0];
      for (int w = 1; w < kSplitWaves; ++w) bm = max(bm, red[w]);
      if (bm > __atomic_load_n(&a.so->amax_bits, __ATOMIC_RELAXED)) atomicMax(&a.so->amax_bits, bm);
      if (bm == 0x7f800000u) atomicOr(&a.so->flags, DFP_FLAG_OUTPUT_INF);
    }
  }
}

inline int64_t align256(int64_t v) { return (v + 255) & ~(int64_t)255; }

}  // namespace

GemmPlan plan_gemm(int32_t m, int32_t n, int32_t k) {
  GemmPlan p{};
  p.KB = (k + 31) / 32;
  p.G16 = p.KB * 2;
  p.Mp = (m + kMfmaRowTile - 1) / kMfmaRowTile * kMfmaRowTile;
  p.a_bytes = align256((int64_t)p.KB * p.Mp * 64);
  p.b_bytes = align256((int64_t)n * p.G16 * 32);
  p.t_bytes = align256((int64_t)p.KB * 8);
  p.bytes = p.a_bytes + p.b_bytes + p.t_bytes;
  return p;
}

// Row subtiles per split-chunk workgroup, 0 where the tiled kernels run.  The
// tiled kernels take about 0.7 us per 32 indices however few their tiles, up
// to two per CU; the split kernel's operand traffic grows with its tiles:
// 256 x 4096 x 4096 (128 tiles of 64 x 128) 106 us split and 130 us tiled with
// both operands read as INT16, 113 and 112 us with one prepared.  One subtile
// while the 16 x 16 tiles are few (252: 11.8 / 12.0 / 17.0 us for 1 / 2 / 4),
// more where they are many, since each workgroup re-reads its operands (512:
// 17.7 / 15.6 / 17.1; 1008: 27 / 21 / 19).
// Between them by estimates in us, fitted to 450 products (1 to 5800 rows, 2 to
// 8200 columns, k to 10000) on both sides, off by 7% tiled and 20% split: few
// chunks leave most of a split workgroup's 16 waves idle, and Blocked-DFP
// gathers a chunk's exponents per output (533 x 1046 x 64 at L = 32 10.8 us tiled
// and 15.9 split, blocked 11.3 and 35).
static int32_t split_rt(int32_t m, int32_t n) {
  const int64_t t16 = (int64_t)((m + 15) / 16) * ((n + 15) / 16);
  const int32_t rt = t16 <= 320 ? 1 : t16 <= 600 ? 2 : 4;
  return m <= 16 ? 1 : m <= 32 ? std::min(rt, 2) : rt;
}
// araw, braw: the operand would be read as INT16.
static bool split_pays(int32_t m, int32_t n, int32_t k, int32_t L, int32_t rt, bool blocked, bool araw, bool braw) {
  const int64_t J = ((int64_t)k + L - 1) / L;
  const int64_t tiles = (int64_t)((m + 63) / 64) * ((n + 127) / 128);
  if ((L != 32 && L % 64 != 0) || J < 2 || tiles > 96) return false;
  const double KB = (k + 31) / 32, A = 1e-6 * (double)m * k, B = 1e-6 * (double)n * k, D = 1e-6 * (double)m * n;
  const double wgs = (double)((n + 15) / 16) * ((m + 16 * rt - 1) / (16 * rt));
  const double rounds = (double)((J + kSplitWaves - 1) / kSplitWaves) * std::max(1.0, wgs / 110);
  const double groups = std::max(1, L / 64) * std::sqrt((double)rt);
  const double prep = (araw ? 0 : A) + (braw ? 0 : B);
  const double tiled = blocked ? 7.5 + 0.73 * KB + 1.9 * (A + B) + 3.6 * D : 7.4 + 0.62 * KB + 1.7 * (A + B) + 4.3 * D;
  const double split = blocked ? 7.1 + rounds * (0.29 + groups) + 0.5 * prep + 1.7 * wgs / 256 * rt
                               : 7.5 + rounds * (0.83 + 0.42 * groups) + prep + 0.09 * wgs / 256 * rt;
  return split < tiled;
}

template <int RT, bool BLOCKED>
static dfp_status launch_split(const SplitArgs& a, bool araw, bool braw, hipStream_t st) {
  const dim3 grid((unsigned)((a.n + 15) / 16), (unsigned)((a.m + 16 * RT - 1) / (16 * RT))), block(64 * kSplitWaves);
  const int kid = BLOCKED ? K_GEMM_BLOCKED : K_GEMM;
  if (araw && braw) DFP_LAUNCH(kid, (k_gemm_split<RT, true, true, BLOCKED>), grid, block, 0, st, a);
  else if (araw) DFP_LAUNCH(kid, (k_gemm_split<RT, true, false, BLOCKED>), grid, block, 0, st, a);
  else if (braw) DFP_LAUNCH(kid, (k_gemm_split<RT, false, true, BLOCKED>), grid, block, 0, st, a);
  else DFP_LAUNCH(kid, (k_gemm_split<RT, false, false, BLOCKED>), grid, block, 0, st, a);
  return DFP_OK;
}

dfp_status launch_gemm_mfma(int32_t m, int32_t n, int32_t k, int32_t trans_a, int32_t trans_b, int32_t L,
                            const int16_t* a, const dfp_scale* sa, const int16_t* b, const dfp_scale* sb,
                            float* d, dfp_scale* so, int32_t* partials, void* ws, hipStream_t st,
                            const int8_t* exa, const int8_t* exb, int32_t bk) {
  const GemmPlan p = plan_gemm(m, n, k);
  uint8_t* wsa = reinterpret_cast<uint8_t*>(ws);
  uint8_t* xs = wsa + p.a_bytes;
  int2* boff = reinterpret_cast<int2*>(xs + p.b_bytes);
  // Split kernel: an operand whose reduction is contiguous is read as INT16, with
  // no preparation, where every row is 4-byte aligned or, since unaligned loads
  // split, one workgroup reads it (1 x 2934 x 9175 33 us so and 68 prepared; 37 x 80
  // x 7999, whose operands 5 and 3 workgroups read, 56 and 14).
  int32_t rt = split_rt(m, n);
  auto aligned_rows = [&](const int16_t* x) { return k % 2 == 0 && (reinterpret_cast<uintptr_t>(x) & 3) == 0; };
  bool araw = !trans_a && (aligned_rows(a) || n <= 16), braw = trans_b && (aligned_rows(b) || m <= 16 * rt);
  if (partials || !split_pays(m, n, k, L, rt, exa != nullptr, araw, braw)) {
    rt = 0;
    araw = braw = false;
  }
  if (araw && braw) {
    if (so) {
      const dfp_status rc = launch_scale_reset(so, st);
      if (rc != DFP_OK) return rc;
    }
  } else {
    // opA[i][t] = a[i*k + t] or a[t*m + i]; column j of opB: opB[t][j] = b[t*n + j] or b[j*k + t]
    const DigitOp oa{a, trans_a ? 1 : k, trans_a ? m : 1, wsa, m, p.Mp, 1, trans_a};
    const DigitOp ob{b, trans_b ? k : 1, trans_b ? 1 : n, xs, n, n, 0, !trans_b};
    const int64_t ua = araw ? 0 : (int64_t)p.Mp * p.G16, ub = braw ? 0 : (int64_t)n * p.G16;
    const int64_t na = (ua + kBlock - 1) / kBlock, nb = (ub + kBlock - 1) / kBlock;
    const int64_t nt = rt ? 0 : (p.KB + kBlock - 1) / kBlock;  // workgroups the offset table needs
    DFP_LAUNCH(K_GEMM_PREP, k_gemm_digits, dim3((unsigned)std::max(na + nb, nt)), dim3(kBlock), 0, st, oa, ob,
               (int32_t)na, k, p.G16, so, rt ? (int2*)nullptr : boff);
  }
  if (rt) {
    const SplitArgs sp{a, b, wsa, xs, sa, sb, exa, exb, d, so, m, n, k, L, (k + L - 1) / L, p.Mp, p.G16, bk};
    if (exa)
      return rt == 1   ? launch_split<1, true>(sp, araw, braw, st)
             : rt == 2 ? launch_split<2, true>(sp, araw, braw, st)
                       : launch_split<4, true>(sp, araw, braw, st);
    return rt == 1   ? launch_split<1, false>(sp, araw, braw, st)
           : rt == 2 ? launch_split<2, false>(sp, araw, braw, st)
                     : launch_split<4, false>(sp, araw, braw, st);
  }
  ConvMfmaArgs args{};
  args.xs = xs;
  args.wsa = wsa;
  args.boff = boff;
  args.ea = sa;
  args.eb = sb;
  args.out = d;
  args.so = so;
  args.partials = partials;
  args.M = m; args.Mp = p.Mp; args.Cin = p.KB * 32; args.S = 1; args.T = k; args.KB = p.KB; args.L = L;
  args.CG = p.G16; args.Hp = 1; args.Wp = n; args.Po = 1; args.Qo = n;
  args.NP = n;
  args.O = (int64_t)m * n;
  args.ustride_h = 1; args.ustride_w = 1; args.rsign = 1; args.roff_h = 0; args.roff_w = 0;
  args.exa = exa;
  args.exb = exb;
  args.bk = bk;
  args.nb = exa ? (k + bk - 1) / bk : 0;
  return launch_mfma_main(args, p.b_bytes, exa ? K_GEMM_BLOCKED : K_GEMM, K_GEMM, false, st);
}

dfp_status launch_gemm_blocked_valu(int32_t m, int32_t n, int32_t k, int32_t L, int32_t bk, const int16_t* a,
                                    const int8_t* ea, const int16_t* b, const int8_t* eb, float* d, dfp_scale* so,
                                    int32_t* partials, hipStream_t st) {
  const int64_t O = (int64_t)m * n;
  const dim3 grid((unsigned)((O + kBlock - 1) / kBlock));
  if (partials)
    DFP_LAUNCH(K_GEMM_BLOCKED, k_gemm_blocked_valu<true>, grid, dim3(kBlock), 0, st, a, ea, b, eb, m, n, k, L, bk, d,
               so, partials);
  else
    DFP_LAUNCH(K_GEMM_BLOCKED, k_gemm_blocked_valu<false>, grid, dim3(kBlock), 0, st, a, ea, b, eb, m, n, k, L, bk,
               d, so, partials);
  return DFP_OK;
}

dfp_status launch_gemm_valu(int32_t m, int32_t n, int32_t k, int32_t trans_a, int32_t trans_b, int32_t L,
                            const int16_t* a, const dfp_scale* sa, const int16_t* b, const dfp_scale* sb,
                            float* d, dfp_scale* so, int32_t* partials, hipStream_t st) {
  const int64_t ars = trans_a ? 1 : k, ats = trans_a ? m : 1;
  const int64_t bts = trans_b ? 1 : n, bcs = trans_b ? k : 1;
  const int64_t O = (int64_t)m * n;
  const dim3 grid((unsigned)((O + kBlock - 1) / kBlock));
  if (partials)
    DFP_LAUNCH(K_GEMM, k_gemm_valu<true>, grid, dim3(kBlock), 0, st, a, ars, ats, b, bts, bcs, m, n, k, L, sa, sb, d,
               so, partials);
  else
    DFP_LAUNCH(K_GEMM, k_gemm_valu<false>, grid, dim3(kBlock), 0, st, a, ars, ats, b, bts, bcs, m, n, k, L, sa, sb,
               d, so, partials);
  return DFP_OK;
}

}  // namespace dfp
