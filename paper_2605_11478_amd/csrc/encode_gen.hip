// Encoder for block dimensions k = 4, 8, 16 and 32 (Eq. encode of Sec. 3.1)
// with the nearest-codeword search as a dense contraction on the matrix cores:
// every N, input type, row stride and alignment, d = 64 or 128 (k = 32: 64);
// and for k = 1 and 2 with a scan (scan_kernel below).  Over many rows the tile
// kernels of the specialised codes take over, and for tiny codebooks and dense
// k = 1 codes the general encoder (few_rows and scan_rows in codec_kernels.hip).
//
// A wavefront encodes 16 vectors per batch:
//
//   norm     nu^2 = sum x^2 in float64 (exact squares), header = binary16(nu)
//            rounded once, to nearest even;
//   rotate   y = Pi x / nu with v_mfma_f64_16x16x4_f64, so y carries only
//            float64 rounding; it is then rounded to float32.  Pi's rows are
//            permuted so that a lane ends with whole blocks (k <= 16) or half
//            a block (k = 32) of vector lane % 16;
//   screen   S_j = 2^24 (<y_b, c_j> - |c_j|^2 / 2) for 32 codewords x 32
//            blocks per v_mfma_f32_32x32x16_f16 (k = 8: one, its 16 K slots
//            hold y's binary16 hi and lo parts; k = 4: half of them; k = 16,
//            32: k / 8 products, hi then lo),
//            A = the codeword's binary16 rows, accumulators starting at
//            -2^24 |c_j|^2 / 2;
//   select   a lane holds the scores of 16 of a tile's 32 codewords; it keeps
//            the largest half-tile maximum, that tile's number (in the low
//            mantissa bits of the key) and the largest of the other tiles;
//   rescore  the 16 codewords of the best half-tile again in float32 from
//            float32 y, keeping the best two;
//   certify  if the best beats both its half-tile's second and the best of the
//            other tiles by more than a bound on the errors, it is the float64
//            argmin; otherwise the whole wavefront scores all N codewords of
//            that block in float64 (direct form, lowest index on ties);
//   pack     w-bit indices, little-endian bit stream of P bytes.
//
// Bound: a score tile (32 codewords x 32 blocks) is one 32-clock product and
// 11 vector instructions of 4.4 clocks, 62 clocks together as measured (the
// maxima read what the matrix cores write); at N = 4096 that is two thirds of
// the time, at N <= 1024 the rotation (64 clocks per float64 product) and the
// rescoring are.  147456 fp16 rows, d = 64, k = 8: N = 1024 1124 -> 91 us,
// N = 4096 4450 -> 260 us against one thread per vector; 262144 bf16 rows of
// d = 128, k = 4, N = 4096 1634 -> 1495 us against a float64 rescore of each
// best tile.
//
// The codebook's binary16 rows and norms stay in LDS when they fit; larger
// ones (CH) go through it in chunks that all wavefronts of the workgroup scan
// together.
//
// Error bounds (unscaled; a = |c|_max |y_b| bounds sum |c_i y_i|): float32 y
// 2^-24 a; its binary16 hi + lo 2^-22 a + 2^-28 |c|_1 (low parts may be
// flushed); codewords that are not binary16-exact clo |y_b|, clo the largest
// |c - fp16(c)|_2; the accumulation of the NM products' 16 NM + 1 terms at most
// 32 NM ulps of their sum of magnitudes:
//   e_s = (2^-18 NM + 2^-21) a + (2^-18 NM + 2^-22) |c|^2_max / 2
//         + 2^-28 |c|_1,max + clo |y_b|   (+ the packed bits of the key)
//   e_r = (k + 4) 2^-24 (a + |c|^2_max / 2) + clo |y_b|
// each with a 25 % margin.
#include <hip/hip_runtime.h>

#include "device_common.h"
#include "fibq.h"
#include "fibq_internal.h"

namespace fibq {
namespace dev {
namespace gen {

constexpr int kVec = 16;  // vectors of a wavefront batch
constexpr float kY = 16384.0f, kC = 1024.0f;  // scales of y and c (2^14, 2^10)
constexpr float kS = kY * kC;                 // of the scores
constexpr int kOps = 4;                       // 32-block operands screened together, at most

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f16v __attribute__((ext_vector_type(16)));
typedef double d4 __attribute__((ext_vector_type(4)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));

// LDS rows: k binary16 per codeword, 16 bytes of padding per tile of 32, so
// that lanes reading the same row of different tiles use different banks; norms
// likewise (16 bytes per 32 floats).
template <int K>
__device__ __forceinline__ uint32_t row_at(uint32_t j) { return j * (2 * K) + (j >> 5) * 16; }
// eight binary16 of an A operand; k = 4: the row's four, twice
template <int K>
__device__ __forceinline__ h8 load_a(const unsigned char* p) {
  if constexpr (K == 4) {
    const h4 v = *reinterpret_cast<const h4*>(p);
    return h8{v[0], v[1], v[2], v[3], v[0], v[1], v[2], v[3]};
  } else {
    return *reinterpret_cast<const h8*>(p);
  }
}
__device__ __forceinline__ uint32_t nrm_at(uint32_t j) { return j * 4 + (j >> 5) * 16; }
template <int K>
constexpr size_t rows_bytes(int n) { return (size_t)n * 2 * K + (n / 32) * 16; }
constexpr size_t nrms_bytes(int n) { return (size_t)n * 4 + (n / 32) * 16; }

__device__ __forceinline__ float fmax3(float a, float b, float c) {
  return __builtin_elementwise_maximum(__builtin_elementwise_maximum(a, b), c);
}
__device__ __forceinline__ double shfl64(double v, int src) {
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)u, src, 64);
  const uint32_t hi = (uint32_t)__shfl((int)(uint32_t)(u >> 32), src, 64);
  return __longlong_as_double((long long)((uint64_t)lo | ((uint64_t)hi << 32)));
}
__device__ __forceinline__ double xor64(double v, int m) {
  return shfl64(v, (int)(threadIdx.x & 63) ^ m);
}
// a's upper half-wavefront and b's lower one trade places
__device__ __forceinline__ void swap32(uint32_t& a, uint32_t& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}
__device__ __forceinline__ void swap32(float& a, float& b) {
  uint32_t x = __float_as_uint(a), y = __float_as_uint(b);
  swap32(x, y);
  a = __uint_as_float(x);
  b = __uint_as_float(y);
}
// the value of lane ^ 32
__device__ __forceinline__ float other_half(float v) {
  float a = v, b = v;
  swap32(a, b);  // a: the lower half's values everywhere, b: the upper half's
  return (threadIdx.x & 32) ? a : b;
}

template <typename IN, int NQ>
__device__ __forceinline__ void load_row(const IN* p, float* xf) {
  constexpr int E = 16 / sizeof(IN);
#pragma unroll
  for (int i = 0; i < NQ / E; ++i) {
    IN w[E];
    __builtin_memcpy(w, p + i * E, 16);
#pragma unroll
    for (int e = 0; e < E; ++e) xf[i * E + e] = to_float(w[e]);
  }
}

// E floats as E / 2 dwords of binary16 pairs (hi), and the rest (lo)
template <int E>
__device__ __forceinline__ void split8(const float* y, uint32_t (&hi)[4], uint32_t (&lo)[4]) {
#pragma unroll
  for (int i = 0; i < E / 2; ++i) {
    const h2 h = h2{(_Float16)y[2 * i], (_Float16)y[2 * i + 1]};
    hi[i] = __builtin_bit_cast(uint32_t, h);
    asm("" : "+v"(hi[i]));  // the rest is taken from these bits
    const h2 g = __builtin_bit_cast(h2, hi[i]);
    lo[i] = __builtin_bit_cast(uint32_t, h2{(_Float16)(y[2 * i] - (float)g[0]),
                                            (_Float16)(y[2 * i + 1] - (float)g[1])});
  }
}

// Float64 nearest codeword of block m of one row, by the whole wavefront.
template <typename IN, int D, int K>
__device__ __noinline__ int scan64(const IN* __restrict__ row, const float* __restrict__ R,
                                   const float* __restrict__ C, int N, int m, double inv) {
  const int lane = threadIdx.x & 63;
  double y[K];
#pragma unroll
  for (int r = 0; r < K; ++r) {
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < D; j += 64)
      s = fma((double)R[(m * K + r) * D + j + lane], (double)to_float(row[j + lane]), s);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += xor64(s, o);
    y[r] = s * inv;
  }
  double bd = INFINITY;
  int bj = 0;
  for (int j = lane; j < N; j += 64) {
    double s = 0.0;
#pragma unroll
    for (int r = 0; r < K; ++r) {
      const double t = y[r] - (double)C[(size_t)j * K + r];
      s = fma(t, t, s);
    }
    if (s < bd) { bd = s; bj = j; }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const double od = xor64(bd, o);
    const int oj = __shfl_xor(bj, o, 64);
    if (od < bd || (od == bd && oj < bj)) { bd = od; bj = oj; }
  }
  return bj;
}

// Norm and rotation of 16 vectors: lane group g reads quarter g of row
// lane % 16 (xrow).  Returns nu, sets inv = 1 / nu (0 for a zero row) and
// yf[4 rt + i] = scale times row 4 i + g of rotation tile rt, whose row p is
// Pi's row prow(rt) in the lanes with lane % 16 = p (the float64 product leaves
// output row 4 i + g of a tile in register i of lane group g).
template <typename IN, int D, int NT, typename F>
__device__ __forceinline__ double rotate(const IN* xrow, const float* __restrict__ R, float scale,
                                         F prow, float (&yf)[4 * NT], double& inv) {
  constexpr int NQ = D / 4;  // elements of a row per lane
  const int g = (threadIdx.x & 63) >> 4;
  float xf[NQ];
  load_row<IN, NQ>(xrow + NQ * g, xf);
  double ss = 0.0;
#pragma unroll
  for (int s = 0; s < NQ; ++s) ss = fma((double)xf[s], (double)xf[s], ss);
  ss += xor64(ss, 16);
  ss += xor64(ss, 32);
  const double nu = sqrt(ss);
  inv = nu > 0.0 ? 1.0 / nu : 0.0;
  const double sc = inv * (double)scale;
#pragma unroll
  for (int rt = 0; rt < NT; ++rt) {
    const float* pr = R + (size_t)prow(rt) * D + NQ * g;
    d4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < NQ; s += 4) {
      f4 p;
      __builtin_memcpy(&p, pr + s, 16);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)p[e], (double)xf[s + e], acc, 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      yf[4 * rt + i] = (float)(acc[i] * sc);
      // (keeps the binary16 parts from being converted from float64, which
      // is a software sequence)
      asm("" : "+v"(yf[4 * rt + i]));
    }
  }
  return nu;
}

// Lane v < 16 writes the bit stream of its vector from its indices.
template <int NB>
__device__ __forceinline__ void pack_row(const uint16_t* idx, bool zero, int W, uint8_t* dst) {
  uint64_t bits = 0;
  int nb = 0, at = 0;
#pragma unroll 8
  for (int m = 0; m < NB; ++m) {
    bits |= (uint64_t)(zero ? 0u : (uint32_t)idx[m]) << nb;
    nb += W;
    if (nb >= 32) {
      const uint32_t wv = (uint32_t)bits;
      __builtin_memcpy(dst + at, &wv, 4);
      at += 4;
      bits >>= 32;
      nb -= 32;
    }
  }
  for (; nb > 0; nb -= 8, bits >>= 8) dst[at++] = (uint8_t)bits;
}

// lane groups' blocks: a wavefront's rotation leaves 4 blocks (64 columns, two
// operands) for each of these
constexpr int quads(int D, int K) { return K <= 16 ? D / (4 * K) : 1; }

// NC: codewords in LDS at a time (N rounded up to 64, or a chunk of it when
// CH).  SP: quads(D, K) wavefronts share a batch, one quad of blocks each (few
// rows: more wavefronts, a shorter chain and less code for each).
template <typename IN, int D, int K, int WAVES, bool CH, bool SP>
__global__ __launch_bounds__(64 * WAVES) void encode_kernel(
    const IN* __restrict__ x, int64_t n_vec, int64_t stride, const float* __restrict__ R,
    const float* __restrict__ C, int N, int NC, int W, int P, uint32_t kmask_s,
    uint8_t* __restrict__ payload, uint16_t* __restrict__ norms) {
  constexpr int NB = D / K;                     // blocks per vector
  constexpr int QN = SP ? quads(D, K) : 1;      // wavefronts of a batch
  constexpr int QW = quads(D, K) / QN;          // quads of a wavefront
  constexpr int NT = K <= 16 ? QW * (K / 4) : 4;  // its row tiles of the rotation
  constexpr int NOP = K <= 16 ? 2 * QW : 1;     // its 32-block operands
  static_assert(!(SP && CH), "");
  constexpr int OPS = NOP < kOps ? NOP : kOps;  // screened together
  constexpr int NM = K <= 8 ? 1 : K / 8;        // matrix products per score
  constexpr int NA = K == 32 ? 2 : 1;           // A operands of a tile
  constexpr int ROWB = 2 * K;                   // bytes of a codeword's row
  constexpr int E8 = K < 8 ? K : 8;             // entries of a row read at once
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned char* rows = smem;
  unsigned char* nrms = smem + rows_bytes<K>(NC);
  __shared__ __align__(16) float cst[WAVES][4];                   // each wavefront's constants of the codebook
  __shared__ uint16_t stage[WAVES / QN][kVec][NB];  // chosen indices of a batch
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int q0 = wave % QN, wb = wave / QN;         // quad, batch of the workgroup
  const int h = lane >> 5, c32 = lane & 31, g = lane >> 4, v16 = lane & 15;

  // codewords c0 .. c0 + NC - 1 as scaled binary16 rows and norms (rows past N
  // score lowest; finite: a tile number in -inf's mantissa would be a NaN), and
  // their constants for the bounds
  float c2 = 0.0f, c1 = 0.0f, cl = 0.0f;
  bool odd = false;  // a codeword out of range
  auto stage_rows = [&](int c0, bool put) {
    for (int j = tid; j < (put ? NC : N); j += 64 * WAVES) {
      float n = -3e38f;
      double s = 0.0;
      float s1 = 0.0f, sl = 0.0f;
      const bool in = c0 + j < N;
#pragma unroll
      for (int p = 0; p < K; p += E8) {
        float cv[E8] = {};
        if (in) __builtin_memcpy(cv, C + (size_t)(c0 + j) * K + p, 4 * E8);
        _Float16 r[E8];
#pragma unroll
        for (int e = 0; e < E8; ++e) {
          r[e] = (_Float16)(cv[e] * kC);
          const float l = cv[e] - (float)r[e] * (1.0f / kC);
          s = fma((double)cv[e], (double)cv[e], s);
          s1 += fabsf(cv[e]);
          sl = fmaf(l, l, sl);
        }
        if (put)
          __builtin_memcpy(__builtin_assume_aligned(rows + row_at<K>(j) + 2 * p, 2 * E8), r, 2 * E8);
      }
      if (in) n = (float)(-0.5 * s * (double)kS);
      if (put) *reinterpret_cast<float*>(nrms + nrm_at(j)) = n;
      odd |= !(s <= 256.0);  // |c| <= 16: operands in binary16 range
      c2 = fmaxf(c2, (float)s);
      c1 = fmaxf(c1, s1);
      cl = fmaxf(cl, sl);
    }
  };
  stage_rows(0, !CH);
  c2 = wave_max(c2);
  c1 = wave_max(c1);
  cl = wave_max(cl);
  odd = __any(odd);
  if (lane == 0) *reinterpret_cast<f4*>(cst[wave]) = f4{c2, c1, cl, odd ? 1.0f : 0.0f};
  __syncthreads();
#pragma unroll
  for (int i = 0; i < WAVES; ++i) {
    const f4 v = *reinterpret_cast<const f4*>(cst[i]);
    c2 = fmaxf(c2, v[0]);
    c1 = fmaxf(c1, v[1]);
    cl = fmaxf(cl, v[2]);
    odd |= v[3] != 0.0f;
  }
  // (float32 sums of K terms: 2^-16 covers their rounding)
  const float c2max = c2 * (1.0f + 0x1p-16f);
  const float cn = sqrtf(c2max) * (1.0f + 0x1p-20f);
  const float c1max = c1 * (1.0f + 0x1p-16f);
  const float clo = sqrtf(cl) * (1.0f + 0x1p-16f);
  const bool bad = odd;
  // bounds as (slope) |y_b| + (constant), scaled, with the 25 % margin
  const float a_s = 0x1p-18f * NM + 0x1p-21f, a_n = 0x1p-18f * NM + 0x1p-22f;
  const float a_r = (K + 4) * 0x1p-24f;
  const float es1 = 1.25f * kS * (a_s * cn + clo);
  const float es0 = 1.25f * kS * (a_n * 0.5f * c2max + 0x1p-28f * c1max);
  const float er1 = 1.25f * kS * (a_r * cn + clo);
  const float er0 = 1.25f * kS * (a_r * 0.5f * c2max);
  const float epack = 1.25f * (float)(~kmask_s + 1u) * 0x1p-23f;

  const int64_t nbatch = (n_vec + kVec - 1) / kVec;
  const int64_t nw = (int64_t)gridDim.x * (WAVES / QN);
  for (int64_t b0 = (int64_t)blockIdx.x * (WAVES / QN); b0 < nbatch; b0 += nw) {
    const int64_t bt = b0 + wb;
    if (!CH && !SP && bt >= nbatch) break;  // (otherwise every wavefront reaches the barriers)
    const bool live = bt < nbatch;
    const int64_t v0 = (live ? bt : nbatch - 1) * kVec;
    const int64_t vl = v0 + v16 < n_vec ? v0 + v16 : n_vec - 1;  // clamped (ragged batch)
    const IN* xrow = x + vl * stride;
    // yf, scaled: yf[4 rt + i] is coordinate 4 (rt % (K/4)) + i of block
    // 4 (q0 + rt / (K/4)) + g (k <= 16), or coordinate 16 (g / 2) + 4 rt + i of
    // block g % 2 (k = 32)
    float yf[4 * NT];
    const int pg = v16 & 3, pi = v16 >> 2;
    double inv;
    const double nu = rotate<IN, D, NT>(xrow, R, kY, [&](int rt) {
      return K <= 16 ? K * (4 * (q0 + rt / (K / 4)) + pg) + 4 * (rt % (K / 4)) + pi
                     : 32 * (pg & 1) + 16 * (pg >> 1) + 4 * rt + pi;
    }, yf, inv);
    if (g == 0 && q0 == 0 && live && v0 + v16 < n_vec)
      norms[v0 + v16] = nu > 0.0 ? f64_to_f16_bits(nu) : (uint16_t)0;

#pragma unroll
    for (int o0 = 0; o0 < NOP; o0 += OPS) {
      // ---- B operands: [op][product]; k <= 16: a swap of half-wavefronts
      //      makes the operand of lane groups 0, 1 and that of groups 2, 3
      u4 bop[OPS][NM];
      if constexpr (K <= 16) {
#pragma unroll
        for (int o = 0; o < OPS; o += 2) {
          const float* yb = yf + (o0 + o) / 2 * K;
          constexpr int NP = K == 16 ? 2 : 1;
          uint32_t hi[NP][4], lo[NP][4];
#pragma unroll
          for (int p = 0; p < NP; ++p) split8<E8>(yb + 8 * p, hi[p], lo[p]);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            if constexpr (K == 4) {  // slots 0 .. 7: hi, lo; 8 .. 15: zero
              uint32_t a = i < 2 ? hi[0][i] : lo[0][i - 2], b = 0u;
              swap32(a, b);
              // (a zero above the lower half's parts; the upper half's parts below a zero)
              bop[o][0][i] = a; bop[o + 1][0][i] = b;
            } else if constexpr (K == 8) {
              uint32_t a = hi[0][i], b = lo[0][i];
              swap32(a, b);
              bop[o][0][i] = a; bop[o + 1][0][i] = b;
            } else {
              uint32_t a = hi[0][i], b = hi[1][i];
              swap32(a, b);
              bop[o][0][i] = a; bop[o + 1][0][i] = b;
              a = lo[0][i]; b = lo[1][i];
              swap32(a, b);
              bop[o][1][i] = a; bop[o + 1][1][i] = b;
            }
          }
        }
      } else {
        uint32_t hi[2][4], lo[2][4];
        split8<8>(yf, hi[0], lo[0]);
        split8<8>(yf + 8, hi[1], lo[1]);
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          bop[0][p] = u4{hi[p][0], hi[p][1], hi[p][2], hi[p][3]};
          bop[0][2 + p] = u4{lo[p][0], lo[p][1], lo[p][2], lo[p][3]};
        }
      }

      // ---- screen
      uint32_t kmask = kmask_s;  // in a VGPR: an and-or takes one scalar, the tile number
      asm("" : "+v"(kmask));
      float b1[OPS], b2[OPS];
#pragma unroll
      for (int o = 0; o < OPS; ++o) { b1[o] = -INFINITY; b2[o] = -INFINITY; }
      const unsigned char* arow = rows + row_at<K>(c32) + (K == 16 ? 16 * h : K == 32 ? 32 * h : 0);
      const unsigned char* nrow = nrms + 16 * h;
      for (int c0 = 0; c0 < N; c0 += NC) {
        if (CH) {
          __syncthreads();
          stage_rows(c0, true);
          __syncthreads();
        }
        // Two tiles a round; the maxima of one operand's scores are taken
        // while the matrix cores work on the next operand's (a 32x32x16
        // product and 8 max3 together take 42 clocks, each alone 32 and 35).
        constexpr int TS = ROWB * 32 + 16;  // bytes of a tile of rows
        auto fold = [&](const f16v& s, uint32_t tn, float& t1, float& t2) {
          float m = fmax3(s[0], s[1], s[2]);
          m = fmax3(m, s[3], s[4]);
          m = fmax3(m, s[5], s[6]);
          m = fmax3(m, s[7], s[8]);
          m = fmax3(m, s[9], s[10]);
          m = fmax3(m, s[11], s[12]);
          m = fmax3(m, s[13], s[14]);
          m = __builtin_elementwise_maximum(m, s[15]);
          const float mk = __uint_as_float((__float_as_uint(m) & kmask) | tn);
          t2 = __builtin_amdgcn_fmed3f(t1, t2, mk);
          t1 = __builtin_elementwise_maximum(t1, mk);
        };
#pragma unroll 1
        for (int t = 0; t < NC / 32; t += 2) {
          h8 A[2][NA];
          f16v cn16[2];
#pragma unroll
          for (int u = 0; u < 2; ++u) {
#pragma unroll
            for (int p = 0; p < NA; ++p) A[u][p] = load_a<K>(arow + (t + u) * TS + 16 * p);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const f4 v = *reinterpret_cast<const f4*>(nrow + (t + u) * 144 + 32 * r);
#pragma unroll
              for (int e = 0; e < 4; ++e) cn16[u][4 * r + e] = v[e];
            }
          }
          const uint32_t tn = (uint32_t)((c0 >> 5) + t);
          auto score = [&](int i) {
            f16v s = cn16[i / OPS];
#pragma unroll
            for (int p = 0; p < NM; ++p)
              s = __builtin_amdgcn_mfma_f32_32x32x16_f16(
                  A[i / OPS][p & (NA - 1)], __builtin_bit_cast(h8, bop[i % OPS][p]), s, 0, 0, 0);
            return s;
          };
          f16v sp = score(0);
#pragma unroll
          for (int i = 1; i <= 2 * OPS; ++i) {
            f16v sn{};
            if (i < 2 * OPS) sn = score(i);
            fold(sp, tn + (i - 1) / OPS, b1[(i - 1) % OPS], b2[(i - 1) % OPS]);
            sp = sn;
          }
          if constexpr (D == 64 && NM == 1 && !SP) {  // (elsewhere the compiler's own order is as good)
            __builtin_amdgcn_sched_group_barrier(0x100, 2 * (NA + 4), 0);  // LDS reads
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);             // products
#pragma unroll
            for (int i = 1; i < 2 * OPS; ++i) {
              __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
              __builtin_amdgcn_sched_group_barrier(0x002, 11, 0);          // maxima
            }
          }
        }
      }

      // ---- rescore the best half-tile of each block, certify, fall back
#pragma unroll
      for (int o = 0; o < OPS; ++o) {
        float y[K];  // the block's coordinates, in both lanes of its column
        if constexpr (K <= 16) {
#pragma unroll
          for (int i = 0; i < K; ++i) {
            float a = yf[(o0 + o) / 2 * K + i], b = a;
            swap32(a, b);
            y[i] = (o & 1) ? b : a;
          }
        } else {
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            float a = yf[i], b = a;
            swap32(a, b);
            y[i] = a;
            y[16 + i] = b;
          }
        }
        float yy = 0.0f;
#pragma unroll
        for (int i = 0; i < K; ++i) yy = fmaf(y[i], y[i], yy);
        const float yn = sqrtf(yy) * ((1.0f + 0x1p-16f) / kY);
        const int tb = min((int)(__float_as_uint(b1[o]) & ~kmask_s), (N - 1) >> 5);
        const int jb = 32 * tb + 4 * h;  // rows jb + 8 (r / 4) + r % 4
        float s1 = -INFINITY, s2 = -INFINITY;
        int j1 = 0;
#pragma unroll CH ? 1 : 4
        for (int r4 = 0; r4 < 4; ++r4) {
          f4 sv;
          if constexpr (!CH) {
            sv = *reinterpret_cast<const f4*>(nrms + nrm_at(jb) + 32 * r4);
#pragma unroll
            for (int p = 0; p < K / E8; ++p)
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const h8 c = load_a<K>(rows + row_at<K>(jb) + (8 * r4 + e) * ROWB + 16 * p);
#pragma unroll
                for (int i = 0; i < E8; ++i) sv[e] = fmaf((float)c[i], y[E8 * p + i], sv[e]);
              }
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int j = jb + 8 * r4 + e;
              float dot = 0.0f, n2 = 0.0f;
              if (j < N) {
#pragma unroll
                for (int i = 0; i < K; i += 4) {
                  f4 c;
                  __builtin_memcpy(&c, C + (size_t)j * K + i, 16);
#pragma unroll
                  for (int u = 0; u < 4; ++u) {
                    n2 = fmaf(c[u], c[u], n2);
                    dot = fmaf(c[u], y[i + u], dot);
                  }
                }
              }
              sv[e] = j < N ? fmaf(dot, kC, -0.5f * kS * n2) : -3e38f;
            }
          }
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const bool up = sv[e] > s1;
            s2 = __builtin_amdgcn_fmed3f(s1, s2, sv[e]);
            j1 = up ? 8 * r4 + e : j1;
            s1 = fmaxf(s1, sv[e]);
          }
        }
        int jj = jb + j1;
        {  // the column's other half-tile
          const float os1 = other_half(s1), os2 = other_half(s2), ob2 = other_half(b2[o]);
          const int oj = __float_as_int(other_half(__int_as_float(jj)));
          s2 = fmaxf(fmaxf(s2, os2), fminf(s1, os1));
          jj = os1 > s1 ? oj : jj;
          s1 = fmaxf(s1, os1);
          b2[o] = fmaxf(b2[o], ob2);
        }
        const float er = fmaf(er1, yn, er0), es = fmaf(es1, yn, es0);
        const bool cert = !bad && s1 - s2 > 2.0f * er &&
                          s1 - b2[o] > er + es + epack * fabsf(b2[o]);
        const int m = K <= 16 ? 4 * (q0 + (o0 + o) / 2) + 2 * (o & 1) + (c32 >> 4) : (c32 >> 4);
        uint64_t pend = __ballot(!cert && h == 0 && live && nu > 0.0 && v0 + v16 < n_vec);
        while (pend) {
          const int cl = __builtin_ctzll(pend);
          pend &= pend - 1;
          const int64_t vv = v0 + (cl & 15);
          const int mm = __builtin_amdgcn_readlane(m, cl);
          const int fj = scan64<IN, D, K>(x + vv * stride, R, C, N, mm, shfl64(inv, cl & 15));
          if (c32 == cl) jj = fj;
        }
        if (h == 0) stage[wb][v16][m] = (uint16_t)jj;
      }
    }

    // ---- pack: lane v < 16 writes the bit stream of vector v (without SP this
    //      wavefront's own LDS writes precede its reads)
    if (SP) __syncthreads();
    if (lane < 16 && q0 == 0 && live && v0 + lane < n_vec)
      pack_row<NB>(stage[wb][lane], !(nu > 0.0), W, payload + (v0 + lane) * (int64_t)P);
    if (SP) __syncthreads();
  }
}

// k = 1 and 2: the same norm and rotation, then each lane scans all N codewords
// (float32, broadcast from LDS as (c_0, c_1, -|c|^2 / 2)) for its own blocks;
// near ties as above.  One thread per vector with a float64 rotation on the
// vector units took 55 us for 4095 fp32 rows of k = 2, N = 16 (16 workgroups;
// here 7.5), 147 us for 147456 rows of k = 1, N = 16 (79) and 867 us for
// 147456 fp32 rows of k = 2, N = 256 (212).  Bound by the scan's k + 4 vector
// instructions per codeword and block, at small N by the rotation.
template <typename IN, int D, int K, bool SP>
__global__ __launch_bounds__(64 * (SP ? D / 16 : 4)) void scan_kernel(
    const IN* __restrict__ x, int64_t n_vec, int64_t stride, const float* __restrict__ R,
    const float* __restrict__ C, int N, int W, int P, uint8_t* __restrict__ payload,
    uint16_t* __restrict__ norms) {
  constexpr int WAVES = SP ? D / 16 : 4;
  constexpr int QN = SP ? WAVES : 1;      // wavefronts of a batch
  constexpr int NT = D / 16 / QN;         // row tiles of a wavefront
  constexpr int NB = D / K, BT = 4 / K;   // blocks of a vector, of a lane and tile
  extern __shared__ __align__(16) unsigned char smem[];
  f4* cw = reinterpret_cast<f4*>(smem);   // N codewords
  __shared__ float cmax[WAVES];
  __shared__ uint16_t stage[WAVES / QN][kVec][NB];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int q0 = wave % QN, wb = wave / QN, g = lane >> 4, v16 = lane & 15;
  float c2 = 0.0f;
  for (int j = tid; j < N; j += 64 * WAVES) {
    const float a = C[j * K], b = K == 2 ? C[j * K + K - 1] : 0.0f;
    const double n = (double)a * a + (double)b * b;
    cw[j] = f4{a, b, (float)(-0.5 * n), 0.0f};
    c2 = fmaxf(c2, n <= 3e38 ? (float)n : INFINITY);
  }
  c2 = wave_max(c2);
  if (lane == 0) cmax[wave] = c2;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < WAVES; ++i) c2 = fmaxf(c2, cmax[i]);
  // float32 scores of float32 y: (k + 4) roundings of |c| |y| + |c|^2 / 2, twice
  const float er = 2.0f * 1.25f * (K + 4) * 0x1p-24f;
  const float er1 = er * sqrtf(c2) * (1.0f + 0x1p-16f), er0 = er * 0.5f * c2;

  const int64_t nbatch = (n_vec + kVec - 1) / kVec;
  for (int64_t b0 = (int64_t)blockIdx.x * (WAVES / QN); b0 < nbatch;
       b0 += (int64_t)gridDim.x * (WAVES / QN)) {
    const int64_t bt = b0 + wb;
    if (!SP && bt >= nbatch) break;
    const int64_t v0 = bt * kVec;
    const int64_t vl = v0 + v16 < n_vec ? v0 + v16 : n_vec - 1;  // clamped (ragged batch)
    float yf[4 * NT];
    double inv;
    const double nu = rotate<IN, D, NT>(x + vl * stride, R, 1.0f, [&](int rt) {
      return 16 * (q0 + rt) + 4 * (v16 & 3) + (v16 >> 2);
    }, yf, inv);
    if (g == 0 && q0 == 0 && v0 + v16 < n_vec)
      norms[v0 + v16] = nu > 0.0 ? f64_to_f16_bits(nu) : (uint16_t)0;
    float s1[NT * BT], s2[NT * BT];
    int j1[NT * BT];
#pragma unroll
    for (int b = 0; b < NT * BT; ++b) { s1[b] = -INFINITY; s2[b] = -INFINITY; j1[b] = 0; }
#pragma unroll 2
    for (int j = 0; j < N; ++j) {
      const f4 c = cw[j];
#pragma unroll
      for (int b = 0; b < NT * BT; ++b) {
        float s = fmaf(c[0], yf[b * K], c[2]);
        if (K == 2) s = fmaf(c[1], yf[b * K + K - 1], s);
        j1[b] = s > s1[b] ? j : j1[b];
        s2[b] = __builtin_amdgcn_fmed3f(s1[b], s2[b], s);
        s1[b] = fmaxf(s1[b], s);
      }
    }
#pragma unroll
    for (int b = 0; b < NT * BT; ++b) {
      const float y0 = yf[b * K], y1 = K == 2 ? yf[b * K + K - 1] : 0.0f;
      const float yn = sqrtf(fmaf(y0, y0, y1 * y1)) * (1.0f + 0x1p-16f);
      const bool cert = s1[b] - s2[b] > fmaf(er1, yn, er0);
      const int m = (16 * (q0 + b / BT) + 4 * g) / K + b % BT;
      uint64_t pend = __ballot(!cert && nu > 0.0 && v0 + v16 < n_vec);
      while (pend) {
        const int cl = __builtin_ctzll(pend);
        pend &= pend - 1;
        const int fj = scan64<IN, D, K>(x + (v0 + (cl & 15)) * stride, R, C, N,
                                        __builtin_amdgcn_readlane(m, cl), shfl64(inv, cl));
        if (lane == cl) j1[b] = fj;
      }
      stage[wb][v16][m] = (uint16_t)j1[b];
    }
    if (SP) __syncthreads();
    if (lane < 16 && q0 == 0 && v0 + lane < n_vec)
      pack_row<NB>(stage[wb][lane], !(nu > 0.0), W, payload + (v0 + lane) * (int64_t)P);
    if (SP) __syncthreads();
  }
}

constexpr size_t kLds = 160 * 1024 - 8192;  // dynamic, beside the static arrays
// Rows that leave at most this many wavefronts per SIMD when a batch is shared:
// (d, k, N) = (64, 4, 256), 16384 rows 18.4 us shared, 19.5 not, 32768 rows
// 27.3 / 24.4; (128, 4, 4096) 8192 rows 106 / 214, 32768 rows 330 / 228.
constexpr int kSplitWaves = 4;
constexpr int kScanN = 2048;  // k <= 2: codewords of 16 bytes in 32 KB of LDS

template <typename IN, int D, int K, int WAVES, bool CH, bool SP>
static int launch_w(const void* x, int64_t n_vec, int64_t stride, const Shape& s, const float* R,
                    const float* C, uint8_t* payload, uint16_t* norms, int nc, int wgs,
                    hipStream_t st) {
  const size_t lds = rows_bytes<K>(nc) + nrms_bytes(nc);
  auto kern = encode_kernel<IN, D, K, WAVES, CH, SP>;
  if (lds > 65536) {  // above the default dynamic LDS limit
    const hipError_t e = hipFuncSetAttribute((const void*)kern,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return (int)e;
  }
  constexpr int PER = WAVES / (SP ? quads(D, K) : 1);  // batches of a workgroup
  const int64_t nbatch = (n_vec + kVec - 1) / kVec;
  const int64_t want = (nbatch + PER - 1) / PER;
  const int grid = (int)(want < wgs ? want : wgs);
  const uint32_t kmask = s.N <= 4096 ? ~127u : ~511u;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * WAVES), lds, st, static_cast<const IN*>(x), n_vec,
                     stride, R, C, s.N, nc, s.w, s.P, kmask, payload, norms);
  return (int)hipGetLastError();
}

template <typename IN, int D, int K>
static int launch_k(const void* x, int64_t n_vec, int64_t stride, const Shape& s, const float* R,
                    const float* C, uint8_t* payload, uint16_t* norms, int n_cu, hipStream_t st) {
  const int nc = (s.N + 63) & ~63;  // whole pairs of tiles
  const size_t lds = rows_bytes<K>(nc) + nrms_bytes(nc);
  constexpr int Q = quads(D, K);
  if constexpr (Q > 1) {
    if (lds <= kLds && n_vec * Q <= (int64_t)kSplitWaves * kVec * 4 * n_cu)
      return launch_w<IN, D, K, (Q < 4 ? 4 : Q), false, true>(x, n_vec, stride, s, R, C, payload, norms,
                                                             nc, 1 << 30, st);
  }
  if (lds <= 40 * 1024)  // small codebooks: 4-wavefront workgroups, several per compute unit
    return launch_w<IN, D, K, 4, false, false>(x, n_vec, stride, s, R, C, payload, norms, nc,
                                               3 * n_cu, st);
  if (lds <= kLds)
    return launch_w<IN, D, K, 8, false, false>(x, n_vec, stride, s, R, C, payload, norms, nc, n_cu, st);
  return launch_w<IN, D, K, 8, true, false>(x, n_vec, stride, s, R, C, payload, norms, 65536 / (2 * K),
                                            n_cu, st);
}

template <typename IN, int D, int K, bool SP>
static int launch_scan(const void* x, int64_t n_vec, int64_t stride, const Shape& s, const float* R,
                       const float* C, uint8_t* payload, uint16_t* norms, int n_cu,
                       hipStream_t st) {
  const int64_t nbatch = (n_vec + kVec - 1) / kVec, want = SP ? nbatch : (nbatch + 3) / 4;
  const int grid = (int)(SP || want < 4 * n_cu ? want : 4 * n_cu);
  hipLaunchKernelGGL((scan_kernel<IN, D, K, SP>), dim3(grid), dim3(64 * (SP ? D / 16 : 4)),
                     (size_t)s.N * 16, st, static_cast<const IN*>(x), n_vec, stride, R, C, s.N, s.w,
                     s.P, payload, norms);
  return (int)hipGetLastError();
}

template <typename IN, int D, int K>
static int launch_s(const void* x, int64_t n_vec, int64_t stride, const Shape& s, const float* R,
                    const float* C, uint8_t* payload, uint16_t* norms, int n_cu, hipStream_t st) {
  if (n_vec * (D / 16) <= (int64_t)kSplitWaves * kVec * 4 * n_cu)
    return launch_scan<IN, D, K, true>(x, n_vec, stride, s, R, C, payload, norms, n_cu, st);
  return launch_scan<IN, D, K, false>(x, n_vec, stride, s, R, C, payload, norms, n_cu, st);
}

template <typename IN>
static int launch_t(const void* x, int64_t n_vec, int64_t stride, const Shape& s, const float* R,
                    const float* C, uint8_t* payload, uint16_t* norms, int n_cu, hipStream_t st) {
#define FIBQ_GEN_CASE(DD, KK)   \
  if (s.d == DD && s.k == KK) \
    return launch_k<IN, DD, KK>(x, n_vec, stride, s, R, C, payload, norms, n_cu, st);
  FIBQ_GEN_CASE(64, 4) FIBQ_GEN_CASE(64, 8) FIBQ_GEN_CASE(64, 16) FIBQ_GEN_CASE(64, 32)
  FIBQ_GEN_CASE(128, 4) FIBQ_GEN_CASE(128, 8) FIBQ_GEN_CASE(128, 16)
#undef FIBQ_GEN_CASE
#define FIBQ_SCAN_CASE(DD, KK)  \
  if (s.d == DD && s.k == KK) \
    return launch_s<IN, DD, KK>(x, n_vec, stride, s, R, C, payload, norms, n_cu, st);
  FIBQ_SCAN_CASE(64, 1) FIBQ_SCAN_CASE(64, 2) FIBQ_SCAN_CASE(128, 1) FIBQ_SCAN_CASE(128, 2)
#undef FIBQ_SCAN_CASE
  return (int)hipErrorInvalidValue;
}

}  // namespace gen

bool encode_gen_applies(const Shape& s) {
  if (s.k <= 2) return (s.d == 64 || s.d == 128) && s.N <= gen::kScanN;
  return ((s.d == 64 || s.d == 128) && (s.k == 4 || s.k == 8 || s.k == 16)) ||
         (s.d == 64 && s.k == 32);
}

int launch_encode_gen(const void* x, int dtype, int64_t n_vec, int64_t stride, const Shape& s,
                      const float* R, const float* C, uint8_t* payload, uint16_t* norms,
                      void* stream, int n_cu) {
  hipStream_t st = static_cast<hipStream_t>(stream);
  switch (dtype) {
    case FIBQ_F32:
      return gen::launch_t<float>(x, n_vec, stride, s, R, C, payload, norms, n_cu, st);
    case FIBQ_F16:
      return gen::launch_t<f16_t>(x, n_vec, stride, s, R, C, payload, norms, n_cu, st);
    default:
      return gen::launch_t<bf16_t>(x, n_vec, stride, s, R, C, payload, norms, n_cu, st);
  }
}

}  // namespace dev
}  // namespace fibq
