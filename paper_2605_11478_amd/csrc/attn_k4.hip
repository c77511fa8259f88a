// Fused dequantisation + single-query decode attention on the matrix cores
// (Eq. lattn over the decoded cache of Sec. 3.1, evaluated in rotated space)
// for d = 64 or 128, k a multiple of 4 (a codeword is k / 4 rows of 4 dims) or
// k = 2, G <= 8 query heads per KV head, and codebooks whose binary16 rows and
// residuals fit in LDS.
//
// Block dimension k = 2 with w = 4 or 6 bits (N = 16 or 64) runs through the
// same kernels: its payload, read as a stream of 2w-bit indices, is exactly
// the payload of a k = 4 code over the pair codebook whose row i + N j is
// (c_i, c_j) (index i of block 2p sits in the low w bits of pair p).  The main
// kernel stages that N^2-row table instead of the codebook.
//
// Per wavefront, 32 cached tokens per step (two 16-token tiles):
//   loads   the payload of a token is read as four contiguous quarters of
//           P / 4 bytes, one per lane of a 4-lane set, so a wavefront's loads
//           cover 16 whole payloads per instruction (no lane reads bytes it
//           does not use).  The MFMA K slots are assigned to dimensions to
//           match: in the score product, lane group g (lanes 16 g .. 16 g + 15)
//           owns the blocks of quarter g; in the value product, the lane with
//           lane % 4 = a supplies rows of quarter a;
//   scores  S[t][.] = K_hat[t][:] . [q~_hi | q~_lo]  (v_mfma_f32_16x16x32_f16,
//           A = two gathered 4-dim codeword rows per lane from an fp16 copy of
//           the codebook in LDS; the 16 columns are the heads' products with
//           the binary16 high and low parts of the rotated query, summed by
//           one DPP add; a codebook that is not binary16-exact adds its
//           residual rows' products);
//   softmax online, base 2 (q~ carries scale * log2 e and a power of two that
//           puts it in the upper binary16 range); the running maximum of a
//           head moves only when a token exceeds it;
//   values  acc[(part, h)][dims] += W[(part, h)][tokens] V_hat[tokens][dims]
//           (v_mfma_f32_16x16x32_f16; the weights p nu_V in two binary16
//           parts of 22 bits together, which fill the 16 rows; plus the residual rows when the
//           codebook is not binary16-exact), B from transposing LDS reads
//           (ds_read_b64_tr_b16: in each 16-lane row, lane 4 a + e receives
//           element e of the rows addressed by lanes a, a + 4, a + 8, a + 12).
// Units of 32 tokens over all groups laid end to end are split into equal
// contiguous ranges, one per wavefront.  Each workgroup stages the binary16
// codebook itself and, when it meets few groups, also the rotated query's
// operands (otherwise prep_kernel writes them to the workspace).  At the end
// the wavefronts whose ranges end in the same group combine their states
// (m, l, acc) in LDS, so a workgroup leaves one record per group; the merge
// kernel combines the records by log-sum-exp and applies Pi^T once per head.
// When every group is one workgroup's ("whole"), that workgroup does this
// itself and there is no second launch.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "attn_split.h"
#include "device_common.h"
#include "fibq.h"
#include "fibq_internal.h"

namespace fibq {
namespace dev {
namespace k4 {

constexpr int K = 4;
constexpr int kMaxG = 8;
constexpr int kWaves = 8;       // wavefronts per workgroup, split plans
constexpr int kWavesWhole = 16;  // one workgroup per group: as many as registers allow
constexpr int whole_waves(int D) { return D == 64 ? kWavesWhole : kWaves; }
constexpr int kMaxWgs = 512;     // split plans: two workgroups per compute unit
constexpr int kStep = 32;        // tokens per unit
constexpr int kHeadBlocks = 2048;  // merge: a block per head up to so many heads
constexpr float kCs = 4096.0f;   // scale of the codebook's binary16 rows
constexpr float kVs = 16384.0f;  // scale of the weights while all value norms are below 2

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef short s4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef uint32_t u4v __attribute__((ext_vector_type(4)));

struct Plan {
  Split sp;       // 32-token units over all groups, their wavefronts
  int upg;        // units per group
  int wgs, wpg;   // workgroups, wavefronts per workgroup
  int slots;      // groups that a workgroup's range can meet
  bool whole;     // workgroup b holds exactly group b
  bool pro;       // query operands built by the main kernel
  size_t off_bq, off_qs, off_rec, total;
};

static inline size_t al(size_t x) { return (x + 255) & ~(size_t)255; }
constexpr int rec_floats(int D) { return kMaxG * (D + 2); }
// groups whose query operands a workgroup builds: 8 KB of operands at most
constexpr int pro_groups(int D) { return 256 / D; }

// Records of a split plan: slot (workgroup, group met by it), then kWaves - 1
// per workgroup for the wavefronts that run past the end of a group that an
// earlier wavefront of the workgroup also meets.
__host__ __device__ inline int64_t rec_cross(int wgs, int slots, int64_t wg, int i) {
  return (int64_t)wgs * slots + wg * (kWaves - 1) + (i - 1);
}

static Plan make_plan(int64_t n_groups, int64_t T, int D, int max_wgs) {
  Plan p{};
  p.upg = (int)((T + kStep - 1) / kStep);
  if (p.upg < 1) p.upg = 1;
  const int64_t units = n_groups * p.upg;
  // One workgroup per group saves the merge launch (4 us) and the records; it
  // pays while all groups run at once and a wavefront has at most two units
  // (one at d = 128, whose workgroups have half the wavefronts).  k = 4,
  // N = 256, d = 64, whole / split: 144 groups of 1024 tokens 13.3 / 17.6 us,
  // 256 of 500 13.0 / 16.2, 512 of 250 14.5 / 17.4; but 32 of 1999
  // 19.7 / 14.9 and 512 of 1000 29.7 / 22.7.
  p.whole = n_groups <= max_wgs &&
            p.upg <= (D == 64 && n_groups <= kMaxWgs / 2 ? 2 * kWavesWhole : kWaves);
  if (p.whole) {
    p.wgs = n_groups > 0 ? (int)n_groups : 1;
    p.wpg = p.upg <= kWaves ? kWaves : whole_waves(D);
    p.slots = 1;
    p.pro = true;
  } else {
    const int64_t want = (units + kWaves - 1) / kWaves;
    p.wgs = (int)(want < max_wgs ? want : max_wgs);
    if (p.wgs < 1) p.wgs = 1;  // (no groups)
    p.wpg = kWaves;
    const int64_t per = (units + p.wgs - 1) / p.wgs;  // units of a workgroup, at most
    p.slots = (int)(per <= 1 ? 1 : (per - 2) / p.upg + 2);
    p.pro = p.slots <= pro_groups(D);
  }
  const uint32_t waves = (uint32_t)(p.wgs * p.wpg);
  p.sp = make_split(units, waves, p.upg);
  size_t off = 0;
  p.off_bq = off;
  if (!p.pro) off = al(off + (size_t)n_groups * (D / 32) * 64 * 8 * 2);
  p.off_qs = off;
  if (!p.pro) off = al(off + (size_t)n_groups * 4);
  p.off_rec = off;
  if (!p.whole) off = al(off + (size_t)p.wgs * (p.slots + kWaves - 1) * rec_floats(D) * 4);
  p.total = off;
  return p;
}

// maximum over the wavefront of v >= 0, in registers
__device__ __forceinline__ float wave_max_dpp(float v) {
  float x = v;
#define FIBQ_ROR(n) x = fmaxf(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x120 + n, 0xf, 0xf, false)));
  FIBQ_ROR(8) FIBQ_ROR(4) FIBQ_ROR(2) FIBQ_ROR(1)
#undef FIBQ_ROR
  const int i = __float_as_int(x);
  return fmaxf(fmaxf(__int_as_float(__builtin_amdgcn_readlane(i, 0)), __int_as_float(__builtin_amdgcn_readlane(i, 16))),
               fmaxf(__int_as_float(__builtin_amdgcn_readlane(i, 32)), __int_as_float(__builtin_amdgcn_readlane(i, 48))));
}

// ---------------------------------------------------------------- query ----
// All threads of the block build the operands of groups g0 .. g0 + ng - 1:
// q~ = Pi q * scale * log2(e) divided by the power of two that takes the
// group's largest entry to [2^13, 2^14) (so that the low parts are normal
// numbers), split into binary16 hi + lo in the B-operand order of the score
// MFMA.  The rotation runs on v_mfma_f32_16x16x4_f32 (float32
// products and sums): a wavefront takes 16 rows of Pi and the 16 heads of two
// groups; K slot kk of lane group gq is column (D / 4) gq + kk, so a lane
// reads contiguous pieces of its row and of its head.
// qt: ng * kMaxG * D floats of LDS; bq, qsc: the destination (LDS or workspace).
template <typename IN, int PC>
__device__ __forceinline__ void load_q(const void* q, int64_t at, f4 (&v)[PC]) {
#pragma unroll
  for (int p = 0; p < PC; ++p) {
    IN w[4];
    __builtin_memcpy(w, static_cast<const IN*>(q) + at + 4 * p, sizeof(w));
    v[p] = f4{to_float(w[0]), to_float(w[1]), to_float(w[2]), to_float(w[3])};
  }
}
template <int D>
__device__ __forceinline__ void build_queries(const void* __restrict__ q, int q_dtype, int G,
                                              int64_t g0, int ng, const float* __restrict__ R,
                                              float qscale, float* qt, _Float16* bq, float* qsc) {
  constexpr int NB = D / K, Q = NB / 4, KQ = D / 4;
  const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63;
  const int n = lane & 15, gq = lane >> 4;
  const int items = (D / 16) * ((ng + 1) / 2);
  for (int it = tid >> 6; it < items; it += nt >> 6) {
    const int rt = it % (D / 16), gi = 2 * (it / (D / 16)) + (n >> 3), h = n & 7;
    const bool live = gi < ng && h < G;
    const int64_t at = ((g0 + gi) * G + h) * D + KQ * gq;
    const float* row = R + (16 * rt + n) * D + KQ * gq;
    f4 a[KQ / 4], b[KQ / 4] = {};  // (every load is issued before the first product)
#pragma unroll
    for (int p = 0; p < KQ / 4; ++p) __builtin_memcpy(&a[p], row + 4 * p, 16);
    if (live) {
      if (q_dtype == FIBQ_F32) load_q<float>(q, at, b);
      else if (q_dtype == FIBQ_F16) load_q<f16_t>(q, at, b);
      else load_q<bf16_t>(q, at, b);
    }
    f4 acc = {0, 0, 0, 0};
#pragma unroll
    for (int p = 0; p < KQ / 4; ++p)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[p][e], b[p][e], acc, 0, 0, 0);
    if (live) {  // lane: column n, rows 4 gq + e
#pragma unroll
      for (int e = 0; e < 4; ++e) qt[(gi * kMaxG + h) * D + 16 * rt + 4 * gq + e] = acc[e] * qscale;
    }
  }
  __syncthreads();
  // B operand of K-step kap: lane l holds B[k = 8 (l / 16) + e][n = l % 16];
  // the K slots of lane group gq are dims 4 (gq Q + 2 kap + e / 4) + e % 4;
  // column n < 8 is the high part of head n, n >= 8 the low part of head n - 8
  for (int gi = 0; gi < ng; ++gi) {
    const float* qg = qt + gi * kMaxG * D;
    float top = 0.0f;  // (every wavefront for itself)
#pragma unroll
    for (int e = 0; e < kMaxG * D; e += 256) {
      if (e + 4 * lane < G * D) {
        const f4 v = *reinterpret_cast<const f4*>(qg + e + 4 * lane);
        top = fmaxf(fmaxf(top, fmaxf(fabsf(v[0]), fabsf(v[1]))), fmaxf(fabsf(v[2]), fabsf(v[3])));
      }
    }
    top = wave_max_dpp(top);
    float sc = 1.0f, inv = 1.0f;
    if (top > 0.0f && top < INFINITY) {
      int e2 = 0;
      frexpf(top, &e2);
      e2 = max(e2 - 14, -100);
      sc = ldexpf(1.0f, e2);
      inv = ldexpf(1.0f, -e2);
    }
    if (tid == 0) qsc[gi] = sc;
    for (int x = tid; x < (D / 32) * 512; x += nt) {
      const int kap = x / 512, l = (x / 8) % 64, e = x % 8, c = l % 16, h = c & 7;
      const int dim = 4 * ((l / 16) * Q + 2 * kap + e / 4) + (e % 4);
      _Float16 o = (_Float16)0.0f;
      if (h < G) {
        const float v = qg[h * D + dim] * inv;
        const _Float16 hi = (_Float16)v;
        o = (c < 8) ? hi : (_Float16)(v - (float)hi);
      }
      bq[gi * (D / 32) * 512 + x] = o;
    }
  }
}

// One block per group, for plans whose workgroups meet more than
// pro_groups(D) groups (caches of many short groups).
template <int D>
__global__ __launch_bounds__(256) void prep_kernel(const void* __restrict__ q, int q_dtype, int G,
                                                   const float* __restrict__ R, float qscale,
                                                   _Float16* __restrict__ bq,
                                                   float* __restrict__ qsc) {
  __shared__ float qt[kMaxG * D];
  __shared__ float sc;
  const int64_t g = blockIdx.x;
  build_queries<D>(q, q_dtype, G, g, 1, R, qscale, qt, bq + g * (D / 32) * 512, &sc);
  if (threadIdx.x == 0) qsc[g] = sc;
}

// ----------------------------------------------------------------- main ----
__device__ __forceinline__ h4 tr_read(const unsigned char* lds_byte_addr) {
  s4 r = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) s4*)(lds_byte_addr));
  return __builtin_bit_cast(h4, r);
}
__device__ __forceinline__ float dpp_ror8(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xf, 0xf, false));
}
__device__ __forceinline__ uint32_t dpp_ror8u(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xf, 0xf, false);
}
__device__ __forceinline__ float xmax(float v, int mask) {
  return fmaxf(v, __shfl_xor(v, mask, 64));
}
__device__ __forceinline__ float xsum(float v, int mask) { return v + __shfl_xor(v, mask, 64); }

// One lane's raw loads of a unit: a payload quarter of the token whose K rows
// it gathers in each tile, a quarter of the token whose V rows it addresses
// in each tile, and the binary16 norms of the four tokens of its softmax work.
template <int QW>
struct Unit {
  uint32_t kq[2][QW], vq[2][QW];  // [tile][dword of the quarter]
  uint32_t nk[2], nv[2];          // two binary16 norms per word
};

// LDS byte offset of the 4-dim row b of a quarter: index b / KB of the quarter
// (w-bit indices, little-endian), row b % KB of its codeword.
template <int QW, int W, int KB>
__device__ __forceinline__ uint32_t qrow(const uint32_t (&qq)[QW], int b, int w) {
  if constexpr (W == 8 && KB == 1) {
    return ((qq[b >> 2] >> (8 * (b & 3))) & 0xFFu) * 8u;
  } else if constexpr (W == 12 && KB == 1) {  // bits 12 b .. 12 b + 11 of the quarter
    const int bit = 12 * b, wd = bit >> 5, sh = bit & 31;
    uint32_t v = qq[wd] >> sh;
    if (sh > 20) v |= qq[wd + 1] << (32 - sh);
    return (v & 0xFFFu) * 8u;
  } else {  // the quarter starts at bit 0 of qq
    const int i = b / KB;
    uint32_t v;
    if constexpr (QW == 1) {
      v = qq[0] >> (i * w);
    } else {
      const uint64_t u = (uint64_t)qq[0] | ((uint64_t)qq[1] << 32);
      v = (uint32_t)(u >> (i * w));
    }
    return (v & ((1u << w) - 1u)) * (8u * KB) + 8u * (b % KB);
  }
}

// Codewords of KB 4-dim rows (k = 4 KB); W > 0: compile-time index width,
// W == 0: width `wr` at run time.
template <int D, int W, int KB>
__global__ __launch_bounds__(64 * whole_waves(D)) void main_kernel(
    const uint8_t* __restrict__ kp, const uint16_t* __restrict__ kn,
    const uint8_t* __restrict__ vp, const uint16_t* __restrict__ vn, int G, int T,
    int64_t T_stride, int N, int wr, int pair_n, Split sp, int slots, int whole, int pro,
    const void* __restrict__ q, int q_dtype, float qscale, const float* __restrict__ R,
    const float* __restrict__ C, const _Float16* __restrict__ bq, const float* __restrict__ qsc,
    float* __restrict__ rec, float* __restrict__ out, int lds_qry) {
  constexpr int NB = D / K, Q = NB / 4;      // 4-dim rows per quarter
  constexpr int NI = Q / KB;                 // indices per quarter
  constexpr int KS = D / 32;                 // score K-steps
  constexpr int VM = D / 16;                 // value MFMAs (16 dims each)
  constexpr int REC = rec_floats(D);
  constexpr bool kBits = KB > 1 || W == 0;   // quarters that need not be whole bytes
  constexpr int QW = kBits ? (NI * (W > 0 ? W : KB == 1 ? 16 : 12) + 31) / 32 : (Q * W / 8 + 3) / 4;
  const int w = W > 0 ? W : wr;
  const int P = (4 * NI * w + 7) / 8;        // payload bytes
  // otherwise they are whole dwords, except d = 64 with 12-bit indices
  // (6 bytes, read as three 16-bit halves)
  constexpr int QB = kBits ? 0 : NB * W / 32;
  static_assert(kBits || QB % 4 == 0 || QB == 6, "unsupported payload quarter");
  extern __shared__ __align__(16) unsigned char smem[];  // rows hi [N KB][4], lo [N KB][4]; states
  __shared__ float qss[4];                               // query divisors of this workgroup's groups
  __shared__ int lastg[kWavesWhole];                     // last group of each wavefront, relative
  __shared__ float cmax[kWavesWhole];                    // each wavefront's largest codebook entry,
  __shared__ int clo[kWavesWhole];                       // whether it met a residual
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nthr = blockDim.x;
  const int wpg = nthr >> 6;
  const int g16 = lane >> 4, c = lane & 15;
  const int nrow = N * KB;
  const int upg = sp.upg;
  const uint32_t wv = blockIdx.x * wpg + __builtin_amdgcn_readfirstlane(wave);
  const uint32_t u0 = first_unit(wv, sp), u1 = first_unit(wv + 1, sp);
  const uint32_t U0 = first_unit(blockIdx.x * wpg, sp);
  const int64_t g_wg = U0 / sp.upg;  // first group of the workgroup
  const bool some = u0 < u1;  // (a wavefront with an empty range goes on to the barriers)
  const int64_t g_first = u0 / sp.upg;
  const int step0 = (int)(u0 - (uint32_t)g_first * sp.upg);
  const bool norms_aligned = ((T_stride & 3) == 0) &&
                             ((reinterpret_cast<uintptr_t>(kn) | reinterpret_cast<uintptr_t>(vn)) & 7) == 0;
  const int mytile = c >> 3;                     // tile of this lane's softmax tokens
  const int sm_tok = 16 * mytile + 4 * g16;      // first of its four tokens (unit-relative)
  const int kq_tok = c, kq_q = g16;              // K loads: token c of each tile, quarter g16
  const int vq_tok = 4 * g16 + (c >> 2), vq_q = c & 3;  // V loads: quarter c % 4
  // kBits: a quarter's bits read as 4 QW unaligned bytes that stay inside the
  // row (P >= 4 QW), then shifted down
  const int kbit = kq_q * NI * w, vbit = vq_q * NI * w;
  const int kst = min(kbit >> 3, P - 4 * QW), vst = min(vbit >> 3, P - 4 * QW);
  const int ksh = kbit - 8 * kst, vsh = vbit - 8 * vst;

  // A unit inside its group is read at wave-uniform bases plus these per-lane
  // offsets; the last unit of a ragged group clamps every token into it.
  const uint32_t ko = kq_tok * P + (kBits ? kst : kq_q * QB), vo = vq_tok * P + (kBits ? vst : vq_q * QB);
  auto quarter = [&](const uint8_t* at, int sh, uint32_t (&d)[QW]) {
    if constexpr (kBits) {
      __builtin_memcpy(d, at, 4 * QW);
      if constexpr (QW == 1) {
        d[0] >>= sh;
      } else {
        const uint64_t u = ((uint64_t)d[0] | ((uint64_t)d[1] << 32)) >> sh;
        d[0] = (uint32_t)u;
        d[1] = (uint32_t)(u >> 32);
      }
    } else if constexpr (QB % 4 == 0) {
#pragma unroll
      for (int i = 0; i < QW; ++i) d[i] = reinterpret_cast<const uint32_t*>(at)[i];
    } else {
      const uint16_t* h = reinterpret_cast<const uint16_t*>(at);
      d[0] = (uint32_t)h[0] | ((uint32_t)h[1] << 16);
      d[1] = h[2];
    }
  };
  auto load = [&](int64_t grp, int step) -> Unit<QW> {
    Unit<QW> b;
    const int tb = step * kStep, tm = T - 1;
    const uint8_t* kpg = kp + grp * T_stride * (int64_t)P;
    const uint8_t* vpg = vp + grp * T_stride * (int64_t)P;
    const uint16_t* kng = kn + grp * T_stride;
    const uint16_t* vng = vn + grp * T_stride;
    if (tb + kStep <= T) {
      const uint8_t* kb = kpg + (int64_t)tb * P;
      const uint8_t* vb = vpg + (int64_t)tb * P;
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        quarter(kb + 16 * t * P + ko, ksh, b.kq[t]);
        quarter(vb + 16 * t * P + vo, vsh, b.vq[t]);
      }
      if (norms_aligned) {
        const uint2 k4v = *reinterpret_cast<const uint2*>(kng + tb + sm_tok);
        const uint2 v4v = *reinterpret_cast<const uint2*>(vng + tb + sm_tok);
        b.nk[0] = k4v.x; b.nk[1] = k4v.y; b.nv[0] = v4v.x; b.nv[1] = v4v.y;
        return b;
      }
    } else {
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int tk = min(tb + 16 * t + kq_tok, tm), tv = min(tb + 16 * t + vq_tok, tm);
        quarter(kpg + (int64_t)tk * P + (ko - kq_tok * P), ksh, b.kq[t]);
        quarter(vpg + (int64_t)tv * P + (vo - vq_tok * P), vsh, b.vq[t]);
      }
    }
    uint32_t kk[4], vv[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int t = min(tb + sm_tok + e, tm);
      kk[e] = kng[t];
      vv[e] = vng[t];
    }
    b.nk[0] = kk[0] | (kk[1] << 16); b.nk[1] = kk[2] | (kk[3] << 16);
    b.nv[0] = vv[0] | (vv[1] << 16); b.nv[1] = vv[2] | (vv[3] << 16);
    return b;
  };

  // the first unit's loads go out before the codebook and the query are built
  Unit<QW> cur{};
  if (some) cur = load(g_first, step0);
  // ---- binary16 rows of the codebook times cs (k = 2: of the pair codebook,
  //      whose row j holds codewords j % pair_n and j / pair_n) and their
  //      residuals.  Rows of unit vectors' blocks have entries up to 1; times
  //      2^12 an entry above 2^-14 keeps 22 bits or more (unscaled, the residual
  //      of one below 1/8 is a subnormal number, and a float32 codebook's
  //      results were up to 1.5 times as far from float64 as the general
  //      kernels').  Codebooks outside that range are staged once more, with
  //      the power of two that takes their largest entry to [2^13, 2^14).
  const unsigned char* cbhi = smem;
  const unsigned char* cblo = smem + (size_t)nrow * 8;
  _Float16* bqs = reinterpret_cast<_Float16*>(smem + lds_qry);  // [slots][KS * 512]
  bool has_lo = false;
  float cs = kCs, ci = 1.0f / kCs;
#pragma unroll 1
  for (bool again = false;; again = true) {
    bool lo_any = false;
    float top = 0.0f;
    for (int i = tid; i < nrow; i += nthr) {
      float cv[4];
      if (pair_n > 0) {
        __builtin_memcpy(cv, C + 2 * (i % pair_n), 8);
        __builtin_memcpy(cv + 2, C + 2 * (i / pair_n), 8);
      } else {
        __builtin_memcpy(cv, C + (size_t)i * 4, 16);
      }
      h4 hi, lo;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        hi[e] = (_Float16)(cv[e] * cs);
        lo[e] = (_Float16)fmaf(cv[e], cs, -(float)hi[e]);
        lo_any |= (float)lo[e] != 0.0f;
        top = fmaxf(top, fabsf(cv[e]));
      }
      reinterpret_cast<h4*>(smem)[i] = hi;
      reinterpret_cast<h4*>(smem)[nrow + i] = lo;
    }
    top = wave_max_dpp(top);
    lo_any = __any(lo_any);
    if (lane == 0) {
      cmax[wave] = top;
      clo[wave] = lo_any;
    }
    if (pro && !again) {
      float* qt = reinterpret_cast<float*>(bqs + slots * KS * 512);
      const uint32_t U1 = first_unit((blockIdx.x + 1) * wpg, sp);
      const int ng = (int)((U1 - 1) / sp.upg - g_wg) + 1;  // at most slots
      build_queries<D>(q, q_dtype, G, g_wg, ng, R, qscale, qt, bqs, qss);
    }
    __syncthreads();
    has_lo = __any(lane < wpg && clo[lane & (kWavesWhole - 1)] != 0);
    top = wave_max_dpp(lane < wpg ? cmax[lane & (kWavesWhole - 1)] : 0.0f);
    if (again || top == 0.0f || (top >= 0x1p-6f && top < 15.9f)) break;
    int e2 = 0;
    frexpf(top, &e2);
    e2 = top < INFINITY ? min(max(14 - e2, -100), 100) : 0;
    cs = ldexpf(1.0f, e2);
    ci = ldexpf(1.0f, -e2);
    __syncthreads();  // (the flags are written again)
  }
  h8 bqv[KS];
  f4 acc[VM];
  float m_run = -INFINITY, l_run = 0.0f, qsg = 1.0f;
  // Scale of the weights p nu_V: a binary16 part holds 11 bits only above
  // 2^-14, and value norms go down to 2^-24.  In every group it is 2^14 up to
  // the first unit with a norm of 2 or more, then 1.
  bool small = true, drop = false;  // drop: at the present unit
  int64_t cur_group = -1;

  auto flush = [&](auto* r) {
    // rows h and h + 8 (high parts of the weights, rest times 2^11) sit in
    // lanes l and l ^ 32
    const float avs = small ? ci / kVs : ci;  // undoes the scales
    float l = l_run;
    l = xsum(l, 8);
    l = xsum(l, 16);
    l = xsum(l, 32);
#pragma unroll
    for (int mu = 0; mu < VM; ++mu) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float a = fmaf(__shfl_xor(acc[mu][e], 32, 64), 0x1p-11f, acc[mu][e]) * avs;
        // row 4 g16 + e is head 4 g16 + e; column c is dim
        // 4 ((c / 4) (D / 16) + mu) + c % 4
        const int h = 4 * g16 + e;
        if (g16 < 2 && h < G) r[2 * kMaxG + h * D + 4 * ((c >> 2) * (D / 16) + mu) + (c & 3)] = a;
      }
    }
    if (lane < G) {
      r[lane] = m_run * qsg;  // true log2 units
      r[kMaxG + lane] = l;
    }
  };

  // compiled once per codebook kind (residual rows or not): the hot body
  // has no branch on it
  auto compute = [&](const Unit<QW>& b, int tb, auto lo_tag) {
    constexpr bool HL = decltype(lo_tag)::value;
    const bool full = tb + kStep <= T;
    // ---- scores: two tiles x KS K-steps
    f4 s[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      s[t] = f4{0, 0, 0, 0};
#pragma unroll
      for (int kap = 0; kap < KS; ++kap) {
        const uint32_t r0 = qrow<QW, W, KB>(b.kq[t], 2 * kap, w);
        const uint32_t r1 = qrow<QW, W, KB>(b.kq[t], 2 * kap + 1, w);
        const h4 a0 = *reinterpret_cast<const h4*>(cbhi + r0);
        const h4 a1 = *reinterpret_cast<const h4*>(cbhi + r1);
        const h8 av = h8{a0[0], a0[1], a0[2], a0[3], a1[0], a1[1], a1[2], a1[3]};
        s[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(av, bqv[kap], s[t], 0, 0, 0);
        if (HL) {
          const h4 d0 = *reinterpret_cast<const h4*>(cblo + r0);
          const h4 d1 = *reinterpret_cast<const h4*>(cblo + r1);
          const h8 dv = h8{d0[0], d0[1], d0[2], d0[3], d1[0], d1[1], d1[2], d1[3]};
          s[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(dv, bqv[kap], s[t], 0, 0, 0);
        }
      }
    }
    // ---- this lane's (tile, head) scores for its four tokens, relative to
    //      the running maximum: t = S nu_K - m
    const int ts = tb + sm_tok;
    float f4s[4], t4[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float own = mytile ? s[1][e] : s[0][e];
      const float oth = mytile ? s[0][e] : s[1][e];
      f4s[e] = own + dpp_ror8(oth);  // hi + lo parts of the head
      const h2 nk2 = __builtin_bit_cast(h2, b.nk[e >> 1]);
      t4[e] = fmaf(f4s[e], (float)nk2[e & 1], -m_run);
    }
    if (!full) {
#pragma unroll
      for (int e = 0; e < 4; ++e) t4[e] = (ts + e < T) ? t4[e] : -INFINITY;
    }
    const float tmx = fmaxf(fmaxf(t4[0], t4[1]), fmaxf(t4[2], t4[3]));
    // a token beats the running maximum, or (not a number) no finite score has
    // come yet and an infinite key norm scores -inf
    if (__any(!(tmx <= 0.0f)) || drop) {
      // the maximum first, then every score against it in one fma (a score
      // of 100 rounded by itself would move its weight by 4e-6)
      const bool first = m_run == -INFINITY;  // nothing accumulated yet for this group
      float mh = tmx;
      if (first) {
        mh = -INFINITY;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const h2 nk2 = __builtin_bit_cast(h2, b.nk[e >> 1]);
          if (full || ts + e < T) mh = fmaxf(mh, f4s[e] * (float)nk2[e & 1]);
        }
      }
      mh = xmax(mh, 8);
      mh = xmax(mh, 16);
      mh = xmax(mh, 32);
      const float m_new = first ? mh : m_run + fmaxf(mh, 0.0f);
      const float delta = first ? INFINITY : m_new - m_run;
      m_run = m_new;
      const float m_sub = m_run == -INFINITY ? 0.0f : m_run;  // (scores of -inf keep weight 0)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const h2 nk2 = __builtin_bit_cast(h2, b.nk[e >> 1]);
        const float t = fmaf(f4s[e], (float)nk2[e & 1], -m_sub);
        t4[e] = (full || ts + e < T) ? t : -INFINITY;
      }
      const float alpha = __builtin_amdgcn_exp2f(-delta * qsg);
      l_run *= alpha;
      const float beta = drop ? alpha * (1.0f / kVs) : alpha;
#pragma unroll
      for (int e = 0; e < 4; ++e) {  // accumulator row 4 g16 + e belongs to head (4 g16 + e) & 7
        const float ar = __shfl(beta, (4 * g16 + e) & 7, 64);
#pragma unroll
        for (int mu = 0; mu < VM; ++mu) acc[mu][e] *= ar;
      }
    }
    // ---- weights p nu_V (binary16) as the value MFMA's A operand
    float p[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      p[e] = __builtin_amdgcn_exp2f(t4[e] * qsg);  // exp2(-inf) = 0
      l_run += p[e];
    }
    // Row h of A holds the high binary16 part of head h's weights p nu_V, row
    // h + 8 the rest times 2^11 (so that it stays in the normal range): the
    // two halves of a 16-lane row trade a tile's parts.
    u4v au;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const h2 nv2 = __builtin_bit_cast(h2, b.nv[i]);
      const float w0 = p[2 * i] * (float)nv2[0], w1 = p[2 * i + 1] * (float)nv2[1];
      uint32_t uh = __builtin_bit_cast(uint32_t, h2{(_Float16)w0, (_Float16)w1});
      asm("" : "+v"(uh));  // the rest is taken from these bits (not from a conversion fused anew)
      const h2 wh = __builtin_bit_cast(h2, uh);
      const h2 wl = h2{(_Float16)((w0 - (float)wh[0]) * 2048.0f),
                       (_Float16)((w1 - (float)wh[1]) * 2048.0f)};
      const uint32_t ul = __builtin_bit_cast(uint32_t, wl);
      const uint32_t got = dpp_ror8u(mytile ? uh : ul);  // tile 1's high parts, tile 0's low parts
      au[i] = mytile ? got : uh;
      au[2 + i] = mytile ? ul : got;
    }
    const h8 aw = __builtin_bit_cast(h8, au);
    // ---- values: MFMA mu covers local block mu of every quarter
#pragma unroll
    for (int mu = 0; mu < VM; ++mu) {
      const uint32_t ra = qrow<QW, W, KB>(b.vq[0], mu, w);
      const uint32_t rb = qrow<QW, W, KB>(b.vq[1], mu, w);
      const h4 b0 = tr_read(cbhi + ra);
      const h4 b1 = tr_read(cbhi + rb);
      const h8 bv = h8{b0[0], b0[1], b0[2], b0[3], b1[0], b1[1], b1[2], b1[3]};
      acc[mu] = __builtin_amdgcn_mfma_f32_16x16x32_f16(aw, bv, acc[mu], 0, 0, 0);
      if (HL) {  // residual rows of a codebook that is not binary16-exact
        const h4 d0 = tr_read(cblo + ra);
        const h4 d1 = tr_read(cblo + rb);
        const h8 dv = h8{d0[0], d0[1], d0[2], d0[3], d1[0], d1[1], d1[2], d1[3]};
        acc[mu] = __builtin_amdgcn_mfma_f32_16x16x32_f16(aw, dv, acc[mu], 0, 0, 0);
      }
    }
  };

  // record of a group that this wavefront runs past the end of
  auto past = [&](int64_t grp) -> float* {
    const uint32_t s0 = max(U0, (uint32_t)grp * sp.upg);  // the workgroup's first unit of the group
    const int64_t at = u0 <= s0 ? (int64_t)blockIdx.x * slots + (grp - g_wg)
                                : rec_cross(gridDim.x, slots, blockIdx.x, wave);
    return rec + at * REC;
  };
  int64_t grp = g_first;
  if (some) {
    int step = step0;
    for (uint32_t it = u0; it < u1; ++it) {
      if (grp != cur_group) {
        if (cur_group >= 0) flush(past(cur_group));
        cur_group = grp;
        const _Float16* bqg = pro ? bqs + (grp - g_wg) * KS * 512 : bq + grp * KS * 512;
        qsg = (pro ? qss[grp - g_wg] : qsc[grp]) * ci;
#pragma unroll
        for (int kap = 0; kap < KS; ++kap) {
          bqv[kap] = *reinterpret_cast<const h8*>(bqg + kap * 512 + lane * 8);
        }
#pragma unroll
        for (int mu = 0; mu < VM; ++mu) acc[mu] = f4{0, 0, 0, 0};
        m_run = -INFINITY;
        l_run = 0.0f;
        small = true;
      }
      drop = false;
      if (small) {  // (uniform)
        drop = __any(((cur.nv[0] | cur.nv[1]) & 0x40004000u) != 0);  // an exponent of 1 or more
        small = !drop;
        if (small) {
#pragma unroll
          for (int i = 0; i < 2; ++i)  // (exact)
            cur.nv[i] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(h2, cur.nv[i]) * (_Float16)kVs);
        }
      }
      int64_t ngrp = grp;
      int nstep = step + 1;
      if (nstep == upg) {
        nstep = 0;
        ++ngrp;
      }
      Unit<QW> nxt = cur;
      if (it + 1 < u1) nxt = load(ngrp, nstep);  // prefetch the next unit
      if (has_lo) compute(cur, step * kStep, std::true_type{});
      else compute(cur, step * kStep, std::false_type{});
      cur = nxt;
      grp = ngrp;
      step = nstep;
    }
  }

  // ---- the states of the wavefronts that end in the same group are combined
  //      (float32, in LDS, over the codebook) into the workgroup's record
  const int nstr = nthr / D, rows = D / nstr;     // whole: stripes of Pi's rows, rows each
  __syncthreads();
  float* states = reinterpret_cast<float*>(smem);
  if (lane == 0) lastg[wave] = some ? (int)(cur_group - g_wg) : -1;
  if (some) flush(states + wave * REC);
  __syncthreads();
  float* ar = states + wpg * REC;                // whole: [kMaxG][D], then [stripes][kMaxG][D]
  for (int a = 0; a < wpg;) {                    // runs of wavefronts a .. b - 1 (uniform)
    const int ga = lastg[a];
    int b = a + 1;
    while (b < wpg && (lastg[b] == ga || lastg[b] < 0)) ++b;
    if (ga < 0) { a = b; continue; }             // (no state before the first range)
    float* r = rec + ((int64_t)blockIdx.x * slots + ga) * REC;
    for (int e = tid; e < G * D; e += nthr) {
      const int h = e / D;
      float M = -INFINITY, l = 0.0f, s = 0.0f;
      for (int x0 = a; x0 < b; x0 += 8) {        // eight states' values are read at once
        float mx[8], lx[8], sx[8];
#pragma unroll
        for (int x = 0; x < 8; ++x) {
          const bool ok = x0 + x < b && lastg[min(x0 + x, wpg - 1)] >= 0;
          const float* sp = states + min(x0 + x, wpg - 1) * REC;
          mx[x] = sp[h]; lx[x] = sp[kMaxG + h]; sx[x] = sp[2 * kMaxG + e];
          if (!ok) { mx[x] = -INFINITY; lx[x] = 0.0f; sx[x] = 0.0f; }
        }
        float Mn = M;
#pragma unroll
        for (int x = 0; x < 8; ++x) Mn = fmaxf(Mn, mx[x]);
        if (Mn == -INFINITY) continue;
        const float f0 = __builtin_amdgcn_exp2f(M - Mn);  // exp2(-inf) = 0
        l *= f0;
        s *= f0;
#pragma unroll
        for (int x = 0; x < 8; ++x) {
          const float f = __builtin_amdgcn_exp2f(mx[x] - Mn);
          l = fmaf(lx[x], f, l);
          s = fmaf(sx[x], f, s);
        }
        M = Mn;
      }
      if (whole) {
        ar[e] = (l > 0.0f) ? s / l : 0.0f;
      } else {
        r[2 * kMaxG + e] = s;
        if (e % D == 0) {
          r[h] = M;
          r[kMaxG + h] = l;
        }
      }
    }
    a = b;
  }
  if (!whole) return;
  constexpr int kRows = D * D / (64 * kWaves);  // (at most)
  float pi[kRows];
#pragma unroll
  for (int i = 0; i < kRows; ++i)
    pi[i] = i < rows ? R[((tid / D) * rows + i) * D + tid % D] : 0.0f;
  __syncthreads();
  // ---- whole: o = Pi^T (acc / l), the rows of Pi in stripes over the threads
  float* part = states;  // [stripes][G][D]: nthr G floats, no more than the states took
  for (int h = 0; h < G; ++h) {
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < kRows; ++i)
      if (i < rows) s = fmaf(pi[i], ar[h * D + (tid / D) * rows + i], s);
    part[((tid / D) * G + h) * D + tid % D] = s;
  }
  __syncthreads();
  for (int e = tid; e < G * D; e += nthr) {
    float s = 0.0f;
    for (int x = 0; x < nstr; ++x) s += part[x * G * D + e];
    out[(int64_t)blockIdx.x * G * D + e] = s;
  }
}

// ---------------------------------------------------------------- merge ----

// Block (group, HB heads): log-sum-exp over the group's records, then
// o = Pi^T (acc / l).  The records' places are listed in LDS first; S stripes
// of threads take every S-th record, each loading kRound records' values
// before using any, and their states are combined in LDS.  Few groups leave
// the chip idle with one block per group (8 groups of 131072 tokens, d = 128:
// 278 us with one block per group and one record per wavefront), so the heads
// of a group go to separate blocks unless the groups alone fill it.
template <int D, int HB>
__global__ __launch_bounds__(256) void merge_kernel(const float* __restrict__ rec, Split u,
                                                    int wgs, int slots, int G,
                                                    const float* __restrict__ R,
                                                    float* __restrict__ out) {
  constexpr int REC = rec_floats(D), HD = HB * D;
  constexpr int EPT = HD > 256 ? HD / 256 : 1;   // outputs per thread
  constexpr int S = HD > 256 ? 1 : 256 / HD;     // stripes over the records
  constexpr int kRound = 16 / EPT;
  constexpr int SI = 256 / D, RI = D / SI;       // stripes over Pi's rows, rows each
  __shared__ int list[kMaxWgs + 1];
  __shared__ float sp[3][S > 1 ? 256 : 1];
  __shared__ float ar[HD];
  __shared__ float part[SI][HD];
  const int64_t g = blockIdx.x;
  const int h0 = blockIdx.y * HB, tid = threadIdx.x;
  const int nh = min(HB, G - h0);
  float* og = out + (g * G + h0) * D;
  if (u.units == 0) {  // no cached tokens: the output is zero
    for (int e = tid; e < nh * D; e += 256) og[e] = 0.0f;
    return;
  }
  float pi[RI];
#pragma unroll
  for (int i = 0; i < RI; ++i) pi[i] = R[((tid / D) * RI + i) * D + tid % D];
  const uint32_t first = (uint32_t)g * u.upg, last = first + u.upg - 1;
  const int blo = wave_of(first, u) / kWaves, whi = wave_of(last, u);
  const int bhi = whi / kWaves, nrec = bhi - blo + 2;
  for (int i = tid; i < nrec; i += 256) {
    // the record that workgroup blo + i leaves for g; behind them that of the
    // wavefront that runs past g's end, if another one came before it
    const int wg = min(blo + i, bhi);
    const uint32_t U0 = first_unit(wg * kWaves, u);
    int64_t at = (int64_t)wg * slots + ((uint32_t)g - U0 / u.upg);
    if (i == nrec - 1) {
      const bool past = first_unit(whi + 1, u) > last + 1 && first_unit(whi, u) > max(U0, first);
      at = past ? rec_cross(wgs, slots, bhi, whi % kWaves) : -1;
    }
    list[i] = (int)at;
  }
  __syncthreads();
  const int st = S > 1 ? tid / HD : 0, lt = S > 1 ? tid % HD : tid;
  float M[EPT], L[EPT], a[EPT];
#pragma unroll
  for (int u = 0; u < EPT; ++u) { M[u] = -INFINITY; L[u] = 0.0f; a[u] = 0.0f; }
  for (int base = st; base < nrec; base += S * kRound) {
    float mk[kRound][EPT], lk[kRound][EPT], xk[kRound][EPT];
#pragma unroll
    for (int k = 0; k < kRound; ++k) {
      const int i = base + S * k;
      const int at = i < nrec ? list[i] : -1;
      const float* rr = rec + (int64_t)(at < 0 ? 0 : at) * REC;
#pragma unroll
      for (int u = 0; u < EPT; ++u) {
        const int e = lt + 256 * u, h = e / D;
        const bool ok = at >= 0 && h < nh;
        mk[k][u] = ok ? rr[h0 + h] : -INFINITY;
        lk[k][u] = ok ? rr[kMaxG + h0 + h] : 0.0f;
        xk[k][u] = ok ? rr[2 * kMaxG + h0 * D + e] : 0.0f;
      }
    }
#pragma unroll
    for (int u = 0; u < EPT; ++u) {
      float Mn = M[u];
#pragma unroll
      for (int k = 0; k < kRound; ++k) Mn = fmaxf(Mn, mk[k][u]);
      if (Mn == -INFINITY) continue;
      const float fo = __builtin_amdgcn_exp2f(M[u] - Mn);  // exp2(-inf) = 0
      L[u] *= fo;
      a[u] *= fo;
#pragma unroll
      for (int k = 0; k < kRound; ++k) {
        const float f = __builtin_amdgcn_exp2f(mk[k][u] - Mn);
        L[u] = fmaf(lk[k][u], f, L[u]);
        a[u] = fmaf(xk[k][u], f, a[u]);
      }
      M[u] = Mn;
    }
  }
  if constexpr (S == 1) {
#pragma unroll
    for (int u = 0; u < EPT; ++u) ar[lt + 256 * u] = (L[u] > 0.0f) ? a[u] / L[u] : 0.0f;
  } else {
    sp[0][tid] = M[0];
    sp[1][tid] = L[0];
    sp[2][tid] = a[0];
    __syncthreads();
    if (st == 0) {
      float Mn = -INFINITY;
#pragma unroll
      for (int x = 0; x < S; ++x) Mn = fmaxf(Mn, sp[0][x * HD + lt]);
      float Ls = 0.0f, As = 0.0f;
      if (Mn != -INFINITY) {
#pragma unroll
        for (int x = 0; x < S; ++x) {
          const float mx = sp[0][x * HD + lt];
          const float f = __builtin_amdgcn_exp2f(mx - Mn);
          Ls = fmaf(sp[1][x * HD + lt], f, Ls);
          As = fmaf(sp[2][x * HD + lt], f, As);
        }
      }
      ar[lt] = (Ls > 0.0f) ? As / Ls : 0.0f;
    }
  }
  __syncthreads();
#pragma unroll
  for (int h = 0; h < HB; ++h) {  // o = Pi^T a, Pi's rows in stripes over the threads
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < RI; ++i) s = fmaf(pi[i], ar[h * D + (tid / D) * RI + i], s);
    part[tid / D][h * D + tid % D] = s;
  }
  __syncthreads();
  for (int e = tid; e < nh * D; e += 256) {
    float s = 0.0f;
#pragma unroll
    for (int x = 0; x < SI; ++x) s += part[x][e];
    og[e] = s;
  }
}

}  // namespace k4

// the k = 4 shape a k = 2 code (w = 4 or 6) is read as: pairs of blocks with
// 2w-bit indices over the N^2-row pair codebook
static Shape k4_shape(const Shape& s) {
  if (s.k != 2) return s;
  return Shape{s.d, 4, s.N * s.N, 2 * s.w, s.P};
}

bool attn_k4_applies(int G, const Shape& s0) {
  if (G < 1 || G > k4::kMaxG) return false;
  if (s0.k == 2 && !(s0.w == 4 || s0.w == 6)) return false;
  const Shape s = k4_shape(s0);
  if (s.d != 64 && s.d != 128) return false;
  if (s.k == 4 && (s.w == 8 || s.w == 12)) return true;
  // index width at run time: the binary16 rows and residuals of the codebook
  // have to fit in 128 KB of LDS, and a payload quarter is read as 4 or 8
  // bytes that have to lie inside the row
  if ((int64_t)s.N * s.k > 32768 || s.w > 12) return false;
  const bool two = (s.d == 64 && s.k == 4) || (s.d == 128 && s.k == 8);
  const bool one = (s.d == 64 && (s.k == 8 || s.k == 16)) || (s.d == 128 && s.k == 16);
  return (two && s.P >= 8) || (one && s.P >= 4);
}

static k4::Plan k4_plan(int64_t n_groups, int64_t T, const Shape& s) {
  // (registers at d = 128, and codebooks above 64 KB, leave room for one
  // workgroup per compute unit: a second round would stage everything again)
  const bool one = s.d == 128 || (int64_t)s.N * s.k * 4 > 65536;
  int wgs = one ? k4::kMaxWgs / 2 : k4::kMaxWgs;
  k4::Plan p = k4::make_plan(n_groups, T, s.d, wgs);
  // fewer workgroups (and records) where that makes the problem fit the
  // static scratch: tens of thousands of short groups
  while (p.total > FIBQ_ATTN_SCRATCH_BYTES && wgs > 64)
    p = k4::make_plan(n_groups, T, s.d, wgs /= 2);
  return p;
}

size_t attn_k4_workspace_bytes(int64_t n_groups, int64_t T, const Shape& s0) {
  return k4_plan(n_groups, T, k4_shape(s0)).total;
}

// 32-bit token indices and unit numbers
bool attn_k4_fits(int64_t n_groups, int64_t T) {
  return T < (1LL << 30) && n_groups < (1LL << 31) &&
         n_groups * ((T + k4::kStep) / k4::kStep) < (1LL << 31);
}

namespace k4 {

template <int D, int W, int KB>
static int launch(const void* q, int q_dtype, const uint8_t* kp, const uint16_t* kn,
                  const uint8_t* vp, const uint16_t* vn, int64_t n_groups, int G, int64_t T,
                  int64_t T_stride, const Shape& s, int pair_n, const float* R, const float* C,
                  float scale, float* out, void* ws, hipStream_t st) {
  const Plan p = k4_plan(n_groups, T, s);
  unsigned char* b = static_cast<unsigned char*>(ws);
  _Float16* bq = reinterpret_cast<_Float16*>(b + p.off_bq);
  float* qsc = reinterpret_cast<float*>(b + p.off_qs);
  float* rec = reinterpret_cast<float*>(b + p.off_rec);
  const float qscale = scale * 1.4426950408889634f;  // base-2 softmax
  hipError_t e = hipSuccess;
  if (T > 0) {
    if (!p.pro) {
      hipLaunchKernelGGL(prep_kernel<D>, dim3((unsigned)n_groups), dim3(256), 0, st, q, q_dtype, G,
                         R, qscale, bq, qsc);
      if ((e = hipGetLastError()) != hipSuccess) return (int)e;
    }
    // codebook rows and residuals, then query operands and scratch; at the end
    // the wavefronts' states (and the whole plan's merged heads) over them
    const size_t qry = (size_t)s.N * s.k * 4;
    size_t lds = qry + (p.pro ? (size_t)p.slots * ((D / 32) * 1024 + kMaxG * D * 4) : 0);
    const size_t end = ((size_t)p.wpg * rec_floats(D) + (p.whole ? kMaxG * D : 0)) * 4;
    if (end > lds) lds = end;
    auto kern = main_kernel<D, W, KB>;
    if (lds > 65536) {  // above the default dynamic LDS limit
      e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)lds);
      if (e != hipSuccess) return (int)e;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)p.wgs), dim3(64 * p.wpg), lds, st, kp, kn, vp, vn, G,
                       (int)T, T_stride, s.N, s.w, pair_n, p.sp, p.slots, (int)p.whole, (int)p.pro, q,
                       q_dtype, qscale, R, C, bq, qsc, rec, out, (int)qry);
    if ((e = hipGetLastError()) != hipSuccess) return (int)e;
    if (p.whole) return 0;
  }
  const Split sp = T > 0 ? p.sp : Split{};
  if (G == 1 || n_groups * G <= kHeadBlocks) {
    hipLaunchKernelGGL((merge_kernel<D, 1>), dim3((unsigned)n_groups, G), dim3(256), 0, st, rec,
                       sp, p.wgs, p.slots, G, R, out);
  } else {
    hipLaunchKernelGGL((merge_kernel<D, 4>), dim3((unsigned)n_groups, (G + 3) / 4), dim3(256), 0,
                       st, rec, sp, p.wgs, p.slots, G, R, out);
  }
  return (int)hipGetLastError();
}

}  // namespace k4

int launch_attn_k4(const void* q, int q_dtype, const uint8_t* kp, const uint16_t* kn,
                   const uint8_t* vp, const uint16_t* vn, int64_t n_groups, int G, int64_t T,
                   int64_t T_stride, const Shape& s0, const float* R, const float* C, float scale,
                   float* out, void* ws, hipStream_t st) {
  const Shape s = k4_shape(s0);
  const int pair_n = s0.k == 2 ? s0.N : 0;
#define FIBQ_K4_CASE(DD, WW, KK)                                                                  \
  if (s.d == DD && s.k == 4 * KK && (WW == 0 || s.w == WW))                                       \
    return k4::launch<DD, WW, KK>(q, q_dtype, kp, kn, vp, vn, n_groups, G, T, T_stride, s, pair_n, \
                                  R, C, scale, out, ws, st);
  FIBQ_K4_CASE(64, 8, 1) FIBQ_K4_CASE(64, 12, 1) FIBQ_K4_CASE(128, 8, 1) FIBQ_K4_CASE(128, 12, 1)
  FIBQ_K4_CASE(64, 6, 2) FIBQ_K4_CASE(64, 0, 1) FIBQ_K4_CASE(64, 0, 2) FIBQ_K4_CASE(64, 0, 4) FIBQ_K4_CASE(128, 0, 2)
  FIBQ_K4_CASE(128, 0, 4)
#undef FIBQ_K4_CASE
  return (int)hipErrorInvalidValue;
}

}  // namespace dev
}  // namespace fibq
