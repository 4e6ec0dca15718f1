// One-token attention over a key/value cache, with the cache held as INT8
// codes and per-row scales or as bf16 rows (Sec. 4 names the INT8 key/value
// cache among the further speed-ups; Sec. 2: four query heads share one
// key/value head of 256, grouped-query attention).
//
// The cache of one layer is a row-major array of t_max rows of 256: INT8
// codes (256 B a row) with one binary32 scale per row, or bf16 (512 B a row).
// A decode step appends the current token's key and value at row pos and
// attends rows t0 .. pos with every query head.  The work is split over the
// rows: each workgroup walks its range 128 rows at a time, its four waves each
// 32 of them with a running maximum and sum per head (the softmax is formed
// exactly as one pass would form it, up to binary32 rounding), and a second
// launch merges the workgroups' partial results.  The workgroup whose range
// holds row pos quantises (or copies) the new key and value, stores them in
// the cache and uses them from LDS, so no other workgroup reads the row being
// written.
#include <algorithm>

#include "device.h"
#include "kernels.h"

namespace w8a8 {

namespace {

constexpr int kHd = 256;       // head dimension
constexpr int kStep = 32;      // cached rows a wave takes at a time
constexpr int kPass = 4 * kStep;  // ... and a workgroup
constexpr int kMaxHeads = 8;

// Codes of one 256-wide row held 4 per lane by one wave: the per-token rule
// (s = max |x| / 127, codes rne(x / s) clamped to +-127, zero row -> s = 0).
__device__ __forceinline__ uint32_t quant_row4(const float (&v)[4], float* s_out) {
  float a = fmaxf(fmaxf(fabsf(v[0]), fabsf(v[1])), fmaxf(fabsf(v[2]), fabsf(v[3])));
  const float amax = wave_max(a);
  const float s = amax / 127.0f;
  uint32_t packed = 0;
  if (s != 0.0f) {
    const float inv = 1.0f / s;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      packed |= (uint32_t)(uint8_t)code_of(v[e], s, inv, true) << (8 * e);
  }
  *s_out = s;
  return packed;
}

__device__ __forceinline__ void load_bf16x4(const uint16_t* p, float (&v)[4]) {
  const uint2 raw = *reinterpret_cast<const uint2*>(p);
  v[0] = bf16_bits_to_float(raw.x & 0xffffu);
  v[1] = bf16_bits_to_float(raw.x >> 16);
  v[2] = bf16_bits_to_float(raw.y & 0xffffu);
  v[3] = bf16_bits_to_float(raw.y >> 16);
}

// INT8 code e of a word (exact in bf16)
__device__ __forceinline__ float byte_f(uint32_t w, int e) {
  return (float)(int8_t)(uint8_t)(w >> (8 * e));
}
// the bf16 pair of two binary32 values whose low 16 bits are zero
__device__ __forceinline__ int pair_hi(float lo, float hi) {
  return (int)__builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u);
}

}  // namespace

// One wave per row of 256 bf16 values (stride ld elements): INT8 codes
// (row-major, 256 a row) and the row's scale.
__global__ __launch_bounds__(256) void kv_quant_kernel(const uint16_t* __restrict__ src,
                                                       int64_t rows, int64_t ld,
                                                       int8_t* __restrict__ codes,
                                                       float* __restrict__ scales) {
  const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= rows) return;  // whole wave
  const int l = lane_id();
  float v[4];
  load_bf16x4(src + r * ld + 4 * l, v);
  float s;
  const uint32_t packed = quant_row4(v, &s);
  *reinterpret_cast<uint32_t*>(codes + r * kHd + 4 * l) = packed;
  if (l == 0) scales[r] = s;
}

// Partial results of one workgroup: per head the running maximum m and sum l
// of exp(score - m), and the unnormalised output o (256 values).
constexpr int kPartFloats = 2 * kMaxHeads + kMaxHeads * kHd;

// Both products run on the matrix cores: in vector instructions the products,
// the conversions and the LDS reads of the query outlasted the loads (32768 INT8
// rows, 4 heads: kernel 10.5 -> 8.9 us, call 16.1 -> 12.0 us; 131072 rows 30.0 ->
// 21.9 us; bf16 17.8 -> 13.6 and 39.9 -> 35.7 us; up to 4096 rows, where the
// launches bound it, unchanged).  Scores: a 16-row tile of keys is the first
// operand, the query heads are the columns of the second, both read straight
// from memory (any assignment of the 256 dimensions to the K positions serves,
// so a lane's 16-byte pieces are what is contiguous in a row; codes become bf16
// exactly).  A lane then holds head n % HN's scores of the rows 4 g .. + 3 of
// both tiles (n = lane % 16, g = lane / 16), which is the layout the first
// operand of the value product wants once K position (g, 4 t + i) stands for row
// 16 t + 4 g + i: no exchange between lanes.  The weights stay binary32: each is
// the sum of three bf16 values (8 significant bits apiece), in three row groups
// of the operand, and the three products are added at the end.  Values: lane n
// loads dimensions 16 n .. 16 n + 15 of its rows, one output column per byte (or
// half word).
//
// A wave keeps its own maximum and sum; nothing crosses waves before the end.
// The keys (values) of the next step are loaded as soon as the registers of this
// step's are free.  Two workgroups a CU; the bf16 cache, whose steps hold twice
// the bytes in registers, one.
template <bool I8, int NH>
__global__ __launch_bounds__(256, I8 ? 2 : 1) void attn_decode_kernel(AttnParams p) {
  constexpr int HN = NH > 4 ? 8 : 4;  // heads side by side in a row group
  constexpr int KI = I8 ? 4 : 8;      // 16-byte pieces of a lane's quarter of a row
  constexpr int VW = I8 ? 1 : 2;      // 16-byte pieces of a lane's 16 dimensions
  __shared__ __attribute__((aligned(16))) float ored[4][NH][kHd];  // the four waves' outputs, maxima and sums
  __shared__ float om[4][kMaxHeads], ol[4][kMaxHeads];
  __shared__ __attribute__((aligned(16))) float scl[4][64];  // INT8: key and value scales of a step
  __shared__ uint4 knew[kHd / 8], vnew[kHd / 8];             // the new row (codes or bf16 bits)
  __shared__ float knew_s, vnew_s;

  const int tid = threadIdx.x, w = tid >> 6, l = lane_id(), n = l & 15, g = l >> 4;
  const int64_t r_begin = p.t0 + (int64_t)blockIdx.x * p.rows_per_wg;
  const int64_t r_end = min(r_begin + p.rows_per_wg, p.pos + 1);  // exclusive
  const int64_t lim = min(r_end, p.pos);                          // rows below it are in the cache
  constexpr int ROWB = I8 ? kHd : 2 * kHd;                        // bytes of a cached row
  const int8_t* kbase = reinterpret_cast<const int8_t*>(p.k) + 16 * g;
  const int8_t* vbase = reinterpret_cast<const int8_t*>(p.v) + 16 * VW * n;

  uint4 kc[2][KI];      // key row 16 t + n, bytes 64 i + 16 g .. + 15
  uint4 vc[8][VW];      // value row 16 t + 4 g + i (at 4 t + i), dimensions 16 n .. + 15
  float srow = 0.0f;    // INT8: scale of key row l (l < 32), of value row l - 32
  // Rows from lim on are not read: the new row comes from LDS, rows past the end are 0.
  auto load_k = [&](int64_t r0) {
    const bool whole = r0 + kStep <= lim;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int64_t row = r0 + 16 * t + n;
      if (whole || row < lim) {
#pragma unroll
        for (int i = 0; i < KI; ++i)
          kc[t][i] = *reinterpret_cast<const uint4*>(kbase + row * ROWB + 64 * i);
      } else {
#pragma unroll
        for (int i = 0; i < KI; ++i) kc[t][i] = row == p.pos ? knew[4 * i + g] : make_uint4(0, 0, 0, 0);
      }
    }
    if constexpr (I8) {
      const int64_t row = r0 + (l & 31);
      if (whole || row < lim)
        srow = (l < 32 ? p.sk : p.sv)[row];
      else
        srow = row == p.pos ? (l < 32 ? knew_s : vnew_s) : 0.0f;
    }
  };
  auto load_v = [&](int64_t r0) {
    const bool whole = r0 + kStep <= lim;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int64_t row = r0 + 16 * (i >> 2) + 4 * g + (i & 3);
      if (whole || row < lim) {
#pragma unroll
        for (int c = 0; c < VW; ++c)
          vc[i][c] = *reinterpret_cast<const uint4*>(vbase + row * ROWB + 16 * c);
      } else {
#pragma unroll
        for (int c = 0; c < VW; ++c) vc[i][c] = row == p.pos ? vnew[VW * n + c] : make_uint4(0, 0, 0, 0);
      }
    }
  };

  const bool has_new = r_end == p.pos + 1;
  if (has_new) {  // whole workgroup; wave 0: the key, wave 1: the value
    if (w < 2) {
      const uint16_t* src = p.qkv + NH * kHd + w * kHd + 4 * l;
      if constexpr (I8) {
        float v[4], s;
        load_bf16x4(src, v);
        const uint32_t packed = quant_row4(v, &s);
        int8_t* dst = reinterpret_cast<int8_t*>(w == 0 ? p.k : p.v) + p.pos * kHd;
        *reinterpret_cast<uint32_t*>(dst + 4 * l) = packed;
        reinterpret_cast<uint32_t*>(w == 0 ? knew : vnew)[l] = packed;
        if (l == 0) {
          (w == 0 ? p.sk : p.sv)[p.pos] = s;
          if (w == 0) knew_s = s; else vnew_s = s;
        }
      } else {
        const uint2 raw = *reinterpret_cast<const uint2*>(src);
        uint16_t* dst = reinterpret_cast<uint16_t*>(w == 0 ? p.k : p.v) + p.pos * kHd;
        *reinterpret_cast<uint2*>(dst + 4 * l) = raw;
        reinterpret_cast<uint2*>(w == 0 ? knew : vnew)[l] = raw;
      }
    }
    __syncthreads();
  }
  int64_t r0 = r_begin + kStep * w;
  if (r0 < r_end) {
    load_k(r0);
    load_v(r0);
  }
  v4i q[8];  // head n % HN: the dimensions of key piece i, 8 a step
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const int d0 = I8 ? 64 * (c >> 1) + 16 * g + 8 * (c & 1) : 32 * c + 8 * g;
    q[c] = *reinterpret_cast<const v4i*>(p.qkv + min(n % HN, NH - 1) * kHd + d0);
  }

  float run_m = -INFINITY, run_l = 0.0f;
  v4f acc[16];  // rows 4 g .. + 3 of the weight operand's row groups, dimension 16 n + e
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = v4f{0.f, 0.f, 0.f, 0.f};

  for (; r0 < r_end; r0 += kPass) {
    // ---- scores
    v4f s[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      s[t] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        v4i kf;
        if constexpr (I8) {
          const uint4 u = kc[t][c >> 1];
          const uint32_t a = c & 1 ? u.z : u.x, b = c & 1 ? u.w : u.y;
          kf = v4i{pair_hi(byte_f(a, 0), byte_f(a, 1)), pair_hi(byte_f(a, 2), byte_f(a, 3)),
                   pair_hi(byte_f(b, 0), byte_f(b, 1)), pair_hi(byte_f(b, 2), byte_f(b, 3))};
        } else {
          kf = __builtin_bit_cast(v4i, kc[t][c]);
        }
        s[t] = mma_bf16(kf, q[c], s[t]);
      }
    }
    float ks[8], vs[8];
    if constexpr (I8) {
      scl[w][l] = srow;  // this wave's own part: no barrier between waves
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const float4 a = *reinterpret_cast<const float4*>(&scl[w][16 * t + 4 * g]);
        const float4 b = *reinterpret_cast<const float4*>(&scl[w][32 + 16 * t + 4 * g]);
        ks[4 * t] = a.x; ks[4 * t + 1] = a.y; ks[4 * t + 2] = a.z; ks[4 * t + 3] = a.w;
        vs[4 * t] = b.x; vs[4 * t + 1] = b.y; vs[4 * t + 2] = b.z; vs[4 * t + 3] = b.w;
      }
      __builtin_amdgcn_wave_barrier();
    }
    if (r0 + kPass < r_end) load_k(r0 + kPass);
    // ---- running softmax of this wave's rows
    float sc[8], mx = run_m;
    const int rows = (int)min(r_end - r0, (int64_t)kStep);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      sc[i] = s[i >> 2][i & 3];
      if constexpr (I8) sc[i] *= ks[i];
      sc[i] = 16 * (i >> 2) + 4 * g + (i & 3) < rows ? sc[i] * 0.0625f : -INFINITY;
      mx = fmaxf(mx, sc[i]);
    }
    mx = fmaxf(mx, lane_xor<16>(mx));
    mx = fmaxf(mx, lane_xor<32>(mx));
    const float ref = mx == -INFINITY ? 0.0f : mx;  // scores of -inf only: weights of 0
    const float corr = expf(run_m - ref);  // 0 on the first step
    float sum = 0.0f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      sc[i] = expf(sc[i] - ref);  // 0 for rows past the end
      sum += sc[i];
    }
    sum += lane_xor<16>(sum);
    sum += lane_xor<32>(sum);
    run_l = run_l * corr + sum;
    run_m = mx;
    // ---- the weights as three bf16 values
    v4i pa, pb;
#pragma unroll
    for (int i = 0; i < 8; i += 2) {
      float x0[2], x1[2];
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const float wt = I8 ? sc[i + k] * vs[i + k] : sc[i + k];
        const float hi = bf16_bits_to_float(float_to_bf16_bits(wt));
        const float r1 = wt - hi;
        const float mid = bf16_bits_to_float(float_to_bf16_bits(r1));
        const float lo = bf16_bits_to_float(float_to_bf16_bits(r1 - mid));
        if constexpr (HN == 4) {
          x0[k] = n < 4 ? hi : n < 8 ? mid : n < 12 ? lo : 0.0f;
        } else {
          x0[k] = n < 8 ? hi : mid;
          x1[k] = n < 8 ? lo : 0.0f;
        }
      }
      pa[i >> 1] = pair_hi(x0[0], x0[1]);
      if constexpr (HN == 8) pb[i >> 1] = pair_hi(x1[0], x1[1]);
    }
    // ---- weighted values
    v4f cr;  // correction of the head of accumulator row 4 g + r
#pragma unroll
    for (int r = 0; r < 4; ++r) cr[r] = __shfl(corr, (l & 48) + (HN == 8 ? 4 * (g & 1) : 0) + r);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      v4i vf;
#pragma unroll
      for (int i = 0; i < 8; i += 2) {
        if constexpr (I8) {
          const uint32_t a = (e >> 2) == 0 ? vc[i][0].x : (e >> 2) == 1 ? vc[i][0].y : (e >> 2) == 2 ? vc[i][0].z : vc[i][0].w;
          const uint32_t b = (e >> 2) == 0 ? vc[i + 1][0].x : (e >> 2) == 1 ? vc[i + 1][0].y
                             : (e >> 2) == 2 ? vc[i + 1][0].z : vc[i + 1][0].w;
          vf[i >> 1] = pair_hi(byte_f(a, e & 3), byte_f(b, e & 3));
        } else {
          const uint4 ua = vc[i][VW * e / 16], ub = vc[i + 1][VW * e / 16];
          const int wd = (e >> 1) & 3;
          const uint32_t a = wd == 0 ? ua.x : wd == 1 ? ua.y : wd == 2 ? ua.z : ua.w;
          const uint32_t b = wd == 0 ? ub.x : wd == 1 ? ub.y : wd == 2 ? ub.z : ub.w;
          vf[i >> 1] = (int)__builtin_amdgcn_perm(b, a, e & 1 ? 0x07060302u : 0x05040100u);
        }
      }
      acc[e] = mma_bf16(pa, vf, acc[e] * cr);
      if constexpr (HN == 8) acc[e] = mma_bf16(pb, vf, acc[e]);
    }
    if (r0 + kPass < r_end) load_v(r0 + kPass);
  }

  // ---- the row groups' sums: a head's rows sit HN apart.  Each exchange adds
  // the two halves and leaves each half of the lanes with half of the dimensions.
  auto add32 = [](float a, float b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
  };
  auto add16 = [](float a, float b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
  };
  float finite = 0.0f;  // NaN once a sum is infinite or NaN
  auto check = [&](const float4& o) {
    finite = __builtin_fmaf(o.x, 0.0f, finite);
    finite = __builtin_fmaf(o.y, 0.0f, finite);
    finite = __builtin_fmaf(o.z, 0.0f, finite);
    finite = __builtin_fmaf(o.w, 0.0f, finite);
  };
  float half[8][4];  // dimension 16 n + 8 (g / 2) + e
#pragma unroll
  for (int e = 0; e < 8; ++e)
#pragma unroll
    for (int r = 0; r < 4; ++r) half[e][r] = add32(acc[e][r], acc[e + 8][r]);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    if constexpr (HN == 4) {
      if (r < NH) {
        const float4 o = make_float4(add16(half[0][r], half[4][r]), add16(half[1][r], half[5][r]),
                                     add16(half[2][r], half[6][r]), add16(half[3][r], half[7][r]));
        *reinterpret_cast<float4*>(&ored[w][r][16 * n + 8 * (g >> 1) + 4 * (g & 1)]) = o;
        check(o);
      }
    } else {
      float* dst = &ored[w][4 * (g & 1) + r][16 * n + 8 * (g >> 1)];
      const float4 lo = make_float4(half[0][r], half[1][r], half[2][r], half[3][r]);
      const float4 hi = make_float4(half[4][r], half[5][r], half[6][r], half[7][r]);
      *reinterpret_cast<float4*>(dst) = lo;
      *reinterpret_cast<float4*>(dst + 4) = hi;
      check(lo);
      check(hi);
    }
  }
  if (l < NH) {  // lane h < HN holds head h
    om[w][l] = run_m;
    ol[w][l] = run_l;
  }
  // Where a value (or a weight) is infinite, the zeros and the signs of the three
  // parts make NaN of what one product would leave infinite: such a wave takes its
  // rows again, one by one, each weight whole.
  if (__builtin_expect(__any(!(finite == 0.0f)) != 0, 0)) {
    float m[NH], den[NH], o[NH][4];  // dimensions 4 l .. + 3
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      m[h] = -INFINITY;
      den[h] = 0.0f;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[h][e] = 0.0f;
    }
    for (r0 = r_begin + kStep * w; r0 < r_end; r0 += kPass)
      for (int64_t row = r0; row < min(r0 + kStep, r_end); ++row) {
        const bool cached = row < p.pos;
        float kf[4], vf[4], ks = 1.0f, vs = 1.0f;
        if constexpr (I8) {
          const uint32_t kw = cached ? reinterpret_cast<const uint32_t*>(p.k)[row * (kHd / 4) + l]
                                     : reinterpret_cast<const uint32_t*>(knew)[l];
          const uint32_t vw = cached ? reinterpret_cast<const uint32_t*>(p.v)[row * (kHd / 4) + l]
                                     : reinterpret_cast<const uint32_t*>(vnew)[l];
          ks = cached ? p.sk[row] : knew_s;
          vs = cached ? p.sv[row] : vnew_s;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            kf[e] = byte_f(kw, e);
            vf[e] = byte_f(vw, e);
          }
        } else {
          load_bf16x4(cached ? reinterpret_cast<const uint16_t*>(p.k) + row * kHd + 4 * l
                             : reinterpret_cast<const uint16_t*>(knew) + 4 * l, kf);
          load_bf16x4(cached ? reinterpret_cast<const uint16_t*>(p.v) + row * kHd + 4 * l
                             : reinterpret_cast<const uint16_t*>(vnew) + 4 * l, vf);
        }
#pragma unroll
        for (int h = 0; h < NH; ++h) {
          float qf[4], dot = 0.0f;
          load_bf16x4(p.qkv + h * kHd + 4 * l, qf);
#pragma unroll
          for (int e = 0; e < 4; ++e) dot = __builtin_fmaf(qf[e], kf[e], dot);
          const float sc = (wave_sum(dot) * ks) * 0.0625f;
          const float mx = fmaxf(m[h], sc), ref = mx == -INFINITY ? 0.0f : mx;
          const float corr = expf(m[h] - ref), wt = expf(sc - ref);
          m[h] = mx;
          den[h] = den[h] * corr + wt;
#pragma unroll
          for (int e = 0; e < 4; ++e) o[h][e] = __builtin_fmaf(wt * vs, vf[e], o[h][e] * corr);
        }
      }
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      *reinterpret_cast<float4*>(&ored[w][h][4 * l]) = make_float4(o[h][0], o[h][1], o[h][2], o[h][3]);
      if (l == 0) {
        om[w][h] = m[h];
        ol[w][h] = den[h];
      }
    }
  }
  __syncthreads();
  // ---- the four waves (one without rows has maximum -inf and sums of 0), then
  // the result or this workgroup's partial
#pragma unroll
  for (int h = 0; h < NH; ++h) {
    const float m = fmaxf(fmaxf(om[0][h], om[1][h]), fmaxf(om[2][h], om[3][h]));
    const float ref = m == -INFINITY ? 0.0f : m;  // no row of weight: sums of 0
    float od = 0.0f, den = 0.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float f = expf(om[i][h] - ref);
      od += ored[i][h][tid] * f;
      den += ol[i][h] * f;
    }
    if (p.n_wg == 1) {
      p.out[h * kHd + tid] = float_to_bf16_bits(od / den);
    } else {
      float* part = p.part + (int64_t)blockIdx.x * kPartFloats;
      part[2 * kMaxHeads + h * kHd + tid] = od;
      if (tid == 0) {
        part[h] = m;
        part[kMaxHeads + h] = den;
      }
    }
  }
}

// Merge of at most 32 * CPT partial results: eight workgroups a head, each over
// 32 output dimensions with 32 groups of threads, group j taking the chunks j,
// j + 32, ...  Every partial's maximum, sum and output value is loaded at once
// (one memory round trip: 256 partials of 4 heads 6.1 -> 4.0 us), then come the maximum over the chunks, each
// thread's factors exp(m_c - M), and the sums over the waves in wave order.
template <int CPT>
__global__ __launch_bounds__(1024) void attn_merge_kernel(AttnParams p) {
  __shared__ float wmax[16], wden[16];
  __shared__ float red[16][32];
  const int h = blockIdx.x >> 3, tid = threadIdx.x, dl = tid & 31, d = (blockIdx.x & 7) * 32 + dl;
  const int c0 = tid >> 5, g = tid >> 6, n = p.n_wg;
  float mc[CPT], lc[CPT], oc[CPT];
#pragma unroll
  for (int j = 0; j < CPT; ++j) {
    const int c = c0 + 32 * j;
    mc[j] = -INFINITY;
    lc[j] = 0.0f;
    oc[j] = 0.0f;
    if (c < n) {
      const float* part = p.part + (int64_t)c * kPartFloats;
      mc[j] = part[h];
      lc[j] = part[kMaxHeads + h];
      oc[j] = part[2 * kMaxHeads + h * kHd + d];
    }
  }
  float m = mc[0];
#pragma unroll
  for (int j = 1; j < CPT; ++j) m = fmaxf(m, mc[j]);
  m = fmaxf(m, lane_xor<32>(m));
  if ((tid & 63) == 0) wmax[g] = m;
  __syncthreads();
  m = wmax[0];
#pragma unroll
  for (int i = 1; i < 16; ++i) m = fmaxf(m, wmax[i]);
  float den = 0.0f, num = 0.0f;
#pragma unroll
  for (int j = 0; j < CPT; ++j) {
    const float f = expf(mc[j] - m);  // 0 past the last chunk
    den += lc[j] * f;
    num += oc[j] * f;
  }
  den += lane_xor<32>(den);
  num += lane_xor<32>(num);
  if ((tid & 63) == 0) wden[g] = den;
  if ((tid & 63) < 32) red[g][dl] = num;
  __syncthreads();
  if (tid < 32) {
    float t = 0.0f, dn = 0.0f;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      t += red[i][dl];
      dn += wden[i];
    }
    p.out[h * kHd + d] = float_to_bf16_bits(t / dn);
  }
}

hipError_t launch_kv_quant(const uint16_t* src, int64_t rows, int64_t ld, int8_t* codes,
                           float* scales, hipStream_t st) {
  if (rows <= 0) return hipSuccess;
  kv_quant_kernel<<<dim3((unsigned)((rows + 3) / 4)), 256, 0, st>>>(src, rows, ld, codes, scales);
  return hipGetLastError();
}

// Rows per workgroup: whole passes of 128, at most kAttnWgTarget workgroups
// (two per CU: more would only add partial results to merge).
void attn_plan(int64_t rows, int target, int* rows_per_wg, int* n_wg) {
  target = std::max(1, std::min(target, kAttnWgTarget));
  const int64_t passes = (rows + kPass - 1) / kPass;
  const int64_t per = (passes + target - 1) / target;  // passes per workgroup
  *rows_per_wg = (int)(per * kPass);
  *n_wg = (int)((passes + per - 1) / per);
}

size_t attn_ws_bytes(int64_t rows, int target) {
  int rpw = 0, n = 0;
  attn_plan(rows, target, &rpw, &n);
  return n > 1 ? (size_t)n * kPartFloats * sizeof(float) : 0;
}

// Enough for every row count up to t_max: a launch uses min(passes,
// kAttnWgTarget) workgroups or fewer, and more rows never mean fewer passes.
size_t attn_ws_bytes_max(int64_t t_max) {
  const int64_t passes = (t_max + kPass - 1) / kPass;
  const int64_t n = std::min<int64_t>(passes, kAttnWgTarget);
  return n > 1 ? (size_t)n * kPartFloats * sizeof(float) : 0;
}

template <bool I8>
static hipError_t attn_launch(const AttnParams& p, int nh, hipStream_t st) {
  const dim3 grid((unsigned)p.n_wg);
  switch (nh) {
    case 1: attn_decode_kernel<I8, 1><<<grid, 256, 0, st>>>(p); break;
    case 2: attn_decode_kernel<I8, 2><<<grid, 256, 0, st>>>(p); break;
    case 4: attn_decode_kernel<I8, 4><<<grid, 256, 0, st>>>(p); break;
    case 8: attn_decode_kernel<I8, 8><<<grid, 256, 0, st>>>(p); break;
    default: return hipErrorInvalidValue;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || p.n_wg == 1) return e;
  static_assert(kAttnWgTarget <= 512, "the merge loads every partial at once");
  const dim3 mg((unsigned)(8 * nh));
  if (p.n_wg <= 64)
    attn_merge_kernel<2><<<mg, 1024, 0, st>>>(p);
  else if (p.n_wg <= 256)
    attn_merge_kernel<8><<<mg, 1024, 0, st>>>(p);
  else
    attn_merge_kernel<16><<<mg, 1024, 0, st>>>(p);
  return hipGetLastError();
}

hipError_t launch_attn_decode(AttnParams p, int nh, bool i8, int target, hipStream_t st) {
  attn_plan(p.pos + 1 - p.t0, target, &p.rows_per_wg, &p.n_wg);
  return i8 ? attn_launch<true>(p, nh, st) : attn_launch<false>(p, nh, st);
}

}  // namespace w8a8
