// GEMM whose waves split K (gfx950): C[M x N] = A[M x K] B[N x K]^T for
// products with few output tiles.
//
// Every wave of a workgroup computes the whole (16 TM) x (16 TN) tile over its
// own fragment columns (wave w takes w, w + NW, ...), loading both operands
// from the packed fragment layout straight into registers; the waves' sums
// meet once, in LDS, after the K loop.  No operand passes through LDS and no
// barrier stands in the K loop, so the waves' loads and matrix instructions
// overlap freely, and a long K needs no split over workgroups: no partial sums
// in memory and no reduction launch.  (Where the consumer adds partial sums by
// itself, raw sums can be split over workgroups all the same.)
//
// What bounds it: the register-return path of a CU (64 B a cycle), at
// (TM + TN) KiB per fragment column against 16 TM TN / 4 matrix cycles, so the
// tile is as large as leaves one workgroup for every CU.
#include "device.h"
#include "kernels.h"

namespace w8a8 {

namespace {

template <int DT, int EPI, int TM, int TN, int NW, int PD>
__global__ __launch_bounds__(64 * NW, NW / 4) void gemm_kwave_kernel(GemmParams p) {
  constexpr bool GLU = EPI == EPI_GLU;
  constexpr bool BF16 = DT == DT_BF16;
  constexpr int KP = frags_per_mma<DT>();   // fragment columns a step consumes
  constexpr int TH = GLU ? TN / 2 : TN;     // column blocks of the output
  constexpr int STEP = KP * NW;             // fragment columns between a wave's steps
  typedef typename Acc<DT>::T AccT;
  extern __shared__ v4i lds[];

  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int m_tiles = (p.M + 16 * TM - 1) / (16 * TM);
  const int n_tiles = (p.rb_b + TH - 1) / TH;
  // XCD blockIdx % 8 takes a contiguous range of tiles; the walk goes through
  // bands of group_m tile rows, so a range is a compact block of both operands
  // (with K splits the ranges of every tile's first split come first, and so on)
  const int tiles = m_tiles * n_tiles, total = tiles * p.splits, per_xcd = (total + 7) / 8;
  const int item = (int)(blockIdx.x % 8) * per_xcd + (int)(blockIdx.x / 8);
  if (item >= total) return;  // whole workgroup, before any barrier
  const int z = item / tiles, tile = item % tiles;
  const int kb0 = z * p.kchunk, kbs = min(p.kchunk, p.kb_count - kb0);  // this split's columns
  const int band_tiles = p.group_m * n_tiles, band = tile / band_tiles, in_band = tile % band_tiles;
  const int gm = min(p.group_m, m_tiles - band * p.group_m);
  const int mt = band * p.group_m + in_band % gm, nt = in_band / gm;

  // operand streams: a scalar base per fragment row, one running lane offset
  const int8_t* pa[TM];
  const int8_t* pb[TN];
  unsigned arow[BF16 ? TM : 1];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    if (BF16 && !p.a_packed) {  // row-major: lane l reads row l % 16, columns (l / 16) * 8 .. + 7
      pa[i] = reinterpret_cast<const int8_t*>(reinterpret_cast<const uint16_t*>(p.A) +
                                              (int64_t)mt * TM * 16 * p.lda + kb0 * kFragK16);
      const int r = min((mt * TM + i) * 16 + (lane & 15), p.M - 1) - mt * TM * 16;
      arow[BF16 ? i : 0] = (unsigned)r * (unsigned)(p.lda * 2) + (lane >> 4) * 16;
    } else {
      arow[BF16 ? i : 0] = lane * 16;
      pa[i] = reinterpret_cast<const int8_t*>(p.A) +
              frag_offset(min(mt * TM + i, p.rb_a - 1), kb0, p.kb_count);
    }
  }
#pragma unroll
  for (int t = 0; t < TN; ++t) {
    const void* base = GLU && t >= TH ? p.B2 : p.B;
    pb[t] = reinterpret_cast<const int8_t*>(base) +
            frag_offset(min(nt * TH + (GLU && t >= TH ? t - TH : t), p.rb_b - 1), kb0, p.kb_count);
  }

  const unsigned a_step = BF16 && !p.a_packed ? kFragK16 * 2 : kFragBytes;

  // this wave's steps: fragment columns KP (wave + NW j) .. + KP - 1
  const int all = (kbs + KP - 1) / KP;
  const int n = all > wave ? (all - wave + NW - 1) / NW : 0;
  AccT acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int t = 0; t < TN; ++t) acc[i][t] = Acc<DT>::zero();
  struct Frags {
    v4i a[KP][TM], b[KP][TN];
  };
  Frags F[PD];
  // loads past the last step repeat it (a fixed number of loads, never used)
  int col = KP * wave;
  const int col_last = KP * (wave + NW * max(n - 1, 0));
  auto load = [&](Frags& f) {
#pragma unroll
    for (int k = 0; k < KP; ++k) {
      const unsigned off = (unsigned)(min(col, kbs - KP) + k) * kFragBytes + lane * 16;
#pragma unroll
      for (int t = 0; t < TN; ++t) f.b[k][t] = *reinterpret_cast<const v4i*>(pb[t] + off);
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const unsigned aoff =
            BF16 ? arow[BF16 ? i : 0] + (unsigned)min(col, kbs - 1) * a_step : off;
        f.a[k][i] = *reinterpret_cast<const v4i*>(pa[i] + aoff);
      }
    }
    col = min(col + STEP, col_last);
  };
  auto mma = [&](const Frags& f) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int t = 0; t < TN; ++t) {
        // operands swapped: lane l holds row l % 16, columns 4 (l / 16) .. + 3
        if constexpr (DT == DT_F8)
          acc[i][t] = Acc<DT>::mma2(f.b[0][t], f.b[1][t], f.a[0][i], f.a[1][i], acc[i][t]);
        else
          acc[i][t] = Acc<DT>::mma(f.b[0][t], f.a[0][i], acc[i][t]);
      }
  };
#pragma unroll
  for (int d = 0; d < PD - 1; ++d) load(F[d]);
  int j = 0;
  for (; j + PD <= n; j += PD) {
#pragma unroll
    for (int d = 0; d < PD; ++d) {
      load(F[(d + PD - 1) % PD]);
      mma(F[d]);
      // spread the loads between the matrix instructions
      constexpr int NL = KP * (TM + TN), NM = TM * TN;
#pragma unroll
      for (int q = 0; q < NL; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x20, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x8, NM / NL > 0 ? NM / NL : 1, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int d = 0; d < PD - 1; ++d)
    if (j + d < n) mma(F[d]);

  // ---- the waves' sums: wave w's block (i, t) at ((w TM + i) TN + t) KiB.
  // Then a wave finishes units of 16 rows x 32 columns: lane l row l % 16,
  // columns 8 (l / 16) .. + 7 (quarter-waves read 256 contiguous bytes).
  // Their scales are requested before the exchange.
  constexpr int PAIRS = (TH + 1) / 2, UNITS = TM * PAIRS, PER = (UNITS + NW - 1) / NW;
  constexpr bool SCALED = !BF16 && EPI != EPI_I32;
  float sa[PER], sb[PER][8], sb2[GLU ? PER : 1][8];
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int unit = wave + u * NW;
    if constexpr (SCALED) {
      const int row = min((mt * TM + unit / PAIRS) * 16 + (lane & 15), p.M - 1);
      const int c0 = (nt * TH + (unit % PAIRS) * 2) * 16 + (lane >> 4) * 8;
      sa[u] = p.s_a[row];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        sb[u][e] = p.s_b[min(c0 + e, p.N - 1)];
        if constexpr (GLU) sb2[u][e] = p.s_b2[min(c0 + e, p.N - 1)];
      }
    }
  }
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int t = 0; t < TN; ++t)
      lds[((wave * TM + i) * TN + t) * 64 + lane] = __builtin_bit_cast(v4i, acc[i][t]);
  __syncthreads();
  constexpr int ESZ = (EPI == EPI_GLU || EPI == EPI_BF16) ? 2 : 4;
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int unit = wave + u * NW;
    if (unit >= UNITS) break;
    const int i = unit / PAIRS, t = (unit % PAIRS) * 2 + (lane >> 5);
    const int row = (mt * TM + i) * 16 + (lane & 15);
    const int c0 = (nt * TH + (unit % PAIRS) * 2) * 16 + (lane >> 4) * 8;
    if (t >= TH || row >= p.M || c0 >= p.N) continue;
    auto sums = [&](int tt, AccT (&s)[2]) {  // K slices in wave order
      const v4i* src = lds + (i * TN + tt) * 64 + (lane & 15) + 32 * ((lane >> 4) & 1);
#pragma unroll
      for (int h = 0; h < 2; ++h) s[h] = __builtin_bit_cast(AccT, src[16 * h]);
#pragma unroll
      for (int w = 1; w < NW; ++w)
#pragma unroll
        for (int h = 0; h < 2; ++h) s[h] += __builtin_bit_cast(AccT, src[w * TM * TN * 64 + 16 * h]);
    };
    AccT s[2], s2[2];
    sums(t, s);
    if constexpr (GLU) sums(TH + t, s2);
    uint32_t o[2 * ESZ];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if constexpr (EPI == EPI_I32) {
        if constexpr (DT == DT_I8) o[e] = (uint32_t)s[e >> 2][e & 3];
        else o[e] = __float_as_uint((float)s[e >> 2][e & 3]);
      } else {
        float y = (float)s[e >> 2][e & 3];
        if constexpr (!BF16) y = (y * sa[u]) * sb[u][e];
        if constexpr (GLU) {
          float v = (float)s2[e >> 2][e & 3];
          if constexpr (!BF16) v = (v * sa[u]) * sb2[u][e];
          y = gelu_tanh(y) * v;
        }
        if constexpr (EPI == EPI_F32) {
          o[e] = __float_as_uint(y);
        } else {
          const uint32_t b = float_to_bf16_bits(y);
          o[e >> 1] = (e & 1) ? (o[e >> 1] | (b << 16)) : b;
        }
      }
    }
    char* dst = reinterpret_cast<char*>(p.out) +
                (((int64_t)z * p.M + row) * p.ldo + c0) * ESZ;  // partial sums: one plane a split
    if (BF16 && ESZ == 2 && p.out_packed)  // packed bf16 layout (the next GEMM's A operand)
      dst = reinterpret_cast<char*>(p.out) + frag_offset(row >> 4, c0 / kFragK16, p.ldo / kFragK16) +
            ((row & 15) + 16 * ((c0 % kFragK16) / 8)) * 16;
    if (c0 + 8 <= p.N && (reinterpret_cast<uintptr_t>(dst) & 15) == 0) {
#pragma unroll
      for (int h = 0; h < ESZ / 2; ++h)
        reinterpret_cast<uint4*>(dst)[h] = make_uint4(o[4 * h], o[4 * h + 1], o[4 * h + 2], o[4 * h + 3]);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (c0 + e < p.N) {
          if constexpr (ESZ == 2)
            reinterpret_cast<uint16_t*>(dst)[e] = (uint16_t)(o[e >> 1] >> (16 * (e & 1)));
          else
            reinterpret_cast<uint32_t*>(dst)[e] = o[e];
        }
    }
  }
}

template <int DT, int EPI, int TM, int TN, int NW, int PD>
hipError_t launch_kwave(const GemmParams& p, hipStream_t st) {
  // an E4M3 step holds two fragment columns: half the steps for the same bytes
  constexpr int STEPS = DT == DT_F8 ? (PD + 2) / 2 : PD;
  auto kern = gemm_kwave_kernel<DT, EPI, TM, TN, NW, STEPS>;
  // the waves' sums; when the tiles number no more than the CUs, enough more
  // LDS that no CU takes two workgroups while others have none
  constexpr int sums = NW * TM * TN * kFragBytes, spread = 84 * 1024;
  static_assert(sums <= 160 * 1024, "the waves' sums must fit in LDS");
  static bool attr_set = false;  // benign race: every caller sets the same value
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                       sums > spread ? sums : spread);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  constexpr int TH = EPI == EPI_GLU ? TN / 2 : TN;
  // partial sums are raw
  if (p.splits > 1 && ((EPI != EPI_I32 && !(DT == DT_BF16 && EPI == EPI_F32)) || !p.out ||
                       p.kchunk % frags_per_mma<DT>()))
    return hipErrorInvalidValue;
  const int64_t tiles =
      (int64_t)((p.M + 16 * TM - 1) / (16 * TM)) * ((p.rb_b + TH - 1) / TH) * p.splits;
  const int lds = tiles <= device_cus() && sums < spread ? spread : sums;
  GemmParams q = p;
  if (q.group_m < 1) q.group_m = 8;
  kern<<<(unsigned)((tiles + 7) / 8 * 8), 64 * NW, lds, st>>>(q);
  return hipGetLastError();
}

template <int DT, int EPI>
hipError_t kwave_tile(int tile, const GemmParams& p, hipStream_t st) {
  switch (tile) {
#define KW(NAME, TM, TN, NW, PD) \
    case NAME: return launch_kwave<DT, EPI, TM, TN, NW, PD>(p, st)
    KW(TILE_KW_64x144, 4, 9, 4, 3);
    KW(TILE_KW_64x96, 4, 6, 4, 3);
    KW(TILE_KW_64x64, 4, 4, 4, 4);
    KW(TILE_KW_64x64_W8, 4, 4, 8, 3);
    KW(TILE_KW_32x64_W8, 2, 4, 8, 3);
    KW(TILE_KW_32x32_W8, 2, 2, 8, 4);
    KW(TILE_KW_64x32_W8, 4, 2, 8, 3);
    KW(TILE_KW_32x64, 2, 4, 4, 5);
    KW(TILE_KW_32x32, 2, 2, 4, 6);
    KW(TILE_KW_16x32, 1, 2, 8, 5);
    KW(TILE_KW_16x64, 1, 4, 8, 4);
    KW(TILE_KW_16x16_W16, 1, 1, 16, 4);
#undef KW
    default: return hipErrorInvalidValue;
  }
}

template <int DT>
hipError_t kwave_epi(int epi, int tile, const GemmParams& p, hipStream_t st) {
  switch (epi) {
    case EPI_I32: return kwave_tile<DT, EPI_I32>(tile, p, st);
    case EPI_F32: return kwave_tile<DT, EPI_F32>(tile, p, st);
    case EPI_BF16: return kwave_tile<DT, EPI_BF16>(tile, p, st);
    case EPI_GLU:
      switch (tile) {  // columns: half gate, half up
        case TILE_KW_64x64: return launch_kwave<DT, EPI_GLU, 4, 4, 4, 4>(p, st);
        case TILE_KW_64x128: return launch_kwave<DT, EPI_GLU, 4, 8, 4, 3>(p, st);
        case TILE_KW_128x64: return launch_kwave<DT, EPI_GLU, 8, 4, 4, 3>(p, st);
        case TILE_KW_32x64: return launch_kwave<DT, EPI_GLU, 2, 4, 4, 5>(p, st);
        case TILE_KW_32x128: return launch_kwave<DT, EPI_GLU, 2, 8, 4, 3>(p, st);
        case TILE_KW_16x64: return launch_kwave<DT, EPI_GLU, 1, 4, 4, 5>(p, st);
        case TILE_KW_16x32: return launch_kwave<DT, EPI_GLU, 1, 2, 4, 6>(p, st);
        case TILE_KW_32x32: return launch_kwave<DT, EPI_GLU, 2, 2, 4, 6>(p, st);
        default: return hipErrorInvalidValue;
      }
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_gemm_kwave(int dt, int epi, int tile, const GemmParams& p, hipStream_t st) {
  switch (dt) {
    case DT_I8: return kwave_epi<DT_I8>(epi, tile, p, st);
    case DT_BF16: return kwave_epi<DT_BF16>(epi, tile, p, st);
    case DT_F8: return kwave_epi<DT_F8>(epi, tile, p, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace w8a8
