// Persistent MFMA GEMM for large products (gfx950): C[M x N] = A[M x K] B[N x K]^T
// on tiles of 64 TM x 16 (TNA + TNB), one workgroup of 8 waves per CU.
//
// Waves stand 4 x 2: wave w takes 16 TM rows (w % 4) and TNA (w < 4) or TNB
// column blocks, so each SIMD holds one wave of either width and the widths
// need not be equal: the tile width is chosen so that the tiles divide evenly
// over the CUs.  Operand fragments arrive by LDS-DMA in a ring of S stages of
// KS fragment columns, S stages ahead; the ring runs on across tiles, so a
// tile's first stages arrive during the tile before it and its epilogue.  The
// fragments of step j + 1 are read from LDS into registers between the matrix
// instructions of step j; a stage's slot is free for step j + S as soon as the
// barrier of step j has passed, one barrier per step.
//
// The products run with the operands swapped (weights as the first operand),
// so a lane holds four consecutive columns of one row: two lane exchanges
// (permlane32_swap, permlane16_swap) turn a pair of column blocks into 16-byte
// row pieces and the epilogue needs no LDS.
#include <type_traits>

#include "device.h"
#include "kernels.h"

namespace w8a8 {

namespace {

constexpr int kRingWaves = 8;

__device__ __forceinline__ void ring_dma16(const void* g, v4i* l) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)g,
                                   (__attribute__((address_space(3))) void*)l, 16, 0, 0);
}
__device__ __forceinline__ void ring_dma4(const void* g, float* l) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)g,
                                   (__attribute__((address_space(3))) void*)l, 4, 0, 0);
}
template <int N>
__device__ __forceinline__ void ring_wait() {  // at most N vector-memory operations outstanding
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}
// barrier that waits for this wave's LDS reads but not for its LDS-DMA
__device__ __forceinline__ void ring_barrier() {
  __builtin_amdgcn_s_waitcnt(0xF | (7 << 4) | (0 << 8) | (3 << 14));
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
}
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  return (uint32_t)float_to_bf16_bits(lo) | ((uint32_t)float_to_bf16_bits(hi) << 16);
}

// Sets of scales in LDS.  At a tile's epilogue the producer stands S steps ahead
// and has fetched the next tile's scales as well: with nk steps a tile the live
// tiles are S / nk + 2, so S + 2 sets serve the shortest K.
constexpr int ring_scale_sets(int S) { return S + 2; }

// The order of producer and consumer, replayed: whether every tile's set still
// holds its own scales at the tile's epilogue (only nk <= S needs more than two).
constexpr bool ring_scales_live(int S, int sets) {
  for (int nk = 1; nk <= S + 1; ++nk) {
    const int tiles = 3 * S + 6;
    int owner[16] = {}, pq = 0, pj = 0;
    auto advance = [&]() {  // after an issue, as in ring_body
      if (++pj < nk) return;
      if (pq + 1 < tiles) {
        ++pq;
        pj = 0;
        owner[pq % sets] = pq;
      } else {
        --pj;
      }
    };
    for (int j = 0; j < S; ++j) advance();
    for (int q = 0; q < tiles; ++q) {
      for (int j = 0; j < nk; ++j) advance();
      if (owner[q % sets] != q) return false;
    }
  }
  return true;
}

template <int DT, int EPI, int TM, int TNA, int TNB, int S, int KS>
struct Ring {
  static constexpr bool GLU = EPI == EPI_GLU, BF16 = DT == DT_BF16;
  static constexpr bool SCALED = !BF16 && EPI != EPI_I32;
  static constexpr int NA = 4 * TM, NB = TNA + TNB, NF = NA + NB;
  static constexpr int BM = 16 * NA, BNH = 16 * NB / (GLU ? 2 : 1);
  static constexpr int PIECES = NF * KS, PF = (PIECES + kRingWaves - 1) / kRingWaves;
  static constexpr int NC = (BNH + 63) / 64;                    // 64-wide pieces of the column scales
  static constexpr int NSC = SCALED ? TM + NC * (GLU ? 2 : 1) : 0;
  static constexpr int SETS = ring_scale_sets(S);
  static constexpr int LDS = S * PIECES * kFragBytes + SETS * NSC * 256;
  static_assert(ring_scales_live(S, SETS), "a tile's scales must live until its epilogue");
  static_assert(NSC <= kRingWaves, "one scale piece per wave");
  static_assert(KS % frags_per_mma<DT>() == 0, "a stage must hold whole MFMA K steps");
  static_assert(LDS <= 160 * 1024, "LDS");
};

// The whole kernel for a wave of TN column blocks (C0: its first one).
template <int DT, int EPI, int TM, int TNA, int TNB, int S, int KS, int TN>
__device__ __forceinline__ void ring_body(const GemmParams& p, v4i* lds, int wave, int lane) {
  typedef Ring<DT, EPI, TM, TNA, TNB, S, KS> R;
  typedef typename Acc<DT>::T AccT;
  constexpr bool GLU = R::GLU, BF16 = R::BF16;
  constexpr int KP = frags_per_mma<DT>();
  constexpr int TH = GLU ? TN / 2 : TN;
  constexpr int PF = R::PF, NB = R::NB;
  const int wm = wave & 3;
  const int c0 = wave < 4 ? 0 : (GLU ? TNA / 2 : TNA);  // this wave's first column block
  float* sc = reinterpret_cast<float*>(lds + S * R::PIECES * 64);  // R::SETS sets of scales

  // tiles: XCD blockIdx % 8 takes a contiguous range of a walk through bands of
  // group_m tile rows (M fastest), its workgroups take them in turn
  const int mts = (p.M + R::BM - 1) / R::BM, nts = (p.N + R::BNH - 1) / R::BNH, tot = mts * nts;
  const int per = (tot + 7) / 8, slots = (int)gridDim.x / 8;
  const int first = (int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8);
  const int limit = min(tot, (int)(blockIdx.x % 8 + 1) * per);
  const int n_items = limit > first ? (limit - first + slots - 1) / slots : 0;
  if (n_items == 0) return;  // whole workgroup, before any barrier
  auto item = [&](int q, int& mt, int& nt) {
    const int t = first + q * slots, band_tiles = p.group_m * nts;
    const int band = t / band_tiles, in = t % band_tiles, gm = min(p.group_m, mts - band * p.group_m);
    mt = band * p.group_m + in % gm;
    nt = in / gm;
  };

  // ---- producer: this wave's pieces of a stage, S stages ahead
  const int nk = (p.kb_count + KS - 1) / KS;  // steps per tile (KS = 2: kb_count is even)
  const int rot = p.rotate ? (int)((blockIdx.x * 5u) % (unsigned)nk) : 0;
  const int8_t* src[PF];
  unsigned voff[BF16 ? PF : 1], step_bytes[BF16 ? PF : 1];
  int pq = 0, pj = 0, pslot = 0, pset = 0;
  auto producer_item = [&]() {
    int mt, nt;
    item(pq, mt, nt);
#pragma unroll
    for (int i = 0; i < PF; ++i) {
      const int piece = min(wave + kRingWaves * i, R::PIECES - 1);  // the last ones load it twice
      const int f = piece / KS, k = piece % KS;
      if (f < R::NA) {
        const int rb = min(mt * R::NA + f, p.rb_a - 1);
        if (BF16 && !p.a_packed) {  // row-major: lane l reads row l % 16, columns (l / 16) * 8 .. + 7
          const int64_t row0 = (int64_t)mt * R::BM;
          src[i] = reinterpret_cast<const int8_t*>(reinterpret_cast<const uint16_t*>(p.A) + row0 * p.lda);
          const int r = (int)(min((int64_t)rb * 16 + (lane & 15), (int64_t)p.M - 1) - row0);
          voff[BF16 ? i : 0] = (unsigned)r * (unsigned)(p.lda * 2) + (lane >> 4) * 16;
          step_bytes[BF16 ? i : 0] = kFragK16 * 2;
        } else {
          src[i] = reinterpret_cast<const int8_t*>(p.A) + frag_offset(rb, k, p.kb_count);
          if constexpr (BF16) {
            voff[i] = lane * 16;
            step_bytes[i] = kFragBytes;
          }
        }
      } else {
        int fb = f - R::NA;
        const void* base = p.B;
        if (GLU && fb >= NB / 2) {
          fb -= NB / 2;
          base = p.B2;
        }
        src[i] = reinterpret_cast<const int8_t*>(base) +
                 frag_offset(min(nt * (R::BNH / 16) + fb, p.rb_b - 1), k, p.kb_count);
        if constexpr (BF16) {
          voff[i] = lane * 16;
          step_bytes[i] = kFragBytes;
        }
      }
    }
    if constexpr (R::SCALED) {  // the tile's scales, 64 a wave (indexes clamped into range)
      const int piece = min(wave, R::NSC - 1);
      const float* g;
      if (piece < TM) {
        g = p.s_a + min(mt * R::BM + piece * 64 + lane, p.M - 1);
      } else {
        const bool up = GLU && piece >= TM + R::NC;
        const int c = (piece - TM - (up ? R::NC : 0)) * 64 + lane;
        g = (up ? p.s_b2 : p.s_b) + min(nt * R::BNH + c, p.N - 1);
      }
      ring_dma4(g, sc + pset * R::NSC * 64 + piece * 64);
    }
  };
  auto issue = [&]() {
    int jj = pj + rot;
    if (jj >= nk) jj -= nk;
#pragma unroll
    for (int i = 0; i < PF; ++i) {
      const int piece = min(wave + kRingWaves * i, R::PIECES - 1);
      const int8_t* g = BF16 ? src[i] + (voff[BF16 ? i : 0] + (unsigned)jj * step_bytes[BF16 ? i : 0])
                             : src[i] + ((unsigned)(jj * KS) * kFragBytes + lane * 16);
      ring_dma16(g, &lds[(pslot * R::PIECES + piece) * 64]);
    }
  };
  auto advance = [&]() {
    pslot = pslot + 1 == S ? 0 : pslot + 1;
    if (++pj == nk) {
      if (pq + 1 < n_items) {
        ++pq;
        pj = 0;
        pset = pset + 1 == R::SETS ? 0 : pset + 1;
        producer_item();
      } else {
        --pj;  // past the last tile: its last stage again, never read
      }
    }
  };

  AccT acc[TM][TN];
  struct Frags {
    v4i a[KS][TM], b[KS][TN];
  };
  auto read_frags = [&](int slot, Frags& F) {
    const v4i* St = lds + slot * R::PIECES * 64 + lane;
#pragma unroll
    for (int k = 0; k < KS; ++k) {
#pragma unroll
      for (int t = 0; t < TN; ++t) {
        const int f = R::NA + (GLU && t >= TH ? NB / 2 + t - TH : t) + c0;
        F.b[k][t] = St[(f * KS + k) * 64];
      }
#pragma unroll
      for (int i = 0; i < TM; ++i) F.a[k][i] = St[((wm * TM + i) * KS + k) * 64];
    }
  };

  producer_item();
#pragma unroll
  for (int j = 0; j < S; ++j) {
    issue();
    advance();
  }
  Frags F0, F1;
  ring_wait<PF*(S - 1)>();
  ring_barrier();
  read_frags(0, F0);
  // Before step j's barrier the stages up to j + S - 1 have been issued and
  // stage j + 1 must be complete: the S - 2 stages after it may be
  // outstanding, and, while stage j + 1 was issued before the last epilogue,
  // that epilogue's stores as well (operations complete in order).
  constexpr int AHEAD = PF * (S - 2);
  constexpr int STORES = (EPI == EPI_I32 || EPI == EPI_F32) ? TM * TN : TM * ((TH + 1) / 2);
  constexpr int AHEAD_ST = AHEAD + STORES < 63 ? AHEAD + STORES : 63;
  int cslot = 0, after_epilogue = 0;
  auto step = [&](const Frags& Fc, Frags& Fn) {
    if (after_epilogue > 0) {
      --after_epilogue;
      ring_wait<AHEAD_ST>();
    } else {
      ring_wait<AHEAD>();
    }
    ring_barrier();
    cslot = cslot + 1 == S ? 0 : cslot + 1;
    read_frags(cslot, Fn);
    issue();
#pragma unroll
    for (int k = 0; k < KS; k += KP)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int t = 0; t < TN; ++t) {
          if constexpr (DT == DT_F8)
            acc[i][t] = Acc<DT>::mma2(Fc.b[k][t], Fc.b[k + 1][t], Fc.a[k][i], Fc.a[k + 1][i], acc[i][t]);
          else
            acc[i][t] = Acc<DT>::mma(Fc.b[k][t], Fc.a[k][i], acc[i][t]);
        }
    // spread the LDS reads, then the DMA issues, between the matrix instructions
    constexpr int NL = KS * (TM + TN), NM = KS / KP * TM * TN, EACH = NM / (NL + PF) > 0 ? NM / (NL + PF) : 1;
#pragma unroll
    for (int q = 0; q < NL; ++q) {
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x8, EACH, 0);
    }
#pragma unroll
    for (int q = 0; q < PF; ++q) {
      __builtin_amdgcn_sched_group_barrier(0x10, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x8, EACH, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    advance();
  };

  const bool vec = (p.ldo & (EPI == EPI_I32 || EPI == EPI_F32 ? 3 : 7)) == 0;
  int cset = 0;
  for (int q = 0; q < n_items; ++q, cset = cset + 1 == R::SETS ? 0 : cset + 1) {
    int mt, nt;
    item(q, mt, nt);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int t = 0; t < TN; ++t) acc[i][t] = Acc<DT>::zero();
    int j = 0;
    for (; j + 1 < nk; j += 2) {
      step(F0, F1);
      step(F1, F0);
    }
    if (j < nk) {
      step(F0, F1);
      F0 = F1;
    }

    // ---- epilogue: lane l holds row l % 16, columns 4 (l / 16) .. + 3 of a block
    const int g = lane >> 4;
    const int rloc = wm * TM * 16 + (lane & 15);
    const int row0 = mt * R::BM + rloc, col0 = nt * R::BNH + c0 * 16;
    const bool full = vec && mt * R::BM + R::BM <= p.M && nt * R::BNH + R::BNH <= p.N;
    const float* ss = sc + cset * R::NSC * 64;
    float4 sb[TH], sb2[GLU ? TH : 1];
    if constexpr (R::SCALED) {
#pragma unroll
      for (int t = 0; t < TH; ++t) {
        const int c = (c0 + t) * 16 + 4 * g;
        sb[t] = *reinterpret_cast<const float4*>(ss + TM * 64 + c);
        if constexpr (GLU) sb2[t] = *reinterpret_cast<const float4*>(ss + (TM + R::NC) * 64 + c);
      }
    }
    auto value = [&](int i, int t, float sa, float (&y)[4]) {
      const float s[4] = {sb[t].x, sb[t].y, sb[t].z, sb[t].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        y[e] = (float)acc[i][t][e];
        if constexpr (!BF16) y[e] = (y[e] * sa) * s[e];
      }
      if constexpr (GLU) {
        const float s2[4] = {sb2[t].x, sb2[t].y, sb2[t].z, sb2[t].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float u = (float)acc[i][TH + t][e];
          if constexpr (!BF16) u = (u * sa) * s2[e];
          y[e] = gelu_tanh(y[e]) * u;
        }
      }
    };
    auto store = [&](auto full_tile) {
      constexpr bool FULL = decltype(full_tile)::value;
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int row = row0 + i * 16;
        const float sa = R::SCALED ? ss[rloc + i * 16] : 0.0f;
        if constexpr (EPI == EPI_I32 || EPI == EPI_F32) {
#pragma unroll
          for (int t = 0; t < TN; ++t) {
            v4i o;
            if constexpr (EPI == EPI_I32) {
              o = __builtin_bit_cast(v4i, acc[i][t]);
            } else {
              float y[4];
              value(i, t, sa, y);
              o = v4i{__float_as_int(y[0]), __float_as_int(y[1]), __float_as_int(y[2]), __float_as_int(y[3])};
            }
            const int col = col0 + t * 16 + 4 * g;
            int32_t* d = reinterpret_cast<int32_t*>(p.out) + (int64_t)row * p.ldo + col;
            if constexpr (FULL) {
              if (p.nt_out)
                __builtin_nontemporal_store(o, reinterpret_cast<v4i*>(d));
              else
                *reinterpret_cast<v4i*>(d) = o;
            } else if (row < p.M) {
#pragma unroll
              for (int e = 0; e < 4; ++e)
                if (col + e < p.N) d[e] = o[e];
            }
          }
        } else {
#pragma unroll
          for (int t = 0; t < TH; t += 2) {
            uint32_t x[2][2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              float y[4] = {0.f, 0.f, 0.f, 0.f};
              if (t + h < TH) value(i, t + h, sa, y);
              x[h][0] = pack_bf16x2(y[0], y[1]);
              x[h][1] = pack_bf16x2(y[2], y[3]);
            }
            // lane group g takes columns 8 g .. 8 g + 7 of the block pair
            v4i o;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              const auto r = __builtin_amdgcn_permlane32_swap(x[0][h], x[1][h], false, false);
              const auto r2 = __builtin_amdgcn_permlane16_swap(r[0], r[1], false, false);
              o[h] = (int)r2[0];
              o[2 + h] = (int)r2[1];
            }
            const bool mine = t + 1 < TH || g < 2;  // the last block of an odd count stands alone
            const int col = col0 + t * 16 + 8 * g;
            uint16_t* d;
            if (BF16 && p.out_packed)  // packed bf16 layout (the next GEMM's A operand)
              d = reinterpret_cast<uint16_t*>(p.out) +
                  (frag_offset(row >> 4, col / kFragK16, p.ldo / kFragK16) +
                   ((row & 15) + 16 * ((col % kFragK16) / 8)) * 16) / 2;
            else
              d = reinterpret_cast<uint16_t*>(p.out) + (int64_t)row * p.ldo + col;
            if constexpr (FULL) {
              if (mine) {
                if (p.nt_out)
                  __builtin_nontemporal_store(o, reinterpret_cast<v4i*>(d));
                else
                  *reinterpret_cast<v4i*>(d) = o;
              }
            } else if (mine && row < p.M) {
              if (vec && col + 8 <= p.N) {
                *reinterpret_cast<v4i*>(d) = o;
              } else {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                  if (col + e < p.N) d[e] = (uint16_t)((uint32_t)o[e >> 1] >> (16 * (e & 1)));
              }
            }
          }
        }
      }
    };
    if (full) {
      store(std::true_type{});
      after_epilogue = S - 1;
    } else {
      store(std::false_type{});
      ring_wait<0>();  // a masked tile's store count is not known
      after_epilogue = 0;
    }
  }
  ring_wait<0>();  // no LDS-DMA may be in flight when the workgroup ends
}

template <int DT, int EPI, int TM, int TNA, int TNB, int S, int KS>
__global__ __launch_bounds__(64 * kRingWaves, 1) void gemm_ring_kernel(GemmParams p) {
  extern __shared__ v4i lds[];
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  if (TNA == TNB || wave < 4)
    ring_body<DT, EPI, TM, TNA, TNB, S, KS, TNA>(p, lds, wave, lane);
  else
    ring_body<DT, EPI, TM, TNA, TNB, S, KS, TNB>(p, lds, wave, lane);
}

template <int DT, int EPI, int TM, int TNA, int TNB, int S, int KS>
hipError_t launch_ring(const GemmParams& p, int cus, hipStream_t st) {
  typedef Ring<DT, EPI, TM, TNA, TNB, S, KS> R;
  auto kern = gemm_ring_kernel<DT, EPI, TM, TNA, TNB, S, KS>;
  if constexpr (R::LDS > 64 * 1024) {
    static bool attr_set = false;  // benign race: every caller sets the same value
    if (!attr_set) {
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, R::LDS);
      if (e != hipSuccess) return e;
      attr_set = true;
    }
  }
  const int64_t tiles = (int64_t)((p.M + R::BM - 1) / R::BM) * ((p.N + R::BNH - 1) / R::BNH);
  const int64_t per = (tiles + 7) / 8;
  GemmParams q = p;
  if (q.group_m < 1) q.group_m = 8;
  kern<<<(unsigned)(8 * (per < cus / 8 ? per : cus / 8)), 64 * kRingWaves, R::LDS, st>>>(q);
  return hipGetLastError();
}

template <int DT, int EPI>
hipError_t ring_tile(int tile, const GemmParams& p, int cus, hipStream_t st) {
  if constexpr (DT != DT_F8) {
    switch (tile) {
      case TILE_RING_256: return launch_ring<DT, EPI, 4, 8, 8, 4, 1>(p, cus, st);
      case TILE_RING_224: return launch_ring<DT, EPI, 4, 8, 6, 4, 1>(p, cus, st);
      case TILE_RING_192: return launch_ring<DT, EPI, 4, 6, 6, 4, 1>(p, cus, st);
      case TILE_RING_160: return launch_ring<DT, EPI, 4, 6, 4, 5, 1>(p, cus, st);
      case TILE_RING_128: return launch_ring<DT, EPI, 4, 4, 4, 5, 1>(p, cus, st);
      default: return hipErrorInvalidValue;
    }
  } else {
    switch (tile) {
      case TILE_RING_128: return launch_ring<DT, EPI, 4, 4, 4, 3, 2>(p, cus, st);
      default: return hipErrorInvalidValue;
    }
  }
}

template <int DT>
hipError_t ring_epi(int epi, int tile, const GemmParams& p, int cus, hipStream_t st) {
  switch (epi) {
    case EPI_I32: return ring_tile<DT, EPI_I32>(tile, p, cus, st);
    case EPI_F32: return ring_tile<DT, EPI_F32>(tile, p, cus, st);
    case EPI_BF16: return ring_tile<DT, EPI_BF16>(tile, p, cus, st);
    case EPI_GLU: return ring_tile<DT, EPI_GLU>(tile, p, cus, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_gemm_ring(int dt, int epi, int tile, const GemmParams& p, int cus, hipStream_t st) {
  if (cus < 8) return hipErrorInvalidValue;
  switch (dt) {
    case DT_I8: return ring_epi<DT_I8>(epi, tile, p, cus, st);
    case DT_BF16: return ring_epi<DT_BF16>(epi, tile, p, cus, st);
    case DT_F8: return ring_epi<DT_F8>(epi, tile, p, cus, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace w8a8
