// Multi-channel convolution on the bf16 matrix cores (paper, Section 2.1, Eq. 1;
// Section 3.2): an implicit GEMM whose fp32 operands are split into three
// bf16 parts (split.h), six v_mfma_f32_32x32x16_bf16 per product of tiles.
//
// What bounds the fp32 kernel (multi_kernels.h) on large layers is the fp32
// matrix rate: six bf16 instructions do the work of eight fp32 ones in 192
// clocks where those take 512.  The price is the split, 52 vector
// instructions per eight values and lane, so each value is split as few
// times as possible and its parts are reused:
//   * Input: a workgroup's halo tile of CC channels is loaded into registers
//     (eight channels of one pixel per lane), split and written to LDS as
//     B[part][group of 8 channels][pixel], 16 bytes per pixel: a lane's operand
//     for any tap is then one 16-byte read per part, and a value split once
//     serves K * K taps and all filters of the workgroup.
//   * Filters: F[m][c0 : c0 + CC] is copied to LDS as it is (direct 16-byte
//     copies, rows at an odd float4 pitch); a wave reads the eight channels of a tap
//     of its 32 filters, splits them and uses them for NB tiles of 32 pixels.
//     With NB = 2 the split (52 instructions against 12 matrix instructions)
//     hides behind the matrix pipe, which leaves about six issue slots per
//     instruction.
// The 16 values of k of an instruction are two items of eight channels: item
// (group, tap) for lanes 0-31 and the next item for lanes 32-63.  A stage of CC
// channels has CC / 8 * K * K items; WK wave groups share out its pairs, and
// their sums are added through LDS in a fixed order.
#pragma once
#include <type_traits>

#include "multi_kernels.h"
#include "split.h"

namespace dconv {
namespace {

typedef float floatx4s __attribute__((ext_vector_type(4)));

// Pixels a stage's input tile may hold: that of tiles 32 wide, in whole
// 64-lane chunks.
constexpr int split_pix(int K, int PT) {
  return 64 * ceil_div((PT / 32 + K - 1) * (32 + K - 1), 64);
}
constexpr int split_frow(int K, int CC) { return CC * K * K; }
constexpr int split_pitch(int K, int CC) { return mfma_frwp(split_frow(K, CC)); }
constexpr int split_a_floats(int K, int MT, int CC) { return ceil_div(MT * split_pitch(K, CC), 256) * 256; }
constexpr int split_b_vec(int K, int PT, int CC) { return 3 * (CC / 8) * split_pix(K, PT); }
constexpr int split_lds(int K, int MT, int PT, int CC) {
  return 2 * (4 * split_a_floats(K, MT, CC) + 16 * split_b_vec(K, PT, CC));
}
// Channels per stage: the most of 8, 16, 32, 64, 128 whose two buffers fit the
// 160 KB of LDS (0: none).
constexpr int split_cc(int K, int MT, int PT) {
  int best = 0;
  for (int cc = 8; cc <= 128; cc *= 2)
    if (split_lds(K, MT, PT, cc) <= 160 * 1024) best = cc;
  return best;
}

template <int K, int NB, int WM, int WN, int WK>
struct SplitCfg {
  static constexpr int KK = K * K;
  static constexpr int NW = WM * WN * WK, NTHR = 64 * NW;
  static constexpr int MT = 32 * WM, PT = 32 * NB * WN;
  static constexpr int CC = split_cc(K, MT, PT);
  static constexpr int G = CC / 8;
  static constexpr int FROW = split_frow(K, CC), FP = split_pitch(K, CC);
  static constexpr int AF = split_a_floats(K, MT, CC);      // floats of a filter buffer
  static constexpr int NA = ceil_div(AF / 256, NW);         // 1 KB copies per wave
  static constexpr int PIX = split_pix(K, PT);
  static constexpr int NU = ceil_div(G * (PIX / 64), NW);   // input units (64 pixels x 8 channels) per wave
  static constexpr int ITEMS = G * KK, KS = (ITEMS + 1) / 2;
  static constexpr int BV = split_b_vec(K, PT, CC);
  static constexpr int LDS_BYTES = split_lds(K, MT, PT, CC);
  // the wave groups' sums go through the larger of the two kinds of buffer
  static constexpr bool RED_IN = 4 * BV > AF;
  static constexpr int RED = RED_IN ? 4 * BV : AF;
};

typedef float floatx16s __attribute__((ext_vector_type(16)));

// A wave group's part (one of WK) of the sums of a 32 x 32 tile, straight from
// memory with fp32 matrix instructions: taken where the sum of the triples is
// not finite, it gives what the fp32 kernels give.  Every lane of the wave
// takes part: its filter m + lane % 32, its pixel (y, x), inside the map, and
// every second channel.  Bound by the loads of the filters (64 lines each): one
// infinity in 512 -> 512 channels, 40 x 40, K = 3: 205 us (545 where one wave
// group sums alone, 2898 with a sum per lane and filter in turn; a finite
// input 67), 64 -> 64 channels of 512 x 512 NaN 344 us (2442; finite 119).
template <int K, int WK>
__device__ __forceinline__ floatx16s sum_again(const float *__restrict__ I,
                                               const float *__restrict__ F, const TileArgs &a,
                                               int m, int y, int x, int wk) {
  constexpr int KK = K * K, CB = K >= 8 ? 1 : 8 / K;  // channel pairs loaded at once
  const int lane = threadIdx.x & 63, g = lane >> 5;
  const size_t plane = (size_t)a.Wy * a.Wx;
  const float *Fm = F + (size_t)min(m + (lane & 31), a.M - 1) * a.C * KK;
  const float *Ip = I + (size_t)y * a.Wx + x;
  floatx16s f;
#pragma unroll
  for (int v = 0; v < 16; ++v) f[v] = 0.f;
#pragma unroll 1
  for (int c0 = 2 * CB * wk; c0 < a.C; c0 += 2 * CB * WK)
#pragma unroll 1
    for (int r = 0; r < K; ++r) {
      float iv[CB][K], fv[CB][K];
#pragma unroll
      for (int q = 0; q < CB; ++q) {
        const int c = c0 + 2 * q + g, cl = min(c, a.C - 1);
#pragma unroll
        for (int s = 0; s < K; ++s) {
          iv[q][s] = Ip[cl * plane + (size_t)r * a.Wx + s];
          fv[q][s] = Fm[cl * KK + r * K + s];
          if (c >= a.C) iv[q][s] = fv[q][s] = 0.f;
        }
      }
#pragma unroll
      for (int q = 0; q < CB; ++q)
#pragma unroll
        for (int s = 0; s < K; ++s)
          f = __builtin_amdgcn_mfma_f32_32x32x2f32(fv[q][s], iv[q][s], f, 0, 0, 0);
    }
  return f;
}

template <int K, int NB, int WM, int WN, int WK>
__global__ __launch_bounds__(64 * WM * WN * WK, WM *WN *WK / 4) void multi_split(
    const float *__restrict__ I, const float *__restrict__ F, float *__restrict__ O, TileArgs a) {
  using Cfg = SplitCfg<K, NB, WM, WN, WK>;
  constexpr int KK = Cfg::KK, NW = Cfg::NW, NTHR = Cfg::NTHR, MT = Cfg::MT, CC = Cfg::CC;
  constexpr int G = Cfg::G, FROW = Cfg::FROW, FP = Cfg::FP, AF = Cfg::AF, NA = Cfg::NA;
  constexpr int PIX = Cfg::PIX, NU = Cfg::NU, ITEMS = Cfg::ITEMS, KS = Cfg::KS;
  // one object per buffer, so that the copies into one are not waited for
  // when the other is read
  __shared__ float fa0[AF], fa1[AF];
  __shared__ uintx4 in0[Cfg::BV], in1[Cfg::BV];
  DCONV_POISON(poison_lds(fa0, AF), poison_lds(fa1, AF), poison_lds(in0, Cfg::BV),
               poison_lds(in1, Cfg::BV));

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // Stage trace (trace builds): lane 0 of wave 0 and of the last wave writes
  // the shader clock into word idx of its record: in a stage, its start, the
  // first, middle and last step, and the end of its matrix instructions.
  auto mark = [&](int idx) __attribute__((always_inline)) {
#ifdef DCONV_STAGE_TRACE
    const long long t = clock64();
    if (a.trace && (wave == 0 || wave == NW - 1) && lane == 0 && idx < kStageTraceWords) {
      long long *rec = a.trace + ((size_t)blockIdx.x * 2 + (wave != 0)) * kStageTraceWords;
      rec[idx] = idx == 0 || idx == 5 ? wall_clock64() : t;
    }
#else
    (void)idx;
#endif
  };
  mark(0);
  mark(1);
  int tile, mt;
  block_coords(a, tile, mt);
  const int py0 = (tile / a.tiles_x) * a.tpy;
  const int px0 = (tile % a.tiles_x) * a.tpx;
  const int m0 = mt * MT;
  const int Hout = a.Wy - K + 1, Wout = a.Wx - K + 1;
  const int wk = wave % WK;
  const int wm = (wave / WK) % WM;
  const int wn = wave / WK / WM;
  const int col = lane & 31, g = lane >> 5;
  const int npix = a.tpy * a.tpx;
  const float inv_tpx = rcp(a.tpx), inv_iw = rcp(a.IW);

  // Filter copies: chunk j of this wave covers buffer floats
  // [256 (wave + j NW), + 256); the source of lane's 16 bytes relative to
  // filter m0's stage.  Rows past M re-read filter M - 1, a row's padding its
  // start.
  //   A row starts shift(row) floats into its first 16 bytes, so that the 32
  // rows a wave reads one value of lie in different banks (rows that all start
  // on 16 bytes share a quarter of them: 72 conflict clocks per pair of items
  // on 512 x 512 maps, K = 3).  The copies of a shifted row begin up to three
  // floats before it and end after it, inside the filters next to it; filter
  // M - 1, the last in memory, is not shifted.
  auto shift = [&](int row) __attribute__((always_inline)) {
    return m0 + row >= a.M - 1 ? 0 : (row >> 3) & 3;
  };
  const int ckk = a.C * KK;
  uint32_t va[NA];
#pragma unroll
  for (int j = 0; j < NA; ++j) {
    const int e = 256 * (wave + j * NW) + 4 * lane;
    const int row = e / FP;
    int eo = e - row * FP - shift(row);
    if (eo >= FROW || row >= MT) eo = 0;
    const int rr = min(m0 + min(row, MT - 1), a.M - 1) - m0;
    va[j] = 4u * ((uint32_t)rr * (uint32_t)ckk + (uint32_t)eo);
  }
  // Input units: unit u = wave + i NW is channel group u % G, pixels
  // [64 (u / G), + 64); the lane's pixel, clamped into the map (pixels past the
  // tile or the map reach no stored output).
  const int nunits = G * ((a.IH * a.IW + 63) / 64);
  const size_t plane = (size_t)a.Wy * a.Wx;
  uint32_t vp[NU];
#pragma unroll
  for (int i = 0; i < NU; ++i) {
    const int p = 64 * ((wave + i * NW) / G) + lane;
    const int iy = fdiv(p, a.IW, inv_iw);
    const int gy = min(py0 + iy, a.Wy - 1);
    const int gx = min(px0 + p - mul24(iy, a.IW), a.Wx - 1);
    vp[i] = 4u * ((uint32_t)gy * (uint32_t)a.Wx + (uint32_t)gx);
  }

  const int a_base = (wm * 32 + col) * FP + shift(wm * 32 + col);
  int b_base[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int p = (wn * NB + nb) * 32 + col;
    const int ty = fdiv(p, a.tpx, inv_tpx);
    b_base[nb] = p < npix ? mul24(ty, a.IW) + p - mul24(ty, a.tpx) : 0;
  }

  typedef floatx16s acc_t;
  acc_t acc[NB], cor[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[nb][v] = cor[nb][v] = 0.f;

  // stage c0's filter slice into fa
  auto copy_filters = [&](int c0, float *fa) __attribute__((always_inline)) {
    const float *src = F + (size_t)m0 * ckk + (size_t)c0 * KK;
    if (c0 + CC <= a.C) {
#pragma unroll
      for (int j = 0; j < NA; ++j)
        if (wave + j * NW < AF / 256) dma_f128_at<0>(src, va[j], fa + 256 * (wave + j * NW));
    } else {
      // the last channels: nothing past a filter's end is read, zeros instead
      const int flen = (a.C - c0) * KK;
      for (int base = threadIdx.x; base < MT * FROW; base += 8 * NTHR) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int i = base + u * NTHR, row = i / FROW, e = i - row * FROW;
          const bool ok = i < MT * FROW && e < flen;
          const int rr = min(m0 + row, a.M - 1) - m0;
          v[u] = ok ? src[(size_t)(i < MT * FROW ? rr : 0) * ckk + e] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int i = base + u * NTHR, row = i / FROW;
          if (i < MT * FROW) fa[row * FP + shift(row) + i - row * FROW] = v[u];
        }
      }
    }
  };
  // input unit i of stage c0 into registers, and its parts into LDS
  float raw[NU][8];
  auto load_unit = [&](int c0, auto UNIT) __attribute__((always_inline)) {
    constexpr int i = decltype(UNIT)::value;
    const int u = wave + i * NW;
    if (u < nunits) {
      const int c = c0 + 8 * (u % G);
      if (c + 8 <= a.C) {
        const float *src = I + (size_t)c * plane;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          raw[i][e] = *reinterpret_cast<const float *>(reinterpret_cast<const char *>(src) + vp[i]);
          src += plane;
        }
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float *src = I + (size_t)min(c + e, a.C - 1) * plane;
          raw[i][e] = *reinterpret_cast<const float *>(reinterpret_cast<const char *>(src) + vp[i]);
        }
      }
    }
  };
  auto store_unit = [&](int c0, uintx4 *in, auto UNIT) __attribute__((always_inline)) {
    constexpr int i = decltype(UNIT)::value;
    const int u = wave + i * NW;
    if (u < nunits) {
      const int gr = u % G, c = c0 + 8 * gr;
      if (c + 8 > a.C) {
#pragma unroll
        for (int e = 0; e < 8; ++e) raw[i][e] = c + e < a.C ? raw[i][e] : 0.f;
      }
      const Split8 s = split8(raw[i]);
      uintx4 *dst = in + gr * PIX + 64 * (u / G) + lane;
      dst[0] = __builtin_bit_cast(uintx4, s.h);
      dst[G * PIX] = __builtin_bit_cast(uintx4, s.m);
      dst[2 * G * PIX] = __builtin_bit_cast(uintx4, s.l);
    }
  };

  // The pairs of items wk, wk + WK, ... of a stage.  While the matrix
  // instructions of a pair run, the filter values of the next pair are split
  // between them, and the LDS reads of the next pair's input parts and of the
  // filter values after that are in flight.  (A wave that read, split and
  // multiplied in turn took 2.7 times the matrix instructions' time.)
  struct Item { int fo, po; bool ok; };  // floats into a filter row, pixels into the tile
  auto item = [&](int k) __attribute__((always_inline)) {
    const int i = 2 * min(k, KS - 1) + g;
    // divisions by constants through 24-bit multiplies (i < 2^11, t < 2^6)
    const int gr = KK == 1 ? i : mul24(i, (65536 + KK - 1) / KK) >> 16;
    const int t = i - gr * KK;
    const int r = K == 1 ? 0 : mul24(t, (1024 + K - 1) / K) >> 10;
    const bool ok = ITEMS % 2 == 0 || i < ITEMS;
    return Item{ok ? gr * (7 * KK) + i : 0, ok ? gr * PIX + mul24(r, a.IW - K) + t : 0, ok};
  };
  auto read_a = [&](const Item &t, const float *fa, float (&av)[8]) __attribute__((always_inline)) {
    const float *ap = fa + a_base + t.fo;
#pragma unroll
    for (int e = 0; e < 8; ++e) av[e] = ap[e * KK];
    if (ITEMS % 2 != 0) {
#pragma unroll
      for (int e = 0; e < 8; ++e) av[e] = t.ok ? av[e] : 0.f;
    }
  };
  auto read_b = [&](const Item &t, const uintx4 *in, uintx4 (&b)[NB][3]) __attribute__((always_inline)) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int c = 0; c < 3; ++c) b[nb][c] = in[b_base[nb] + t.po + c * G * PIX];
  };
  auto compute = [&](const float *fa, const uintx4 *in, auto &&at_step) __attribute__((always_inline)) {
    constexpr int NK = ceil_div(KS, WK);
    float av[2][8];
    uintx4 bv[2][NB][3];
    Split8 s[2];
    Item t0 = item(wk), t1 = item(wk + WK);
    read_a(t0, fa, av[0]);
    read_b(t0, in, bv[0]);
    read_a(t1, fa, av[1]);
    s[0] = split8(av[0]);
    Item t2 = item(wk + 2 * WK);
    static_for<0, NK>([&](auto STEP) __attribute__((always_inline)) {
      constexpr int i = decltype(STEP)::value, j = i & 1;
      at_step(STEP);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (i + 1 < NK) read_b(t1, in, bv[1 - j]);
      if constexpr (i + 2 < NK) read_a(t2, fa, av[j]);
      __builtin_amdgcn_sched_barrier(0);
      // only the last step may have no pair left for some of the waves
      if (i + 1 < NK || KS % WK == 0 || wk + i * WK < KS) {
#pragma unroll
        for (int part = 0; part < 6; ++part)
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) {
            const bf16x8 x = part == 0 ? s[j].l : (part == 2 || part == 3) ? s[j].m : s[j].h;
            const bf16x8 y = __builtin_bit_cast(
                bf16x8, bv[j][nb][part == 1 ? 2 : (part == 2 || part == 4) ? 1 : 0]);
            acc_t &c = part == 5 ? acc[nb] : cor[nb];
            c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, y, c, 0, 0, 0);
          }
      }
      if constexpr (i + 1 < NK) {
        s[1 - j] = split8(av[1 - j]);
        t1 = t2;
        if constexpr (i + 3 < NK) t2 = item(wk + (i + 3) * WK);
#pragma unroll
        for (int q = 0; q < 6 * NB; ++q) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, NB == 2 ? 5 : 10, 0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    });
  };

  mark(2);
  copy_filters(0, fa0);
  static_for<0, NU>([&](auto U) { load_unit(0, U); });
  static_for<0, NU>([&](auto U) { store_unit(0, in0, U); });
  wait_lds_dma();
  __syncthreads();
  mark(3);
  // The next stage is fetched between the steps of this one: input unit u is
  // loaded before step u NK / NU, split and written to LDS before the step
  // that loads the next unit (the last one before the last step), and the
  // filters' copies go out before step 1.  (All of it at the start of the stage
  // held the matrix instructions back by 1,100 clocks, and by 10,000 where the
  // eight waves had more than 64 loads to issue: a compute unit takes about
  // that many before it waits for the first to return.)
  auto stage = [&](auto J, int c0) __attribute__((always_inline)) {
    constexpr int j = decltype(J)::value;
    constexpr int NK = ceil_div(KS, WK);
    const bool more = c0 + CC < a.C;
    const int tw = 6 + 5 * (c0 / CC);
    mark(tw);
    uintx4 *nin = j == 0 ? in1 : in0;
    auto at_step = [&](auto STEP) __attribute__((always_inline)) {
      constexpr int i = decltype(STEP)::value;
      if constexpr (i == 0) mark(tw + 1);
      if constexpr (i == NK / 2) mark(tw + 2);
      if constexpr (i == NK - 1) mark(tw + 3);
      if (more) {
        static_for<0, NU>([&](auto U) {
          constexpr int u = decltype(U)::value;
          constexpr int at = u + 1 < NU ? (u + 1) * NK / NU : NK - 1;
          if constexpr (i == at && at > u * NK / NU) store_unit(c0 + CC, nin, U);
        });
        static_for<0, NU>([&](auto U) {
          if constexpr (i == decltype(U)::value * NK / NU) load_unit(c0 + CC, U);
        });
        if constexpr (i == (NK > 1 ? 1 : 0)) copy_filters(c0 + CC, j == 0 ? fa1 : fa0);
      }
    };
    compute(j == 0 ? fa0 : fa1, j == 0 ? in0 : in1, at_step);
    mark(tw + 4);
    if (more) {  // units without a later step to be stored at
      static_for<0, NU>([&](auto U) {
        constexpr int u = decltype(U)::value;
        constexpr int at = u + 1 < NU ? (u + 1) * NK / NU : NK - 1;
        if constexpr (at <= u * NK / NU) store_unit(c0 + CC, nin, U);
      });
    }
    wait_lds_dma();
    lds_barrier();
  };
  for (int c0 = 0; c0 < a.C; c0 += 2 * CC) {
    stage(std::integral_constant<int, 0>{}, c0);
    if (c0 + CC >= a.C) break;
    stage(std::integral_constant<int, 1>{}, c0 + CC);
  }

  mark(4);
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) acc[nb] += cor[nb];
  struct Pixel { int y, x; bool ok; };
  auto pixel = [&](int nb) __attribute__((always_inline)) {
    const int p = (wn * NB + nb) * 32 + col;
    const int ty = fdiv(p, a.tpx, inv_tpx);
    const int gy = py0 + ty, gx = px0 + p - mul24(ty, a.tpx);
    return Pixel{gy, gx, p < npix && gy < Hout && gx < Wout};
  };
  // whether a sum that is stored is not finite
  auto any_bad = [&](int nb) __attribute__((always_inline)) {
    float z = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) z = fmaf(0.f, acc[nb][v], z);
    return kSumAgain && __any(pixel(nb).ok && !(z == 0.f));
  };
  // this wave group's part of the sums again
  auto again = [&](int nb) __attribute__((always_inline)) {
    const Pixel p = pixel(nb);
    return sum_again<K, WK>(I, F, a, m0 + wm * 32, min(p.y, Hout - 1), min(p.x, Wout - 1), wk);
  };
  auto replace = [&](int nb, const acc_t &f) __attribute__((always_inline)) {
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[nb][v] = 0.f * acc[nb][v] == 0.f ? acc[nb][v] : f[v];
  };
  // Fixed-order sum of the WK wave groups, in as many passes as one buffer
  // takes.
  if constexpr (WK > 1) {
    constexpr int TILE = WM * WN * 1024;
    constexpr int PER = Cfg::RED / TILE;  // wave groups per pass
    static_assert(PER >= 1, "a wave group's sums fit a buffer");
    float *red = Cfg::RED_IN ? reinterpret_cast<float *>(in0) : fa0;
    const int wmn = wm + WM * wn;
    auto add_groups = [&](acc_t &sum, auto &&added) __attribute__((always_inline)) {
      for (int g0 = 1; g0 < WK; g0 += PER) {
        if (wk >= g0 && wk < g0 + PER) {
#pragma unroll
          for (int v = 0; v < 16; ++v)
            red[(wk - g0) * TILE + (wmn * 16 + v) * 64 + lane] = sum[v];
        }
        lds_barrier();
        if (wk == 0) {
          for (int q = g0; q < min(g0 + PER, WK); ++q)
#pragma unroll
            for (int v = 0; v < 16; ++v)
              sum[v] += red[(q - g0) * TILE + (wmn * 16 + v) * 64 + lane];
          if (g0 + PER >= WK) added();
        }
        lds_barrier();
      }
    };
    // Group 0 tells the others, which otherwise are done here, of sums that are
    // not finite: all groups sum those again.
    int *flags = reinterpret_cast<int *>(in1);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
      add_groups(acc[nb], [&]() __attribute__((always_inline)) {
        acc[nb] *= kSplitUnscale;
        const int bad = any_bad(nb);
        if (lane == 0) flags[nb * WM * WN + wmn] = bad;
      });
    int bad = 0;
#pragma unroll
    for (int i = 0; i < NB * WM * WN; ++i) bad |= flags[i];
    if (__builtin_amdgcn_readfirstlane(bad)) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        acc_t f;
#pragma unroll
        for (int v = 0; v < 16; ++v) f[v] = 0.f;
        const int mine = __builtin_amdgcn_readfirstlane(flags[nb * WM * WN + wmn]);
        if (mine) f = again(nb);
        add_groups(f, [&]() __attribute__((always_inline)) { if (mine) replace(nb, f); });
      }
    }
    if (wk != 0) return;
  } else {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      acc[nb] *= kSplitUnscale;
      if (any_bad(nb)) replace(nb, again(nb));
    }
  }

#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const Pixel p = pixel(nb);
    if (p.ok) {
      // one offset per lane, the filters' planes in scalar registers
      const size_t map = (size_t)Hout * Wout;
      const int mw = m0 + wm * 32;
      float *Ol = O + ((size_t)p.y * Wout + p.x) + 4 * g * map;
      if (mw + 32 <= a.M) {
#pragma unroll
        for (int v = 0; v < 16; ++v)
          Ol[(size_t)(mw + 8 * (v >> 2) + (v & 3)) * map] = acc[nb][v];
      } else {
#pragma unroll
        for (int v = 0; v < 16; ++v)
          if (mw + Mfma<32>::row(lane, v) < a.M)
            Ol[(size_t)(mw + 8 * (v >> 2) + (v & 3)) * map] = acc[nb][v];
      }
    }
  }
  mark(5);
}

// Workgroup shapes: 32 WM filters x 32 NB WN pixels, WK wave groups sharing a
// stage's items.
struct SplitShape { int NB, WM, WN, WK; };
constexpr SplitShape kSplitShapes[] = {
    {2, 2, 4, 1},  // 64 x 256
    {2, 2, 2, 2},  // 64 x 128
    {2, 1, 2, 4},  // 32 x 128
    {2, 2, 1, 4},  // 64 x 64
    {2, 1, 1, 8},  // 32 x 64
    {1, 1, 1, 8},  // 32 x 32
};
constexpr int kNumSplit = sizeof(kSplitShapes) / sizeof(kSplitShapes[0]);

template <int K, int S>
using SplitShapeCfg = SplitCfg<K, kSplitShapes[S].NB, kSplitShapes[S].WM, kSplitShapes[S].WN,
                               kSplitShapes[S].WK>;

template <int K, int S>
hipError_t launch_split_shape(const MultiPlan &p, const float *I, const float *F, float *O,
                              const TileArgs &a, hipStream_t st) {
  constexpr SplitShape sh = kSplitShapes[S];
  if constexpr (SplitShapeCfg<K, S>::CC == 0) {
    return hipErrorInvalidValue;
  } else {
    auto kern = multi_split<K, sh.NB, sh.WM, sh.WN, sh.WK>;
    hipLaunchKernelGGL(kern, dim3(p.grid_x), dim3(64 * sh.WM * sh.WN * sh.WK), 0, st, I, F, O, a);
    return hipGetLastError();
  }
}

template <int K, int... S>
hipError_t launch_split_k(const MultiPlan &p, const float *I, const float *F, float *O,
                          const TileArgs &a, hipStream_t st, std::integer_sequence<int, S...>) {
  hipError_t e = hipErrorInvalidValue;
  ((p.kernel == kSplitKernel + S ? (e = launch_split_shape<K, S>(p, I, F, O, a, st), 0) : 0), ...);
  return e;
}

}  // namespace
}  // namespace dconv
