// Single-map convolution on the bf16 matrix cores (paper, Section 2.1, Eq. 2):
// fp32 values split into three bf16 parts (split.h), the filter in banded
// form over two dimensions.
//
// v_mfma_f32_16x16x32_bf16 multiplies A[16][32] by B[32][16].  The 16 rows of
// A are the outputs of one PH x PW patch, the 16 columns of B are 16 patches
// side by side, and the 32 values of k are two input rows of 16 columns: step
// q of a patch takes input rows 2q and 2q + 1 (u) and columns t = 0..15 of its
// window,
//   A[(dy, dx)][(u, t)] = F[u - dy][t - dx]   (zero outside 0..K-1)
//   B[(u, t)][j]        = I[y + u][x_j + t]
// (on the strip at a map's right edge the second eight columns start at T2 <= 8,
// so that the last one is the last one the patch needs and no load leaves the
// row; A is zero where the two eights overlap)
// and NQ = ceil((PH + K - 1) / 2) steps finish the patch: 2 x 8 patches
// (K <= 9, whose window is at most 16 wide) use 0.38 / 0.51 of the products at
// K = 7 / 9, 4 x 4 patches (K <= 13) 0.54 at K = 11; at six instructions a
// product that is 1.2 to 2.9 times the rate of one fp32 FMA per lane per
// clock.  The filter sits in registers for the whole kernel (A is the same
// for every patch).
//
// A wave owns a strip of 16 * PW columns and walks down it two input rows a
// step, straight from memory into registers (no LDS, no barrier): each lane
// loads the eight values it supplies to B, splits them, and the instructions
// of that step feed every patch row the two rows touch (NS of them in
// flight).  The next two steps' loads are in flight meanwhile.  A float is
// loaded by up to four lanes of a wave, which the vector L1 absorbs, and
// rows need no alignment (4-byte alignment suffices for 16-byte loads), so
// odd widths run at the same speed.
#include "internal.h"
#include "split.h"

namespace dconv {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t uintx2 __attribute__((ext_vector_type(2)));
typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));

constexpr int kBlock = 256, kLanes = 64;
constexpr int kDepth = 2;  // steps loaded ahead
constexpr uint32_t kOutOfRange = 0xffffff00u;  // a buffer offset past every row
constexpr int kNT = 2;     // non-temporal (buffer store)

template <int K> struct Patch {
  static constexpr int PW = K <= 9 ? 8 : 4;   // outputs of a patch: PH rows of PW
  static constexpr int PH = 16 / PW;
  static constexpr int SW = 16 * PW;          // columns of a wave's strip
  static constexpr int NQ = (PH + K) / 2;     // steps (row pairs) per patch
  static constexpr int ADV = PH / 2;          // steps between patch rows
  static constexpr int NS = (NQ + ADV - 1) / ADV;  // patch rows in flight
  static constexpr int P = NS * ADV;          // steps until the registers repeat
  // the zero-bordered filter: rows -(PH-1) .. 2 NQ - 1, columns -(PW-1) .. 15
  static constexpr int ZH = 2 * NQ + PH - 1, ZW = 16 + PW - 1;
  // Neighbouring windows overlap by 16 - PW columns.  At PW = 4 a float would
  // be split by four lanes; instead each lane splits one group of four columns
  // and the lanes read their windows back from LDS (SHARE).
  static constexpr bool SHARE = PW == 4;
  static constexpr int NF = SHARE ? 4 : 8;    // floats a lane loads per step
  // At the right edge: first column of the second eight of a window; SHARE:
  // how far the last group of four is moved left to end on the map's last
  // column.  (Elsewhere 8 and 0: the loads of K = 6 and 7 at T2 = 5 and 6
  // measured 12% slower.)
  static constexpr int T2 = SHARE ? 8 : PW + K - 9;
  static constexpr int BACK = SHARE ? 13 - K : 0;
  static constexpr int QUADS = SHARE ? 20 : 0;     // groups of four per row (19 used)
  static_assert(PW + K - 1 <= 16, "a patch's window is 16 columns wide");
  static_assert(2 * NQ >= PH + K - 1, "the steps cover the window");
};

// The sums of a strip (its patches from column x0 and row y0 of map O, the columns
// from x_own stored) that came out non-finite, again from memory, one fp32 FMA
// per tap.  It runs once the strip is stored and reads the stored values back,
// so that the strip's own code only gathers a flag.  A window's row is loaded
// at once, 16 bytes at a time (bound by the vector L1): a 4096 x 4096 map of
// NaN 164 us at K = 7 and 205 at K = 11 (543 and 592 with 4-byte loads; 1374 and
// 1815 with a load and an FMA after the other at each patch row).
template <int K>
__device__ __forceinline__ void sum_again(const float *I, const float *F, float *O, int Wx, int Wy,
                                          int x0, int x_own, int y0, int nv) {
  constexpr int PW = Patch<K>::PW, PH = Patch<K>::PH;
  const int Hout = Wy - K + 1, Wout = Wx - K + 1;
  // the lane's outputs of a patch row, as in the strip's stores; the lane number
  // read anew, so that nothing per lane stays in registers through the strip
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int j = tid & 15, g = (tid & 63) >> 4;
  const int oy = PW == 8 ? g >> 1 : g, x = x0 + PW * j + (PW == 8 ? 4 * (g & 1) : 0);
  __threadfence_block();
#pragma unroll 1
  for (int y = y0 + oy; y < min(y0 + nv * PH, Hout); y += PH) {
    float *Or = O + (size_t)y * Wout + x;
    bool bad[4], any = false;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      bad[e] = x + e >= x_own && x + e < Wout && !(0.f * Or[e] == 0.f);
      any = any || bad[e];
    }
    if (!any) continue;
    const float *Ir = I + (size_t)y * Wx;
    float f[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int r = 0; r < K; ++r, Ir += Wx) {
      float w[K + 3];
      if (x + 4 <= Wout) {
        constexpr int V = (K + 3) / 4;
#pragma unroll
        for (int q = 0; q < V; ++q) {
          const floatx4u p = *reinterpret_cast<const floatx4u *>(Ir + x + 4 * q);
#pragma unroll
          for (int i = 0; i < 4; ++i) w[4 * q + i] = p[i];
        }
#pragma unroll
        for (int i = 4 * V; i < K + 3; ++i) w[i] = Ir[x + i];
      } else {
#pragma unroll
        for (int i = 0; i < K + 3; ++i) w[i] = Ir[min(x + i, Wx - 1)];
      }
#pragma unroll
      for (int s = 0; s < K; ++s)
#pragma unroll
        for (int e = 0; e < 4; ++e) f[e] = fmaf(w[s + e], F[r * K + s], f[e]);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (bad[e]) Or[e] = f[e];
  }
}

// Strips of `nv` patch rows, numbered along x, then y; a workgroup's waves take
// four in turn.  nstrips: all of them.
template <int K>
__global__ __launch_bounds__(kBlock, 2) void single_split(
    const float *__restrict__ I, const float *__restrict__ F, float *__restrict__ O, int Wx,
    int Wy, int M, int strips_x, int nstrips, int m_per_block, int nv) {
  using S = Patch<K>;
  constexpr int PW = S::PW, PH = S::PH, NQ = S::NQ, ADV = S::ADV, NS = S::NS, P = S::P, NF = S::NF;
  const int Hout = Wy - K + 1, Wout = Wx - K + 1;
  const int nwg = gridDim.x;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int j = lane & 15;       // patch (B, D) or output of a patch (A)
  const int g = lane >> 4;       // group of eight k: row g / 2, columns 8 (g % 2) ...
  const int m_begin = blockIdx.y * m_per_block;
  const int m_end = min(M, m_begin + m_per_block);
  __shared__ float zf[2][S::ZH * S::ZW];
  __shared__ uintx2 shared[4][3][2][S::SHARE ? S::QUADS : 1];  // per wave: part, row, group
  DCONV_POISON(poison_lds(&zf[0][0], 2 * S::ZH * S::ZW),
               poison_lds(&shared[0][0][0][0], 24 * (S::SHARE ? S::QUADS : 1)));

  // The border is zeroed once; thread i < K * K copies element i of each
  // filter, loaded while the filter before it is in use.
  for (int i = threadIdx.x; i < 2 * S::ZH * S::ZW; i += kBlock) (&zf[0][0])[i] = 0.f;
  const int zpos = ((int)threadIdx.x / K + PH - 1) * S::ZW + (int)threadIdx.x % K + PW - 1;
  float fnext = threadIdx.x < K * K ? F[(size_t)m_begin * K * K + threadIdx.x] : 0.f;
  __syncthreads();
  for (int m = m_begin; m < m_end; ++m) {
    const float *Fm = F + (size_t)m * K * K;
    // The filter with a border of zeros, from which each lane reads its rows
    // of A at constant offsets.  Two copies: while some waves still walk their
    // strips with one filter, others may write the next one.
    float *z = zf[(m - m_begin) & 1];
    if (threadIdx.x < K * K) z[zpos] = fnext;
    __syncthreads();
    if (threadIdx.x < K * K && m + 1 < m_end) fnext = Fm[K * K + threadIdx.x];
    Split8 a[NQ];
    int t2 = 0;  // first column of the second eight that `a` stands for
    for (int t = 4 * xcd_remap(blockIdx.x, nwg) + wave; t < nstrips; t += 4 * nwg) {
      const int y0 = (t / strips_x) * nv * PH;
      int x0 = (t % strips_x) * S::SW;
      // A strip that would pass the right edge starts further left and stores
      // its own columns only (from x_own: the order of an output's sum depends
      // on its place in a patch, so its neighbour's may differ in a rounding).
      const int x_own = x0;
      constexpr int REACH = S::SW + 16 - PW;  // columns the windows span
      constexpr int FULL = 0, EDGE = 1, NARROW = 2, NARROW_END = 3;
      const bool edge = Wout >= S::SW && x0 + REACH > Wx;
      if (edge) x0 = min(x0, Wout - S::SW);
      // patch rows of this strip that hold outputs, and its steps
      const int n_patch = min(nv, (Hout - y0 + PH - 1) / PH);
      const int n_step = ADV * (n_patch - 1) + NQ;

      // Loads: lane (j, g) takes its eight columns of row 2w + g / 2 of the
      // strip.  Past the strip's last rows (or the map's) the last ones are
      // read again: they meet only zeros of A or outputs that are never
      // stored.  On maps narrower than a strip a window runs past its row (which
      // reaches no stored output either), and strips whose last rows would be
      // read past the whole map load one float at a time, the index clamped.
      const float *Is = I + (size_t)y0 * Wx + x0;
      const int last_row = Wy - 1 - y0;
      const int row_cap = min(2 * n_step - 1, last_row);
      const int64_t left = (int64_t)(last_row + 1) * Wx - x0;  // floats to the end of the map
      const int quad = S::SHARE ? ((g & 1) ? 16 + min(j, 2) : j) : 0;  // SHARE: group of four
      const int back = edge && quad == 18 ? S::BACK : 0;
      const int t2_want = edge ? S::T2 : 8;
      const int col = S::SHARE ? 4 * quad - back : PW * j + t2_want * (g & 1);
      if (t2 != t2_want) {
        t2 = t2_want;
        const float *za = z + ((g >> 1) - j / PW + PH - 1) * S::ZW + t2 * (g & 1) - j % PW + PW - 1;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          float v[8];
#pragma unroll
          for (int e = 0; e < 8; ++e)
            v[e] = (g & 1) && t2 + e < 8 ? 0.f : za[2 * q * S::ZW + e];
          a[q] = split8(v);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      float *Os = O + ((size_t)m * Hout + y0) * Wout + x0;
      const int oy = PW == 8 ? g >> 1 : g, ox = PW * j + (PW == 8 ? 4 * (g & 1) : 0);
      // 32-bit byte offsets from the row pair's and the patch row's start
      const uint32_t off_even = 4u * (uint32_t)col;
      const uint32_t off_pair = off_even + ((g >> 1) ? 4u * (uint32_t)Wx : 0u);
      const uint32_t off_out = 4u * (uint32_t)(oy * Wout + ox);

      const bool whole = x0 + ox >= x_own, part = !whole && x0 + ox + 4 > x_own;
      int bad = 0;  // 1: a sum was not finite

      // FULL: every column of the strip is stored; EDGE: those from x_own;
      // NARROW: the map is narrower than a strip (NARROW_END: loads clamped).
      auto strip = [&](auto KIND) __attribute__((always_inline)) {
        constexpr int kind = decltype(KIND)::value;
        int row = 0;             // the row pair the next load takes
        const float *Ir = Is;
        float *Or = Os;          // the patch row the next store writes
        auto load = [&](float (&v)[NF]) __attribute__((always_inline)) {
          const uint32_t off = row < row_cap ? off_pair : off_even;
          if constexpr (kind != NARROW_END) {
            const char *src = reinterpret_cast<const char *>(Ir) + off;
#pragma unroll
            for (int q = 0; q < NF / 4; ++q) {
              const floatx4u p = *reinterpret_cast<const floatx4u *>(src + 16 * q);
#pragma unroll
              for (int e = 0; e < 4; ++e) v[4 * q + e] = p[e];
            }
          } else {
            const int64_t at = (int64_t)row * Wx + off / 4u;
#pragma unroll
            for (int e = 0; e < NF; ++e) {
              const int64_t i = at + e;
              v[e] = Is[i < left ? i : left - 1];
            }
          }
          if (row + 2 <= row_cap) {
            row += 2;
            Ir += 2 * (size_t)Wx;
          }
        };
        // a lane's operand of B from the floats it loaded
        auto operand = [&](const float (&v)[NF]) __attribute__((always_inline)) {
          if constexpr (S::SHARE) {
            Split8 r;
            // the group moved left, put back in place
            float u[4];
#pragma unroll
            for (int e = 0; e < 4; ++e)
              u[e] = kind == EDGE && quad == 18 ? (e + S::BACK < 4 ? v[(e + S::BACK) & 3] : 0.f)
                                                  : v[e];
            uint32_t parts[3][2];
#pragma unroll
            for (int i = 0; i < 2; ++i)
              split2(u[2 * i], u[2 * i + 1], parts[0][i], parts[1][i], parts[2][i]);
#pragma unroll
            for (int c = 0; c < 3; ++c)
              shared[wave][c][g >> 1][quad] = (uintx2){parts[c][0], parts[c][1]};
            __builtin_amdgcn_wave_barrier();
            uintx4 w[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
              const uintx2 lo = shared[wave][c][g >> 1][j + 2 * (g & 1)];
              const uintx2 hi = shared[wave][c][g >> 1][j + 2 * (g & 1) + 1];
              w[c] = (uintx4){lo[0], lo[1], hi[0], hi[1]};
            }
            __builtin_amdgcn_wave_barrier();
            r.h = __builtin_bit_cast(bf16x8, w[0]);
            r.m = __builtin_bit_cast(bf16x8, w[1]);
            r.l = __builtin_bit_cast(bf16x8, w[2]);
            return r;
          } else {
            return split8(v);
          }
        };
        float buf[kDepth][NF];
#pragma unroll
        for (int d = 0; d < kDepth; ++d) load(buf[d]);
        Split8 b = operand(buf[0]);
        auto advance = [&]() __attribute__((always_inline)) {
#pragma unroll
          for (int d = 0; d + 1 < kDepth; ++d)
#pragma unroll
            for (int e = 0; e < NF; ++e) buf[d][e] = buf[d + 1][e];
          load(buf[kDepth - 1]);
        };
        advance();

        // Patch row v starts at step ADV v and lives in accumulator slot
        // v % NS: the products of the high parts in acc, the others in cor.
        floatx4 acc[NS], cor[NS];
        // One period of P steps from step `base`.  FIRST: the patch rows
        // above the strip are left out; GUARD: steps past the end too.
        auto period = [&](int base, auto FIRST, auto GUARD) __attribute__((always_inline)) {
          constexpr bool first = decltype(FIRST)::value, guard = decltype(GUARD)::value;
#pragma unroll
          for (int jj = 0; jj < P; ++jj) {
            const int w = base + jj;
            if (guard && w >= n_step) break;
            // the next step's operand is split while this step's products run
            const Split8 nb = operand(buf[0]);
            advance();
            if (jj % ADV == 0) {
#pragma unroll
              for (int v = 0; v < 4; ++v) acc[jj / ADV][v] = cor[jj / ADV][v] = 0.f;
            }
            // the patch rows this step feeds: q = jj % ADV, + ADV, ...
#pragma unroll
            for (int part = 0; part < 6; ++part) {
#pragma unroll
              for (int q = jj % ADV; q < NQ; q += ADV) {
                if (first && jj < q) continue;
                const int s = ((jj - q) / ADV + NS * ((jj < q) ? 1 : 0)) % NS;
                const bf16x8 av = part == 0 ? a[q].l : (part == 2 || part == 3) ? a[q].m : a[q].h;
                const bf16x8 bv = part == 1 ? b.l : (part == 2 || part == 4) ? b.m : b.h;
                floatx4 &c = part == 5 ? acc[s] : cor[s];
                c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv, c, 0, 0, 0);
              }
            }
            // K >= 8: the split of the next operand spread between the products
            if constexpr (K >= 8) {
#pragma unroll
              for (int i = 0; i < 6 * NQ / ADV; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
              }
            }
            // the patch row that ends with this step
            constexpr int QL = NQ - 1;
            if ((jj - QL % ADV + ADV) % ADV == 0 && !(first && jj < QL)) {
              const int s = ((jj - QL) / ADV + NS * ((jj < QL) ? 1 : 0)) % NS;
              const floatx4 sum = (acc[s] + cor[s]) * kSplitUnscale;
              floatx4u r = {sum[0], sum[1], sum[2], sum[3]};
              const int y = y0 + PH * ((w - QL) / ADV) + oy, x = x0 + ox;
              const bool ok = (!guard || y < Hout) &&
                              (kind == FULL || (kind == EDGE ? whole || part : x < Wout));
              // zero times a finite value is zero, anything else NaN
              const float z = fmaf(0.f, r[0], fmaf(0.f, r[1], fmaf(0.f, r[2], 0.f * r[3])));
              // (a branch, which the compiler keeps for the statement in it: without
              // one it takes 6 more registers at K = 7, and so a third less waves)
              if (__ballot(!(z == 0.f)) != 0) {
                asm volatile("" : "+s"(bad));
                bad = 1;
              }
              if constexpr (kind == FULL) {
                if (ok)
                  __builtin_nontemporal_store(r, reinterpret_cast<floatx4u *>(
                                reinterpret_cast<char *>(Or) + off_out));
              } else {
                // Whole groups of four, then the floats of a partial one: of
                // a shifted strip's first group, or of the row's last one.
                // Buffer stores drop the lanes whose offset is out of range,
                // so no store is skipped by a branch and every wait for a
                // load knows how many stores follow it (the partial stores
                // behind branches: 28.6 against 24.3 us for a 4096 x 4096 map
                // at K = 7, the waits for loads held by the edge strips' stores).
                const __amdgpu_buffer_rsrc_t rows =
                    __builtin_amdgcn_make_buffer_rsrc(Or, 0, kOutOfRange, 0x00027000);
                const bool all = kind == EDGE ? whole : x + 4 <= Wout;
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(uintx4, (floatx4)r), rows,
                                                       ok && all ? off_out : kOutOfRange, 0, kNT);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                  if (e == (kind == EDGE ? 0 : 3)) continue;
                  const bool in = ok && !all && (kind == EDGE ? x + e >= x_own : x + e < Wout);
                  __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(r[e]), rows,
                                                        in ? off_out + 4u * e : kOutOfRange, 0, 0);
                }
              }
              Or += (size_t)PH * Wout;
            }
            b = nb;
            __builtin_amdgcn_sched_barrier(0);
          }
        };
        period(0, std::true_type{}, std::true_type{});
        int base = P;
        for (; base + P < n_step; base += P) period(base, std::false_type{}, std::false_type{});
        if (base < n_step) period(base, std::false_type{}, std::true_type{});
      };
      if (edge)
        strip(std::integral_constant<int, EDGE>{});
      else if (Wout >= S::SW)
        strip(std::integral_constant<int, FULL>{});
      else if ((int64_t)row_cap * Wx + REACH <= left)
        strip(std::integral_constant<int, NARROW>{});
      else
        strip(std::integral_constant<int, NARROW_END>{});
      if (kSumAgain && bad != 0)
        sum_again<K>(I, Fm, O + (size_t)m * Hout * Wout, Wx, Wy, x0, x_own, y0, nv);
    }
  }
}

template <int K>
hipError_t launch_k(const SinglePlan &p, const float *I, const float *F, float *O, int Wx, int Wy,
                    int M, hipStream_t st) {
  hipLaunchKernelGGL(single_split<K>, dim3(p.grid, p.grid_z), dim3(kBlock), 0, st, I, F, O, Wx, Wy,
                     M, p.tiles_x, p.tiles_x * p.tiles_y, p.m_per_block, p.rows);
  return hipGetLastError();
}

}  // namespace

// Where the kernel is the automatic choice, from times of both kernels on
// random maps (28 to 4096 wide and high, 1 to 512 filters), vector kernel
// against this one:
//   K >= 10   faster on every map (4096 x 4096, K = 11: 55.5 -> 37.1 us; K = 12
//             and 13 had a kernel of one output per thread: 18 -> 5 us on
//             256 x 256 with four filters)
//   K = 7, 9  faster (34.9 -> 25.0, 40.4 -> 27.0 us) but for small outputs less
//             than half a strip wide, where a wave is mostly empty (32 x 55, 16
//             filters: 4.9 against 6.0 us)
//   K = 8     (the steps of K = 9 for fewer taps) faster on tall maps (35.2 ->
//             27.9 us); short ones up to 1.35x slower (1755 x 39, 272 filters)
//   K = 6     faster from about 1.5M outputs (4096 x 4096: 29.0 -> 25.3 us;
//             below, up to 1.4x slower), and wherever rows are not whole float4
//   K = 5     only where rows are not whole float4, which the vector kernel
//             stages float by float (1021 x 1003, 8 filters: 17.3 -> 12.5 us)
bool single_takes_split(int Wx, int Wy, int K, int M, bool aligned) {
  if (K < kSplitMinK || K > kSplitMaxK) return false;
  const bool vec4 = aligned && Wx % 4 == 0;
  const int64_t outputs = (int64_t)M * (Wy - K + 1) * (Wx - K + 1);
  if (K >= 10) return true;
  if (K == 8) return vec4 ? Wy >= 512 && outputs >= 3000000 : Wy >= 64;
  if (K >= 7) return !(vec4 && Wx - K + 1 < 64 && outputs < 32768);
  if (K == 6) return !vec4 || outputs >= 1500000;
  return !vec4;
}

void plan_single_split(int Wx, int Wy, int K, int M, int num_cu, int force_splits, SinglePlan *p) {
  *p = SinglePlan{};
  const int Hout = Wy - K + 1, Wout = Wx - K + 1;
  const int pw = K <= 9 ? 8 : 4, ph = 16 / pw, sw = 16 * pw;
  const int nq = (ph + K) / 2, adv = ph / 2;
  // workgroups per compute unit: the kernels up to K = 7 fit three (K = 9
  // measured 26.7 us at two, 31 at three)
  const int slots = (K <= 7 ? 3 : 2) * num_cu;
  const int strips_x = (Wout + sw - 1) / sw;
  const int wave_rows = (Hout + ph - 1) / ph;   // patch rows of the map
  // Clocks: a step of a lone wave, and of a SIMD's issue (six instructions
  // per patch row and the operand's split); setting up a filter and starting a
  // strip each cost about a load latency and more.
  const double busy = 6.0 * nq / adv * 16 + 130, lone = busy + 150;
  double best = 0;
  for (int splits = force_splits > 0 ? force_splits : 1;;
       splits = splits * 2 < M ? splits * 2 : M) {
    const int mpb = (M + splits - 1) / splits, groups = (M + mpb - 1) / mpb;
    if (groups > slots && splits > 1 && force_splits == 0) break;
    const int cap = slots / groups > 0 ? slots / groups : 1;
    for (int nv : {1, 2, 3, 4, 5, 6, 8, 10, 12, 16, 20, 24, 28, 32, 40, 48, 64}) {
      const int strips = strips_x * ((wave_rows + nv - 1) / nv);
      const int tiles = (strips + 3) / 4;
      const int nwg = tiles < cap ? tiles : cap;
      const int64_t wgs = (int64_t)nwg * groups;
      const double share = wgs <= num_cu ? 1.0 : wgs >= slots ? (double)wgs / num_cu
                                                              : (double)((wgs + num_cu - 1) / num_cu);
      const double step = share * busy > lone ? share * busy : lone;
      const double cost = mpb * (3000.0 + ((tiles + nwg - 1) / nwg) *
                                              (2000.0 + (adv * (nv - 1) + nq) * step));
      if (best == 0 || cost < best) {
        best = cost;
        p->rows = nv;
        p->tiles_y = strips / strips_x;
        p->m_per_block = mpb;
        p->grid_z = groups;
        p->grid = nwg;
      }
    }
    if (splits >= M || force_splits > 0) break;
  }
  p->kernel = 3;
  p->K = K;
  p->lanes = kLanes;
  p->tile_w = sw;
  p->tile_h = p->rows * ph;
  p->tiles_x = strips_x;
  p->block = kBlock;
  p->lds_bytes = 4 * (2 * (2 * nq + ph - 1) * (15 + pw) + 2 * 24 * (pw == 4 ? 20 : 1));
}

hipError_t launch_single_split(const SinglePlan &p, const float *I, const float *F, float *O,
                               int Wx, int Wy, int M, hipStream_t st) {
  switch (p.K) {
#define DCONV_SPLIT_K(k) \
  case k:                \
    return launch_k<k>(p, I, F, O, Wx, Wy, M, st);
    DCONV_SPLIT_K(5) DCONV_SPLIT_K(6) DCONV_SPLIT_K(7) DCONV_SPLIT_K(8) DCONV_SPLIT_K(9) 
    DCONV_SPLIT_K(10) DCONV_SPLIT_K(11) DCONV_SPLIT_K(12) DCONV_SPLIT_K(13)
#undef DCONV_SPLIT_K
    default:
      return hipErrorInvalidValue;
  }
}

}  // namespace dconv
