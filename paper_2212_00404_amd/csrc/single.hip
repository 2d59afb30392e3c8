// Single-map direct convolution (paper, Section 2.1, Eq. 2; Section 3.1).
//
// One input map I[Wy][Wx], M filters F[M][K][K], output O[M][Hout][Wout].
//
// Design for gfx950 (the paper's SM partitioning for Pascal is prior art):
//  * The output is cut into TH x 256 tiles (TH = 4 waves x R rows; R = 4 or 8,
//    4 where tall tiles would leave compute units idle), or for outputs up to
//    128 columns wide into 64-column tiles whose waves split into four row
//    groups.  A tile needs its input rows plus K-1 halo rows and columns
//    (Section 3.1 adds the same K-1 extra lines to each map piece).
//  * Workgroups are persistent: each walks every nwg-th tile and, while it
//    computes one tile from LDS, the global loads of its next tile are
//    already in flight into registers (the prefetching of Section 2.2,
//    method 1, done per workgroup).  After the compute the prefetched tile is
//    written to LDS.  Blocks are remapped per XCD so that neighbouring tiles,
//    which share halo rows, run on the same L2.
//  * Each lane owns 4 adjacent output columns x R output rows and streams the
//    input rows of its strip through registers G output rows at a time: one
//    16-byte LDS read per 4 input columns feeds up to K filter rows x K taps x
//    4 columns of FMAs, so LDS traffic stays far below the FMA rate.
//  * The filter is wave-uniform: up to 7x7 it stays in scalar registers and
//    every FMA takes it as an operand; larger filters are held in VGPRs.
//  * The filters of a workgroup (its share of the M filters) are applied to
//    each staged tile in turn, so the map is read from HBM once per filter
//    group (the map-split method of Section 3.1).
//  * Each lane writes its 4 columns of a row with one 16-byte store at any
//    row alignment, non-temporal except in one case chosen on the host.
#include <type_traits>

#include "internal.h"

namespace dconv {
namespace {

constexpr int kW = 4;           // output columns per lane
constexpr int kLanes = 64;
constexpr int kWaves = 4;
constexpr int kBlock = kLanes * kWaves;

// A lane's 4 output columns, stored as one 16-byte write.  Rows of O start
// wherever Wout puts them, so the type asks for 4-byte alignment only: the
// chip's global stores need dword alignment, and one 16-byte store per lane
// keeps every write a whole run of the row.  (Two 8-byte or four 4-byte
// non-temporal stores per lane, as an odd or 2 (mod 4) width would otherwise
// need, leave partly written lines: measured 1.05x slower at Wout = 4090 and
// 1.8-2.6x slower at Wout = 4089 and 4091.)
typedef float vf4u __attribute__((ext_vector_type(4), aligned(4)));

// Output rows per lane: enough that halo re-reads stay small, few enough that
// accumulators, filter, input rows and the prefetched tile fit in VGPRs (a
// tile prefetched as single floats takes four times the registers of one
// prefetched as float4, so unaligned maps get shorter tiles for large K).
// Small filters are bound by memory traffic: shorter tiles give each
// persistent workgroup more of them, so its first (unhidden) tile load is
// shorter and the loads of later tiles overlap more compute (measured 4-8%
// faster at K = 3 and 5 on a 4096 x 4096 map; no gain at K = 7).
template <int K, bool VEC4> struct Rows {
  static constexpr int value = (K <= 5 || (!VEC4 && K >= 8)) ? 4 : 8;
};
// Rows per lane of the short tiles used where tall ones would not give every
// compute unit a tile.
constexpr int kShortRows = 4;
// Output rows accumulated at once (a divisor of Rows).
template <int K> struct Group { static constexpr int value = 4; };
// Workgroups per compute unit the kernel is compiled for (register budget; a
// tile prefetched as single floats needs four times the registers).
template <int K, bool VEC4> struct Occupancy { static constexpr int value = (VEC4 && K <= 7) ? 4 : 2; };

// Up to 7x7 the filter fits the scalar register file next to the addressing
// state.  Larger filters would spill scalar registers into VGPR lanes inside
// the FMA loop, so they are held in VGPRs instead (one copy per lane).
template <int K> struct FilterInVgpr { static constexpr bool value = K * K > 49; };

// L: lanes across a row.  With L = 64 a wave covers R rows x 256 columns;
// with L < 64 its lanes form 64 / L row groups, each R rows x 4L columns
// (narrow maps, where most of a 256-column tile would hold no outputs).
template <int K, int R, int L = kLanes>
struct TileShape {
  static constexpr int RG = kLanes / L;            // row groups per wave
  static constexpr int TW = kW * L;                // output columns per tile
  static constexpr int TH = kWaves * RG * R;       // output rows per tile
  static constexpr int IH = TH + K - 1;            // staged input rows
  static constexpr int NQ = (kW + K - 1 + 3) / 4;  // float4 reads per lane per row
  static constexpr int IW4 = L + NQ - 1;           // float4 per staged row
  static constexpr int LW4 = IW4;                  // LDS stride of a staged row (float4)
  static constexpr int LDS = IH * LW4 * 16;
};
// Lanes across a row of the narrow tiles, and the widest output they serve.
constexpr int kNarrowLanes = 16;
constexpr int kNarrowMaxWout = 128;
constexpr int kNarrowMaxK = 5;

// s_waitcnt immediate for "vmcnt(0)" alone on gfx9-family chips: vmcnt in
// bits 3:0 and 15:14 (0), expcnt in bits 6:4 and lgkmcnt in bits 11:8 at their
// maxima (no wait).
constexpr int kWaitVmcnt0 = 0x0F70;

// Barrier for LDS hand-over inside a workgroup.  Unlike __syncthreads() it
// does not wait for outstanding global loads (the next tile's prefetch stays
// in flight across it) or global stores.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Loads of one staged tile held in registers between fetch() and commit().
// VEC4: every map row starts on a 16-byte boundary, so whole float4 are
// loaded; otherwise single floats.  Values outside the map are zero.
// S: the tile shape (IH staged rows of IW4 float4, stored LW4 float4 apart).
template <class S, bool VEC4>
struct Stager {
  using T = typename std::conditional<VEC4, float4, float>::type;
  static constexpr int PER_ROW = VEC4 ? S::IW4 : S::IW4 * 4;
  static constexpr int LDS_ROW = VEC4 ? S::LW4 : S::LW4 * 4;
  static constexpr int N = S::IH * PER_ROW;
  static constexpr int NL = (N + kBlock - 1) / kBlock;
  T v[NL];

  __device__ __forceinline__ void fetch(const float *__restrict__ I, int Wx, int Wy, int y0, int x0) {
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      const int idx = threadIdx.x + j * kBlock;
      const int iy = idx / PER_ROW;
      const int ix = idx - iy * PER_ROW;
      const int gy = y0 + iy;
      const bool ok = (NL * kBlock == N || idx < N) && gy < Wy;
      if constexpr (VEC4) {
        const int gx = x0 + 4 * ix;
        v[j] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (ok && gx < Wx) v[j] = *reinterpret_cast<const float4 *>(I + (size_t)gy * Wx + gx);
      } else {
        const int gx = x0 + ix;
        v[j] = 0.f;
        if (ok && gx < Wx) v[j] = I[(size_t)gy * Wx + gx];
      }
    }
  }

  __device__ __forceinline__ void commit(float4 *tile) const {
    T *dst = reinterpret_cast<T *>(tile);
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      const int idx = threadIdx.x + j * kBlock;
      if (NL * kBlock == N || idx < N) {
        if constexpr (LDS_ROW == PER_ROW) {
          dst[idx] = v[j];
        } else {
          const int iy = idx / PER_ROW;
          dst[iy * LDS_ROW + (idx - iy * PER_ROW)] = v[j];
        }
      }
    }
  }
};

template <int NQ>
__device__ __forceinline__ void load_row(const float4 *p, float *v) {
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const float4 t = p[q];
    v[4 * q + 0] = t.x;
    v[4 * q + 1] = t.y;
    v[4 * q + 2] = t.z;
    v[4 * q + 3] = t.w;
  }
}

template <int K>
__device__ __forceinline__ void load_filter(const float *__restrict__ F, int m, float (&f)[K][K]) {
  const float *Fm = F + (size_t)m * K * K;
  if constexpr (FilterInVgpr<K>::value) {
    // Vector loads through a pointer the compiler cannot prove uniform: all
    // K*K loads are in flight together (scalar loads of this many values
    // would be issued and waited for one at a time).
    int zero;
    asm volatile("v_mov_b32 %0, 0" : "=v"(zero));
    const float *p = Fm + zero;
#pragma unroll
    for (int r = 0; r < K; ++r)
#pragma unroll
      for (int s = 0; s < K; ++s) f[r][s] = p[r * K + s];
    // Wait for them here, with an instruction the compiler sees.  Otherwise
    // the first use of the filter, at a point the load may or may not have
    // been issued on every path, gets a wait for all loads in flight, which
    // includes the next tile's prefetch: prefetch and compute would then not
    // overlap even where no filter is reloaded.
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
  } else {
#pragma unroll
    for (int r = 0; r < K; ++r)
#pragma unroll
      for (int s = 0; s < K; ++s) f[r][s] = Fm[r * K + s];
  }
}

// One filter over the staged tile: this lane's R x 4 outputs at (oy0, ox0).
// NT: non-temporal output stores.  L: lanes across a row (TileShape).
template <int K, int R, bool NT, int L>
__device__ __forceinline__ void apply_filter(const float4 *rowp, const float (&f)[K][K],
                                             float *__restrict__ Om, int oy0, int ox0, int Hout,
                                             int Wout) {
  using S = TileShape<K, R, L>;
  constexpr int IW4 = S::IW4, NQ = S::NQ;
  constexpr int G = Group<K>::value;
  static_assert(R % G == 0, "group must divide the strip");
#pragma unroll 1
  for (int g = 0; g < R / G; ++g) {
    const float4 *gp = rowp + g * G * IW4;
    float acc[G][kW];
#pragma unroll
    for (int j = 0; j < G; ++j)
#pragma unroll
      for (int w = 0; w < kW; ++w) acc[j][w] = 0.f;

    // One row of look-ahead: the next input row is requested from LDS
    // before the current one is consumed.  The accumulators pass through an
    // empty asm statement and a scheduling barrier ends each row, which
    // keeps the compiler from hoisting every row's reads (and exhausting the
    // VGPRs).
    float cur[NQ * 4], nxt[NQ * 4];
    load_row<NQ>(gp, cur);
#pragma unroll
    for (int yy = 0; yy < G + K - 1; ++yy) {
      if (yy + 1 < G + K - 1) load_row<NQ>(gp + (yy + 1) * IW4, nxt);
#pragma unroll
      for (int r = 0; r < K; ++r) {
        const int j = yy - r;  // output row fed by filter row r
        if (j < 0 || j >= G) continue;
#pragma unroll
        for (int s = 0; s < K; ++s)
#pragma unroll
          for (int w = 0; w < kW; ++w)
            acc[j][w] = __builtin_fmaf(cur[w + s], f[r][s], acc[j][w]);
      }
#pragma unroll
      for (int j = 0; j < G; ++j)
#pragma unroll
        for (int w = 0; w < kW; ++w) asm volatile("" : "+v"(acc[j][w]));
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < NQ * 4; ++q) cur[q] = nxt[q];
    }

#pragma unroll
    for (int j = 0; j < G; ++j) {
      const int y = oy0 + g * G + j;
      if (y >= Hout) continue;
      // The output is written once and never read back by this kernel:
      // non-temporal stores keep it from displacing the input tiles and
      // halos in the caches (measured: 15-20% faster across K).  The
      // exception (NT false) is chosen by the host.
      float *orow = Om + (size_t)y * Wout + ox0;
      const vf4u v = {acc[j][0], acc[j][1], acc[j][2], acc[j][3]};
      if (ox0 + kW <= Wout) {
        if constexpr (NT)
          __builtin_nontemporal_store(v, reinterpret_cast<vf4u *>(orow));
        else
          *reinterpret_cast<vf4u *>(orow) = v;
      } else {
#pragma unroll
        for (int w = 0; w < kW; ++w)
          if (ox0 + w < Wout) orow[w] = v[w];
      }
    }
  }
}

template <int K, int R, bool VEC4, bool NT, int L>
__global__ __launch_bounds__(kBlock, (Occupancy<K, VEC4>::value)) void single_tiled(
    const float *__restrict__ I, const float *__restrict__ F, float *__restrict__ O,
    int Wx, int Wy, int M, int tiles_x, int ntiles, int m_per_block) {
  using S = TileShape<K, R, L>;
  __shared__ float4 tile[S::IH * S::IW4];
  DCONV_POISON(poison_lds(tile, S::IH * S::IW4));

  const int Hout = Wy - K + 1;
  const int Wout = Wx - K + 1;
  // Persistent workgroup: tiles wg, wg + nwg, wg + 2 nwg, ...  At any moment
  // the workgroups in flight cover one contiguous band of tiles (rows of the
  // map), which measured faster than giving each workgroup its own run.
  const int nwg = gridDim.x;
  const int wg = xcd_remap(blockIdx.x, nwg);
  if (wg >= ntiles) return;
  const int m_begin = blockIdx.y * m_per_block;
  const int m_end = min(M, m_begin + m_per_block);

  const int lane = threadIdx.x & (kLanes - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
  // This lane's row group (first output row within the tile) and column
  // quad.
  const int row0 = (wave * S::RG + lane / L) * R;
  const int cq = lane % L;
  const float4 *rowp = tile + row0 * S::IW4 + cq;

  Stager<S, VEC4> st;
  st.fetch(I, Wx, Wy, (wg / tiles_x) * S::TH, (wg % tiles_x) * S::TW);
  st.commit(tile);
  lds_barrier();

  float f[K][K];
  load_filter<K>(F, m_begin, f);
  for (int t = wg; t < ntiles; t += nwg) {
    const int y0 = (t / tiles_x) * S::TH;
    const int x0 = (t % tiles_x) * S::TW;
    const int tn = t + nwg;
    const bool more = tn < ntiles;
    if (more) st.fetch(I, Wx, Wy, (tn / tiles_x) * S::TH, (tn % tiles_x) * S::TW);

    for (int m = m_begin; m < m_end; ++m) {
      if (m != m_begin) load_filter<K>(F, m, f);
      apply_filter<K, R, NT, L>(rowp, f, O + (size_t)m * Hout * Wout, y0 + row0,
                                x0 + cq * kW, Hout, Wout);
    }
    if (m_end - m_begin > 1) load_filter<K>(F, m_begin, f);

    lds_barrier();  // every wave is done reading this tile
    if (more) st.commit(tile);
    lds_barrier();  // the next tile is in LDS
  }
}

// Any K: one output per thread, operands read through the caches.  Used for
// filters larger than the tiled kernels are instantiated for.
__global__ __launch_bounds__(256) void single_generic(
    const float *__restrict__ I, const float *__restrict__ F, float *__restrict__ O,
    int Wx, int Wy, int K, int M) {
  const int Hout = Wy - K + 1;
  const int Wout = Wx - K + 1;
  const int64_t total = (int64_t)M * Hout * Wout;
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= total) return;
  const int x = (int)(idx % Wout);
  const int64_t my = idx / Wout;
  const int y = (int)(my % Hout);
  const int m = (int)(my / Hout);
  const float *Fm = F + (int64_t)m * K * K;
  float acc = 0.f;
  for (int r = 0; r < K; ++r) {
    const float *irow = I + (int64_t)(y + r) * Wx + x;
    const float *frow = Fm + r * K;
    for (int s = 0; s < K; ++s) acc = __builtin_fmaf(irow[s], frow[s], acc);
  }
  O[idx] = acc;
}

// Persistent workgroups: as many as fit on the chip at once.  Filters reuse
// the staged tile; they are split over workgroups only as far as needed to
// fill the chip when there are fewer tiles than slots (or into `force_splits`
// groups when that is given, for the candidate plans).
void plan_persistent(int Wx, int Wy, int K, int M, int num_cu, int th, int tw, int occupancy,
                     SinglePlan *p, int force_splits = 0) {
  const int Hout = Wy - K + 1, Wout = Wx - K + 1;
  p->tile_h = th;
  p->tile_w = tw;
  p->tiles_x = (Wout + tw - 1) / tw;
  p->tiles_y = (Hout + th - 1) / th;
  const int ntiles = p->tiles_x * p->tiles_y;
  const int slots = occupancy * num_cu;
  int splits = force_splits > 0 ? force_splits : (slots + ntiles - 1) / ntiles;
  if (splits > M) splits = M;
  if (splits < 1) splits = 1;
  p->m_per_block = (M + splits - 1) / splits;
  p->grid_z = (M + p->m_per_block - 1) / p->m_per_block;
  int per_split = slots / p->grid_z;
  if (per_split < 1) per_split = 1;
  p->grid = ntiles < per_split ? ntiles : per_split;
  p->block = kBlock;
}

template <int K, bool VEC4>
void plan_tiled(int Wx, int Wy, int M, int num_cu, SinglePlan *p) {
  constexpr int R = Rows<K, VEC4>::value;
  using S = TileShape<K, R>;
  p->kernel = VEC4 ? 0 : 2;
  p->rows = R;
  p->lanes = kLanes;
  if constexpr (VEC4 && K <= kNarrowMaxK) {
    // Narrow maps: lanes in row groups over 64-column tiles.
    if (Wx - K + 1 <= kNarrowMaxWout) {
      using SN = TileShape<K, R, kNarrowLanes>;
      p->lanes = kNarrowLanes;
      plan_persistent(Wx, Wy, K, M, num_cu, SN::TH, SN::TW, Occupancy<K, VEC4>::value, p);
      p->lds_bytes = SN::LDS;
      return;
    }
  }
  plan_persistent(Wx, Wy, K, M, num_cu, S::TH, S::TW, Occupancy<K, VEC4>::value, p);
  p->lds_bytes = S::LDS;
  if constexpr (R > kShortRows) {
    // Fewer tall tiles than compute units (a small map with few filters):
    // short tiles, twice as many (1024 x 1024, K = 7, M = 1: 128 tall tiles
    // left half the chip idle).
    if ((int64_t)p->tiles_x * p->tiles_y * p->grid_z < num_cu) {
      using SS = TileShape<K, kShortRows>;
      p->rows = kShortRows;
      plan_persistent(Wx, Wy, K, M, num_cu, SS::TH, SS::TW, Occupancy<K, VEC4>::value, p);
      p->lds_bytes = SS::LDS;
    }
  }
}

// Non-temporal output stores, except where rows of O do not start on
// 16-byte boundaries, each workgroup writes four or more filters per tile
// and the output is larger than the L2s together: there ordinary stores,
// which L2 merges into whole lines, measured faster (1024 x 1024 map, K = 3,
// 32 filters: 31.6 vs 39.7 us; 2048 x 2048, 4 filters: 15.4 vs 19.1 us).
// With one or two filters per workgroup or aligned rows the non-temporal
// stores are as fast or faster (4096 x 4096, K = 3, M = 1: 22.3 vs 26.3 us),
// and on small outputs (112 x 112, 128 filters) slightly faster.  The
// ordinary-store kernels exist for K <= kTemporalMaxK (the filter sizes of
// the many-filter layers).
constexpr int kTemporalMaxK = 5;
constexpr int64_t kTemporalMinBytes = 32ll << 20;
bool use_nt_stores(const SinglePlan &p, const float *O, int Wx, int Wy, int M) {
  const int Hout = Wy - p.K + 1, Wout = Wx - p.K + 1;
  const bool aligned_rows = Wout % 4 == 0 && (reinterpret_cast<uintptr_t>(O) & 15) == 0;
  const int64_t out_bytes = (int64_t)M * Hout * Wout * 4;
  return aligned_rows || p.m_per_block < 4 || p.K > kTemporalMaxK ||
         out_bytes < kTemporalMinBytes;
}

template <int K, bool VEC4, int R>
void launch_vector(const SinglePlan &p, const float *I, const float *F, float *O, int Wx, int Wy,
                   int M, bool nt, hipStream_t s) {
  const int ntiles = p.tiles_x * p.tiles_y;
  if constexpr (VEC4 && K <= kNarrowMaxK) {
    if (p.lanes == kNarrowLanes) {
      hipLaunchKernelGGL((single_tiled<K, R, VEC4, true, kNarrowLanes>), dim3(p.grid, p.grid_z),
                         dim3(kBlock), 0, s, I, F, O, Wx, Wy, M, p.tiles_x, ntiles,
                         p.m_per_block);
      return;
    }
  }
  if constexpr (K <= kTemporalMaxK) {
    if (!nt) {
      hipLaunchKernelGGL((single_tiled<K, R, VEC4, false, kLanes>), dim3(p.grid, p.grid_z),
                         dim3(kBlock), 0, s, I, F, O, Wx, Wy, M, p.tiles_x, ntiles,
                         p.m_per_block);
      return;
    }
  }
  hipLaunchKernelGGL((single_tiled<K, R, VEC4, true, kLanes>), dim3(p.grid, p.grid_z),
                     dim3(kBlock), 0, s, I, F, O, Wx, Wy, M, p.tiles_x, ntiles, p.m_per_block);
}

template <int K>
hipError_t launch_tiled(const SinglePlan &p, const float *I, const float *F, float *O,
                        int Wx, int Wy, int M, hipStream_t s) {
  const bool nt = use_nt_stores(p, O, Wx, Wy, M);
  constexpr int RA = Rows<K, true>::value, RU = Rows<K, false>::value;
  if (p.kernel == 0) {
    if (RA > kShortRows && p.rows == kShortRows)
      launch_vector<K, true, kShortRows>(p, I, F, O, Wx, Wy, M, nt, s);
    else
      launch_vector<K, true, RA>(p, I, F, O, Wx, Wy, M, nt, s);
  } else {
    if (RU > kShortRows && p.rows == kShortRows)
      launch_vector<K, false, kShortRows>(p, I, F, O, Wx, Wy, M, nt, s);
    else
      launch_vector<K, false, RU>(p, I, F, O, Wx, Wy, M, nt, s);
  }
  return hipGetLastError();
}

}  // namespace

// Where the matrix-core kernel can be forced (the automatic choice and its plans
// reach it at K = kSplitMinK .. kSplitMaxK and any alignment).
static bool can_force_split(int K, bool vec4) {
  return vec4 && K >= kSplitMinK && K <= kMaxTiledK;
}

int plan_single(int Wx, int Wy, int K, int M, int num_cu, bool aligned, int variant,
                SinglePlan *p) {
  *p = SinglePlan{};
  p->K = K;
  // 16-byte aligned rows: whole float4 staging loads.
  const bool vec4 = aligned && (Wx % 4 == 0);
  if (variant == DCONV_VARIANT_MFMA && !can_force_split(K, vec4)) return DCONV_EUNSUPPORTED;
  if (variant == DCONV_VARIANT_MFMA ||
      (variant == DCONV_VARIANT_AUTO && single_takes_split(Wx, Wy, K, M, aligned))) {
    plan_single_split(Wx, Wy, K, M, num_cu, 0, p);
    return DCONV_OK;
  }
  switch (K) {
#define DCONV_PLAN_K(k)                                              \
  case k:                                                            \
    if (vec4) plan_tiled<k, true>(Wx, Wy, M, num_cu, p);             \
    else plan_tiled<k, false>(Wx, Wy, M, num_cu, p);                 \
    return DCONV_OK;
    DCONV_PLAN_K(1) DCONV_PLAN_K(2) DCONV_PLAN_K(3) DCONV_PLAN_K(4) DCONV_PLAN_K(5)
    DCONV_PLAN_K(6) DCONV_PLAN_K(7) DCONV_PLAN_K(8) DCONV_PLAN_K(9) DCONV_PLAN_K(10)
    DCONV_PLAN_K(11)
#undef DCONV_PLAN_K
    default:
      break;
  }
  const int64_t total = (int64_t)M * (Wy - K + 1) * (Wx - K + 1);
  p->kernel = 1;  // generic
  p->rows = 1;
  p->tile_h = 1;
  p->tile_w = 256;
  p->grid = (int)((total + 255) / 256);
  p->grid_z = 1;
  p->tiles_x = p->grid;
  p->tiles_y = 1;
  p->m_per_block = M;
  p->block = 256;
  p->lds_bytes = 0;
  return DCONV_OK;
}

namespace {

// The filter divisions tried for one tile shape: 1, 2, 4, ... groups up to
// M, M itself, and the planner's own (enough groups to fill the chip).
void add_splits(int Wx, int Wy, int K, int M, int num_cu, int occupancy, const SinglePlan &base,
                std::vector<SinglePlan> &out) {
  const int Hout = Wy - K + 1, Wout = Wx - K + 1;
  const int ntiles = ((Wout + base.tile_w - 1) / base.tile_w) * ((Hout + base.tile_h - 1) / base.tile_h);
  const int slots = occupancy * num_cu;
  std::vector<int> splits;
  for (int s = 1; s < M; s *= 2) splits.push_back(s);
  splits.push_back(M);
  splits.push_back((slots + ntiles - 1) / ntiles);
  const size_t first = out.size();
  for (int s : splits) {
    SinglePlan p = base;
    plan_persistent(Wx, Wy, K, M, num_cu, base.tile_h, base.tile_w, occupancy, &p, s);
    bool dup = false;
    for (size_t i = first; i < out.size(); ++i)
      dup = dup || (out[i].m_per_block == p.m_per_block && out[i].grid == p.grid &&
                    out[i].grid_z == p.grid_z);
    if (!dup) out.push_back(p);
  }
}

template <int K, bool VEC4>
void tiled_candidates(int Wx, int Wy, int M, int num_cu, std::vector<SinglePlan> &out) {
  constexpr int RA = Rows<K, VEC4>::value;
  constexpr int OCC = Occupancy<K, VEC4>::value;
  SinglePlan b{};
  b.kernel = VEC4 ? 0 : 2;
  b.K = K;
  b.block = kBlock;
  // tall (or the only) tiles
  b.rows = RA;
  b.lanes = kLanes;
  b.tile_h = TileShape<K, RA>::TH;
  b.tile_w = TileShape<K, RA>::TW;
  b.lds_bytes = TileShape<K, RA>::LDS;
  add_splits(Wx, Wy, K, M, num_cu, OCC, b, out);
  if constexpr (RA > kShortRows) {
    b.rows = kShortRows;
    b.tile_h = TileShape<K, kShortRows>::TH;
    b.tile_w = TileShape<K, kShortRows>::TW;
    b.lds_bytes = TileShape<K, kShortRows>::LDS;
    add_splits(Wx, Wy, K, M, num_cu, OCC, b, out);
  }
  if constexpr (VEC4 && K <= kNarrowMaxK) {
    using SN = TileShape<K, RA, kNarrowLanes>;
    b.rows = RA;
    b.lanes = kNarrowLanes;
    b.tile_h = SN::TH;
    b.tile_w = SN::TW;
    b.lds_bytes = SN::LDS;
    add_splits(Wx, Wy, K, M, num_cu, OCC, b, out);
  }
}

// The matrix-core kernel's plans for the same divisions of the filters
// (tile_m: those of that many filters per workgroup only, 0: all).
void split_candidates(int Wx, int Wy, int K, int M, int num_cu, int tile_m,
                      std::vector<SinglePlan> &out) {
  std::vector<int> splits{0};
  for (int s = 1; s < M; s *= 2) splits.push_back(s);
  splits.push_back(M);
  const size_t first = out.size();
  for (int s : splits) {
    if (tile_m > 0 && s > 0 && (M + s - 1) / s != tile_m) continue;
    SinglePlan p{};
    plan_single_split(Wx, Wy, K, M, num_cu, s, &p);
    bool dup = false;
    for (size_t i = first; i < out.size(); ++i)
      dup = dup || (out[i].m_per_block == p.m_per_block && out[i].rows == p.rows &&
                    out[i].grid == p.grid && out[i].grid_z == p.grid_z);
    if (!dup) out.push_back(p);
  }
}

}  // namespace

int single_candidates(int Wx, int Wy, int K, int M, int num_cu, bool aligned, int variant,
                      std::vector<SinglePlan> &out) {
  out.clear();
  if (num_cu <= 0) num_cu = 256;
  const bool vec4 = aligned && (Wx % 4 == 0);
  const bool valu = variant != DCONV_VARIANT_MFMA;
  const bool split = variant == DCONV_VARIANT_MFMA
                         ? can_force_split(K, vec4)
                         : variant == DCONV_VARIANT_AUTO && K >= kSplitMinK && K <= kSplitMaxK;
  if (valu && K > kMaxTiledK) {
    SinglePlan p;
    plan_single(Wx, Wy, K, M, num_cu, aligned, DCONV_VARIANT_VALU, &p);
    out.push_back(p);
  }
  switch (K) {
#define DCONV_CANDIDATES_K(k)                                                    \
  case k:                                                                        \
    if (valu) {                                                                  \
      if (vec4) tiled_candidates<k, true>(Wx, Wy, M, num_cu, out);               \
      else tiled_candidates<k, false>(Wx, Wy, M, num_cu, out);                   \
    }                                                                            \
    break;
    DCONV_CANDIDATES_K(1) DCONV_CANDIDATES_K(2) DCONV_CANDIDATES_K(3) DCONV_CANDIDATES_K(4)
    DCONV_CANDIDATES_K(5) DCONV_CANDIDATES_K(6) DCONV_CANDIDATES_K(7) DCONV_CANDIDATES_K(8)
    DCONV_CANDIDATES_K(9) DCONV_CANDIDATES_K(10) DCONV_CANDIDATES_K(11)
#undef DCONV_CANDIDATES_K
    default:
      break;
  }
  if (split) split_candidates(Wx, Wy, K, M, num_cu, 0, out);
  return out.empty() ? DCONV_EUNSUPPORTED : DCONV_OK;
}

void single_candidates_like(int Wx, int Wy, int K, int M, int num_cu, bool aligned,
                            const dconv_plan &like, std::vector<SinglePlan> &out) {
  out.clear();
  if (like.variant == DCONV_VARIANT_VALU)
    single_candidates(Wx, Wy, K, M, num_cu, aligned, DCONV_VARIANT_VALU, out);
  else if (like.variant == DCONV_VARIANT_MFMA && like.tile_m > 0 && K >= kSplitMinK &&
           K <= kSplitMaxK)
    split_candidates(Wx, Wy, K, M, num_cu, like.tile_m, out);
}

void export_single_plan(const SinglePlan &p, dconv_plan *out) {
  *out = dconv_plan{};
  out->variant = p.kernel == 3 ? DCONV_VARIANT_MFMA : DCONV_VARIANT_VALU;
  out->kernel = p.kernel;
  out->tile_m = p.m_per_block;
  out->tile_h = p.tile_h;
  out->tile_w = p.tile_w;
  out->chunk_c = 1;
  out->waves_c = 1;
  out->grid_x = p.grid;
  out->grid_y = p.grid_z;
  out->grid_z = 1;
  out->block = p.block;
  out->lds_bytes = p.lds_bytes;
}

hipError_t launch_single(const SinglePlan &p, const float *I, const float *F, float *O,
                         int Wx, int Wy, int M, hipStream_t s) {
  if (p.kernel == 1) {  // generic
    hipLaunchKernelGGL(single_generic, dim3(p.grid), dim3(256), 0, s, I, F, O, Wx, Wy, p.K, M);
    return hipGetLastError();
  }
  if (p.kernel == 3) return launch_single_split(p, I, F, O, Wx, Wy, M, s);
  switch (p.K) {
#define DCONV_LAUNCH_K(k) \
  case k:                 \
    return launch_tiled<k>(p, I, F, O, Wx, Wy, M, s);
    DCONV_LAUNCH_K(1) DCONV_LAUNCH_K(2) DCONV_LAUNCH_K(3) DCONV_LAUNCH_K(4) DCONV_LAUNCH_K(5)
    DCONV_LAUNCH_K(6) DCONV_LAUNCH_K(7) DCONV_LAUNCH_K(8) DCONV_LAUNCH_K(9) DCONV_LAUNCH_K(10)
    DCONV_LAUNCH_K(11)
#undef DCONV_LAUNCH_K
    default:
      return hipErrorInvalidValue;
  }
}

}  // namespace dconv
