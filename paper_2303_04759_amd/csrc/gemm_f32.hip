// Dense contractions of the full-precision mode on the matrix cores: v_mfma_f32_16x16x4_f32 (float operands, float
// accumulation), operand tiles brought straight from global memory into LDS through a ring, all four operand layouts.
//
// What bounds it: a CU's matrix cores run float products at 256 flops per clock (151 TFLOP/s over the chip, measured with
// nothing else running), and while they do, the SIMD issues no memory instruction of any wavefront: a probe with
// computing and loading wavefronts took 231 000 clocks for its MFMAs alone, 141 000 for its direct loads alone and
// 372 000 for both (with the bf16 16x16x32 MFMA: 240 000, 141 000, 240 000).  The time of a tile is therefore the sum
// of its MFMAs and its loads, about 24 clocks per KiB: 64x48 tiles reach 66 %, 64x192 tiles 79 % of the MFMA rate, and
// loading wavefronts of their own, fragments read one stage ahead and deeper rings all measured the same or worse.
// The tile is chosen so that the 256 CUs get equal work in whole rounds (launch_gemm_f32).  The wavefronts of a block
// split the contraction (KS), which fills the SIMDs without further operand bytes.
// Against the 64x64 FMA kernel before it, 1024 x 768 x 3072: 539 -> 51 us, 1024 x 3072 x 768 with GeLU: 167 -> 55 us.
//
// LDS layout of a k-step of 32 (128 bytes per row, the geometry of the bf16 kernels):
//   K-major tile  [ROWS][32]: 16-byte chunk c of row r at position c ^ ((r >> 1) & 7); a fragment is one ds_read_b128
//                             whose four values feed four MFMAs (the contraction index of MFMA e, lane group g is
//                             4 g + e: any order serves as long as both operands use the same)
//   MN-major tile [32][ROWS]: chunk cc of k-row k at position (cc + 4 ((k >> 2) & 3)) mod (ROWS / 4), so that the four
//                             lane groups of a fragment read hit different banks
#include "gemm_device.hpp"

namespace raf {

constexpr int FK = 32;   // contraction values per ring sub-tile

typedef __attribute__((address_space(3))) void* f32_lds_ptr;

// per-lane source of KiB chunk q of a [ROWS] x 32 operand tile at contraction offset 0
template <int ROWS, bool KMAJOR>
__device__ __forceinline__ const float* f32_src(const float* base, long ld, int row0, int nrows, int q) {
  const int lane = threadIdx.x & 63;
  if (KMAJOR) {
    const int r = q * 8 + (lane >> 3);
    int gr = row0 + r;
    gr = gr < nrows ? gr : nrows - 1;
    return base + (long)gr * ld + (((lane & 7) ^ ((r >> 1) & 7)) << 2);
  } else {
    constexpr int CPR = ROWS / 4;
    const int n = q * 64 + lane, k = n / CPR;
    int cc = n % CPR - (4 * ((k >> 2) & 3)) % CPR;
    cc = cc < 0 ? cc + CPR : cc;
    int col = row0 + cc * 4;
    col = col < nrows ? col : nrows - 4;
    return base + (long)k * ld + col;
  }
}

// byte offset of a lane's first fragment value of 16 rows at row0 (multiple of 16), half kk of the sub-tile
template <int ROWS, bool KMAJOR>
__device__ __forceinline__ int f32_frag_offset(int row0, int kk) {
  const int lane = threadIdx.x & 63, g = lane >> 4;
  if (KMAJOR) {
    const int r = row0 + (lane & 15);
    return r * 128 + (((kk * 4 + g) ^ ((r >> 1) & 7)) << 4);
  } else {
    constexpr int CPR = ROWS / 4;
    const int pos = (((row0 + (lane & 15)) >> 2) + 4 * g) % CPR;
    return (kk * 16 + g * 4) * (ROWS * 4) + pos * 16 + (lane & 3) * 4;
  }
}
template <int ROWS, bool KMAJOR>
__device__ __forceinline__ f32x4_t f32_fragment(const char* p) {
  if (KMAJOR) return *reinterpret_cast<const f32x4_t*>(p);
  f32x4_t v;
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = *reinterpret_cast<const float*>(p + e * (ROWS * 4));
  return v;
}

// columns j .. j+3 of row i, epilogue resolved at compile time
template <int EPI, int TANH>
__device__ __forceinline__ void f32_epilogue_store4(const GemmDev& g, float* __restrict__ c, float* __restrict__ aux, int i,
                                                    int j, f32x4_t v) {
  v = v * g.alpha;
  if constexpr (EPI == EPI_BIAS || EPI == EPI_BIAS_GELU || EPI == EPI_BIAS_GELU_DERIV) {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] += g.bias[j + e];
  }
  f32x4_t* ax = reinterpret_cast<f32x4_t*>(aux + (long)i * g.ldaux + j);
  if constexpr (EPI == EPI_BIAS_GELU) {
    *ax = v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = gelu_f(v[e], TANH);
  } else if constexpr (EPI == EPI_BIAS_GELU_DERIV) {
    f32x4_t dy;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float y, d;
      gelu_and_grad_f(v[e], TANH, y, d);
      v[e] = y;
      dy[e] = d;
    }
    *ax = dy;
  } else if constexpr (EPI == EPI_MUL_GELU_GRAD) {
    const f32x4_t u = *ax;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] *= gelu_grad_f(u[e], TANH);
  } else if constexpr (EPI == EPI_ADD_RES) {
    v = v + *ax;
  } else if constexpr (EPI == EPI_MUL_AUX) {
    v = v * *ax;
  }
  *reinterpret_cast<f32x4_t*>(c + (long)i * g.ldc + j) = v;
}

// One BM x BN output tile, BM = 16 WGM MB and BN = 16 WGN NB, by WGM x WGN blocks of 16 MB x 16 NB outputs with KS
// wavefronts each.  A ring stage holds SUB = KS / 2 sub-tiles of 32 contraction values; wavefront kg of a block takes
// half kg % 2 of sub-tile kg / 2.
template <int WGM, int WGN, int MB, int NB, int KS, int NS, bool AK, bool BK>
__device__ __forceinline__ void f32_tile(const GemmDev& g, int m0, int n0, int z, char* lds) {
  constexpr int NT = WGM * WGN, NW = NT * KS, SUB = KS / 2;
  constexpr int BM = 16 * WGM * MB, BN = 16 * WGN * NB;
  constexpr int ACH = BM / 8, CH = (BM + BN) / 8;      // KiB chunks of a sub-tile: A, then B
  constexpr int SUB_BYTES = CH * 1024, STAGE_BYTES = SUB * SUB_BYTES;
  constexpr int LOADS = (SUB * CH + NW - 1) / NW;      // direct loads per wavefront and stage (the last may be absent)
  static_assert(KS == 2 || KS == 4 || KS == 8, "wavefronts come in pairs, one per half of a sub-tile");
  static_assert(BM % 8 == 0 && BN % 8 == 0, "tiles are loaded in KiB chunks");

  const int zb = z / g.nz_inner, zi = z % g.nz_inner;
  const float* __restrict__ A = (const float*)g.a + zb * g.sa0 + zi * g.sa1;
  const float* __restrict__ B = (const float*)g.b + zb * g.sb0 + zi * g.sb1;
  float* __restrict__ C = (float*)g.c + zb * g.sc0 + zi * g.sc1;
  float* __restrict__ AUX = g.aux ? (float*)g.aux + zb * g.sc0 + zi * g.sc1 : nullptr;

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int wt = wave % NT, kg = wave / NT, sub = kg >> 1;
  const int wm = (wt / WGN) * 16 * MB, wn = (wt % WGN) * 16 * NB;
  const int nsub = g.K / FK, nk = (nsub + SUB - 1) / SUB;

  // chunk f of a stage (sub-tile f / CH, A chunks first) goes to wavefront f % NW
  const float* src[LOADS];
  long step[LOADS];
#pragma unroll
  for (int i = 0; i < LOADS; ++i) {
    int f = i * NW + wave;
    f = f < SUB * CH ? f : SUB * CH - 1;               // an absent load keeps a valid address it never uses
    const int s = f / CH, q = f % CH;
    const bool is_a = q < ACH;
    const long kstep = is_a ? (AK ? FK : (long)FK * g.lda) : (BK ? FK : (long)FK * g.ldb);
    src[i] = (is_a ? f32_src<BM, AK>(A, g.lda, m0, g.M, q) : f32_src<BN, BK>(B, g.ldb, n0, g.N, q - ACH)) + s * kstep;
    step[i] = kstep * SUB;
  }
  // sub-tiles past the end of the contraction (last stage only) are neither loaded nor used
  auto issue = [&](int it, int slot) {
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      const int f = i * NW + wave;
      if (f < SUB * CH && (SUB == 1 || it * SUB + f / CH < nsub))
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src[i] + it * step[i]),
                                         (f32_lds_ptr)(lds + slot * STAGE_BYTES + f * 1024), 16, 0, 0);
    }
  };
  auto loads_of = [&](int it) {                          // loads this wavefront issues for stage `it`
    int n = 0;
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      const int f = i * NW + wave;
      n += (f < SUB * CH && (SUB == 1 || it * SUB + f / CH < nsub)) ? 1 : 0;
    }
    return n;
  };
  const int full_loads = loads_of(0), last_loads = loads_of(nk - 1);

  int fa_off[MB], fb_off[NB];
#pragma unroll
  for (int i = 0; i < MB; ++i) fa_off[i] = sub * SUB_BYTES + f32_frag_offset<BM, AK>(wm + 16 * i, kg & 1);
#pragma unroll
  for (int j = 0; j < NB; ++j) fb_off[j] = sub * SUB_BYTES + ACH * 1024 + f32_frag_offset<BN, BK>(wn + 16 * j, kg & 1);

  f32x4_t acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

#pragma unroll
  for (int s = 0; s < NS - 1; ++s)
    if (s < nk) issue(s, s);
  int stage = 0;
  for (int it = 0; it < nk; ++it) {
    // stages it+1 .. it+NS-2 may stay in flight; stage `it` must have landed
    const int ahead = nk - 1 - it < NS - 2 ? nk - 1 - it : NS - 2;
    wait_vmcnt_dyn(it + ahead == nk - 1 && ahead > 0 ? (ahead - 1) * full_loads + last_loads : ahead * full_loads);
    __builtin_amdgcn_s_barrier();                        // stage `it` is complete for every wavefront; stage it-1 is free
    if (it + NS - 1 < nk) {
      int ns = stage + NS - 1;
      ns = ns >= NS ? ns - NS : ns;
      issue(it + NS - 1, ns);
    }
    if (SUB == 1 || it * SUB + sub < nsub) {
      const char* st = lds + stage * STAGE_BYTES;
      f32x4_t fa[MB], fb[NB];
#pragma unroll
      for (int i = 0; i < MB; ++i) fa[i] = f32_fragment<BM, AK>(st + fa_off[i]);
#pragma unroll
      for (int j = 0; j < NB; ++j) fb[j] = f32_fragment<BN, BK>(st + fb_off[j]);
      // operands swapped: a lane ends with output row (l & 15) and 4 consecutive columns 4*(l>>4) + r
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
          for (int j = 0; j < NB; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[j][e], fa[i][e], acc[i][j], 0, 0, 0);
    }
    stage = stage + 1 == NS ? 0 : stage + 1;
  }

  // the KS partial blocks meet in LDS; wavefront kg adds blocks kg, kg + KS, ... in a fixed order and finishes them
  __builtin_amdgcn_s_barrier();                          // every wavefront is done with the ring
  f32x4_t* xch = reinterpret_cast<f32x4_t*>(lds) + (long)wt * MB * NB * 64;
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) xch[((long)kg * NT * MB * NB + i * NB + j) * 64 + lane] = acc[i][j];
  __syncthreads();
  epilogue_dispatch(g, [&](auto tag, auto form) {
    constexpr int EPI = decltype(tag)::value, TANH = decltype(form)::value;
    for (int b = kg; b < MB * NB; b += KS) {
      f32x4_t v = xch[(long)b * 64 + lane];
#pragma unroll
      for (int s = 1; s < KS; ++s) v = v + xch[((long)s * NT * MB * NB + b) * 64 + lane];
      const int row = m0 + wm + (b / NB) * 16 + (lane & 15), col = n0 + wn + (b % NB) * 16 + 4 * (lane >> 4);
      if (row < g.M && col < g.N) f32_epilogue_store4<EPI, TANH>(g, C, AUX, row, col, v);
    }
  });
}

template <int WGM, int WGN, int MB, int NB, int KS, int NS>
constexpr int f32_lds_bytes() {
  constexpr int ring = NS * (KS / 2) * (16 * WGM * MB + 16 * WGN * NB) / 8 * 1024;
  constexpr int xch = KS * WGM * WGN * MB * NB * 1024;
  return ring > xch ? ring : xch;
}

// The tiles (rows, columns, then the template arguments).  LDS of a CU holds two workgroups of the smaller ones, which
// evens out launches of several rounds (the grouped weight gradients of a 768-wide layer: 156 us against 192 with one).
#define RAF_F32_TILES(X)                                          \
  X(64, 192, 2, 2, 2, 6, 2, 3) X(64, 144, 2, 1, 2, 9, 4, 2)       \
  X(64, 96, 2, 2, 2, 3, 2, 3) X(64, 64, 2, 2, 2, 2, 2, 3)         \
  X(64, 48, 2, 1, 2, 3, 4, 2) X(32, 32, 1, 1, 2, 2, 8, 2)

template <int WGM, int WGN, int MB, int NB, int KS, int NS, bool AK, bool BK>
__global__ __launch_bounds__(64 * WGM * WGN * KS) void gemm_f32_kernel(GemmDev g, int tiles_m, int tiles_n, int remap) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  const int ntile = tiles_m * tiles_n;
  const int per = (ntile + 7) >> 3;
  // one large problem: XCD x takes tiles [x*per, (x+1)*per), so that tiles that share operand panels meet in one L2
  const int t = remap ? (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3) : (int)blockIdx.x;
  if (t >= ntile) return;
  f32_tile<WGM, WGN, MB, NB, KS, NS, AK, BK>(g, (t / tiles_n) * 16 * WGM * MB, (t % tiles_n) * 16 * WGN * NB,
                                             (int)blockIdx.y, lds);
}

// up to four problems of the weight-gradient layout (both operands MN-major) in one launch
template <int WGM, int WGN, int MB, int NB, int KS, int NS>
__global__ __launch_bounds__(64 * WGM * WGN * KS) void gemm_f32_group_kernel(GemmGroupDev grp) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  const int ntile = grp.tile_start[grp.count];
  const int per = (ntile + 7) >> 3;
  const int t = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
  if (t >= ntile) return;
  // the problem is selected with static indices (a run-time index would copy the descriptors to scratch memory)
  GemmDev g = grp.p[0];
  int lt = t, tn = grp.tiles_n[0];
#pragma unroll
  for (int q = 1; q < GEMM_GROUP_MAX; ++q)
    if (q < grp.count && t >= grp.tile_start[q]) {
      g = grp.p[q];
      lt = t - grp.tile_start[q];
      tn = grp.tiles_n[q];
    }
  f32_tile<WGM, WGN, MB, NB, KS, NS, false, false>(g, (lt / tn) * 16 * WGM * MB, (lt % tn) * 16 * WGN * NB, 0, lds);
}

constexpr int F32_CUS = 256;
struct F32Tile { int bm, bn; };
#define RAF_F32_TILE_DIM(BM, BN, ...) F32Tile{BM, BN},
static const F32Tile f32_tiles[] = {RAF_F32_TILES(RAF_F32_TILE_DIM)};
#undef RAF_F32_TILE_DIM
constexpr int F32_NTILES = sizeof(f32_tiles) / sizeof(f32_tiles[0]);

// Every CU works through ceil(tiles / 256) tiles; per 64 contraction values a tile costs its MFMAs (area / 2 clocks) and
// its direct loads (6 clocks per operand row, see above).  The smallest total wins, ties go to the larger tile.  A tile
// that hangs over the edge costs its whole area, which the count takes care of.
static int f32_tile_choice(const GemmDev* ds, int count, int batch) {
  int best = 0;
  long best_cost = 0, best_area = 0;
  for (int i = 0; i < F32_NTILES; ++i) {
    const long area = (long)f32_tiles[i].bm * f32_tiles[i].bn;
    long tiles = 0;
    for (int p = 0; p < count; ++p)
      tiles += (long)((ds[p].M + f32_tiles[i].bm - 1) / f32_tiles[i].bm) * ((ds[p].N + f32_tiles[i].bn - 1) / f32_tiles[i].bn);
    const long cost = (tiles * batch + F32_CUS - 1) / F32_CUS * (area / 2 + 6 * (f32_tiles[i].bm + f32_tiles[i].bn));
    if (i == 0 || cost < best_cost || (cost == best_cost && area > best_area)) {
      best = i;
      best_cost = cost;
      best_area = area;
    }
  }
  return best;
}

template <int WGM, int WGN, int MB, int NB, int KS, int NS, bool AK, bool BK>
static bool launch_f32_inst(const GemmDev& d, int batch, hipStream_t st) {
  constexpr int LDS_BYTES = f32_lds_bytes<WGM, WGN, MB, NB, KS, NS>();
  static_assert(LDS_BYTES <= 160 * 1024, "tile exceeds the LDS of a CU");
  auto kern = gemm_f32_kernel<WGM, WGN, MB, NB, KS, NS, AK, BK>;
  static LdsLimitOnce lds_limit;   // per instantiation
  if (!lds_limit.ensure((const void*)kern, LDS_BYTES)) return false;
  const int tiles_m = (d.M + 16 * WGM * MB - 1) / (16 * WGM * MB), tiles_n = (d.N + 16 * WGN * NB - 1) / (16 * WGN * NB);
  const int ntile = tiles_m * tiles_n, remap = batch == 1 ? 1 : 0;
  hipLaunchKernelGGL(kern, dim3(remap ? ((ntile + 7) / 8) * 8 : ntile, batch), dim3(64 * WGM * WGN * KS), LDS_BYTES, st, d,
                     tiles_m, tiles_n, remap);
  return true;
}

template <int WGM, int WGN, int MB, int NB, int KS, int NS>
static bool launch_f32_layout(const GemmDev& d, int a_kmajor, int b_kmajor, int batch, hipStream_t st) {
  if (a_kmajor && b_kmajor) return launch_f32_inst<WGM, WGN, MB, NB, KS, NS, true, true>(d, batch, st);
  if (a_kmajor) return launch_f32_inst<WGM, WGN, MB, NB, KS, NS, true, false>(d, batch, st);
  if (b_kmajor) return launch_f32_inst<WGM, WGN, MB, NB, KS, NS, false, true>(d, batch, st);
  return launch_f32_inst<WGM, WGN, MB, NB, KS, NS, false, false>(d, batch, st);
}

// Where the LDS limit of the chosen tile cannot be raised, the 64x96 one runs, which needs no raised limit.
#define RAF_F32_FALLBACK 2, 2, 2, 3, 2, 3
static_assert(f32_lds_bytes<RAF_F32_FALLBACK>() <= LDS_LIMIT_UNRAISED, "the fallback tile needs a raised LDS limit");

bool launch_gemm_f32(const GemmDev& d, int a_kmajor, int b_kmajor, int batch, hipStream_t st) {
  const F32Tile t = f32_tiles[f32_tile_choice(&d, 1, batch)];
#define RAF_F32_CASE(BM, BN, WGM, WGN, MB, NB, KS, NS) \
  if (t.bm == BM && t.bn == BN && launch_f32_layout<WGM, WGN, MB, NB, KS, NS>(d, a_kmajor, b_kmajor, batch, st)) return true;
  RAF_F32_TILES(RAF_F32_CASE)
#undef RAF_F32_CASE
  return launch_f32_layout<RAF_F32_FALLBACK>(d, a_kmajor, b_kmajor, batch, st);
}

template <int WGM, int WGN, int MB, int NB, int KS, int NS>
static bool launch_f32_group_inst(const GemmDev* ds, int count, hipStream_t st) {
  constexpr int BM = 16 * WGM * MB, BN = 16 * WGN * NB, LDS_BYTES = f32_lds_bytes<WGM, WGN, MB, NB, KS, NS>();
  auto kern = gemm_f32_group_kernel<WGM, WGN, MB, NB, KS, NS>;
  static LdsLimitOnce lds_limit;   // per instantiation
  if (!lds_limit.ensure((const void*)kern, LDS_BYTES)) return false;
  GemmGroupDev grp{};
  grp.count = count;
  int tiles = 0;
  for (int i = 0; i < count; ++i) {
    grp.p[i] = ds[i];
    grp.tile_start[i] = tiles;
    grp.tiles_n[i] = (ds[i].N + BN - 1) / BN;
    tiles += ((ds[i].M + BM - 1) / BM) * grp.tiles_n[i];
  }
  for (int i = count; i <= GEMM_GROUP_MAX; ++i) grp.tile_start[i] = tiles;
  for (int i = count; i < GEMM_GROUP_MAX; ++i) { grp.p[i] = grp.p[0]; grp.tiles_n[i] = 1; }
  hipLaunchKernelGGL(kern, dim3(((tiles + 7) / 8) * 8), dim3(64 * WGM * WGN * KS), LDS_BYTES, st, grp);
  return true;
}

bool launch_gemm_f32_group(const GemmDev* ds, int count, hipStream_t st) {
  if (count <= 0 || count > GEMM_GROUP_MAX) return false;
  const F32Tile t = f32_tiles[f32_tile_choice(ds, count, 1)];
#define RAF_F32_CASE(BM, BN, WGM, WGN, MB, NB, KS, NS) \
  if (t.bm == BM && t.bn == BN && launch_f32_group_inst<WGM, WGN, MB, NB, KS, NS>(ds, count, st)) return true;
  RAF_F32_TILES(RAF_F32_CASE)
#undef RAF_F32_CASE
  return launch_f32_group_inst<RAF_F32_FALLBACK>(ds, count, st);
}

}  // namespace raf
