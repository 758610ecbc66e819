// Pipelined bf16 MFMA GEMM for gfx950: operand tiles go from global memory
// straight into LDS (global_load_lds, 16 bytes per lane) through an NS-stage
// ring, so several k-steps of loads are in flight while the matrix cores work
// on the oldest stage; one workgroup barrier per k-step.
//
// LDS layout (no padding is possible with direct loads: one instruction fills
// 1 KiB contiguously, 16 bytes per lane, so bank conflicts are avoided by
// permuting which global 16-byte chunk each lane fetches):
//   K-major tile  [ROWS][64]  : chunk c of row r sits at position c ^ ((r>>1)&7)
//   MN-major tile [64][ROWS]  : chunk cc of k-row k sits at position cc ^ ((k&3)<<2)
// K-major fragments are read with ds_read_b128, MN-major ones with the
// transposing ds_read_b64_tr_b16.
#include "gemm_device.hpp"

namespace raf {

constexpr int PBK = 64;

template <int ROWS, bool KMAJOR, int NW>
struct PipeTile {
  static constexpr int BYTES = ROWS * PBK * 2;
  static constexpr int LOADS = BYTES / 1024 / NW;       // direct-load instructions per wave per stage
  static_assert(LOADS >= 1 && LOADS * NW * 1024 == BYTES, "tile must split evenly over the waves");
  static constexpr int CPR = KMAJOR ? 8 : ROWS / 8;     // 16-byte chunks per LDS row
  static __device__ __forceinline__ int swz_k(int r) { return (r >> 1) & 7; }
  static __device__ __forceinline__ int swz_mn(int k) { return CPR >= 16 ? ((k & 3) << 2) : ((k & 1) << 2); }
};

typedef __attribute__((address_space(3))) void* lds_void_ptr;

// per-lane global source addresses of this wave's direct loads for k-step 0
template <int ROWS, bool KMAJOR, int NW>
__device__ __forceinline__ void pipe_src_init(const bf16_t* base, long ld, int row0, int nrows,
                                              const bf16_t* (&src)[PipeTile<ROWS, KMAJOR, NW>::LOADS], int wave) {
  typedef PipeTile<ROWS, KMAJOR, NW> PT;
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int i = 0; i < PT::LOADS; ++i) {
    const int q = wave * PT::LOADS + i;       // which KiB of the tile
    if (KMAJOR) {
      const int r = q * 8 + (lane >> 3);
      const int c = (lane & 7) ^ PT::swz_k(r);
      int gr = row0 + r;
      gr = gr < nrows ? gr : nrows - 1;
      src[i] = base + (long)gr * ld + c * 8;
    } else {
      constexpr int RPK = 64 / PT::CPR;       // k-rows per KiB
      const int k = q * RPK + lane / PT::CPR;
      const int cc = (lane % PT::CPR) ^ PT::swz_mn(k);
      int col = row0 + cc * 8;
      col = col < nrows ? col : nrows - 8;
      src[i] = base + (long)k * ld + col;
    }
  }
}

template <int ROWS, bool KMAJOR, int NW>
__device__ __forceinline__ void pipe_issue(const bf16_t* (&src)[PipeTile<ROWS, KMAJOR, NW>::LOADS], long koff,
                                           char* lds_tile, int wave) {
  typedef PipeTile<ROWS, KMAJOR, NW> PT;
#pragma unroll
  for (int i = 0; i < PT::LOADS; ++i) {
    char* dst = lds_tile + (wave * PT::LOADS + i) * 1024;
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src[i] + koff),
                                     (lds_void_ptr)dst, 16, 0, 0);
  }
}

template <int ROWS, bool KMAJOR>
__device__ __forceinline__ bf16x8_t pipe_fragment(const char* lds_tile, int row, int kk) {
  typedef PipeTile<ROWS, KMAJOR, 1> PT;
  const int lane = threadIdx.x & 63;
  if (KMAJOR) {
    const int r = row + (lane & 31);
    const int c = kk * 2 + (lane >> 5);
    return *reinterpret_cast<const bf16x8_t*>(lds_tile + r * 128 + ((c ^ PT::swz_k(r)) << 4));
  } else {
    const int grp = lane >> 4, s = lane & 15;
    const int k = kk * 16 + (grp >> 1) * 8 + (s >> 2);
    const int col = row + (grp & 1) * 16 + (s & 3) * 4;
    const char* p = lds_tile + k * (ROWS * 2) + (((col >> 3) ^ PT::swz_mn(k)) << 4) + (col & 7) * 2;
    typedef s16x4_t __attribute__((address_space(3))) * lds_v4_ptr;
    const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4_ptr)(p));
    const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4_ptr)(p + 4 * ROWS * 2));
    const s16x8_t both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8_t, both);
  }
}

template <int BM, int BN, int WGM, int WGN, bool A_KMAJOR, bool B_KMAJOR, int NS>
__global__ __launch_bounds__(64 * WGM * WGN) void gemm_bf16_pipe_kernel(GemmDev g, int tiles_m, int tiles_n) {
  constexpr int NW = WGM * WGN;
  constexpr int WM = BM / WGM, WN = BN / WGN;
  constexpr int TM = WM / 32, TN = WN / 32;
  static_assert(TM >= 1 && TN >= 1, "wave tile below one MFMA block");
  typedef PipeTile<BM, A_KMAJOR, NW> PA;
  typedef PipeTile<BN, B_KMAJOR, NW> PB;
  constexpr int STAGE_BYTES = PA::BYTES + PB::BYTES;
  constexpr int LPS = PA::LOADS + PB::LOADS;          // loads per wave per stage
  static_assert(NS == 2 || NS == 3, "the waits below leave at most one k-step in flight");
  extern __shared__ __attribute__((aligned(1024))) char lds[];

  // Tile assignment.  Consecutive workgroup ids go round-robin over the 8
  // XCDs (each with its own L2), so XCD x takes the contiguous range
  // [x*per, (x+1)*per) of the row-major tile list: tiles sharing A rows and B
  // columns meet in one L2.
  const int ntile = tiles_m * tiles_n;
  const int per = (ntile + 7) >> 3;
  const int t = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
  if (t >= ntile) return;
  const int m0 = (t / tiles_n) * BM, n0 = (t % tiles_n) * BN;

  const bf16_t* __restrict__ A = (const bf16_t*)g.a;
  const bf16_t* __restrict__ B = (const bf16_t*)g.b;
  bf16_t* __restrict__ C = (bf16_t*)g.c;
  bf16_t* __restrict__ AUX = (bf16_t*)g.aux;

  const int wave = threadIdx.x >> 6;
  const int wm = (wave / WGN) * WM, wn = (wave % WGN) * WN;

  const bf16_t* srca[PA::LOADS];
  const bf16_t* srcb[PB::LOADS];
  pipe_src_init<BM, A_KMAJOR, NW>(A, g.lda, m0, g.M, srca, wave);
  pipe_src_init<BN, B_KMAJOR, NW>(B, g.ldb, n0, g.N, srcb, wave);
  const long stepa = A_KMAJOR ? PBK : (long)PBK * g.lda;
  const long stepb = B_KMAJOR ? PBK : (long)PBK * g.ldb;

  f32x16_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int nk = g.K / PBK;
#pragma unroll
  for (int s = 0; s < NS - 1; ++s) {
    if (s < nk) {
      pipe_issue<BM, A_KMAJOR, NW>(srca, s * stepa, lds + s * STAGE_BYTES, wave);
      pipe_issue<BN, B_KMAJOR, NW>(srcb, s * stepb, lds + s * STAGE_BYTES + PA::BYTES, wave);
    }
  }

  int stage = 0;
  for (int it = 0; it < nk; ++it) {
    // loads of k-steps it+1 .. it+NS-2 may stay in flight; those of k-step `it` must have landed
    const int ahead = nk - 1 - it;
    if (NS == 3 && ahead >= 1) wait_vmcnt<LPS>();
    else wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();   // stage `it` is complete for every wave; stage it-1 is free
    const int nxt = it + NS - 1;
    if (nxt < nk) {
      int ns = stage + NS - 1;
      ns = ns >= NS ? ns - NS : ns;
      pipe_issue<BM, A_KMAJOR, NW>(srca, nxt * stepa, lds + ns * STAGE_BYTES, wave);
      pipe_issue<BN, B_KMAJOR, NW>(srcb, nxt * stepb, lds + ns * STAGE_BYTES + PA::BYTES, wave);
    }
    const char* ta = lds + stage * STAGE_BYTES;
    const char* tb = ta + PA::BYTES;
    // fragment loads run one sub-step ahead of the MFMAs that consume them
    bf16x8_t fa[2][TM], fb[2][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) fa[0][i] = pipe_fragment<BM, A_KMAJOR>(ta, wm + i * 32, 0);
#pragma unroll
    for (int j = 0; j < TN; ++j) fb[0][j] = pipe_fragment<BN, B_KMAJOR>(tb, wn + j * 32, 0);
#pragma unroll
    for (int kk = 0; kk < PBK / 16; ++kk) {
      const int cur = kk & 1, nx = cur ^ 1;
      if (kk + 1 < PBK / 16) {
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[nx][i] = pipe_fragment<BM, A_KMAJOR>(ta, wm + i * 32, kk + 1);
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[nx][j] = pipe_fragment<BN, B_KMAJOR>(tb, wn + j * 32, kk + 1);
      }
      // operands swapped: the MFMA yields the transposed 32x32 block, so a lane
      // holds 4 consecutive output columns per register group
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[cur][j], fa[cur][i], acc[i][j], 0, 0, 0);
    }
    stage = stage + 1 == NS ? 0 : stage + 1;
  }

  // register r of lane l holds output row (l & 31), column 8*(r/4) + 4*(l/32) + r%4 of its 32x32 block
  epilogue_tile32<bf16_t, TM, TN>(g, C, AUX, acc, m0 + wm, n0 + wn);
}

template <int BM, int BN, int WGM, int WGN, bool AK, bool BKM, int NS>
static bool launch_pipe_inst(const GemmDev& d, hipStream_t st) {
  constexpr int NW = WGM * WGN;
  constexpr int LDS_BYTES = NS * (PipeTile<BM, AK, NW>::BYTES + PipeTile<BN, BKM, NW>::BYTES);
  auto kern = gemm_bf16_pipe_kernel<BM, BN, WGM, WGN, AK, BKM, NS>;
  static LdsLimitOnce lds_limit;   // per instantiation
  if (!lds_limit.ensure((const void*)kern, LDS_BYTES)) return false;
  const int tiles_m = (d.M + BM - 1) / BM, tiles_n = (d.N + BN - 1) / BN;
  const int ntile = tiles_m * tiles_n;
  hipLaunchKernelGGL(kern, dim3(((ntile + 7) / 8) * 8), dim3(64 * NW), LDS_BYTES, st, d, tiles_m, tiles_n);
  return true;
}

// ---------------------------------------------------------------------------
// Producer/consumer form of the ring for a group of problems (the four weight
// gradients of a layer: long contraction, operands contiguous along M and N).
// A wave is held for roughly a hundred cycles per 1-KiB direct load, so loads
// issued by the computing waves serialise with their MFMAs, and loads that go
// through registers are capped near 16 bytes/clock/CU.  Here NP producer waves
// do nothing but issue the direct-to-LDS loads, NS-1 k-steps ahead, while the
// WGM*WGN consumer waves only read fragments and issue MFMAs.  One workgroup
// barrier per k-step keeps both sides in step: after barrier `it` the consumers
// work on stage it while the producers refill the stage that was just freed
// and then wait until stage it+1 has landed.
//
// The MFMA is the 16x16x32 one: while 32x32x16 MFMAs (twice as long per
// instruction) of one wave run back to back, its SIMD issues no memory or LDS
// instruction of any other wave, so that loads and MFMAs add up; the shorter
// ones overlap with both (probe with computing and loading waves: 239 000 clocks
// for the MFMAs, 141 000 for the loads, together 329 000 to 372 000 with 32x32x16
// and 240 000 with 16x16x32).  The group of a 768-wide layer over 4096 rows went from 76
// to 62 us, 1024-wide 126 to 108 us, 2048-wide 406 to 371 us, bit-identical.  What is
// left: per 64 contraction values a 256x128 tile needs 1024 clocks of MFMA, about
// 900 of LDS (131 KiB read transposed at 210 bytes/clock, 48 written) and 850 of
// direct loads (48 KiB at 57), and takes 1900.  On the 768-wide group fragments read
// across the barrier, two wave groups alternating between reading and computing,
// 128x64 wave tiles and 256x256 tiles (108 of them for 256 CUs) all measured slower
// (66 to 70 us, 64, 141), each with whole stages handed over at a barrier.  Half-tile
// buffers as in the ping-pong kernel below, and the wider groups, whose 256x256 tiles
// would fill the CUs, were not measured.
//
// LDS layout of a [64][ROWS] tile: 16-byte chunk cc of k-row k sits at chunk
// cc ^ wg_swz(k), which spreads the eight k-rows x 32 bytes of half a fragment
// read over all banks.
__device__ __forceinline__ int wg_swz(int k) { return ((k & 3) | (((k >> 3) & 1) << 2)) << 1; }

// per-lane source of KiB chunk q of a [64][ROWS] tile for k-step 0
template <int ROWS>
__device__ __forceinline__ const bf16_t* wg_src(const bf16_t* base, long ld, int col0, int ncols, int q) {
  constexpr int CPR = ROWS / 8;
  static_assert(CPR >= 16, "the swizzle permutes 16 chunks");
  const int n = q * 64 + (threadIdx.x & 63), k = n / CPR;
  int col = col0 + ((n % CPR) ^ wg_swz(k)) * 8;
  col = col < ncols ? col : ncols - 8;
  return base + (long)k * ld + col;
}

// operand fragment of 16 tile columns at col0: lane l holds column l & 15, k values 32*kk + 8*(l >> 4) .. +7
template <int ROWS>
__device__ __forceinline__ bf16x8_t wg_fragment(const char* tile, int col0, int kk) {
  const int lane = threadIdx.x & 63, g = lane >> 4, s = lane & 15;
  const int k = kk * 32 + 8 * g + (s >> 2);
  const int col = col0 + (s & 3) * 4;
  const char* p = tile + k * (ROWS * 2) + (((col >> 3) ^ wg_swz(k)) << 4) + (col & 7) * 2;
  typedef s16x4_t __attribute__((address_space(3))) * lds_v4_ptr;
  const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4_ptr)(p));
  const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4_ptr)(p + 4 * ROWS * 2));   // k + 4: same swizzle
  return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// Side work of the grouped launch: worker w of nworkers takes a contiguous range of the 8-column vectors of the
// (concatenated) column space; its threads are dealt to (vector, row group), every row group sums its rows in
// registers, and the row groups are added in a fixed order through LDS, so the sums are reproducible.
constexpr int SIDE_MAX_SLICES = 64;
__device__ __forceinline__ void colsum_side_worker(const ColsumSide& sd, int w, int nworkers, char* lds) {
  const int nvec0 = sd.cols[0] / 8, total = nvec0 + sd.cols[1] / 8;
  const int per = (total + nworkers - 1) / nworkers;
  const int v0 = w * per;
  const int nv = total - v0 < per ? total - v0 : per;
  if (per > (int)blockDim.x) return;               // uniform over the launch; the host never asks for it
  // few enough row groups that adding them up at the end stays short (1024 of them, one vector per worker, took 20 us)
  int ngroups = (int)blockDim.x / per;
  ngroups = ngroups < SIDE_MAX_SLICES ? ngroups : SIDE_MAX_SLICES;
  const int vec = threadIdx.x % per, rg = threadIdx.x / per;
  const bool active = rg < ngroups && vec < nv;     // nv <= 0: a worker beyond the last vector idles through the barrier
  const int uv = v0 + vec;
  const int j = uv < nvec0 ? 0 : 1;
  const bf16_t* __restrict__ x = sd.x[j] + (long)(j ? uv - nvec0 : uv) * 8;
  const long ld = sd.ld[j];
  float acc[8] = {};
  if (active) {
    long r = rg;
    // eight independent 16-byte loads in flight per lane
    for (; r + 7L * ngroups < sd.rows; r += 8L * ngroups) {
      float v[8][8];
#pragma unroll
      for (int u = 0; u < 8; ++u) Vec8<bf16_t>::load(x + (r + (long)u * ngroups) * ld, v[u]);
#pragma unroll
      for (int u = 0; u < 8; ++u)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] += v[u][e];
    }
    for (; r < sd.rows; r += ngroups) {
      float v[8];
      Vec8<bf16_t>::load(x + r * ld, v);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] += v[e];
    }
  }
  float* red = reinterpret_cast<float*>(lds);   // [ngroups][per * 8]
  if (active) {
#pragma unroll
    for (int e = 0; e < 8; ++e) red[(rg * per + vec) * 8 + e] = acc[e];
  }
  __syncthreads();
  bool bad = false;
  for (int c = threadIdx.x; c < nv * 8; c += blockDim.x) {
    float sum = red[c];
    for (int g = 1; g < ngroups; ++g) sum += red[g * per * 8 + c];
    const int u = v0 + c / 8;
    const int jj = u < nvec0 ? 0 : 1;
    sd.out[jj][(long)(jj ? u - nvec0 : u) * 8 + (c & 7)] = sum;
    bad |= !(sum - sum == 0.f);   // x - x is 0 for finite x and nan for inf and nan
  }
  if (bad && sd.nonfinite) *sd.nonfinite = 1;   // every writer stores the same value
}

// out_k[c] = sum_p partial[p][k][c] for the columns of worker w: threads are dealt to (column, slice of the partial
// rows), slices are added in a fixed order through LDS
__device__ __forceinline__ void reduce_side_worker(const ReduceJob& job, int w, int nworkers, char* lds, int* nonfinite) {
  const int chunk = (job.width_out + nworkers - 1) / nworkers;
  const int c0 = w * chunk;
  const int nc = job.width_out - c0 < chunk ? job.width_out - c0 : chunk;
  float* red = reinterpret_cast<float*>(lds);   // [nslices][chunk]
  const bool fits = chunk <= (int)blockDim.x;
  int nslices = fits ? (int)blockDim.x / chunk : 1;
  nslices = nslices < SIDE_MAX_SLICES ? nslices : SIDE_MAX_SLICES;
  const int cl = fits ? threadIdx.x % chunk : 0, slice = fits ? threadIdx.x / chunk : nslices;
  const long width = (long)job.nout * job.ncols;   // stride between partial rows
  __syncthreads();                                 // the previous user of the LDS buffer is done
  if (nc > 0 && fits && slice < nslices) {
    float acc = 0.f;
    if (cl < nc) {
      // eight loads in flight; rows past the end re-read the last row and are not added
      for (int p = slice; p < job.nparts; p += 8 * nslices) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int q = p + u * nslices;
          v[u] = job.partial[(long)(q < job.nparts ? q : job.nparts - 1) * width + c0 + cl];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) acc += p + u * nslices < job.nparts ? v[u] : 0.f;
      }
    }
    red[slice * chunk + cl] = acc;
  }
  __syncthreads();
  if (nc > 0 && fits && slice == 0 && cl < nc) {
    float sum = 0.f;
    for (int sl = 0; sl < nslices; ++sl) sum += red[sl * chunk + cl];
    const int c = c0 + cl;
    const int k = c / job.ncols;
    int cc = c % job.ncols;
    if (job.perm_nvec > 0) cc = (cc % job.perm_nvec) * 8 + cc / job.perm_nvec;   // partial rows stored element-major
    float* o = k == 0 ? job.o0 : (k == 1 ? job.o1 : job.o2);
    if (o) {
      o[cc] = sum;
      if (nonfinite && !(sum - sum == 0.f)) *nonfinite = 1;
    }
  }
}

template <int BM, int BN, int WGM, int WGN, int NS, int NP>
__global__ __launch_bounds__(64 * (WGM * WGN + NP)) void gemm_bf16_spec_kernel(GemmGroupDev grp, ColsumSide side,
                                                                               int tile_blocks) {
  constexpr int NC = WGM * WGN;
  constexpr int WM = BM / WGM, WN = BN / WGN;
  constexpr int MB = WM / 16, NB = WN / 16;
  static_assert(NS >= 3, "the producers need a stage to fill while one is read and one is in flight");
  constexpr int ACH = BM / 8, BCH = BN / 8;            // KiB per operand tile
  constexpr int STAGE_BYTES = (ACH + BCH) * 1024;
  static_assert(ACH % NP == 0 && BCH % NP == 0 && NP % 2 == 0, "loads split evenly; half of the producers load half the k-rows");
  constexpr int LA = ACH / NP, LB = BCH / NP, LPS = LA + LB;   // loads per producer wave per stage
  extern __shared__ __attribute__((aligned(1024))) char lds[];

  if ((int)blockIdx.x >= tile_blocks) {   // a workgroup without a tile: column sums on a CU that the tiles leave idle
    const int w = (int)blockIdx.x - tile_blocks, nworkers = (int)gridDim.x - tile_blocks;
    colsum_side_worker(side, w, nworkers, lds);
    // static indices: a run-time index would copy the descriptors to scratch memory
    if (side.nred > 0) reduce_side_worker(side.red[0], w, nworkers, lds, side.nonfinite);
    if (side.nred > 1) reduce_side_worker(side.red[1], w, nworkers, lds, side.nonfinite);
    if (side.nred > 2) reduce_side_worker(side.red[2], w, nworkers, lds, side.nonfinite);
    return;
  }
  const int ntile = grp.tile_start[grp.count];
  const int per = (ntile + 7) >> 3;
  const int t = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);   // XCD x takes tiles [x*per, (x+1)*per)
  if (t >= ntile) return;
  // the problem is selected with static indices (a run-time index would copy the descriptors to scratch memory)
  GemmDev g = grp.p[0];
  int lt = t, tn = grp.tiles_n[0], tmf = grp.tiles_m_first[0];
#pragma unroll
  for (int q = 1; q < GEMM_GROUP_MAX; ++q)
    if (q < grp.count && t >= grp.tile_start[q]) {
      g = grp.p[q];
      lt = t - grp.tile_start[q];
      tn = grp.tiles_n[q];
      tmf = grp.tiles_m_first[q];
    }
  const int m0 = (tmf ? lt % tmf : lt / tn) * BM, n0 = (tmf ? lt / tmf : lt % tn) * BN;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // a contraction that ends in the middle of a k-step: its second half is neither loaded nor used
  const int nk = (g.K + PBK - 1) / PBK;
  const bool half_last = g.K % PBK != 0;

  if (wave >= NC) {
    // ------------------------------------------------------------ producer
    const int pw = wave - NC;
    const bf16_t* srca[LA];
    const bf16_t* srcb[LB];
#pragma unroll
    for (int i = 0; i < LA; ++i) srca[i] = wg_src<BM>((const bf16_t*)g.a, g.lda, m0, g.M, pw * LA + i);
#pragma unroll
    for (int i = 0; i < LB; ++i) srcb[i] = wg_src<BN>((const bf16_t*)g.b, g.ldb, n0, g.N, pw * LB + i);
    const long stepa = (long)PBK * g.lda, stepb = (long)PBK * g.ldb;
    // chunks are dealt in order, so producers 0 .. NP/2-1 load k-rows 0 .. 31 of both tiles
    const bool in_last = !half_last || pw < NP / 2;
    auto issue = [&](int it, int slot) {
      if (it == nk - 1 && !in_last) return;
      char* base = lds + slot * STAGE_BYTES;
#pragma unroll
      for (int i = 0; i < LA; ++i)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(srca[i] + it * stepa),
                                         (lds_void_ptr)(base + (pw * LA + i) * 1024), 16, 0, 0);
#pragma unroll
      for (int i = 0; i < LB; ++i)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(srcb[i] + it * stepb),
                                         (lds_void_ptr)(base + (ACH + pw * LB + i) * 1024), 16, 0, 0);
    };
#pragma unroll
    for (int s = 0; s < NS - 1; ++s)
      if (s < nk) issue(s, s);
    int stage = 0;
    for (int it = 0; it < nk; ++it) {
      // k-steps it+1 .. it+NS-2 may stay in flight; k-step `it` must have landed
      int ahead = nk - 1 - it < NS - 2 ? nk - 1 - it : NS - 2;
      if (it + ahead == nk - 1 && !in_last) ahead = ahead > 0 ? ahead - 1 : 0;   // the last stage has no load of this wave
      wait_vmcnt_dyn(ahead * LPS);
      __builtin_amdgcn_s_barrier();   // stage `it` handed to the consumers; stage it-1 is free
      const int nxt = it + NS - 1;
      if (nxt < nk) {
        int ns = stage + NS - 1;
        ns = ns >= NS ? ns - NS : ns;
        issue(nxt, ns);
      }
      stage = stage + 1 == NS ? 0 : stage + 1;
    }
    return;
  }

  // -------------------------------------------------------------- consumer
  const int wm = (wave / WGN) * WM, wn = (wave % WGN) * WN;
  f32x4_t acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  int stage = 0;
  for (int it = 0; it < nk; ++it) {
    __builtin_amdgcn_s_barrier();   // stage `it` is complete
    const char* ta = lds + stage * STAGE_BYTES;
    const char* tb = ta + ACH * 1024;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      if (kk == 1 && half_last && it == nk - 1) break;
      bf16x8_t fa[MB], fb[NB];
#pragma unroll
      for (int i = 0; i < MB; ++i) fa[i] = wg_fragment<BM>(ta, wm + i * 16, kk);
#pragma unroll
      for (int j = 0; j < NB; ++j) fb[j] = wg_fragment<BN>(tb, wn + j * 16, kk);
      // operands swapped: a lane ends with output row (l & 15) and 4 consecutive columns 4*(l>>4) + r
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
    }
    stage = stage + 1 == NS ? 0 : stage + 1;
  }

  if (side.nonfinite) {
    // non-finite test of the weight gradients while they are still in registers (rows and columns past the edge of a
    // ragged tile repeat operand rows that also feed real outputs, so they raise the flag only when those do)
    bool bad = false;
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) bad |= !(acc[i][j][r] - acc[i][j][r] == 0.f);
    if (bad) *side.nonfinite = 1;   // every writer stores the same value
  }
  // every consumer has passed the last barrier, so the stage after the last one is read by nobody and no load is in
  // flight to it: each wave stages its blocks in a slice of it
  static_assert(NC * epilogue_stage_f32_bytes<NB>() <= STAGE_BYTES, "staging exceeds a ring stage");
  epilogue_tile16_f32<MB, NB>(g, (float*)g.c, acc, m0 + wm, n0 + wn,
                              lds + stage * STAGE_BYTES + wave * epilogue_stage_f32_bytes<NB>());
}

bool launch_gemm_group_spec(const GemmDev* ds, int count, hipStream_t st, const ColsumSide* side, bool* side_taken) {
  constexpr int BM = 256, BN = 128, WGM = 4, WGN = 2, NS = 3, NP = 8;
  if (side_taken) *side_taken = false;
  if (!ds || count <= 0 || count > GEMM_GROUP_MAX) return false;
  GemmGroupDev grp;
  grp.count = count;
  int tiles = 0;
  for (int i = 0; i < count; ++i) {
    if (ds[i].K % 32 || ds[i].M < 8 || ds[i].N < 8 || (ds[i].M % 8) || (ds[i].N % 8)) return false;
    grp.p[i] = ds[i];
    grp.tile_start[i] = tiles;
    grp.tiles_n[i] = (ds[i].N + BN - 1) / BN;
    const int tiles_m = (ds[i].M + BM - 1) / BM;
    // Each XCD takes a contiguous share of the tile list and its L2 fetches every operand panel its tiles touch:
    // numbering the tiles along the side with fewer tiles first keeps the panels of the long side to one XCD each
    // (the 768 x 3072 gradient: 3 x 24 tiles, 78 -> 42 MB of L2 fills).
    grp.tiles_m_first[i] = tiles_m < grp.tiles_n[i] ? tiles_m : 0;
    tiles += tiles_m * grp.tiles_n[i];
  }
  for (int i = count; i <= GEMM_GROUP_MAX; ++i) grp.tile_start[i] = tiles;
  for (int i = count; i < GEMM_GROUP_MAX; ++i) { grp.p[i] = grp.p[0]; grp.tiles_n[i] = 1; grp.tiles_m_first[i] = 0; }
  constexpr int LDS_BYTES = NS * (BM + BN) * PBK * 2;
  static_assert(LDS_BYTES <= 160 * 1024, "ring exceeds the LDS of a CU");
  auto kern = gemm_bf16_spec_kernel<BM, BN, WGM, WGN, NS, NP>;
  static LdsLimitOnce lds_limit;   // per instantiation
  if (!lds_limit.ensure((const void*)kern, LDS_BYTES)) return false;
  const int tile_blocks = ((tiles + 7) / 8) * 8;
  // Side workers come last in the grid and so take the CUs that the last round of tiles leaves free (one workgroup per
  // CU: the ring takes most of the LDS).
  ColsumSide sd{};
  int workers = 0;
  if (side && side->count > 0) {
    constexpr int NUM_CUS = 256, THREADS = 64 * (WGM * WGN + NP);
    const int total_vecs = (side->cols[0] + side->cols[1]) / 8;
    const int last_round = tile_blocks % NUM_CUS;
    const int free_cus = last_round ? NUM_CUS - last_round : 0;
    if (total_vecs > 0) {
      // Per row of the contraction a worker reads per*16 bytes through registers (about 16 bytes/clock/CU: `per` clocks)
      // while a tile needs about 30 clocks.  Where the free CUs cannot take the sums in a tile's time, all CUs take them
      // after their tiles: at 7 vectors each for the 2048-wide layer 13 us, against 32 us for two launches of their own.
      const bool on_free = free_cus > 0 && (total_vecs + free_cus - 1) / free_cus <= 24;
      const int most = on_free ? free_cus : NUM_CUS;
      const int nw = most < total_vecs ? most : total_vecs;
      const int per = (total_vecs + nw - 1) / nw;
      bool red_ok = side->nred >= 0 && side->nred <= 3;
      for (int i = 0; red_ok && i < side->nred; ++i)
        red_ok = side->red[i].partial && side->red[i].nparts > 0 && side->red[i].ncols > 0 &&
                 side->red[i].nout >= 1 && side->red[i].nout <= 3 && side->red[i].width_out > 0 &&
                 (side->red[i].width_out + nw - 1) / nw <= THREADS;
      if (per <= THREADS && red_ok && (long)(THREADS / per) * per * 32 <= LDS_BYTES) {
        sd = *side;
        workers = nw;
        if (side_taken) *side_taken = true;
      }
    }
  }
  dim3 grid(tile_blocks + workers);
  hipLaunchKernelGGL(kern, grid, dim3(64 * (WGM * WGN + NP)), LDS_BYTES, st, grp, sd, tile_blocks);
  return true;
}

// ---------------------------------------------------------------------------
// Tiles of 64*WGM x 48*WGN outputs for K-major operands.  The widths 48, 96,
// 144 and 192 let the launcher pick a tile count that fills the 256 CUs in
// whole rounds when 128-wide tiles would leave most of the last round idle
// (N = 2304: 16 x 16 tiles of 256x144, one per CU, instead of 576 of 128x128),
// and the tall variants halve the bytes fetched per flop, which is what bounds
// these kernels (direct loads deliver at most about 52 bytes/clock/CU).  Each of the
// WGM x WGN wavefronts owns 64 x 48 outputs as 4 x 3 blocks of
// v_mfma_f32_16x16x32_bf16.  Same direct-to-LDS ring and swizzle as above, NS
// stages deep; the KiB chunks of a stage are dealt round-robin to the waves, so
// some waves issue one load more than others and each wave counts its own.
template <int CHUNKS, int NW>
__device__ __forceinline__ void w48_src_init(const bf16_t* base, long ld, int row0, int nrows, int first,
                                             const bf16_t* (&src)[(CHUNKS + NW - 1) / NW + 1]) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
  for (int i = 0; i < (CHUNKS + NW - 1) / NW + 1; ++i) {
    int q = i * NW + wave - first;            // which KiB (8 rows) of the tile
    q = q < 0 ? 0 : (q < CHUNKS ? q : CHUNKS - 1);   // out-of-range slots keep a valid address they never use
    const int r = q * 8 + (lane >> 3);
    const int c = (lane & 7) ^ ((r >> 1) & 7);
    int gr = row0 + r;
    gr = gr < nrows ? gr : nrows - 1;
    src[i] = base + (long)gr * ld + c * 8;
  }
}

// `first` shifts the dealing so that the B chunks continue where the A chunks stopped
__device__ __forceinline__ int kmajor_tail_shift(int q);
template <int CHUNKS, int NW>
__device__ __forceinline__ void w48_issue(const bf16_t* (&src)[(CHUNKS + NW - 1) / NW + 1], long koff, char* lds_tile,
                                          int first, bool tail) {
  const int wave = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < (CHUNKS + NW - 1) / NW + 1; ++i) {
    const int q = i * NW + wave - first;
    if (q >= 0 && q < CHUNKS)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src[i] + (tail ? koff + kmajor_tail_shift(q) : koff)),
                                       (lds_void_ptr)(lds_tile + q * 1024), 16, 0, 0);
  }
}

// A contraction that ends in the middle of a k-step: in the last step the lanes whose 16-byte chunk lies in its second
// half fetch the chunk half a step earlier instead (a valid address), and that half is not used.  q: KiB of the tile.
__device__ __forceinline__ int kmajor_tail_shift(int q) {
  return ((threadIdx.x & 4) != 0) == ((q & 1) == 0) ? -(PBK / 2) : 0;   // chunk (l & 7) ^ ((r >> 1) & 7), r = 8 q + l / 8
}

// 16 rows x 32 contraction values of a K-major tile: lane l holds row l&15, elements 8*(l>>4) .. +7 of k-half kk
__device__ __forceinline__ bf16x8_t w48_fragment(const char* lds_tile, int row0, int kk) {
  const int lane = threadIdx.x & 63;
  const int r = row0 + (lane & 15);
  const int c = kk * 4 + (lane >> 4);
  return *reinterpret_cast<const bf16x8_t*>(lds_tile + r * 128 + ((c ^ ((r >> 1) & 7)) << 4));
}

// 16 (4 x 4) symmetric wavefronts: each loads, reads and multiplies in turn.
// HALF: the contraction ends in the middle of a k-step.  A template parameter: the test for the last step in the loops
// costs the shapes without one 3 to 12 % (256x192 tiles, 4096 x 6144 x 2048: 116 -> 130 us).
template <int WGM, int WGN, int NS, bool HALF>
__global__ __launch_bounds__(64 * WGM * WGN) void gemm_bf16_w48_kernel(GemmDev g, int tiles_m, int tiles_n) {
  constexpr int NB = 3, NW = WGM * WGN, BM = 64 * WGM, BN = 16 * NB * WGN;
  constexpr int ACH = BM / 8, BCH = BN / 8;           // KiB per operand tile
  constexpr int STAGE_BYTES = (ACH + BCH) * 1024;
  constexpr int BFIRST = ACH % NW;                    // wave that takes B chunk 0
  extern __shared__ __attribute__((aligned(1024))) char lds[];

  const int ntile = tiles_m * tiles_n;
  const int per = (ntile + 7) >> 3;
  const int t = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);   // XCD x takes tiles [x*per, (x+1)*per)
  if (t >= ntile) return;
  const int m0 = (t / tiles_n) * BM, n0 = (t % tiles_n) * BN;

  const bf16_t* __restrict__ A = (const bf16_t*)g.a;
  const bf16_t* __restrict__ B = (const bf16_t*)g.b;
  bf16_t* __restrict__ C = (bf16_t*)g.c;
  bf16_t* __restrict__ AUX = (bf16_t*)g.aux;

  const int wave = threadIdx.x >> 6;
  const int wm = (wave / WGN) * 64, wn = (wave % WGN) * 16 * NB;

  const bf16_t* srca[(ACH + NW - 1) / NW + 1];
  const bf16_t* srcb[(BCH + NW - 1) / NW + 1];
  w48_src_init<ACH, NW>(A, g.lda, m0, g.M, 0, srca);
  w48_src_init<BCH, NW>(B, g.ldb, n0, g.N, BFIRST, srcb);
  // loads this wave issues per stage: chunk f of the ACH+BCH goes to wave f % NW
  const int my_loads = (ACH + BCH) / NW + (wave < (ACH + BCH) % NW ? 1 : 0);

  f32x4_t acc[4][NB];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  const int nk = HALF ? g.K / PBK + 1 : g.K / PBK;
#pragma unroll
  for (int s = 0; s < NS - 1; ++s)
    if (s < nk) {
      w48_issue<ACH, NW>(srca, (long)s * PBK, lds + s * STAGE_BYTES, 0, HALF && s == nk - 1);
      w48_issue<BCH, NW>(srcb, (long)s * PBK, lds + s * STAGE_BYTES + ACH * 1024, BFIRST, HALF && s == nk - 1);
    }
  int stage = 0;
  for (int it = 0; it < nk; ++it) {
    // k-steps it+1 .. it+NS-2 may stay in flight; k-step `it` must have landed
    const int ahead = nk - 1 - it < NS - 2 ? nk - 1 - it : NS - 2;
    wait_vmcnt_dyn(ahead * my_loads);
    __builtin_amdgcn_s_barrier();   // stage `it` is complete for every wave; stage it-1 is free
    if (it + NS - 1 < nk) {
      int ns = stage + NS - 1;
      ns = ns >= NS ? ns - NS : ns;
      char* nxt = lds + ns * STAGE_BYTES;
      const bool tail = HALF && it + NS - 1 == nk - 1;
      w48_issue<ACH, NW>(srca, (long)(it + NS - 1) * PBK, nxt, 0, tail);
      w48_issue<BCH, NW>(srcb, (long)(it + NS - 1) * PBK, nxt + ACH * 1024, BFIRST, tail);
    }
    const char* ta = lds + stage * STAGE_BYTES;
    const char* tb = ta + ACH * 1024;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      if (kk == 1 && HALF && it == nk - 1) break;   // no second half
      bf16x8_t fa[4], fb[NB];
#pragma unroll
      for (int i = 0; i < 4; ++i) fa[i] = w48_fragment(ta, wm + i * 16, kk);
#pragma unroll
      for (int j = 0; j < NB; ++j) fb[j] = w48_fragment(tb, wn + j * 16, kk);
      // operands swapped: a lane ends with output row (l & 15) and 4 consecutive columns 4*(l>>4) + r
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
    }
    stage = stage + 1 == NS ? 0 : stage + 1;
  }

  // wave-private LDS for the staged epilogue: a slice of the ring stage that nobody reads any more (every wave has passed
  // the last barrier, so all reads of the stage before the last one are done and no load is in flight); waves whose slice
  // does not fit that stage any more take one behind the ring (w48_stage_spill)
  constexpr int SB = epilogue_stage_bytes<NB>(), FIT = STAGE_BYTES / SB;
  char* stg = wave < FIT ? lds + stage * STAGE_BYTES + wave * SB : lds + NS * STAGE_BYTES + (wave - FIT) * SB;
  if (epilogue_can_stage(g)) epilogue_tile16_staged<NB>(g, C, AUX, acc, m0 + wm, n0 + wn, 0, 4, stg);
  else epilogue_tile16<bf16_t, NB>(g, C, AUX, acc, m0 + wm, n0 + wn, 0, 4);
}

// Same tiles with the waves specialised: NP producer waves only issue the direct-to-LDS loads (a wave is held for
// roughly a hundred cycles per 1-KiB load instruction, so loads issued by the computing waves serialise with their
// MFMAs), the WGM*WGN*KS consumer waves only read fragments and issue MFMAs.  One workgroup barrier per k-step keeps
// both sides in step: after barrier `it` the consumers work on stage it while the producers refill the stage that was
// freed and then wait until stage it+1 has landed.
// KS = 2 doubles the waves of a workgroup without adding LDS traffic: waves w and w + WGM*WGN share one 64x48
// output block, each takes one 32-deep half of every k-step, and the halves are added through LDS at the end (each
// wave of the pair then finishes half of the rows).  For tiles with only 4-8 waves this gives every SIMD a second
// wave to issue MFMAs while the first waits for its LDS fragments.
template <int WGM, int WGN, int NB, int NS, int KS, int NP, typename TC, bool HALF>
__global__ __launch_bounds__(64 * (WGM * WGN * KS + NP)) void gemm_bf16_w48s_kernel(GemmDev g, int tiles_m, int tiles_n) {
  constexpr int NT = WGM * WGN, NC = NT * KS, BM = 64 * WGM, BN = 16 * NB * WGN;
  constexpr int ACH = BM / 8, BCH = BN / 8;           // KiB per operand tile
  constexpr int STAGE_BYTES = (ACH + BCH) * 1024;
  constexpr int BFIRST = ACH % NP;                    // producer that takes B chunk 0
  static_assert(KS == 1 || KS == 2, "one or two waves per output block");
  static_assert(NS >= 2, "one stage is read while another is filled");
  extern __shared__ __attribute__((aligned(1024))) char lds[];

  const int ntile = tiles_m * tiles_n;
  const int per = (ntile + 7) >> 3;
  const int t = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);   // XCD x takes tiles [x*per, (x+1)*per)
  if (t >= ntile) return;
  const int m0 = (t / tiles_n) * BM, n0 = (t % tiles_n) * BN;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int nk = HALF ? g.K / PBK + 1 : g.K / PBK;

  if (wave >= NC) {
    // ------------------------------------------------------------ producer
    const int pw = wave - NC;
    const bf16_t* __restrict__ A = (const bf16_t*)g.a;
    const bf16_t* __restrict__ B = (const bf16_t*)g.b;
    constexpr int LA = (ACH + NP - 1) / NP + 1, LB = (BCH + NP - 1) / NP + 1;
    const bf16_t* srca[LA];
    const bf16_t* srcb[LB];
#pragma unroll
    for (int i = 0; i < LA; ++i) {
      int q = i * NP + pw;
      q = q < ACH ? q : ACH - 1;
      const int r = q * 8 + (lane >> 3);
      int gr = m0 + r;
      gr = gr < g.M ? gr : g.M - 1;
      srca[i] = A + (long)gr * g.lda + (((lane & 7) ^ ((r >> 1) & 7)) << 3);
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
      int q = i * NP + pw - BFIRST;
      q = q < 0 ? 0 : (q < BCH ? q : BCH - 1);
      const int r = q * 8 + (lane >> 3);
      int gr = n0 + r;
      gr = gr < g.N ? gr : g.N - 1;
      srcb[i] = B + (long)gr * g.ldb + (((lane & 7) ^ ((r >> 1) & 7)) << 3);
    }
    const int my_loads = (ACH + BCH) / NP + (pw < (ACH + BCH) % NP ? 1 : 0);
    auto issue = [&](int kstep, int stage) {
      char* base = lds + stage * STAGE_BYTES;
      const long koff = (long)kstep * PBK;
      const bool tail = HALF && kstep == nk - 1;
#pragma unroll
      for (int i = 0; i < LA; ++i) {
        const int q = i * NP + pw;
        if (q < ACH)
          __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(srca[i] + (tail ? koff + kmajor_tail_shift(q) : koff)),
                                           (lds_void_ptr)(base + q * 1024), 16, 0, 0);
      }
#pragma unroll
      for (int i = 0; i < LB; ++i) {
        const int q = i * NP + pw - BFIRST;
        if (q >= 0 && q < BCH)
          __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(srcb[i] + (tail ? koff + kmajor_tail_shift(q) : koff)),
                                           (lds_void_ptr)(base + (ACH + q) * 1024), 16, 0, 0);
      }
    };
#pragma unroll
    for (int s = 0; s < NS - 1; ++s)
      if (s < nk) issue(s, s);
    int stage = 0;
    for (int it = 0; it < nk; ++it) {
      // k-steps it+1 .. it+NS-2 may stay in flight; k-step `it` must have landed
      const int ahead = nk - 1 - it < NS - 2 ? nk - 1 - it : NS - 2;
      wait_vmcnt_dyn(ahead * my_loads);
      __builtin_amdgcn_s_barrier();   // stage `it` handed to the consumers; stage it-1 is free
      if (it + NS - 1 < nk) {
        int ns = stage + NS - 1;
        ns = ns >= NS ? ns - NS : ns;
        issue(it + NS - 1, ns);
      }
      stage = stage + 1 == NS ? 0 : stage + 1;
    }
    if (KS == 2) {   // the consumers' exchange has two more barriers
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_s_barrier();
    }
    return;
  }

  // -------------------------------------------------------------- consumer
  TC* __restrict__ C = (TC*)g.c;
  bf16_t* __restrict__ AUX = (bf16_t*)g.aux;
  const int wt = wave % NT, kg = wave / NT;           // output block of this wave, its half of each k-step
  const int wm = (wt / WGN) * 64, wn = (wt % WGN) * 16 * NB;
  f32x4_t acc[4][NB];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  int stage = 0;
  for (int it = 0; it < nk; ++it) {
    __builtin_amdgcn_s_barrier();   // stage `it` is complete
    const char* ta = lds + stage * STAGE_BYTES;
    const char* tb = ta + ACH * 1024;
#pragma unroll
    for (int kh = 0; kh < 2 / KS; ++kh) {
      const int kk = KS == 2 ? kg : kh;
      if (kk == 1 && HALF && it == nk - 1) break;   // no second half
      bf16x8_t fa[4], fb[NB];
#pragma unroll
      for (int i = 0; i < 4; ++i) fa[i] = w48_fragment(ta, wm + i * 16, kk);
#pragma unroll
      for (int j = 0; j < NB; ++j) fb[j] = w48_fragment(tb, wn + j * 16, kk);
      // operands swapped: a lane ends with output row (l & 15) and 4 consecutive columns 4*(l>>4) + r
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
    }
    stage = stage + 1 == NS ? 0 : stage + 1;
  }

  int i_begin = 0, i_end = 4;
  // wave-private LDS for the staged epilogue: with one wave per block a slice of the ring stage that nobody reads
  // any more (every consumer has passed the last barrier, so all reads of the stage before the last one are done,
  // and the producers have no load in flight), with wave pairs the slot this wave received its partner's
  // accumulators in
  // (waves whose slice does not fit that stage any more take one behind the ring: w48_stage_spill)
  constexpr int SB = epilogue_stage_bytes<NB>(), FIT = STAGE_BYTES / SB;
  static_assert(epilogue_stage_bytes<NB>() <= 2 * NB * 64 * 16, "staging exceeds an exchange slot");
  char* stg = KS == 2 ? lds + (wt * 2 + kg) * 2 * NB * 64 * 16
                      : (wave < FIT ? lds + stage * STAGE_BYTES + wave * SB : lds + NS * STAGE_BYTES + (wave - FIT) * SB);
  if (KS == 2) {
    // exchange: the wave with kg = 0 finishes row blocks 0-1, its partner row blocks 2-3; each sends the other half
    __builtin_amdgcn_s_barrier();   // every wave is done with the ring
    f32x4_t* xch = reinterpret_cast<f32x4_t*>(lds) + (wt * 2 + (kg ^ 1)) * 2 * NB * 64;   // slot read by the partner
#pragma unroll
    for (int ii = 0; ii < 2; ++ii)
#pragma unroll
      for (int j = 0; j < NB; ++j) xch[(ii * NB + j) * 64 + lane] = kg ? acc[ii][j] : acc[2 + ii][j];   // static indices: no scratch
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0): the writes above have reached LDS
    __builtin_amdgcn_s_barrier();
    const f32x4_t* got = reinterpret_cast<const f32x4_t*>(lds) + (wt * 2 + kg) * 2 * NB * 64;
#pragma unroll
    for (int ii = 0; ii < 2; ++ii)
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const f32x4_t o = got[(ii * NB + j) * 64 + lane];
        // fixed order: first k-half plus second k-half
        if (kg == 0) acc[ii][j] = acc[ii][j] + o;
        else acc[2 + ii][j] = o + acc[2 + ii][j];
      }
    i_begin = kg * 2;
    i_end = i_begin + 2;
  }

  if constexpr (sizeof(TC) == 2) {
    if (epilogue_can_stage(g)) {
      epilogue_tile16_staged<NB>(g, C, AUX, acc, m0 + wm, n0 + wn, i_begin, i_end, stg);
      return;
    }
  }
  epilogue_tile16<TC, NB>(g, C, AUX, acc, m0 + wm, n0 + wn, i_begin, i_end);
}

// LDS behind the ring for the epilogue staging of the waves (of `waves`, one wave per output block) whose slice does
// not fit one ring stage
template <int NB>
constexpr int w48_stage_spill(int stage_bytes, int waves) {
  const int fit = stage_bytes / epilogue_stage_bytes<NB>();
  return waves > fit ? (waves - fit) * epilogue_stage_bytes<NB>() : 0;
}

template <int WGM, int WGN, int NB, int NS, int KS, int NP, typename TC, bool HALF>
static bool launch_w48s_half(const GemmDev& d, hipStream_t st) {
  constexpr int BM = 64 * WGM, BN = 16 * NB * WGN;
  constexpr int RING_BYTES = NS * (BM / 8 + BN / 8) * 1024 +
                             (KS == 1 ? w48_stage_spill<NB>((BM / 8 + BN / 8) * 1024, WGM * WGN) : 0);
  constexpr int XCH_BYTES = KS == 2 ? WGM * WGN * 2 * 2 * NB * 64 * 16 : 0;   // accumulator exchange of the wave pairs
  constexpr int LDS_BYTES = RING_BYTES > XCH_BYTES ? RING_BYTES : XCH_BYTES;
  static_assert(LDS_BYTES <= 160 * 1024, "ring exceeds the LDS of a CU");
  static_assert((NS - 2) * ((BM / 8 + BN / 8 + NP - 1) / NP) <= 24, "in-flight loads exceed wait_vmcnt_dyn");
  static_assert(64 * (WGM * WGN * KS + NP) <= 1024, "workgroup too large");
  auto kern = gemm_bf16_w48s_kernel<WGM, WGN, NB, NS, KS, NP, TC, HALF>;
  static LdsLimitOnce lds_limit;   // per instantiation
  if (!lds_limit.ensure((const void*)kern, LDS_BYTES)) return false;
  const int tiles_m = (d.M + BM - 1) / BM, tiles_n = (d.N + BN - 1) / BN;
  const int ntile = tiles_m * tiles_n;
  dim3 grid(((ntile + 7) / 8) * 8);
  hipLaunchKernelGGL(kern, grid, dim3(64 * (WGM * WGN * KS + NP)), LDS_BYTES, st, d, tiles_m, tiles_n);
  return true;
}

template <int WGM, int WGN, int NB, int NS, int KS, int NP, typename TC>
static bool launch_w48s_inst(const GemmDev& d, hipStream_t st) {
  return d.K % PBK ? launch_w48s_half<WGM, WGN, NB, NS, KS, NP, TC, true>(d, st)
                   : launch_w48s_half<WGM, WGN, NB, NS, KS, NP, TC, false>(d, st);
}

template <int WGM, int WGN, int NS, bool HALF>
static bool launch_w48_half(const GemmDev& d, hipStream_t st) {
  constexpr int BM = 64 * WGM, BN = 48 * WGN;
  constexpr int LDS_BYTES = NS * (BM / 8 + BN / 8) * 1024 + w48_stage_spill<3>((BM / 8 + BN / 8) * 1024, WGM * WGN);
  static_assert(LDS_BYTES <= 160 * 1024, "ring exceeds the LDS of a CU");
  static_assert((NS - 2) * ((BM / 8 + BN / 8 + WGM * WGN - 1) / (WGM * WGN)) <= 24, "in-flight loads exceed wait_vmcnt_dyn");
  auto kern = gemm_bf16_w48_kernel<WGM, WGN, NS, HALF>;
  static LdsLimitOnce lds_limit;   // per instantiation
  if (!lds_limit.ensure((const void*)kern, LDS_BYTES)) return false;
  const int tiles_m = (d.M + BM - 1) / BM, tiles_n = (d.N + BN - 1) / BN;
  const int ntile = tiles_m * tiles_n;
  dim3 grid(((ntile + 7) / 8) * 8);
  hipLaunchKernelGGL(kern, grid, dim3(64 * WGM * WGN), LDS_BYTES, st, d, tiles_m, tiles_n);
  return true;
}

template <int WGM, int WGN, int NS>
static bool launch_w48_inst(const GemmDev& d, hipStream_t st) {
  return d.K % PBK ? launch_w48_half<WGM, WGN, NS, true>(d, st) : launch_w48_half<WGM, WGN, NS, false>(d, st);
}

// ---------------------------------------------------------------------------
// Large tiles on eight wavefronts in two groups of four, one of each per SIMD: while one group issues its 16 (12) MFMAs
// of a phase, the other reads the fragments of its next phase from LDS and requests its next operand pieces, and a
// barrier swaps the roles.  A wave tile is split in 2 x 2 quadrants and a k-step in four phases (quadrant 00: reads the
// upper half of the A fragments and the left half of the B ones, 01: the right half of B, 11: the lower half of A, 10:
// nothing), and each half of an operand tile has a buffer of its own in each of the two stages: it is free
// again as soon as its one phase is over, so its next filling is requested ten half-phases (about 1.6 us) before it is
// waited for and the ring needs no third stage.
//
// What bounds it: per k-step a 256x256 tile takes 2048 clocks of MFMA and the loop about 2800; 8192 x 8192 x 8192 runs at
// 1.57 PFLOP/s (699 us; 912 with 16 symmetric wavefronts that read, request and multiply in turn).  Short contractions
// are bound by the fixed part of 8 us: first stages, and an epilogue of all CUs at once.  Measured against the kernels
// that had these shapes (128x128 producer/consumer tiles, 256x192 and 256x256 tiles): 4096 x 6144 x 2048 113.6 -> 86.7
// us, 4096 x 8192 x 2048 125.9 -> 100.2, 4096 x 2048 x 8192 147.8 -> 109.2, 4096 x 2048 x 2048 43.4 -> 33.5, 8192 x 3072 x
// 768 51.9 -> 43.4, 4096 x 4096 x 1024 33.1 -> 30.7, 896 x 30528 x 768 76.5 -> 48.5 (cold operands).  Requests by buffer
// loads (scalar k offset) instead of 64-bit addresses: 8192 x 8192 x 8192 727 -> 699; reading all of a quadrant row's
// fragments in one phase, and waiting for them before the swap: 749.
template <int WGM, int WGN, int MH, int NH>   // waves along M and N, 16x16 blocks of a quadrant along M and N
struct PingPong {
  static constexpr int BM = 32 * MH * WGM, BN = 32 * NH * WGN;
  static constexpr int ACH = BM / 16, BCH = BN / 16;      // KiB (8 rows x 64 values) of half an operand tile
  static constexpr int STAGE = (2 * ACH + 2 * BCH) * 1024;
  static constexpr int LDS_BYTES = 2 * STAGE;
  static_assert(WGM * WGN == 8, "two groups of four wavefronts");
  static_assert(ACH % 8 == 0 && BCH % 4 == 0, "half tiles deal evenly to the wavefronts of a group");
};

template <int WGM, int WGN, int MH, int NH, bool HALF>
__global__ __launch_bounds__(512) void gemm_bf16_pingpong_kernel(GemmDev g, int tiles_m, int tiles_n) {
  typedef PingPong<WGM, WGN, MH, NH> PP;
  constexpr int BM = PP::BM, BN = PP::BN, ACH = PP::ACH, BCH = PP::BCH, STAGE = PP::STAGE;
  constexpr int LA = ACH / 8, LB = (BCH + 7) / 8;        // loads per wavefront of half a tile (B: at most)
  extern __shared__ __attribute__((aligned(1024))) char lds[];

  // XCD x takes tiles [x*per, (x+1)*per) of a list that runs down 4 rows of tiles before it steps to the next column:
  // the 32 tiles that an XCD works on at a time then share 4 + 8 operand panels instead of 1 + 32
  const int ntile = tiles_m * tiles_n;
  const int per = (ntile + 7) >> 3;
  const int t = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
  if (t >= ntile) return;
  const int grp = t / (4 * tiles_n), in_grp = t - grp * 4 * tiles_n;
  const int rows = tiles_m - 4 * grp < 4 ? tiles_m - 4 * grp : 4;
  // (the divisions run in vector registers: back to scalar ones)
  const int m0 = __builtin_amdgcn_readfirstlane((4 * grp + in_grp % rows) * BM);
  const int n0 = __builtin_amdgcn_readfirstlane((in_grp / rows) * BN);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int wr = wave / WGN, wc = wave % WGN;
  const int nk = HALF ? g.K / PBK + 1 : g.K / PBK;

  // Half h of the A tile holds, for every row of waves, the 16 MH rows of quadrant row h; of the B tile likewise.
  // Per-lane source offsets of this wave's KiB pieces (one piece: 8 rows of 128 bytes, chunk c of row r at c ^ ((r >> 1) & 7)).
  // Buffer loads: the k-step is a scalar offset, so a request costs no vector instruction and no address register.
  const int ma = g.M - m0 < BM ? g.M - m0 : BM, mb = g.N - n0 < BN ? g.N - n0 : BN;   // rows of the panels
  const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)g.a + (long)m0 * g.lda * 2), 0,
                                                                      ((ma - 1) * g.lda + g.K) * 2, 0x00020000);
  const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)g.b + (long)n0 * g.ldb * 2), 0,
                                                                      ((mb - 1) * g.ldb + g.K) * 2, 0x00020000);
  uint32_t offa[2][LA], offb[2][LB];
  const int c8 = lane & 7;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
#pragma unroll
    for (int i = 0; i < LA; ++i) {
      const int r = (i * 8 + wave) * 8 + (lane >> 3);    // row within the half
      int row = (r / (16 * MH)) * 32 * MH + h * 16 * MH + r % (16 * MH);
      row = row < ma ? row : ma - 1;
      offa[h][i] = (uint32_t)row * (uint32_t)(g.lda * 2) + ((c8 ^ ((r >> 1) & 7)) << 4);
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
      int q = i * 8 + wave;
      q = q < BCH ? q : BCH - 1;
      const int r = q * 8 + (lane >> 3);
      int row = (r / (16 * NH)) * 32 * NH + h * 16 * NH + r % (16 * NH);
      row = row < mb ? row : mb - 1;
      offb[h][i] = (uint32_t)row * (uint32_t)(g.ldb * 2) + ((c8 ^ ((r >> 1) & 7)) << 4);
    }
  }
  // requests half h of the A (B) tile of k-step `kstep` into stage s = kstep & 1
  auto load_a = [&](int h, int kstep, int s) {
    char* dst = lds + s * STAGE + h * ACH * 1024;
    const bool tail = HALF && kstep == nk - 1;
#pragma unroll
    for (int i = 0; i < LA; ++i) {
      const int q = i * 8 + wave;
      const uint32_t off = tail ? offa[h][i] + 2 * kmajor_tail_shift(q) : offa[h][i];
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_void_ptr)(dst + q * 1024), 16, off, kstep * (PBK * 2), 0, 0);
    }
  };
  auto load_b = [&](int h, int kstep, int s) {
    char* dst = lds + s * STAGE + (2 * ACH + h * BCH) * 1024;
    const bool tail = HALF && kstep == nk - 1;
#pragma unroll
    for (int i = 0; i < LB; ++i) {
      const int q = i * 8 + wave;
      if (i * 8 + 8 <= BCH || q < BCH) {
        const uint32_t off = tail ? offb[h][i] + 2 * kmajor_tail_shift(q) : offb[h][i];
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (lds_void_ptr)(dst + q * 1024), 16, off, kstep * (PBK * 2), 0, 0);
      }
    }
  };

  f32x4_t acc[2][2][MH][NH];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int i = 0; i < MH; ++i)
#pragma unroll
        for (int j = 0; j < NH; ++j) acc[x][y][i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  bf16x8_t fa[2][MH], fb[2][2][NH];     // A: k-half, block; B: column half, k-half, block
  auto read_a = [&](int h, int s) {
    const char* tile = lds + s * STAGE + h * ACH * 1024;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int i = 0; i < MH; ++i) fa[kk][i] = w48_fragment(tile, wr * 16 * MH + i * 16, kk);
  };
  auto read_b = [&](int h, int s) {
    const char* tile = lds + s * STAGE + (2 * ACH + h * BCH) * 1024;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int j = 0; j < NH; ++j) fb[h][kk][j] = w48_fragment(tile, wc * 16 * NH + j * 16, kk);
  };
  auto swap_roles = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
  // The products of quadrant (x, y); the compiler waits for their fragments, whose reads were issued before the swap.  The
  // fourth phase reads for the next k-step (`drain`), and the last k-step of a contraction with half a step leaves
  // fragments unused: no product waits for those reads, so the phase does, before it hands its turn over.  (In every phase
  // the wait costs 0.5 to 1 % on 8192 x 8192 x 8192, 684 against 691 us and 686 against 689 in the other order, and
  // nothing on layer products; half steps take it, which keeps the rule free of a branch.)
  auto products = [&](int x, int y, bool both, bool drain) {
    swap_roles();
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      if (HALF && kk == 1 && !both) break;
      // operands swapped: a lane ends with output row (l & 15) and 4 consecutive columns 4*(l>>4) + r
#pragma unroll
      for (int i = 0; i < MH; ++i)
#pragma unroll
        for (int j = 0; j < NH; ++j)
          acc[x][y][i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[y][kk][j], fa[kk][i], acc[x][y][i][j], 0, 0, 0);
    }
    if (HALF || drain) {
      __builtin_amdgcn_sched_barrier(0);
      lds_reads_done();
    }
    __builtin_amdgcn_s_setprio(0);
    swap_roles();
  };
  // loads of this wave per half tile of B (the second group may have one less)
  const int lb = BCH % 8 ? (wave < BCH % 8 ? LB : LB - 1) : LB;
  auto wait_halves = [&](auto na, auto nb) {   // that many halves of A and of B may stay in flight
    constexpr int NA = decltype(na)::value, NBH = decltype(nb)::value;
    if constexpr (BCH % 8 == 0) wait_vmcnt<NA * LA + NBH * LB>();
    else if (lb == LB) wait_vmcnt<NA * LA + NBH * LB>();
    else wait_vmcnt<NA * LA + NBH * (LB - 1)>();
  };
  constexpr EpiTag<0> n0h{}; constexpr EpiTag<1> n1h{}; constexpr EpiTag<2> n2h{}; constexpr EpiTag<3> n3h{};

  // k-step `it` of parity F.  Quadrants (0,F) (0,1-F) (1,1-F) (1,F): the last phase leaves the registers of B half 1-F
  // free for the fragments that k-step it + 1 starts with, so that no phase reads more than 2 MH fragments.  A half
  // buffer is refilled two phases after the phase that reads it.  A wave's reads have returned before the swap that closes
  // their phase, and the other group runs half a phase apart: a barrier lies between the last return and the request.
  // Order of a wave's requests: B[F] A[0] B[1-F] A[1] of each k-step; every wait leaves the last five (fewer at the end)
  // in flight and is for what the next phase reads.
  auto kstep = [&](auto parity, int it, int rest) {
    constexpr int F = decltype(parity)::value;
    const bool both = !HALF || rest > 0;
    read_a(0, F);
    if (rest >= 1) {
      load_a(1, it + 1, 1 - F);
      wait_halves(n3h, n2h);                    // B[1-F] of this k-step
    } else {
      wait_halves(n1h, n0h);
    }
    products(0, F, both, false);
    read_b(1 - F, F);
    if (rest >= 2) {
      load_b(F, it + 2, F);
      wait_halves(n2h, n3h);                    // A[1]
    } else if (rest == 1) {
      wait_halves(n2h, n2h);
    } else {
      wait_halves(n0h, n0h);
    }
    products(0, 1 - F, both, false);
    read_a(1, F);
    if (rest >= 2) {
      load_a(0, it + 2, F);
      wait_halves(n3h, n2h);                    // B[1-F] of the next k-step
    } else {
      wait_halves(n2h, n1h);
    }
    products(1, 1 - F, both, false);
    if (rest >= 1) read_b(1 - F, 1 - F);
    if (rest >= 2) {
      load_b(1 - F, it + 2, F);
      wait_halves(n2h, n3h);                    // A[0] of the next k-step
    } else {
      wait_halves(n1h, n1h);
    }
    products(1, F, both, true);
  };
  load_b(0, 0, 0); load_a(0, 0, 0); load_b(1, 0, 0); load_a(1, 0, 0);
  load_b(1, 1, 1); load_a(0, 1, 1); load_b(0, 1, 1);
  wait_halves(n2h, n3h);                        // B[0] and A[0] of k-step 0 have landed
  __builtin_amdgcn_s_barrier();
  read_b(0, 0);
  if (wave >= 4) {                              // the second group runs half a phase behind
    lds_reads_done();
    swap_roles();
  }
  __builtin_amdgcn_sched_barrier(0);

  int it = 0;
  for (; it + 3 < nk; it += 2) {                // without the tests for the end
    kstep(n0h, it, 2);
    kstep(n1h, it + 1, 2);
  }
  for (; it < nk; it += 2) {
    kstep(n0h, it, nk - 1 - it);
    if (it + 1 < nk) kstep(n1h, it + 1, nk - 2 - it);
  }
  if (wave < 4) swap_roles();

  // every fragment read and every load of the workgroup is over: the waves stage their blocks in slices of the ring
  constexpr int SB = epilogue_stage_bytes<2 * NH>();
  static_assert(8 * SB <= PP::LDS_BYTES, "staging exceeds the ring");
  char* stg = lds + wave * SB;
  bf16_t* __restrict__ C = (bf16_t*)g.c;
  bf16_t* __restrict__ AUX = (bf16_t*)g.aux;
  const int row0 = m0 + wr * 32 * MH, col0 = n0 + wc * 32 * NH;
  // 64 rows of the wave tile.  Inlined by force: as a function of its own it gets the kernel's state through memory, and
  // branches too far for one instruction use the registers that hold its return address.
  auto band = [&](auto tag) __attribute__((always_inline)) {
    constexpr int I0 = decltype(tag)::value * 4;
    f32x4_t out[4][2 * NH];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 2 * NH; ++j) out[i][j] = acc[(I0 + i) / MH][j / NH][(I0 + i) % MH][j % NH];
    if (epilogue_can_stage(g)) epilogue_tile16_staged<2 * NH>(g, C, AUX, out, row0 + I0 * 16, col0, 0, 4, stg);
    else epilogue_tile16<bf16_t, 2 * NH>(g, C, AUX, out, row0 + I0 * 16, col0, 0, 4);
  };
  static_assert(MH == 2 || MH == 4, "one or two bands");
  band(EpiTag<0>{});
  if constexpr (MH == 4) band(EpiTag<1>{});
}

template <int WGM, int WGN, int MH, int NH, bool HALF>
static bool launch_pingpong_half(const GemmDev& d, hipStream_t st) {
  typedef PingPong<WGM, WGN, MH, NH> PP;
  auto kern = gemm_bf16_pingpong_kernel<WGM, WGN, MH, NH, HALF>;
  static LdsLimitOnce lds_limit;   // per instantiation
  if (!lds_limit.ensure((const void*)kern, PP::LDS_BYTES)) return false;
  const int tiles_m = (d.M + PP::BM - 1) / PP::BM, tiles_n = (d.N + PP::BN - 1) / PP::BN;
  hipLaunchKernelGGL(kern, dim3(((tiles_m * tiles_n + 7) / 8) * 8), dim3(512), PP::LDS_BYTES, st, d, tiles_m, tiles_n);
  return true;
}
template <int WGM, int WGN, int MH, int NH>
static bool launch_pingpong_inst(const GemmDev& d, hipStream_t st) {
  return d.K % PBK ? launch_pingpong_half<WGM, WGN, MH, NH, true>(d, st)
                   : launch_pingpong_half<WGM, WGN, MH, NH, false>(d, st);
}

// ---------------------------------------------------------------------------
// Products with few output tiles (short batches, narrow layers): every wavefront
// of a workgroup computes the whole 16 MB x 16 NB tile over its own share of the
// contraction (k-steps w, w + NW, ...), from a ring of NS stages of its own, so
// there is no barrier until the NW partial tiles meet in LDS.
//
// What bounds it: lines reach a CU at about 62 GB/s when all of them ask for new
// ones, so a tile takes a fixed part plus 32 ps per operand row and contraction
// value, and the tile is made as small as one round over the 256 CUs allows
// (split_tile_choice).  All of a wavefront's stages are requested at the start:
// with 110 to 144 KiB in flight per CU the latency of cold operands is paid once.
// Direct loads to LDS and not register loads of the fragments: a fragment's 16
// lanes touch 16 lines, and the address unit takes a clock for each (16 bytes per
// clock and CU instead of 57).  Against the register-staged 128x128 kernel and the
// rings above, cold operands: 64 x 768 x 3072 49 -> 5.8 us, 64 x 3072 x 768 15.8 ->
// 4.7, 512 x 768 x 3072 27.7 -> 10.7, 1024 x 768 x 3072 28 -> 14.5, 1824 x 768 x 3072 27.8 -> 21.3.
template <int MB, int NB, int NW, int NS, bool HALF>
__global__ __launch_bounds__(64 * NW) void gemm_bf16_split_kernel(GemmDev g, int tiles_m, int tiles_n) {
  constexpr int BM = 16 * MB, BN = 16 * NB, LA = 2 * MB, LB = 2 * NB;   // KiB of A and of B per stage
  constexpr int LPS = LA + LB, STAGE_BYTES = LPS * 1024;
  static_assert((NS - 1) * LPS <= 24, "in-flight loads exceed wait_vmcnt_dyn");
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  const int ntile = tiles_m * tiles_n;
  const int per = (ntile + 7) >> 3;
  const int t = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);   // XCD x takes tiles [x*per, (x+1)*per)
  if (t >= ntile) return;
  // tiles are numbered along M first: the weights (operand B) are the larger one here, and each of their rows is then
  // fetched by one XCD only
  const int m0 = (t % tiles_m) * BM, n0 = (t / tiles_m) * BN;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  char* ring = lds + wave * (NS * STAGE_BYTES);
  const bf16_t* __restrict__ A = (const bf16_t*)g.a;
  const bf16_t* __restrict__ B = (const bf16_t*)g.b;
  const bf16_t* srca[LA];
  const bf16_t* srcb[LB];
#pragma unroll
  for (int q = 0; q < LA; ++q) {
    const int r = q * 8 + (lane >> 3);
    const int gr = m0 + r < g.M ? m0 + r : g.M - 1;
    srca[q] = A + (long)gr * g.lda + (((lane & 7) ^ ((r >> 1) & 7)) << 3);
  }
#pragma unroll
  for (int q = 0; q < LB; ++q) {
    const int r = q * 8 + (lane >> 3);
    const int gr = n0 + r < g.N ? n0 + r : g.N - 1;
    srcb[q] = B + (long)gr * g.ldb + (((lane & 7) ^ ((r >> 1) & 7)) << 3);
  }
  f32x4_t acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  const int nk = HALF ? g.K / PBK + 1 : g.K / PBK;
  const int mine = wave < nk ? (nk - 1 - wave) / NW + 1 : 0;   // k-steps of this wavefront
  auto issue = [&](int i, int slot) {
    const int kstep = wave + i * NW;
    const long koff = (long)kstep * PBK;
    char* base = ring + slot * STAGE_BYTES;
    const bool tail = HALF && kstep == nk - 1;
#pragma unroll
    for (int q = 0; q < LB; ++q)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(srcb[q] + (tail ? koff + kmajor_tail_shift(q) : koff)),
                                       (lds_void_ptr)(base + (LA + q) * 1024), 16, 0, 0);
#pragma unroll
    for (int q = 0; q < LA; ++q)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(srca[q] + (tail ? koff + kmajor_tail_shift(q) : koff)),
                                       (lds_void_ptr)(base + q * 1024), 16, 0, 0);
  };
#pragma unroll
  for (int i = 0; i < NS; ++i)
    if (i < mine) issue(i, i);
  int slot = 0;
  for (int i = 0; i < mine; ++i) {
    const int ahead = mine - 1 - i < NS - 1 ? mine - 1 - i : NS - 1;
    wait_vmcnt_dyn(ahead * LPS);
    asm volatile("" ::: "memory");                       // the stage is read after the wait
    const char* ta = ring + slot * STAGE_BYTES;
    const char* tb = ta + LA * 1024;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      if (kk == 1 && HALF && wave + i * NW == nk - 1) break;   // no second half
      bf16x8_t fa[MB], fb[NB];
#pragma unroll
      for (int x = 0; x < MB; ++x) fa[x] = w48_fragment(ta, x * 16, kk);
#pragma unroll
      for (int y = 0; y < NB; ++y) fb[y] = w48_fragment(tb, y * 16, kk);
      // operands swapped: a lane ends with output row (l & 15) and 4 consecutive columns 4*(l>>4) + r
#pragma unroll
      for (int x = 0; x < MB; ++x)
#pragma unroll
        for (int y = 0; y < NB; ++y)
          acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[y], fa[x], acc[x][y], 0, 0, 0);
    }
    if (i + NS < mine) {
      lds_reads_done();                                  // this wavefront's reads of the stage have returned: refill it
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      issue(i + NS, slot);
    }
    slot = slot + 1 == NS ? 0 : slot + 1;
  }

  // the partial tiles meet in LDS; wavefront w adds blocks w, w + NW, ... in a fixed order and finishes them
  __syncthreads();                                       // every wavefront is done with its ring
  f32x4_t* xch = reinterpret_cast<f32x4_t*>(lds);
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) xch[(wave * MB * NB + i * NB + j) * 64 + lane] = acc[i][j];
  __syncthreads();
  bf16_t* __restrict__ C = (bf16_t*)g.c;
  bf16_t* __restrict__ AUX = (bf16_t*)g.aux;
  epilogue_dispatch(g, [&](auto tag, auto form) {
    constexpr int EPI = decltype(tag)::value, TANH = decltype(form)::value;
    for (int b = wave; b < MB * NB; b += NW) {
      f32x4_t v = xch[b * 64 + lane];
#pragma unroll
      for (int q = 1; q < NW; ++q) v = v + xch[(q * MB * NB + b) * 64 + lane];
      const int row = m0 + (b / NB) * 16 + (lane & 15), col = n0 + (b % NB) * 16 + 4 * (lane >> 4);
      if (row < g.M && col < g.N) {
        float o[4] = {v[0], v[1], v[2], v[3]};
        epilogue_store4<bf16_t, EPI, TANH>(g, C, AUX, row, col, o);
      }
    }
  });
}

template <int MB, int NB, int NW, int NS, bool HALF>
static bool launch_split_half(const GemmDev& d, hipStream_t st) {
  constexpr int RING_BYTES = NW * NS * 2 * (MB + NB) * 1024, XCH_BYTES = NW * MB * NB * 1024;
  constexpr int LDS_BYTES = RING_BYTES > XCH_BYTES ? RING_BYTES : XCH_BYTES;
  static_assert(LDS_BYTES <= 160 * 1024, "rings exceed the LDS of a CU");
  auto kern = gemm_bf16_split_kernel<MB, NB, NW, NS, HALF>;
  static LdsLimitOnce lds_limit;   // per instantiation
  if (!lds_limit.ensure((const void*)kern, LDS_BYTES)) return false;
  const int tiles_m = (d.M + 16 * MB - 1) / (16 * MB), tiles_n = (d.N + 16 * NB - 1) / (16 * NB);
  hipLaunchKernelGGL(kern, dim3(((tiles_m * tiles_n + 7) / 8) * 8), dim3(64 * NW), LDS_BYTES, st, d, tiles_m, tiles_n);
  return true;
}

template <int MB, int NB, int NW, int NS>
static bool launch_split_inst(const GemmDev& d, hipStream_t st) {
  return d.K % PBK ? launch_split_half<MB, NB, NW, NS, true>(d, st) : launch_split_half<MB, NB, NW, NS, false>(d, st);
}

// Run time of a tiling in picoseconds: rounds over the CUs times (fixed part of a tile + rows per contraction value).
// Decides between the split kernel and the rings, which are both bound by the rate of new lines.
constexpr long CU_LINE_PS = 32;      // per operand row and contraction value: split kernel and rings (ping-pong 34 to 41)
static long tiling_cost(const GemmDev& d, int bm, int bn, long fixed_ps) {
  const long tiles = (long)((d.M + bm - 1) / bm) * ((d.N + bn - 1) / bn);
  return (tiles + 255) / 256 * (fixed_ps + CU_LINE_PS * (bm + bn) * d.K);
}
// The tiles of the split kernel with the fixed part of each (16x16 0.9 us ... 64x64 2.0, 64x96 5.5: six
// blocks per wavefront to add up and store).
struct SplitTile { int bm, bn; long fixed_ps; };
static const SplitTile split_tiles[] = {{16, 16, 900000}, {16, 32, 1000000}, {32, 32, 1200000}, {32, 48, 1600000},
                                        {32, 64, 1600000}, {64, 32, 1600000}, {64, 48, 1800000}, {64, 64, 2000000},
                                        {64, 96, 5500000}};
static int split_tile_choice(const GemmDev& d, long* cost) {
  int best = 0;
  for (int i = 0; i < (int)(sizeof(split_tiles) / sizeof(split_tiles[0])); ++i) {
    const long c = tiling_cost(d, split_tiles[i].bm, split_tiles[i].bn, split_tiles[i].fixed_ps);
    if (i == 0 || c < *cost) { best = i; *cost = c; }
  }
  return best;
}
static bool launch_split(const GemmDev& d, int choice, hipStream_t st) {
  switch (choice) {
    case 0: return launch_split_inst<1, 1, 8, 4>(d, st);
    case 1: return launch_split_inst<1, 2, 8, 3>(d, st);
    case 2: return launch_split_inst<2, 2, 8, 2>(d, st);
    case 3: return launch_split_inst<2, 3, 8, 2>(d, st);
    case 4: return launch_split_inst<2, 4, 4, 3>(d, st);
    case 5: return launch_split_inst<4, 2, 4, 3>(d, st);
    case 6: return launch_split_inst<4, 3, 4, 2>(d, st);
    case 7: return launch_split_inst<4, 4, 4, 2>(d, st);
    default: return launch_split_inst<4, 6, 4, 2>(d, st);
  }
}

// Run time of a tile that one CU works on at a time, in picoseconds, measured on products of whole rounds: fixed part
// (launch, first stages, plain epilogue), time per contraction value, and 200 per output for a GeLU epilogue.  Decides
// between a ring and the ping-pong kernel only: tiling_cost's flat fixed part of 3 us fits the rings beside the split
// kernel, these larger ones hold for rounds that fill the chip.  By both tables together 187 of 2418 layer products
// (hidden 128 to 2048, 64 to 8192 rows) get a tile that another candidate would beat by 5 % or more, most of them by the
// GeLU term, which tiling_cost lacks.
struct RingTile { int bm, bn; long fixed_ps, k_ps; };
static long ring_time(const GemmDev& d, const RingTile& t) {
  const long tiles = (long)((d.M + t.bm - 1) / t.bm) * ((d.N + t.bn - 1) / t.bn);
  const bool gelu = d.epilogue == EPI_BIAS_GELU || d.epilogue == EPI_MUL_GELU_GRAD || d.epilogue == EPI_BIAS_GELU_DERIV;
  return (tiles + 255) / 256 * (t.fixed_ps + t.k_ps * d.K + (gelu ? 200L * t.bm * t.bn : 0));
}

static long tile_count(const GemmDev& d, int bm, int bn) { return (long)((d.M + bm - 1) / bm) * ((d.N + bn - 1) / bn); }

// Where the register-staged kernel, several workgroups per CU, still beats the ring or ping-pong tile `bm` x `bn`:
// * A contraction of half a k-step in several rounds, nothing read beside the operands: its time is that of the stores, which
//   the staged kernel's rounds overlap (39616 x 3840 x 32 113 us against 148, 4608 x 13120 x 32 51 against 57; with a second
//   operand in the epilogue the rings win by a quarter).
// * Outputs of fewer than 128 rows or columns that no single round of split tiles covers (`narrow`: 16384 and more on the
//   long side), where the tile is mostly padding.  Both sides measured over 32, 64 and 96 by 16480 to 131072, K 32 to 2048:
//   in one round the large tile wins from 64 rows on (64 x 24576 x 256 6.6 us against 8.6), with 32 on the 128-row tiles from
//   K = 256 (32 x 36000 x 256 7.6 against 9.1) and on the 256-row ones from K = 1024; plain products, which the staged kernel
//   stores fastest, of K <= 128 do not (64 x 20000 x 64 4.4 against 5.0).  In several rounds staged wins with 32 rows (65536
//   x 32 x 128 8.1 against 11.5), for plain products (64 x 50272 x 512 15.4 against 17.6), with a single k-step on the
//   small tiles (57344 x 64 x 64 7.7 against 9.6), against 256x256 tiles (64 x 131072 x 128 16.4 against 19.5) and from
//   three rounds on (98304 x 64 x 256 14.8 against 18.5).
static bool staged_wins(const GemmDev& d, int bm, int bn, bool narrow) {
  const int side = d.M < d.N ? d.M : d.N;
  const long rounds = (tile_count(d, bm, bn) + 255) / 256;
  if (d.K < PBK && rounds >= 2 && (d.epilogue == EPI_NONE || d.epilogue == EPI_BIAS)) return true;
  if (!narrow) return false;
  if (side <= 32 && (rounds >= 2 || d.K < (bm < 256 ? 256 : 1024))) return true;
  if (d.epilogue == EPI_NONE && side <= 64 && d.K <= 2 * PBK) return true;
  return rounds >= 3 || (rounds == 2 && (d.epilogue == EPI_NONE || bm * bn == 256 * 256 || (d.K <= PBK && bm * bn <= 128 * 128)));
}

bool launch_gemm_pipe(const GemmDev& d, int a_kmajor, int b_kmajor, int out_f32, int batch, hipStream_t st) {
  if (d.K % (PBK / 2) || out_f32 || batch != 1) return false;
  if (a_kmajor && b_kmajor) {
    // Tile choice among the rings.  Every CU has to work through ceil(tiles / 256) tiles.  With work for all CUs the cost
    // of a tiling is that count times the tile area (the fixed parts below are left out of it); among equals the larger
    // tile fetches fewer bytes per flop, then the squarer one.
    static const RingTile cands[] = {{128, 128, 4300000, 8600}, {128, 96, 4500000, 7500}, {128, 144, 6000000, 10000},
                                     {128, 192, 4300000, 11500}, {256, 144, 8500000, 14500}, {256, 192, 10200000, 19200}};
    int best = 0;
    long best_cost = 0, best_area = 0, best_perim = 0;
    for (int i = 0; i < 6; ++i) {
      const RingTile& c = cands[i];
      if (i > 0 && d.N % c.bn) continue;
      const long tl = (long)((d.M + c.bm - 1) / c.bm) * ((d.N + c.bn - 1) / c.bn);
      const long area = (long)c.bm * c.bn, cost = ((tl + 255) / 256) * area, perim = c.bm + c.bn;
      if (i == 0 || cost < best_cost || (cost == best_cost && (area > best_area || (area == best_area && perim < best_perim)))) {
        best = i; best_cost = cost; best_area = area; best_perim = perim;
      }
    }
    // With work for few of them the split kernel's smaller tiles win.  The line lies where its estimate meets that of
    // the tile above, whose fixed part is about 3 us: in a step of 1824 rows the 768-deep products take 10.2 us on the
    // rings and 13.5 on 64x96 split tiles, the 3072-deep ones 26.6 and 26.1.
    long split_cost = 0;
    const int split = split_tile_choice(d, &split_cost);
    // (Rounds of split tiles do not overlap: outputs of fewer than 128 rows or columns take them in one round only.)
    const bool narrow = (d.M < 128 || d.N < 128) && tile_count(d, split_tiles[split].bm, split_tiles[split].bn) > 256;
    if (!narrow && split_cost < tiling_cost(d, cands[best].bm, cands[best].bn, 3000000)) return launch_split(d, split, st);
    // The ping-pong kernel's tiles where their run time, estimated from the same kind of measurements, is below that of
    // the ring's tile: outputs wide enough to fill the CUs with 256-row tiles.  It needs two k-steps, and unsigned 32-bit
    // offsets within an operand panel (a negative leading dimension, rows stored backwards, stays on the rings).
    static const RingTile pp[] = {{256, 128, 7500000, 12200}, {256, 192, 8000000, 17400}, {256, 256, 8000000, 21000}};
    int take = -1;
    if (d.K > PBK && d.lda >= 0 && d.ldb >= 0 && d.lda <= 1 << 20 && d.ldb <= 1 << 20 && d.K <= 1 << 20) {
      long least = ring_time(d, cands[best]);
      for (int i = 0; i < 3; ++i) {
        const long c = ring_time(d, pp[i]);
        if (c < least) { least = c; take = i; }
      }
    }
    const RingTile& chosen = take < 0 ? cands[best] : pp[take];
    if (staged_wins(d, chosen.bm, chosen.bn, narrow)) return false;
    if (take >= 0) {
      if (take == 0) return launch_pingpong_inst<4, 2, 2, 2>(d, st);
      if (take == 1) return launch_pingpong_inst<4, 2, 2, 3>(d, st);
      return launch_pingpong_inst<2, 4, 4, 2>(d, st);
    }
    switch (best) {
      // one 128x96 tile per CU: 8 consumer + 8 producer waves, three stages (measured 24 us against 33 us for the
      // 4096x768x3072 product)
      case 1: return launch_w48s_inst<2, 2, 3, 3, 2, 8, bf16_t>(d, st);
      case 2: return launch_w48s_inst<2, 3, 3, 3, 2, 4, bf16_t>(d, st);   // 128x144: 12 + 4 waves
      case 3: return launch_w48s_inst<2, 4, 3, 3, 1, 8, bf16_t>(d, st);   // 128x192: 8 + 8 waves
      case 4: return launch_w48s_inst<4, 3, 3, 3, 1, 4, bf16_t>(d, st);   // 256x144: 12 + 4 waves
      // 256x192, 16 symmetric waves, two stages: single k-steps and panels beyond the ping-pong kernel's offsets
      case 5: return launch_w48_inst<4, 4, 2>(d, st);
      default: break;
    }
    // 128x128: the same producer/consumer kernel with 64x64 wave tiles
    return launch_w48s_inst<2, 2, 4, 3, 2, 8, bf16_t>(d, st);
  }
  // Both operands MN-major, 64 columns and one or two k-steps: the whole problem fits a three-stage ring, so every load
  // is issued before the first barrier (register-staged kernel: 1024 x 64 x 128 4.5 us against 4.25, 65536 x 64 x 128 9.6
  // against 8.9; with a K-major A the two are level).
  if (!a_kmajor && !b_kmajor && d.N == 64 && d.K % PBK == 0 && d.K <= 2 * PBK && d.M % 128 == 0)
    return launch_pipe_inst<128, 64, 2, 2, false, false, 3>(d, st);
  // A K-major A with an MN-major B (products against an untransposed row-major weight, e.g. the tied decoder of the MLM
  // head): 128x128 tiles, 8 wavefronts (2 x 4), two 32 KiB stages.  The ring only wins when there are enough tiles for
  // two workgroups per CU; below that the register-staged kernel is faster.
  const long tiles = (long)((d.M + 127) / 128) * ((d.N + 127) / 128);
  if (a_kmajor && !b_kmajor && d.K % PBK == 0 && d.M >= 128 && d.N >= 128 && tiles >= 384) return launch_pipe_inst<128, 128, 2, 4, true, false, 2>(d, st);
  return false;
}

}  // namespace raf
