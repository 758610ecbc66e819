// Device-side pieces shared by the GEMM kernels: the launch descriptor and the
// fused epilogues (bias, bias+GeLU with saved pre-activation, GeLU-gradient
// multiply, residual add, scale, fp32 output).
#pragma once
#include "common.hpp"

namespace raf {

struct GemmDev {
  int M, N, K;
  const void* a; long lda;
  const void* b; long ldb;
  void* c; long ldc;
  float alpha;
  int epilogue;
  const float* bias;
  void* aux; long ldaux;
  int gelu_tanh;
  int gelu_exact;   // the staged epilogue, whose GeLU is the one-exponential form, must not be taken
  int nz_inner;
  long sa0, sa1, sb0, sb1, sc0, sc1;
};

// four consecutive columns j..j+3 of row i (j a multiple of 4; all pointers and
// leading dimensions keep 8-byte alignment of such groups)
__device__ __forceinline__ void load4(const bf16_t* p, float (&o)[4]) {
  const uint2 r = *reinterpret_cast<const uint2*>(p);
  o[0] = bf16_bits_to_f32(r.x & 0xffffu); o[1] = __uint_as_float(r.x & 0xffff0000u);
  o[2] = bf16_bits_to_f32(r.y & 0xffffu); o[3] = __uint_as_float(r.y & 0xffff0000u);
}
__device__ __forceinline__ void store4(bf16_t* p, const float (&v)[4]) {
  uint2 r;
  r.x = pack_bf16x2(v[0], v[1]);
  r.y = pack_bf16x2(v[2], v[3]);
  *reinterpret_cast<uint2*>(p) = r;
}
__device__ __forceinline__ void store4(float* p, const float (&v)[4]) {
  *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
}

// The epilogue kind and the form of GeLU are template parameters here and the kernels switch on them once, outside
// their unrolled store loops: a test of the form per element kept the elements' chains from overlapping (with the
// cheaper reciprocal 4096 x 3072 x 768 with GeLU and derivative 37.4 -> 34.5 us on 16 wavefronts, 4096 x 8192 x 2048
// 158 -> 152), and with the run-time switch of the kind inside, every one of the 12-64 store groups of a wave carried
// all cases and the epilogue of the plain-bias GEMMs slowed down by several microseconds when a case was added.
template <typename TC, int EPI, int TANH>
__device__ __forceinline__ void epilogue_store4(const GemmDev& g, TC* __restrict__ c, bf16_t* __restrict__ aux, int i,
                                                int j, float (&v)[4]) {
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] *= g.alpha;
  if constexpr (EPI == EPI_BIAS || EPI == EPI_BIAS_GELU || EPI == EPI_BIAS_GELU_DERIV) {
    const float4 b = *reinterpret_cast<const float4*>(g.bias + j);
    v[0] += b.x; v[1] += b.y; v[2] += b.z; v[3] += b.w;
  }
  if constexpr (EPI == EPI_BIAS_GELU) {
    store4(aux + (long)i * g.ldaux + j, v);
    // GeLU is evaluated on the value the backward pass will read back
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = gelu_f((float)(bf16_t)v[e], TANH);
  } else if constexpr (EPI == EPI_MUL_GELU_GRAD) {
    float u[4];
    load4(aux + (long)i * g.ldaux + j, u);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] *= gelu_grad_f(u[e], TANH);
  } else if constexpr (EPI == EPI_ADD_RES) {
    float r[4];
    load4(aux + (long)i * g.ldaux + j, r);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] += r[e];
  } else if constexpr (EPI == EPI_BIAS_GELU_DERIV) {
    float dy[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) gelu_and_grad_f(v[e], TANH, v[e], dy[e]);
    store4(aux + (long)i * g.ldaux + j, dy);
  } else if constexpr (EPI == EPI_MUL_AUX) {
    float r[4];
    load4(aux + (long)i * g.ldaux + j, r);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] *= r[e];
  }
  store4(c + (long)i * g.ldc + j, v);
}

template <int V>
struct EpiTag {
  static constexpr int value = V;
};
template <typename F>
__device__ __forceinline__ void epilogue_dispatch(const GemmDev& g, F&& f) {
  constexpr EpiTag<0> erf_form{};
  constexpr EpiTag<1> tanh_form{};
  switch (g.epilogue) {
    case EPI_BIAS: f(EpiTag<EPI_BIAS>{}, erf_form); break;
    case EPI_BIAS_GELU:
      if (g.gelu_tanh) f(EpiTag<EPI_BIAS_GELU>{}, tanh_form);
      else f(EpiTag<EPI_BIAS_GELU>{}, erf_form);
      break;
    case EPI_MUL_GELU_GRAD:
      if (g.gelu_tanh) f(EpiTag<EPI_MUL_GELU_GRAD>{}, tanh_form);
      else f(EpiTag<EPI_MUL_GELU_GRAD>{}, erf_form);
      break;
    case EPI_ADD_RES: f(EpiTag<EPI_ADD_RES>{}, erf_form); break;
    case EPI_BIAS_GELU_DERIV:
      if (g.gelu_tanh) f(EpiTag<EPI_BIAS_GELU_DERIV>{}, tanh_form);
      else f(EpiTag<EPI_BIAS_GELU_DERIV>{}, erf_form);
      break;
    case EPI_MUL_AUX: f(EpiTag<EPI_MUL_AUX>{}, erf_form); break;
    default: f(EpiTag<EPI_NONE>{}, erf_form); break;
  }
}

// A wave's TM x TN blocks of the (transposed) 32x32 MFMA result: register r of lane l holds output row (l & 31),
// column 8*(r/4) + 4*(l/32) + r%4 of its block.  row0 / col0: the wave tile's origin.
template <typename TC, int TM, int TN>
__device__ __forceinline__ void epilogue_tile32(const GemmDev& g, TC* __restrict__ C, bf16_t* __restrict__ AUX,
                                                f32x16_t (&acc)[TM][TN], int row0, int col0) {
  const int lane = threadIdx.x & 63;
  epilogue_dispatch(g, [&](auto tag, auto form) {
    constexpr int EPI = decltype(tag)::value, TANH = decltype(form)::value;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int row = row0 + i * 32 + (lane & 31);
      if (row < g.M) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int col = col0 + j * 32 + 8 * q + 4 * (lane >> 5);
            if (col < g.N) {
              float v[4] = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
              epilogue_store4<TC, EPI, TANH>(g, C, AUX, row, col, v);
            }
          }
      }
    }
  });
}

// A wave's 4 x NB blocks of the (transposed) 16x16 MFMA result: a lane holds output row (l & 15) and the 4
// consecutive columns 4*(l>>4) + r of each block; only row blocks [i_begin, i_end) are written.
template <typename TC, int NB>
__device__ __forceinline__ void epilogue_tile16(const GemmDev& g, TC* __restrict__ C, bf16_t* __restrict__ AUX,
                                                f32x4_t (&acc)[4][NB], int row0, int col0, int i_begin, int i_end) {
  const int lane = threadIdx.x & 63;
  epilogue_dispatch(g, [&](auto tag, auto form) {
    constexpr int EPI = decltype(tag)::value, TANH = decltype(form)::value;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (i < i_begin || i >= i_end) continue;
      const int row = row0 + i * 16 + (lane & 15);
      if (row < g.M) {
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          const int col = col0 + j * 16 + 4 * (lane >> 4);
          if (col < g.N) {
            float v[4] = {acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]};
            epilogue_store4<TC, EPI, TANH>(g, C, AUX, row, col, v);
          }
        }
      }
    }
  });
}


// Bytes of LDS one wave needs for epilogue_tile16_staged.
template <int NB>
constexpr int epilogue_stage_bytes() {
  return 2 * 16 * (32 * NB + 16);
}

// True when the output (and aux) rows of a problem can be written 16 bytes at a time (and its GeLU may be the fast form).
__device__ __forceinline__ bool epilogue_can_stage(const GemmDev& g) {
  const unsigned long long p = (unsigned long long)g.c | (unsigned long long)g.aux;
  return !g.gelu_exact && ((g.ldc | g.ldaux | (long)g.N) & 7) == 0 && (p & 15) == 0;
}

// Same result as epilogue_tile16 for bf16 outputs, written through a wave-private LDS buffer: the accumulator
// layout gives a lane 4 columns of one row, so a direct store instruction touches 16 rows with 32 bytes each, and
// such stores cost several times the time of full-row ones (5.5 us against 0.7 us for the 19-MB output of a
// 4096 x 2304 product).  The blocks are therefore finished in registers, laid out row-major in LDS and written
// (aux operands: read) as 16-byte pieces that run along the rows of the wave tile: two 16-row blocks per trip, an
// aux operand being replaced in place by the result; one block per trip with two buffers for the epilogues that
// write a second output.  LDS operations of one wave execute in order, so no barrier is needed; `stg` must not be
// touched by any other wave.
template <int NB>
__device__ __forceinline__ void epilogue_tile16_staged(const GemmDev& g, bf16_t* __restrict__ C,
                                                       bf16_t* __restrict__ AUX, f32x4_t (&acc)[4][NB], int row0,
                                                       int col0, int i_begin, int i_end, char* stg) {
  constexpr int P = 32 * NB + 16;         // row pitch in LDS, bytes
  constexpr int CPR = 2 * NB;             // 16-byte pieces per row
  const int lane = threadIdx.x & 63;
  const int lr = lane & 15, lg = lane >> 4;
  epilogue_dispatch(g, [&](auto tag, auto form) {
    constexpr int EPI = decltype(tag)::value, TANH = decltype(form)::value;
    constexpr bool AUX_IN = EPI == EPI_MUL_GELU_GRAD || EPI == EPI_ADD_RES || EPI == EPI_MUL_AUX;
    constexpr bool AUX_OUT = EPI == EPI_BIAS_GELU || EPI == EPI_BIAS_GELU_DERIV;
    constexpr bool BIAS = EPI == EPI_BIAS || EPI == EPI_BIAS_GELU || EPI == EPI_BIAS_GELU_DERIV;
    constexpr int BLK = AUX_OUT ? 1 : 2;  // row blocks per trip through LDS
    constexpr int ROWS = 16 * BLK, NCH = ROWS * CPR, IT = (NCH + 63) / 64;
    char* s_out = stg;
    char* s_aux = AUX_OUT ? stg + 16 * P : stg;
    // piece `it` of this lane: row and 16-byte column within a trip
    int pr[IT], pc[IT];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int q = it * 64 + lane;
      pr[it] = q / CPR;
      pc[it] = q - pr[it] * CPR;
    }
    // aux pieces of one trip; the next trip's are requested as soon as these have gone to LDS
    uint4 ain[IT];
    auto load_aux = [&](int t) {
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        const int row = row0 + t * ROWS + pr[it], col = col0 + pc[it] * 8;
        ain[it] = make_uint4(0u, 0u, 0u, 0u);
        if (pr[it] < ROWS && row < g.M && col < g.N)
          ain[it] = *reinterpret_cast<const uint4*>(AUX + (long)row * g.ldaux + col);
      }
    };
    if constexpr (AUX_IN) load_aux(i_begin / BLK);
    float4 bias[BIAS ? NB : 1];
    if constexpr (BIAS) {
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const int col = col0 + j * 16 + 4 * lg;
        bias[j] = col < g.N ? *reinterpret_cast<const float4*>(g.bias + col) : make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }
#pragma unroll
    for (int t = 0; t < 4 / BLK; ++t) {
      if (t * BLK < i_begin || t * BLK >= i_end) continue;
      if constexpr (AUX_IN) {
#pragma unroll
        for (int it = 0; it < IT; ++it)
          if (pr[it] < ROWS) *reinterpret_cast<uint4*>(s_aux + pr[it] * P + pc[it] * 16) = ain[it];
        if ((t + 1) * BLK < i_end) load_aux(t + 1);
      }
#pragma unroll
      for (int b = 0; b < BLK; ++b)
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          const int i = t * BLK + b;
          const int off = (b * 16 + lr) * P + j * 32 + lg * 8;
          float v[4] = {acc[i][j][0] * g.alpha, acc[i][j][1] * g.alpha, acc[i][j][2] * g.alpha, acc[i][j][3] * g.alpha};
          if constexpr (BIAS) {
            v[0] += bias[j].x; v[1] += bias[j].y; v[2] += bias[j].z; v[3] += bias[j].w;
          }
          if constexpr (EPI == EPI_BIAS_GELU) {
            store4(reinterpret_cast<bf16_t*>(s_aux + off), v);
            // GeLU is evaluated on the value the backward pass will read back
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = gelu_fast((float)(bf16_t)v[e], TANH);
          } else if constexpr (EPI == EPI_BIAS_GELU_DERIV) {
            float dy[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) gelu_and_grad_fast(v[e], TANH, v[e], dy[e]);
            store4(reinterpret_cast<bf16_t*>(s_aux + off), dy);
          } else if constexpr (AUX_IN) {
            float u[4];
            load4(reinterpret_cast<const bf16_t*>(s_aux + off), u);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              if constexpr (EPI == EPI_MUL_GELU_GRAD) v[e] *= gelu_grad_fast(u[e], TANH);
              else if constexpr (EPI == EPI_ADD_RES) v[e] += u[e];
              else v[e] *= u[e];
            }
          }
          store4(reinterpret_cast<bf16_t*>(s_out + off), v);
          // four chains at a time: with all of a trip's in flight at once some instantiations spill registers
          if constexpr (AUX_OUT || EPI == EPI_MUL_GELU_GRAD) __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        const int row = row0 + t * ROWS + pr[it], col = col0 + pc[it] * 8;
        if (pr[it] < ROWS && row < g.M && col < g.N) {
          *reinterpret_cast<uint4*>(C + (long)row * g.ldc + col) =
              *reinterpret_cast<const uint4*>(s_out + pr[it] * P + pc[it] * 16);
          if constexpr (AUX_OUT)
            *reinterpret_cast<uint4*>(AUX + (long)row * g.ldaux + col) =
                *reinterpret_cast<const uint4*>(s_aux + pr[it] * P + pc[it] * 16);
        }
      }
    }
  });
}

// Float outputs of the 16x16 layout without elementwise epilogue (weight gradients), one row of blocks per trip
// through a wave-private LDS buffer of epilogue_stage_f32_bytes: a direct store instruction writes 64-byte pieces of
// 16 rows, the staged one runs along whole rows of the wave tile.
template <int NB>
constexpr int epilogue_stage_f32_bytes() {
  return 16 * (64 * NB + 16);
}
template <int MB, int NB>
__device__ __forceinline__ void epilogue_tile16_f32(const GemmDev& g, float* __restrict__ C, f32x4_t (&acc)[MB][NB],
                                                    int row0, int col0, char* stg) {
  constexpr int P = 64 * NB + 16, CPR = 4 * NB;   // row pitch in bytes, 16-byte pieces per row
  const int lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
#pragma unroll
  for (int i = 0; i < MB; ++i) {
#pragma unroll
    for (int j = 0; j < NB; ++j) *reinterpret_cast<f32x4_t*>(stg + lr * P + j * 64 + lg * 16) = acc[i][j] * g.alpha;
#pragma unroll
    for (int it = 0; it < 16 * CPR / 64; ++it) {
      const int q = it * 64 + lane, r = q / CPR, c = q % CPR;
      const int row = row0 + i * 16 + r, col = col0 + c * 4;
      if (row < g.M && col < g.N)   // N is a multiple of 8: a piece is inside or outside as a whole
        *reinterpret_cast<f32x4_t*>(C + (long)row * g.ldc + col) = *reinterpret_cast<const f32x4_t*>(stg + r * P + c * 16);
    }
  }
}

// s_waitcnt on the vector-memory counter only (expcnt / lgkmcnt left at max)
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

// s_waitcnt lgkmcnt(0): this wave's LDS reads have returned
__device__ __forceinline__ void lds_reads_done() { __builtin_amdgcn_s_waitcnt(0xc07f); }

// s_waitcnt vmcnt(n) for a wave-uniform run-time n (conservative above 24)
__device__ __forceinline__ void wait_vmcnt_dyn(int n) {
  switch (n) {
#define RAF_VMCNT_CASE(N) case N: wait_vmcnt<N>(); break;
    RAF_VMCNT_CASE(1) RAF_VMCNT_CASE(2) RAF_VMCNT_CASE(3) RAF_VMCNT_CASE(4) RAF_VMCNT_CASE(5) RAF_VMCNT_CASE(6)
    RAF_VMCNT_CASE(7) RAF_VMCNT_CASE(8) RAF_VMCNT_CASE(9) RAF_VMCNT_CASE(10) RAF_VMCNT_CASE(11) RAF_VMCNT_CASE(12)
    RAF_VMCNT_CASE(13) RAF_VMCNT_CASE(14) RAF_VMCNT_CASE(15) RAF_VMCNT_CASE(16) RAF_VMCNT_CASE(17) RAF_VMCNT_CASE(18)
    RAF_VMCNT_CASE(19) RAF_VMCNT_CASE(20) RAF_VMCNT_CASE(21) RAF_VMCNT_CASE(22) RAF_VMCNT_CASE(23) RAF_VMCNT_CASE(24)
#undef RAF_VMCNT_CASE
    default: wait_vmcnt<0>(); break;
  }
}

typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef short s16x8_t __attribute__((ext_vector_type(8)));

// Several independent problems of one layout in a single launch; tile_start[p]
// is the first linear tile of problem p, tiles_n[p] its tile columns.
constexpr int GEMM_GROUP_MAX = 4;
struct GemmGroupDev {
  GemmDev p[GEMM_GROUP_MAX];
  int tile_start[GEMM_GROUP_MAX + 1];
  int tiles_n[GEMM_GROUP_MAX];
  // > 0: the problem's tiles are numbered along M first (that many row tiles), so that a contiguous share of the tile
  // list covers whole strips of the side with fewer tiles; 0: along N first
  int tiles_m_first[GEMM_GROUP_MAX];
  int count;
};


// Column sums out[j][c] = sum_r x[j][r*ld + c] of up to two bf16 matrices with the same row count (the bias
// gradients next to the weight gradients), taken by workgroups of the weight-gradient launch that would otherwise
// find no tile: the grouped launch of a BERT-base layer has 216 tiles for 256 CUs.
struct ColsumSide {
  const bf16_t* x[2];
  float* out[2];
  long ld[2];
  int cols[2];     // multiples of 8; cols[1] = 0 for a single matrix
  long rows;
  int count;       // 0: no side work
  // second stages of earlier two-stage column sums (sums over partial rows, see ReduceJob), taken after the above
  ReduceJob red[3];
  int nred;
  // not null: set to 1 when any sum written here, or any weight-gradient value of the launch's tiles, is inf or nan
  int* nonfinite;
};

// Weight-gradient group (both operands MN-major, float output) on the
// producer/consumer direct-to-LDS kernel (gemm_pipe.hip); false when a problem
// does not fit it (K % 32, M or N not a multiple of 8) or its LDS limit could not be raised.  side: optional column sums;
// *side_taken tells whether the launch computed them, otherwise the caller has to (sums wider than its workers hold).
// side->nonfinite is honoured only when the side work is taken (*side_taken).
bool launch_gemm_group_spec(const GemmDev* ds, int count, hipStream_t st, const ColsumSide* side = nullptr,
                            bool* side_taken = nullptr);

// Pipelined direct-to-LDS kernel family (gemm_pipe.hip).  Returns false when
// the problem does not meet its requirements (layout, bf16 output, no batch) and
// the caller must use the staged kernel instead.
bool launch_gemm_pipe(const GemmDev& d, int a_kmajor, int b_kmajor, int out_f32, int batch, hipStream_t st);

// Full-precision products on the matrix cores (gemm_f32.hip), one problem (batched or not) of any layout, or up to
// GEMM_GROUP_MAX of the weight-gradient layout in one launch.  False: nothing was launched (count out of range).
bool launch_gemm_f32(const GemmDev& d, int a_kmajor, int b_kmajor, int batch, hipStream_t st);
bool launch_gemm_f32_group(const GemmDev* ds, int count, hipStream_t st);

}  // namespace raf
