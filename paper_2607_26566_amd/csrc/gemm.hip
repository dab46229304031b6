// Linear layers y = A W^T + b of the DiT block (qkv, out, cross-q, cross-out,
// fc1, fc2, text projections) on gfx950.
//
//  * gemm_bf16_kernel: bf16 operands, fp32 accumulation on MFMA
//    (v_mfma_f32_16x16x32_bf16).  A workgroup of 4 waves owns a BM x BN output
//    tile; each wave a (BM/2) x (BN/2) quadrant.  K advances 64 at a time
//    through double-buffered LDS tiles (row pitch 72 bf16 = 144 B, so the 16
//    rows a fragment load touches fall in distinct bank groups); the next K
//    tile is fetched from HBM into registers while MFMA works on the current
//    one.  Workgroups are numbered so that each XCD (dispatched round-robin)
//    receives a contiguous run of output tiles: tiles sharing A rows share
//    that XCD's L2.
//  * gemm_f32_kernel: fp32 matrix cores (v_mfma_f32_16x16x4_f32) for the fp32
//    model's layers.
//  * linear_rows_kernel: the conditioning GEMMs (timestep MLP, adaLN table),
//    8 timesteps per pass, weight-streaming and HBM-bound; its per-element
//    summation order does not depend on the number of timesteps, so a
//    sample's batched table equals the per-step tables bitwise.
//
// Epilogues (bias always added): store, GELU-tanh, SiLU, residual add,
// gated residual add (gate row chosen by the row's sequence), and split-store
// for fused q|k|v projections: q and k row-major, v transposed (V^T[d][token],
// four tokens per 8-byte store) so attention can stage V^T tiles directly.
#include <algorithm>
#include <cstring>

#include "t2i_internal.h"

namespace t2i {

hipError_t launch_gemm_dma(const bf16* A, int lda, const bf16* W, int ldw, const bf16* bias,
                           int M, int N, int K, int kind, const Epi& epi, int vec_ok,
                           hipStream_t st, int splits = 1);
bool gemm_dma_fits(int M, int N);

// Map launch order -> tile order so XCD x (blocks b with b % 8 == x) owns the
// contiguous tile range of its share.
__device__ __forceinline__ int xcd_remap(int b, int nb) {
  const int q = nb >> 3, r = nb & 7;
  const int x = b & 7, j = b >> 3;
  return (x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q) + j;
}

// s_waitcnt with only vmcnt constrained
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// one 16-byte-per-lane buffer load into LDS at the wave-uniform address lds
__device__ __forceinline__ void load_lds16(__amdgpu_buffer_rsrc_t r, void* lds, uint32_t voff,
                                           int soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)lds, 16,
                                           voff, soff, 0, 0);
}

// Epilogue on four consecutive columns nb..nb+3 of row m (vector path).
template <int KIND>
__device__ __forceinline__ void epi_store4(const Epi& e, int m, int nb, const float v[4]) {
  if (KIND == EPI_STORE_F32) {
    *(float4*)((float*)e.out + (size_t)m * e.ldo + nb) = float4{v[0], v[1], v[2], v[3]};
  } else if (KIND == EPI_STORE || KIND == EPI_GELU || KIND == EPI_SILU) {
    bf16x4 w;
    const float qs = KIND == EPI_STORE && nb < e.qcols ? e.qscale : 1.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float y = v[r];
      if (KIND == EPI_GELU) y = gelu_tanh(y);
      if (KIND == EPI_SILU) y = silu(y);
      if (KIND == EPI_STORE) y *= qs;
      w[r] = (bf16)y;
    }
    *(bf16x4*)((bf16*)e.out + (size_t)m * e.ldo + nb) = w;
  } else {
    float4 g4 = float4{1.f, 1.f, 1.f, 1.f};
    if (KIND == EPI_RESID_GATED)
      g4 = *(const float4*)(e.gate + (size_t)e.map.modrow[seq_of_row(e.map, m)] * e.ld_gate + nb);
    float4* xp = (float4*)(e.x + (size_t)m * e.ldx + nb);
    float4 x4 = *xp;
    x4.x += g4.x * v[0];
    x4.y += g4.y * v[1];
    x4.z += g4.z * v[2];
    x4.w += g4.w * v[3];
    *xp = x4;
    if (e.xb) {
      bf16x4 w{(bf16)x4.x, (bf16)x4.y, (bf16)x4.z, (bf16)x4.w};
      *(bf16x4*)(e.xb + (size_t)m * e.ldx + nb) = w;
    }
  }
}

// BM x BN tile per workgroup of 4 waves arranged WGM x (4 / WGM).  Except for
// the split q|k|v store, the MFMA computes C^T fragments (operands swapped),
// so a lane ends with four consecutive output columns of one row and the
// epilogue issues one 8-byte (bf16) or 16-byte (fp32) access per lane.
template <int BM, int BN, int WGM, int KIND>
__device__ __forceinline__ void gemm_bf16_body(const bf16* __restrict__ A, int lda,
                                               const bf16* __restrict__ W, int ldw,
                                               const bf16* __restrict__ bias, int M, int N, int K,
                                               const Epi& epi, int tiles_n, int vec_ok, int tile) {
  constexpr bool PART = KIND == EPI_PARTIAL;
  constexpr int EK = PART ? EPI_STORE_F32 : KIND;
  constexpr int BK = 64;
  constexpr int LDK = BK + 8;
  constexpr int WGN = 4 / WGM;
  constexpr int WM = BM / WGM, WN = BN / WGN;
  constexpr int TM = WM / 16, TN = WN / 16;
  constexpr int ACH = BM * (BK / 8), BCH = BN * (BK / 8);   // 16-byte chunks per tile
  constexpr int APT = (ACH + 255) / 256, BPT = (BCH + 255) / 256;
  constexpr bool CT = KIND != EPI_SPLIT_VT;
  static_assert(WM % 16 == 0 && WN % 16 == 0, "wave tile");
  __shared__ bf16 As[2][BM * LDK];
  __shared__ bf16 Bs[2][BN * LDK];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN;
  const int m0 = (tile / tiles_n) * BM, n0 = (tile % tiles_n) * BN;

  const bf16* Ap[APT];
  const bf16* Bp[BPT];
#pragma unroll
  for (int i = 0; i < APT; ++i) {
    const int c = min(tid + 256 * i, ACH - 1);
    Ap[i] = A + (size_t)min(m0 + (c >> 3), M - 1) * lda + (c & 7) * 8;
  }
#pragma unroll
  for (int i = 0; i < BPT; ++i) {
    const int c = min(tid + 256 * i, BCH - 1);
    Bp[i] = W + (size_t)min(n0 + (c >> 3), N - 1) * ldw + (c & 7) * 8;
  }

  bf16x8 ra[APT], rb[BPT];
  auto gload = [&](int k0) {
#pragma unroll
    for (int i = 0; i < APT; ++i)
      if (ACH % 256 == 0 || tid + 256 * i < ACH) ra[i] = *(const bf16x8*)(Ap[i] + k0);
#pragma unroll
    for (int i = 0; i < BPT; ++i)
      if (BCH % 256 == 0 || tid + 256 * i < BCH) rb[i] = *(const bf16x8*)(Bp[i] + k0);
  };
  auto sstore = [&](int buf) {
#pragma unroll
    for (int i = 0; i < APT; ++i) {
      const int c = tid + 256 * i;
      if (ACH % 256 == 0 || c < ACH) *(bf16x8*)&As[buf][(c >> 3) * LDK + (c & 7) * 8] = ra[i];
    }
#pragma unroll
    for (int i = 0; i < BPT; ++i) {
      const int c = tid + 256 * i;
      if (BCH % 256 == 0 || c < BCH) *(bf16x8*)&Bs[buf][(c >> 3) * LDK + (c & 7) * 8] = rb[i];
    }
  };

  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Epilogue operands of a tile that is whole in N (as in gemm_dma.hip): the
  // BN bias values and, for a gated update whose rows all belong to one
  // sequence, the BN gate values, fetched with the first tile and kept in LDS,
  // so that the epilogue's stores never wait behind a global load.
  constexpr bool GATED = KIND == EPI_RESID_GATED;
  __shared__ __attribute__((aligned(16))) float ebias[BN];
  __shared__ __attribute__((aligned(16))) float egate[GATED ? BN : 4];
  const bool whole_n = !PART && vec_ok && n0 + BN <= N;
  bool one_seq = false;
  int grow = 0;
  if constexpr (GATED) {
    const int s0 = seq_of_row(epi.map, m0), s1 = seq_of_row(epi.map, min(m0 + BM, M) - 1);
    one_seq = whole_n && s0 == s1;
    grow = epi.map.modrow[s0];
  }
  const bool stager = tid < BN / 4;
  bf16x4 sbias{};
  float4 sgate{};
  if (whole_n && stager) sbias = *(const bf16x4*)(bias + n0 + 4 * tid);
  if (GATED && one_seq && stager)
    sgate = *(const float4*)(epi.gate + (size_t)grow * epi.ld_gate + n0 + 4 * tid);

  const int KT = K / BK;
  gload(0);
  sstore(0);
  if (whole_n && stager) {
    *(float4*)&ebias[4 * tid] =
        float4{(float)sbias[0], (float)sbias[1], (float)sbias[2], (float)sbias[3]};
    if (GATED && one_seq) *(float4*)&egate[4 * tid] = sgate;
  }
  __syncthreads();
  const int fr = lane & 15, fk = (lane >> 4) * 8;
  for (int kt = 0; kt < KT; ++kt) {
    const int buf = kt & 1;
    if (kt + 1 < KT) gload((kt + 1) * BK);
#pragma unroll
    for (int kk = 0; kk < BK; kk += 32) {
      bf16x8 af[TM], bfr[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i)
        af[i] = *(const bf16x8*)&As[buf][(wm * WM + i * 16 + fr) * LDK + kk + fk];
#pragma unroll
      for (int j = 0; j < TN; ++j)
        bfr[j] = *(const bf16x8*)&Bs[buf][(wn * WN + j * 16 + fr) * LDK + kk + fk];
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = CT ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[j], af[i], acc[i][j], 0, 0, 0)
                         : __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
    }
    if (kt + 1 < KT) sstore(buf ^ 1);
    __syncthreads();
  }

  if (CT && whole_n) {
    // C^T fragment: lane holds row m = (lane & 15), columns 4*(lane >> 4) + 0..3
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int m = m0 + wm * WM + i * 16 + fr;
      if (m >= M) continue;
      if constexpr (KIND == EPI_RESID || KIND == EPI_RESID_GATED) {
        // this row's residual values fetched together, then updated
        float4 xl[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j)
          xl[j] = *(const float4*)(epi.x + (size_t)m * epi.ldx + n0 + wn * WN + j * 16 + (lane >> 4) * 4);
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const int col = wn * WN + j * 16 + (lane >> 4) * 4;
          const float4 b4 = *(const float4*)&ebias[col];
          float4 g4 = float4{1.f, 1.f, 1.f, 1.f};
          if (GATED) {
            g4 = one_seq ? *(const float4*)&egate[col]
                         : *(const float4*)(epi.gate + (size_t)epi.map.modrow[seq_of_row(epi.map, m)] *
                                                           epi.ld_gate + n0 + col);
          }
          float4 x4 = xl[j];
          x4.x += g4.x * (acc[i][j][0] + b4.x);
          x4.y += g4.y * (acc[i][j][1] + b4.y);
          x4.z += g4.z * (acc[i][j][2] + b4.z);
          x4.w += g4.w * (acc[i][j][3] + b4.w);
          *(float4*)(epi.x + (size_t)m * epi.ldx + n0 + col) = x4;
          if (epi.xb) {
            bf16x4 w{(bf16)x4.x, (bf16)x4.y, (bf16)x4.z, (bf16)x4.w};
            *(bf16x4*)(epi.xb + (size_t)m * epi.ldx + n0 + col) = w;
          }
        }
      } else {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const int col = wn * WN + j * 16 + (lane >> 4) * 4;
          const float4 b4 = *(const float4*)&ebias[col];
          const float v[4] = {acc[i][j][0] + b4.x, acc[i][j][1] + b4.y, acc[i][j][2] + b4.z,
                              acc[i][j][3] + b4.w};
          epi_store4<EK>(epi, m, n0 + col, v);
        }
      }
    }
  } else if (CT) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int m = m0 + wm * WM + i * 16 + fr;
      if (m >= M) continue;
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int nb = n0 + wn * WN + j * 16 + (lane >> 4) * 4;
        if (vec_ok && nb + 3 < N) {
          const bf16x4 b4 = PART ? bf16x4{} : *(const bf16x4*)(bias + nb);
          const float v[4] = {acc[i][j][0] + (float)b4[0], acc[i][j][1] + (float)b4[1],
                              acc[i][j][2] + (float)b4[2], acc[i][j][3] + (float)b4[3]};
          epi_store4<EK>(epi, m, nb, v);
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (nb + r < N)
              epi_apply<bf16>(epi, EK, m, nb + r, acc[i][j][r] + (PART ? 0.f : (float)bias[nb + r]));
        }
      }
    }
  } else if (KIND == EPI_SPLIT_VT && whole_n && m0 + BM <= M && n0 >= epi.vcol0) {
    // a whole V tile: four consecutive tokens of one V column per store
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = n0 + wn * WN + j * 16 + fr;
      const float b = ebias[n - n0];
      bf16* vt = epi.vt + (size_t)(n - epi.vcol0) * epi.ldvt;
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int mb = m0 + wm * WM + i * 16 + (lane >> 4) * 4;
        bf16x4 v4;
#pragma unroll
        for (int r = 0; r < 4; ++r) v4[r] = (bf16)(acc[i][j][r] + b);
        *(bf16x4*)(vt + mb) = v4;
      }
    }
  } else if (KIND == EPI_SPLIT_VT && whole_n && m0 + BM <= M && n0 + BN <= epi.vcol0) {
    // a whole q|k tile: no per-element bounds or column-range tests (the
    // query columns scaled exactly as epi_apply scales them)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = n0 + wn * WN + j * 16 + fr;
      const float b = ebias[n - n0];
      const float qs = n < epi.qcols ? epi.qscale : 1.f;
      bf16* o = (bf16*)epi.out + n;
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int mb = m0 + wm * WM + i * 16 + (lane >> 4) * 4;
#pragma unroll
        for (int r = 0; r < 4; ++r) o[(size_t)(mb + r) * epi.ldo] = (bf16)((acc[i][j][r] + b) * qs);
      }
    }
  } else {
    // C fragment: lane holds column (lane & 15), rows 4*(lane >> 4) + 0..3
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = n0 + wn * WN + j * 16 + fr;
      if (n >= N) continue;
      const float b = whole_n ? ebias[n - n0] : (float)bias[n];
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int mb = m0 + wm * WM + i * 16 + (lane >> 4) * 4;
        if (KIND == EPI_SPLIT_VT && n >= epi.vcol0 && mb + 3 < M) {
          // four consecutive tokens of one V column: one 8-byte store into V^T
          bf16x4 v4;
#pragma unroll
          for (int r = 0; r < 4; ++r) v4[r] = (bf16)(acc[i][j][r] + b);
          *(bf16x4*)(epi.vt + (size_t)(n - epi.vcol0) * epi.ldvt + mb) = v4;
          continue;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int m = mb + r;
          if (m < M) epi_apply<bf16>(epi, KIND, m, n, acc[i][j][r] + b);
        }
      }
    }
  }
}

template <int BM, int BN, int WGM, int KIND>
__global__ __launch_bounds__(256, 1) void gemm_bf16_kernel(
    const bf16* __restrict__ A, int lda, const bf16* __restrict__ W, int ldw,
    const bf16* __restrict__ bias, int M, int N, int K, Epi epi, int tiles_n, int vec_ok) {
  // split-K: workgroup row blockIdx.y takes K columns [y K, (y+1) K) and
  // writes its partial sums to slice y of the fp32 output
  if (KIND == EPI_PARTIAL) {
    A += (size_t)blockIdx.y * K;
    W += (size_t)blockIdx.y * K;
    epi.out = (float*)epi.out + (size_t)blockIdx.y * M * epi.ldo;
  }
  gemm_bf16_body<BM, BN, WGM, KIND>(A, lda, W, ldw, bias, M, N, K, epi, tiles_n, vec_ok,
                                    xcd_remap(blockIdx.x, gridDim.x));
}

// One launch for several GEMMs that share A and the shape: group blockIdx.y
// takes its weight, bias and output pointers from the table.  Each tile is
// computed exactly as by gemm_bf16_kernel.
template <int BM, int BN, int WGM, int KIND>
__global__ __launch_bounds__(256, 1) void gemm_bf16_group_kernel(
    const bf16* __restrict__ A, int lda, PtrGroup g, int ldw, int M, int N, int K, Epi epi,
    int tiles_n, int vec_ok) {
  const int grp = blockIdx.y;
  epi.out = g.out[grp];
  epi.vt = g.vt[grp];
  gemm_bf16_body<BM, BN, WGM, KIND>(A, lda, (const bf16*)g.W[grp], ldw, (const bf16*)g.bias[grp],
                                    M, N, K, epi, tiles_n, vec_ok,
                                    xcd_remap(blockIdx.x, gridDim.x));
}

template <int BM, int BN, int WGM>
static hipError_t gemm_bf16_dispatch(const bf16* A, int lda, const bf16* W, int ldw,
                                     const bf16* bias, int M, int N, int K, int kind,
                                     const Epi& epi, int vec_ok, hipStream_t st, int splits = 1) {
  const int tn = (N + BN - 1) / BN, tm = (M + BM - 1) / BM;
  dim3 grid(tm * tn, splits), block(256);
#define T2I_GEMM_CASE(K_)                                                                       \
  case K_:                                                                                      \
    hipLaunchKernelGGL((gemm_bf16_kernel<BM, BN, WGM, K_>), grid, block, 0, st, A, lda, W, ldw, \
                       bias, M, N, K, epi, tn, vec_ok);                                         \
    break;
  switch (kind) {
    T2I_GEMM_CASE(EPI_STORE)
    T2I_GEMM_CASE(EPI_GELU)
    T2I_GEMM_CASE(EPI_SILU)
    T2I_GEMM_CASE(EPI_RESID)
    T2I_GEMM_CASE(EPI_RESID_GATED)
    T2I_GEMM_CASE(EPI_SPLIT_VT)
    T2I_GEMM_CASE(EPI_STORE_F32)
    T2I_GEMM_CASE(EPI_PARTIAL)
    default: return hipErrorInvalidValue;
  }
#undef T2I_GEMM_CASE
  return hipGetLastError();
}

// Split-K reduction: y = bias + sum over slices (fixed order), then the
// epilogue; four consecutive columns per thread.
template <int KIND>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float* __restrict__ part,
                                                            int splits, const bf16* __restrict__ bias,
                                                            int M, int N, Epi epi, int vec_ok) {
  const int nq = (N + 3) / 4;
  const long total = (long)M * nq;
  const size_t slice = (size_t)M * N;
  for (long i = blockIdx.x * 256L + threadIdx.x; i < total; i += (long)gridDim.x * 256) {
    const int m = (int)(i / nq), nb = (int)(i - (long)m * nq) * 4;
    const float* p = part + (size_t)m * N + nb;
    if (vec_ok && nb + 3 < N && KIND != EPI_SPLIT_VT) {
      const bf16x4 b4 = *(const bf16x4*)(bias + nb);
      float v[4] = {(float)b4[0], (float)b4[1], (float)b4[2], (float)b4[3]};
      for (int z = 0; z < splits; ++z) {
        const float4 q = *(const float4*)(p + z * slice);
        v[0] += q.x;
        v[1] += q.y;
        v[2] += q.z;
        v[3] += q.w;
      }
      epi_store4<KIND>(epi, m, nb, v);
    } else {
      for (int r = 0; r < 4 && nb + r < N; ++r) {
        float v = (float)bias[nb + r];
        for (int z = 0; z < splits; ++z) v += p[z * slice + r];
        epi_apply<bf16>(epi, KIND, m, nb + r, v);
      }
    }
  }
}

// Number of K slices (1 = no split) for a layer whose caller allows
// splitting: narrow outputs (N <= 4096) against K >= 2048, one slice per
// 1024 columns, at most 4.  It depends on the layer's shape only.  The launcher
// drops the split from 2048 rows on, and where the workspace does not hold the
// slices: a row's sums are those of any other row count on the same side of
// that line, and differ across it in their last bits.
static int splitk_factor(int N, int K) {
  if (N > 4096 || K < 2048) return 1;
  int s = std::min(4, K / 1024);
  while (s > 1 && K % (64 * s) != 0) --s;
  return s;
}

hipError_t launch_gemm_bf16(const bf16* A, int lda, const bf16* W, int ldw, const bf16* bias,
                            int M, int N, int K, int kind, const Epi& epi, float* splitk_ws,
                            size_t splitk_floats, hipStream_t st) {
  if (M <= 0 || N <= 0) return hipSuccess;
  auto al = [](const void* p, int a) { return ((uintptr_t)p % a) == 0; };
  const int vec_ok = (epi.ldo % 4 == 0) && (epi.ldx % 4 == 0) && (epi.ld_gate % 4 == 0) &&
                     al(bias, 8) && al(epi.out, kind == EPI_STORE_F32 ? 16 : 8) &&
                     al(epi.x, 16) && al(epi.xb, 8) && al(epi.gate, 16);
  // Direct HBM->LDS loads (gemm_dma.hip) for widths of whole tiles, with K
  // split over several workgroups where the caller allows it and a layer of
  // few rows against a long K would leave CUs idle (e.g. the 512-row text
  // stream against K = 3072 or 12288); register-staged tiles for other widths,
  // for operands past the direct loads' 32-bit byte offsets and for operands
  // that are not 16-byte aligned (a lane's direct load moves 16 bytes).
  const bool dma = (size_t)2 * M * lda < 0x7fffffff && (size_t)2 * N * ldw < 0x7fffffff &&
                   al(A, 16) && al(W, 16) && gemm_dma_fits(M, N);
  // (from 2048 rows on there are tiles enough without splitting K)
  int splits = splitk_ws && kind != EPI_SILU && !(dma && M >= 2048) ? splitk_factor(N, K) : 1;
  if ((size_t)splits * M * N > splitk_floats) splits = 1;
  if (splits == 1 && dma)
    return launch_gemm_dma(A, lda, W, ldw, bias, M, N, K, kind, epi, vec_ok, st);
  if (splits > 1) {
    Epi pe;
    std::memset(&pe, 0, sizeof(pe));
    pe.out = splitk_ws;
    pe.ldo = N;
    const int pvec = N % 4 == 0;
    // 64 x 64 register-staged tiles where 128-row tiles would leave most CUs
    // idle; same K order, same sums
    const long t128 = (long)((M + 127) / 128) * ((N + 127) / 128);
    hipError_t err =
        dma ? launch_gemm_dma(A, lda, W, ldw, bias, M, N, K / splits, EPI_PARTIAL, pe, pvec, st,
                              splits)
        : t128 * splits < 256
            ? gemm_bf16_dispatch<64, 64, 2>(A, lda, W, ldw, bias, M, N, K / splits, EPI_PARTIAL,
                                            pe, pvec, st, splits)
            : gemm_bf16_dispatch<128, 128, 2>(A, lda, W, ldw, bias, M, N, K / splits, EPI_PARTIAL,
                                              pe, pvec, st, splits);
    if (err != hipSuccess) return err;
    const long work = (long)M * ((N + 3) / 4);
    const int grid = (int)std::min<long>((work + 255) / 256, 4096);
#define T2I_RED_CASE(K_)                                                                   \
  case K_:                                                                                 \
    hipLaunchKernelGGL(splitk_reduce_kernel<K_>, dim3(grid), dim3(256), 0, st, splitk_ws, \
                       splits, bias, M, N, epi, vec_ok && pvec);                           \
    break;
    switch (kind) {
      T2I_RED_CASE(EPI_STORE)
      T2I_RED_CASE(EPI_GELU)
      T2I_RED_CASE(EPI_RESID)
      T2I_RED_CASE(EPI_RESID_GATED)
      T2I_RED_CASE(EPI_SPLIT_VT)
      T2I_RED_CASE(EPI_STORE_F32)
      default: return hipErrorInvalidValue;
    }
#undef T2I_RED_CASE
    return hipGetLastError();
  }
  // 128-row tiles unless they would leave CUs idle (e.g. 1024 rows x 1152
  // columns = 64 tiles); 64 x 64 tiles then (same K order, same results)
  const long tiles128 = (long)((M + 127) / 128) * ((N + (N % 144 == 0 ? 143 : 127)) /
                                                    (N % 144 == 0 ? 144 : 128));
  if (tiles128 < 256)
    return gemm_bf16_dispatch<64, 64, 2>(A, lda, W, ldw, bias, M, N, K, kind, epi, vec_ok, st);
  if (N % 144 == 0)
    return gemm_bf16_dispatch<128, 144, 4>(A, lda, W, ldw, bias, M, N, K, kind, epi, vec_ok, st);
  return gemm_bf16_dispatch<128, 128, 2>(A, lda, W, ldw, bias, M, N, K, kind, epi, vec_ok, st);
}

bool gemm_bf16_groupable(int M, int N, int kind) {
  // a grouped launch runs the register-staged tiles, with the sums of the single
  // launches; from 2048 rows on a launch of direct-load tiles fills the chip by
  // itself
  return M > 0 && N > 0 && !(M >= 2048 && (N % 144 == 0 || N % 128 == 0) && kind != EPI_SILU) &&
         (kind == EPI_STORE || kind == EPI_SPLIT_VT);
}

hipError_t launch_gemm_bf16_group(const bf16* A, int lda, const PtrGroup& g, int groups, int ldw,
                                  int M, int N, int K, int kind, const Epi& epi, hipStream_t st) {
  if (groups <= 0) return hipSuccess;
  if (groups > kMaxGroups || !gemm_bf16_groupable(M, N, kind)) return hipErrorInvalidValue;
  auto al = [](const void* p, int a) { return ((uintptr_t)p % a) == 0; };
  int vec_ok = (epi.ldo % 4 == 0) && (epi.ldx % 4 == 0) && (epi.ld_gate % 4 == 0);
  for (int i = 0; i < groups; ++i)
    vec_ok = vec_ok && al(g.bias[i], 8) && al(g.out[i], 8);
  dim3 block(256);
#define T2I_GRP(BM_, BN_, WGM_, K_)                                                          \
  {                                                                                          \
    const int tn = (N + BN_ - 1) / BN_, tm = (M + BM_ - 1) / BM_;                            \
    hipLaunchKernelGGL((gemm_bf16_group_kernel<BM_, BN_, WGM_, K_>), dim3(tm * tn, groups),  \
                       block, 0, st, A, lda, g, ldw, M, N, K, epi, tn, vec_ok);              \
  }
  if (N % 144 == 0) {
    if (kind == EPI_STORE) T2I_GRP(128, 144, 4, EPI_STORE) else T2I_GRP(128, 144, 4, EPI_SPLIT_VT)
  } else {
    if (kind == EPI_STORE) T2I_GRP(128, 128, 2, EPI_STORE) else T2I_GRP(128, 128, 2, EPI_SPLIT_VT)
  }
#undef T2I_GRP
  return hipGetLastError();
}

// ---------------------------------------------------------------------------

// fp32 GEMM on the fp32 matrix cores (v_mfma_f32_16x16x4_f32: fp32 products,
// fp32 accumulation), for the fp32 model's layers.  Bound by the matrix cores
// (157 TFLOP/s fp32) at the model's 1024 rows and by load latency at the
// smallest (64 rows).  1024 x 4608 x 1152 takes 91 us (119 TFLOP/s)
// where vector FMAs took 213, 1024 x 1152 x 4608 114 against 620, and 64 x 128
// x 512 6.8 against 62.
//
// 4 waves as 2 x 2 own a (32 TM) x (32 TN) tile.  K advances 32 floats (128
// bytes, 8 chunks of 16) at a time through a ring of four LDS stages filled by
// direct loads (buffer_load_dwordx4 ... lds: 8 rows per wave instruction), the
// 16-byte chunk c of row r in slot c ^ ((r >> 1) & 7) so that the 16 rows of a
// fragment read spread over the banks.  A lane reads four consecutive k of its
// row (chunk 4 kk + g) and MFMA e of the four takes component e: its k are
// {16 kk + 4 g + e, g = 0 .. 3} for both operands, so the products are those
// of k = 16 kk .. 16 kk + 15 and the order of the sums depends on K alone, not
// on the tile.  DMA = false: the same tiles and sums for operands that the
// direct loads cannot take (K % 32, unaligned rows, operands past 2 GiB),
// staged through registers with zeros past K.
constexpr int kF32Stages = 4;

template <int TM, int TN, bool DMA, int KIND>
__global__ __launch_bounds__(256) void gemm_f32_kernel(
    const float* __restrict__ A, int lda, const float* __restrict__ W, int ldw,
    const float* __restrict__ bias, int M, int N, int K, Epi epi, int tiles_m, int vec_ok) {
  constexpr int BM = 32 * TM, BN = 32 * TN, ST = DMA ? kF32Stages : 1;
  constexpr int BPW = (BM + BN) / 32;   // direct loads per wave and stage
  constexpr int STAGE = (BM + BN) * 32;  // floats
  __shared__ __attribute__((aligned(1024))) float smem[ST * STAGE];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int fr = lane & 15, g = lane >> 4;
  // row blocks vary fastest within an XCD's range of tiles: its workgroups
  // share few W rows, and A stays in its L2
  const int tile = xcd_remap(blockIdx.x, gridDim.x);
  const int m0 = (tile % tiles_m) * BM, n0 = (tile / tiles_m) * BN;
  const int wm0 = (wave >> 1) * 16 * TM, wn0 = (wave & 1) * 16 * TN;
  const int KT = (K + 31) / 32;

  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto frag = [&](const float* base, int row, int c) {
    return *(const f32x4*)((const char*)base + row * 128 + ((c ^ ((row >> 1) & 7)) << 4));
  };
  auto compute = [&](int slot) {
    const float* sA = smem + slot * STAGE;
    const float* sB = sA + BM * 32;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      f32x4 af[TM], bfr[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) af[i] = frag(sA, wm0 + i * 16 + fr, kk * 4 + g);
#pragma unroll
      for (int j = 0; j < TN; ++j) bfr[j] = frag(sB, wn0 + j * 16 + fr, kk * 4 + g);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(bfr[j][e], af[i][e], acc[i][j], 0, 0, 0);
    }
  };

  if constexpr (DMA) {
    uint32_t src[BPW];
    const __amdgpu_buffer_rsrc_t ra =
        __builtin_amdgcn_make_buffer_rsrc((void*)A, 0, 0x7fffffff, 0x00020000);
    const __amdgpu_buffer_rsrc_t rw =
        __builtin_amdgcn_make_buffer_rsrc((void*)W, 0, 0x7fffffff, 0x00020000);
#pragma unroll
    for (int i = 0; i < BPW; ++i) {
      const int blk = wave + 4 * i, lr = (i < TM ? blk : blk - BM / 8) * 8 + (lane >> 3);
      const int c = (lane & 7) ^ ((lr >> 1) & 7);
      // rows past the operand repeat its last one; their results are not stored
      src[i] = 4u * (uint32_t)(i < TM ? min(m0 + lr, M - 1) * lda : min(n0 + lr, N - 1) * ldw) +
               16u * (uint32_t)c;
    }
    auto issue = [&](int t, int slot) {
#pragma unroll
      for (int i = 0; i < BPW; ++i)
        load_lds16(i < TM ? ra : rw, (char*)(smem + slot * STAGE) + (wave + 4 * i) * 1024, src[i],
                   t * 128);
    };
#pragma unroll
    for (int s = 0; s < ST - 1; ++s)
      if (s < KT) issue(s, s);
    for (int t0 = 0; t0 < KT; t0 += ST) {
#pragma unroll
      for (int i = 0; i < ST; ++i) {
        const int t = t0 + i;
        if (t >= KT) break;
        // stage t landed (the stages after it may fly), and every wave is done
        // with stage t - 1, which is refilled now
        const int younger = min(ST - 2, KT - 1 - t);
        if (younger == 2) wait_vm<2 * BPW>();
        else if (younger == 1) wait_vm<BPW>();
        else wait_vm<0>();
        __builtin_amdgcn_s_waitcnt(0xC07F);   // this wave's LDS reads
        asm volatile("s_barrier" ::: "memory");
        if (t + ST - 1 < KT) issue(t + ST - 1, (i + ST - 1) % ST);
        compute(i);
      }
    }
  } else {
    for (int t = 0; t < KT; ++t) {
      for (int idx = tid; idx < (BM + BN) * 8; idx += 256) {
        const int row = idx >> 3, c = idx & 7, k = t * 32 + 4 * c;
        const bool is_a = row < BM;
        const int lr = is_a ? row : row - BM;
        const float* p = is_a ? A + (size_t)min(m0 + lr, M - 1) * lda
                              : W + (size_t)min(n0 + lr, N - 1) * ldw;
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = k + e < K ? p[k + e] : 0.f;
        *(f32x4*)((char*)smem + row * 128 + ((c ^ ((lr >> 1) & 7)) << 4)) = v;
      }
      __syncthreads();
      compute(0);
      __syncthreads();
    }
  }

  // a lane owns four consecutive columns of one row per fragment
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int m = m0 + wm0 + i * 16 + fr;
    if (m >= M) continue;
    const float* grow = nullptr;
    if constexpr (KIND == EPI_RESID_GATED)
      grow = epi.gate + (size_t)epi.map.modrow[seq_of_row(epi.map, m)] * epi.ld_gate;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = n0 + wn0 + j * 16 + g * 4;
      if (vec_ok && n + 3 < N) {
        const f32x4 b4 = *(const f32x4*)(bias + n);
        f32x4 y;
#pragma unroll
        for (int r = 0; r < 4; ++r) y[r] = acc[i][j][r] + b4[r];
        if constexpr (KIND == EPI_RESID || KIND == EPI_RESID_GATED) {
          float* xp = epi.x + (size_t)m * epi.ldx + n;
          f32x4 x4 = *(const f32x4*)xp;
          f32x4 g4 = f32x4{1.f, 1.f, 1.f, 1.f};
          if constexpr (KIND == EPI_RESID_GATED) g4 = *(const f32x4*)(grow + n);
#pragma unroll
          for (int r = 0; r < 4; ++r) x4[r] += g4[r] * y[r];
          *(f32x4*)xp = x4;
          if (epi.xb)
            *(bf16x4*)(epi.xb + (size_t)m * epi.ldx + n) =
                bf16x4{(bf16)x4[0], (bf16)x4[1], (bf16)x4[2], (bf16)x4[3]};
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            if (KIND == EPI_STORE && n + r < epi.qcols) y[r] *= epi.qscale;
            if (KIND == EPI_GELU) y[r] = gelu_tanh(y[r]);
            if (KIND == EPI_SILU) y[r] = silu(y[r]);
          }
          *(f32x4*)((float*)epi.out + (size_t)m * epi.ldo + n) = y;
        }
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (n + r < N) epi_apply<float>(epi, KIND, m, n + r, acc[i][j][r] + bias[n + r]);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Small-M linear layer (conditioning: timestep MLP and adaLN table, M = number
// of timesteps).  HBM-bound on the weights: each wave owns 4 output columns,
// lanes stream 16-byte chunks of the 4 weight rows once, multiply them with up
// to MT activation rows (fp32, L2-resident), and reduce across the wave.
// Weight reads are contiguous 1 KB per wave instruction.

// NC columns per wave.  With one column (the timestep MLP: few workgroups) all
// loads of a step, weights and every row, rows past the last repeated, are
// issued before its arithmetic, so that they cost one latency and not one per
// row (1152 x 1152: 13.9 -> 7.1 us for 5 rows, 19.8 -> 11.0 for 20, with one
// column per wave 6.4 -> 5.1 for one).  With four (the adaLN table, a workgroup
// for every 16 of its columns) the chip is full and the waves per SIMD hide the
// latency: rows are loaded where they are used, 86 registers and 5 waves for
// 8 rows.  Loading them first took 142 and left 3 waves: the table of 28 blocks
// of width 1152 took 729 instead of 513 us for 20 rows, 296 instead of 232 for
// 8, 82 instead of 80 for one; 40 blocks of width 3072 5876 instead of 4416 for
// 28; four rows at a time lie between (559 us for 20 rows).
template <typename TW, int MT, int NC, int KIND>
__device__ __forceinline__ void linear_rows_body(const float* __restrict__ A, int lda,
                                                 const TW* __restrict__ W, int ldw,
                                                 const TW* __restrict__ bias, int M, int N, int K,
                                                 const Epi& epi) {
  const int lane = threadIdx.x & 63;
  const int n0 = (blockIdx.y * 4 + (threadIdx.x >> 6)) * NC;
  const int m0 = blockIdx.x * MT;
  if (n0 >= N) return;
  const int mt = min(MT, M - m0);
  float acc[MT][NC];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int j = 0; j < NC; ++j) acc[m][j] = 0.f;
#pragma unroll(NC == 1 && MT <= 2 ? 4 : 1)
  for (int k = lane * 8; k < K; k += 64 * 8) {
    float wv[NC][8];
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      const int n = min(n0 + j, N - 1);
      const TW* wp = W + (size_t)n * ldw + k;
      if constexpr (sizeof(TW) == 2) {
        const bf16x8 v = *(const bf16x8*)wp;
#pragma unroll
        for (int e = 0; e < 8; ++e) wv[j][e] = (float)v[e];
      } else {
        const float4 a = *(const float4*)wp, b = *(const float4*)(wp + 4);
        wv[j][0] = a.x; wv[j][1] = a.y; wv[j][2] = a.z; wv[j][3] = a.w;
        wv[j][4] = b.x; wv[j][5] = b.y; wv[j][6] = b.z; wv[j][7] = b.w;
      }
    }
    auto add_row = [&](int m, float4 a, float4 b) {
      const float av[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
      for (int j = 0; j < NC; ++j)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[m][j] = fmaf(av[e], wv[j][e], acc[m][j]);
    };
    if constexpr (NC == 1) {
      float4 a[MT], b[MT];
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        const float* ap = A + (size_t)(m0 + min(m, mt - 1)) * lda + k;
        a[m] = *(const float4*)ap;
        b[m] = *(const float4*)(ap + 4);
      }
#pragma unroll
      for (int m = 0; m < MT; ++m)
        if (m < mt) add_row(m, a[m], b[m]);
    } else {
#pragma unroll
      for (int m = 0; m < MT; ++m)
        if (m < mt) {
          const float* ap = A + (size_t)(m0 + m) * lda + k;
          add_row(m, *(const float4*)ap, *(const float4*)(ap + 4));
        }
    }
  }
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    if (m >= mt) break;
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      const float v = wave_sum(acc[m][j]);
      if (lane == 0 && n0 + j < N) epi_apply<float>(epi, KIND, m0 + m, n0 + j, v + to_f32(bias[n0 + j]));
    }
  }
}

template <typename TW, int MT, int NC, int KIND>
__global__ __launch_bounds__(256) void linear_rows_kernel(const float* __restrict__ A, int lda,
                                                          const TW* __restrict__ W, int ldw,
                                                          const TW* __restrict__ bias, int M,
                                                          int N, int K, Epi epi) {
  linear_rows_body<TW, MT, NC, KIND>(A, lda, W, ldw, bias, M, N, K, epi);
}

// Several weight matrices against the same rows in one launch: group
// blockIdx.z takes its weight, bias and output from the table.
template <typename TW, int MT, int KIND>
__global__ __launch_bounds__(256) void linear_rows_group_kernel(const float* __restrict__ A,
                                                                int lda, PtrGroup g, int ldw,
                                                                int M, int N, int n_last, int K,
                                                                Epi epi) {
  const int grp = blockIdx.z;
  epi.out = g.out[grp];
  linear_rows_body<TW, MT, 4, KIND>(A, lda, (const TW*)g.W[grp], ldw, (const TW*)g.bias[grp], M,
                                    grp + 1 == (int)gridDim.z ? n_last : N, K, epi);
}

// Rows per weight pass: as few as hold M (fewer registers, so more waves
// stream weights at once), at most 8.  Each row's sums are the same in all.
inline int rows_per_pass(int M) { return M <= 2 ? 2 : M <= 4 ? 4 : 8; }

template <typename TW, int MT>
static hipError_t linear_rows_dispatch(const float* A, int lda, const TW* W, int ldw,
                                       const TW* bias, int M, int N, int K, int kind,
                                       const Epi& epi, hipStream_t st) {
  // consecutive workgroups share weight rows (row passes vary fastest).  Four
  // columns per wave read the rows once for all of them, but up to 4096
  // columns (the timestep MLP) that leaves most CUs idle: one there
  const int nc = N > 4096 && kind == EPI_STORE ? 4 : 1;
  dim3 grid((M + MT - 1) / MT, (N + 4 * nc - 1) / (4 * nc)), block(256);
  switch (kind) {
    case EPI_STORE:
      if (nc == 4)
        hipLaunchKernelGGL((linear_rows_kernel<TW, MT, 4, EPI_STORE>), grid, block, 0, st, A, lda, W, ldw, bias, M, N, K, epi);
      else
        hipLaunchKernelGGL((linear_rows_kernel<TW, MT, 1, EPI_STORE>), grid, block, 0, st, A, lda, W, ldw, bias, M, N, K, epi);
      break;
    case EPI_SILU:
      hipLaunchKernelGGL((linear_rows_kernel<TW, MT, 1, EPI_SILU>), grid, block, 0, st, A, lda, W, ldw, bias, M, N, K, epi);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_linear_rows_group(const float* A, int lda, const PtrGroup& g, int groups,
                                    int ldw, bool w_bf16, int M, int N, int n_last, int K,
                                    const Epi& epi, hipStream_t st) {
  if (groups <= 0 || M <= 0 || N <= 0) return hipSuccess;
  if (groups > kMaxGroups || n_last > N || K % 8 || lda % 4 || ldw % 8 || ((uintptr_t)A & 15))
    return hipErrorInvalidValue;
  for (int i = 0; i < groups; ++i)
    if ((uintptr_t)g.W[i] & 15) return hipErrorInvalidValue;
  const int mt = rows_per_pass(M);
  dim3 grid((M + mt - 1) / mt, (N + 15) / 16, groups), block(256);
#define T2I_ROWS(TW_, MT_)                                                                      \
  hipLaunchKernelGGL((linear_rows_group_kernel<TW_, MT_, EPI_STORE>), grid, block, 0, st, A, lda, \
                     g, ldw, M, N, n_last, K, epi)
  if (w_bf16) {
    if (mt == 2) T2I_ROWS(bf16, 2);
    else if (mt == 4) T2I_ROWS(bf16, 4);
    else T2I_ROWS(bf16, 8);
  } else {
    if (mt == 2) T2I_ROWS(float, 2);
    else if (mt == 4) T2I_ROWS(float, 4);
    else T2I_ROWS(float, 8);
  }
#undef T2I_ROWS
  return hipGetLastError();
}

hipError_t launch_linear_rows(const float* A, int lda, const void* W, int ldw, bool w_bf16,
                              const void* bias, int M, int N, int K, int kind, const Epi& epi,
                              hipStream_t st) {
  if (M <= 0 || N <= 0) return hipSuccess;
  if ((kind != EPI_STORE && kind != EPI_SILU) || K % 8 || lda % 4 || ldw % 8 ||
      ((uintptr_t)A & 15) || ((uintptr_t)W & 15))
    return hipErrorInvalidValue;
#define T2I_ROWS(TW_, MT_)                                                                       \
  return linear_rows_dispatch<TW_, MT_>(A, lda, (const TW_*)W, ldw, (const TW_*)bias, M, N, K, kind, \
                                        epi, st)
  const int mt = rows_per_pass(M);
  if (w_bf16) {
    if (mt == 2) T2I_ROWS(bf16, 2);
    if (mt == 4) T2I_ROWS(bf16, 4);
    T2I_ROWS(bf16, 8);
  }
  if (mt == 2) T2I_ROWS(float, 2);
  if (mt == 4) T2I_ROWS(float, 4);
  T2I_ROWS(float, 8);
#undef T2I_ROWS
}

template <int TM, int TN, bool DMA>
static hipError_t gemm_f32_dispatch(const float* A, int lda, const float* W, int ldw,
                                    const float* bias, int M, int N, int K, int kind,
                                    const Epi& epi, int vec_ok, hipStream_t st) {
  const int tm = (M + 32 * TM - 1) / (32 * TM), tn = (N + 32 * TN - 1) / (32 * TN);
  dim3 grid(tm * tn), block(256);
#define T2I_F32_CASE(K_)                                                                       \
  case K_:                                                                                     \
    hipLaunchKernelGGL((gemm_f32_kernel<TM, TN, DMA, K_>), grid, block, 0, st, A, lda, W, ldw, \
                       bias, M, N, K, epi, tm, vec_ok);                                        \
    break;
  switch (kind) {
    T2I_F32_CASE(EPI_STORE)
    T2I_F32_CASE(EPI_GELU)
    T2I_F32_CASE(EPI_SILU)
    T2I_F32_CASE(EPI_RESID)
    T2I_F32_CASE(EPI_RESID_GATED)
    default: return hipErrorInvalidValue;
  }
#undef T2I_F32_CASE
  return hipGetLastError();
}

hipError_t launch_gemm_f32(const float* A, int lda, const float* W, int ldw, const float* bias,
                           int M, int N, int K, int kind, const Epi& epi, hipStream_t st) {
  if (M <= 0 || N <= 0) return hipSuccess;
  auto al = [](const void* p) { return ((uintptr_t)p % 16) == 0; };
  const int vec_ok = epi.ldo % 4 == 0 && epi.ldx % 4 == 0 && epi.ld_gate % 4 == 0 && al(bias) &&
                     al(epi.out) && al(epi.x) && al(epi.xb) && al(epi.gate);
  // the direct loads take whole 128-byte K steps of 16-byte aligned rows and
  // address each operand with 32-bit byte offsets
  const bool dma = K % 32 == 0 && lda % 4 == 0 && ldw % 4 == 0 && al(A) && al(W) &&
                   (size_t)4 * M * lda < 0x7fffffff && (size_t)4 * N * ldw < 0x7fffffff;
  if (!dma) {
    // 64 x 64 tiles from two per CU on (4096 x 1024 x 1001: 146 us, 205 on 32 x
    // 32; 1024 x 1024 x 1001, one per CU: 81 against 55)
    if ((long)((M + 63) / 64) * ((N + 63) / 64) < 512)
      return gemm_f32_dispatch<1, 1, false>(A, lda, W, ldw, bias, M, N, K, kind, epi, vec_ok, st);
    return gemm_f32_dispatch<2, 2, false>(A, lda, W, ldw, bias, M, N, K, kind, epi, vec_ok, st);
  }
  // The CU with the most tiles decides: the matrix time of its tiles, which is
  // their area.  (Charging their loads too, at 20 bytes per clock, takes larger
  // tiles and was slower at 1024 rows and fewer: 1024 x 3456 x 1152 79 against
  // 72 us, 333 x 2048 x 2048 43 against 32; faster only at some shapes of 2048
  // rows, 2048 x 3456 x 1152 138 against 157.)
  auto cost = [&](long bm, long bn) {
    const long tiles = ((M + bm - 1) / bm) * ((N + bn - 1) / bn);
    return (tiles + 255) / 256 * bm * bn;
  };
  const long c22 = cost(64, 64), c12 = cost(32, 64), c11 = cost(32, 32);
  if (c22 <= c12 && c22 <= c11)
    return gemm_f32_dispatch<2, 2, true>(A, lda, W, ldw, bias, M, N, K, kind, epi, vec_ok, st);
  if (c12 <= c11)
    return gemm_f32_dispatch<1, 2, true>(A, lda, W, ldw, bias, M, N, K, kind, epi, vec_ok, st);
  return gemm_f32_dispatch<1, 1, true>(A, lda, W, ldw, bias, M, N, K, kind, epi, vec_ok, st);
}

}  // namespace t2i
