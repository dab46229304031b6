// HBM-bound kernels of the denoising step on gfx950: patch + position
// embedding, timestep sinusoid, LayerNorm fused with adaLN modulation, the
// final layer fused with unpatchify + classifier-free guidance + Euler update,
// and the step-skip cache reductions.
//
// Row kernels use one 64-lane wave per row with float4 loads (a row of
// D = 1152 floats is 4.5 KB: lane i reads float4 i, i+64, ...), so every load
// instruction of a wave covers 1 KB of contiguous memory.  Reductions run in
// registers with a fixed butterfly order, so results are bitwise reproducible.
#include <algorithm>

#include "t2i_internal.h"

namespace t2i {

constexpr int kMaxV4 = 12;   // float4 per lane: rows up to 3072 wide

// ---------------------------------------------------------------------------
// LayerNorm (biased variance, no affine) + modulation.

// Sum over the 64 lanes of a wave, the same value in every lane: DPP steps
// inside each 16-lane row, then the four row sums read out in a fixed order.
__device__ __forceinline__ float wave_sum_dpp(float v) {
  auto add_dpp = [](float x, int y) { return x + __int_as_float(y); };
  v = add_dpp(v, __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, false));  // quad_perm 1,0,3,2
  v = add_dpp(v, __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xF, 0xF, false));  // quad_perm 2,3,0,1
  v = add_dpp(v, __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x124, 0xF, 0xF, false)); // row_ror 4
  v = add_dpp(v, __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xF, 0xF, false)); // row_ror 8
  const int b = __float_as_int(v);
  return (__int_as_float(__builtin_amdgcn_readlane(b, 0)) +
          __int_as_float(__builtin_amdgcn_readlane(b, 16))) +
         (__int_as_float(__builtin_amdgcn_readlane(b, 32)) +
          __int_as_float(__builtin_amdgcn_readlane(b, 48)));
}

// One wave per row, four rows per workgroup: many small independent waves
// keep enough loads in flight (the kernel is bound by memory latency).
constexpr int kLnRows = 4;

// NV: float4 per row known at compile time (0 = any width up to kMaxV4 * 256),
// so that registers are sized for the row.  The modulation rows are loaded
// together with the row, before the reductions that they do not depend on.
template <typename OutT, int NV>
__global__ __launch_bounds__(256) void ln_mod_kernel(const float* __restrict__ x, int ldx, int rows,
                                                     int D, const float* __restrict__ mod,
                                                     int ld_mod, int shift_off, int scale_off,
                                                     SeqMap map, OutT* __restrict__ out, int ldo,
                                                     float eps) {
  constexpr int NI = NV ? (NV + 63) / 64 : kMaxV4;
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * kLnRows + (threadIdx.x >> 6);
  if (row >= rows) return;
  const int nv = NV ? NV : D >> 2;
  const float4* xr = (const float4*)(x + (size_t)row * ldx);
  const float* md = mod + (size_t)map.modrow[seq_of_row(map, row)] * ld_mod;
  const float4* sh = (const float4*)(md + shift_off);
  const float4* sc = (const float4*)(md + scale_off);
  // (any-width instances load the modulation rows at their use, which keeps
  // their register count down)
  constexpr bool PRE = NV != 0;
  float4 v[NI], shv[PRE ? NI : 1], scv[PRE ? NI : 1];
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int c = lane + 64 * i;
    if (c < nv) {
      v[i] = xr[c];
      if constexpr (PRE) {
        shv[i] = sh[c];
        scv[i] = sc[c];
      }
    }
  }
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int c = lane + 64 * i;
    if (c < nv) s += (v[i].x + v[i].y) + (v[i].z + v[i].w);
  }
  const float mean = wave_sum_dpp(s) / (float)D;
  float q = 0.f;
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int c = lane + 64 * i;
    if (c < nv) {
      const float a = v[i].x - mean, b = v[i].y - mean, cc = v[i].z - mean, d = v[i].w - mean;
      q += (a * a + b * b) + (cc * cc + d * d);
    }
  }
  const float rstd = 1.0f / sqrtf(wave_sum_dpp(q) / (float)D + eps);
  OutT* orow = out + (size_t)row * ldo;
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int c = lane + 64 * i;
    if (c < nv) {
      const float4 a = PRE ? shv[PRE ? i : 0] : sh[c], b = PRE ? scv[PRE ? i : 0] : sc[c];
      const float y0 = (v[i].x - mean) * rstd * (1.f + b.x) + a.x;
      const float y1 = (v[i].y - mean) * rstd * (1.f + b.y) + a.y;
      const float y2 = (v[i].z - mean) * rstd * (1.f + b.z) + a.z;
      const float y3 = (v[i].w - mean) * rstd * (1.f + b.w) + a.w;
      if constexpr (sizeof(OutT) == 2)     // one 8-byte store of four bf16
        *(bf16x4*)(orow + 4 * c) = bf16x4{(bf16)y0, (bf16)y1, (bf16)y2, (bf16)y3};
      else
        *(float4*)(orow + 4 * c) = float4{y0, y1, y2, y3};
    }
  }
}

// RW consecutive rows per wave (D = 1152, RW = 2): the first row and the
// modulation rows are loaded first, then each row's successor before its
// reductions and stores, so the first row's arithmetic starts as early as
// possible and reads and writes overlap.  With two rows per wave the launch
// fits one round of the chip's wave slots (one wave per row leaves a partial
// second round; more rows per wave measured slower: 4 rows as fast as the
// two-row kernel that loaded both rows first, 8 rows 25 % slower).  The
// modulation rows are reloaded only when the sequence changes.  Per-row
// arithmetic as in ln_mod_kernel (bitwise equal).
template <typename OutT, int NV, int RW>
__global__ __launch_bounds__(256) void ln_modr_kernel(const float* __restrict__ x, int ldx, int rows,
                                                      int D, const float* __restrict__ mod,
                                                      int ld_mod, int shift_off, int scale_off,
                                                      SeqMap map, OutT* __restrict__ out, int ldo,
                                                      float eps) {
  constexpr int NI = (NV + 63) / 64;
  const int lane = threadIdx.x & 63;
  const int r0 = (blockIdx.x * kLnRows + (threadIdx.x >> 6)) * RW;
  if (r0 >= rows) return;
  const int rn = min(RW, rows - r0);
  float4 v[2][NI], shv[NI], scv[NI];
  auto load_row = [&](float4 (&b)[NI], int row) {
    const float4* xr = (const float4*)(x + (size_t)row * ldx);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = lane + 64 * i;
      if (c < NV) b[i] = xr[c];
    }
  };
  auto load_mod = [&](int mr) {
    const float4* sh = (const float4*)(mod + (size_t)mr * ld_mod + shift_off);
    const float4* sc = (const float4*)(mod + (size_t)mr * ld_mod + scale_off);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = lane + 64 * i;
      if (c < NV) {
        shv[i] = sh[c];
        scv[i] = sc[c];
      }
    }
  };
  load_row(v[0], r0);
  int mcur = map.modrow[seq_of_row(map, r0)];
  load_mod(mcur);
#pragma unroll
  for (int r = 0; r < RW; ++r) {
    if (r >= rn) break;
    if (r + 1 < rn) load_row(v[(r + 1) & 1], r0 + r + 1);
    if (r > 0) {
      const int mr = map.modrow[seq_of_row(map, r0 + r)];
      if (mr != mcur) {
        load_mod(mr);
        mcur = mr;
      }
    }
    const float4* vr = v[r & 1];
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = lane + 64 * i;
      if (c < NV) s += (vr[i].x + vr[i].y) + (vr[i].z + vr[i].w);
    }
    const float mean = wave_sum_dpp(s) / (float)D;
    float q = 0.f;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = lane + 64 * i;
      if (c < NV) {
        const float a = vr[i].x - mean, b = vr[i].y - mean, cc = vr[i].z - mean, d = vr[i].w - mean;
        q += (a * a + b * b) + (cc * cc + d * d);
      }
    }
    const float rstd = 1.0f / sqrtf(wave_sum_dpp(q) / (float)D + eps);
    OutT* orow = out + (size_t)(r0 + r) * ldo;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = lane + 64 * i;
      if (c < NV) {
        const float4 a = shv[i], b = scv[i];
        const float y0 = (vr[i].x - mean) * rstd * (1.f + b.x) + a.x;
        const float y1 = (vr[i].y - mean) * rstd * (1.f + b.y) + a.y;
        const float y2 = (vr[i].z - mean) * rstd * (1.f + b.z) + a.z;
        const float y3 = (vr[i].w - mean) * rstd * (1.f + b.w) + a.w;
        if constexpr (sizeof(OutT) == 2)
          *(bf16x4*)(orow + 4 * c) = bf16x4{(bf16)y0, (bf16)y1, (bf16)y2, (bf16)y3};
        else
          *(float4*)(orow + 4 * c) = float4{y0, y1, y2, y3};
      }
    }
  }
}

hipError_t launch_ln_modulate(bool bf16_out, int rows, int D, const float* x, int ldx,
                              const float* mod, int ld_mod, int shift_off, int scale_off,
                              const SeqMap& map, void* out, int ldo, float eps, hipStream_t st) {
  if (rows <= 0) return hipSuccess;
  dim3 grid((rows + kLnRows - 1) / kLnRows), block(256);
#define T2I_LN(T_, NV_)                                                                      \
  hipLaunchKernelGGL((ln_mod_kernel<T_, NV_>), grid, block, 0, st, x, ldx, rows, D, mod, ld_mod, \
                     shift_off, scale_off, map, (T_*)out, ldo, eps)
  if (bf16_out) {
    if (D == 1152) {
      constexpr int RW = 2;
      hipLaunchKernelGGL((ln_modr_kernel<bf16, 288, RW>), dim3((rows + RW * kLnRows - 1) / (RW * kLnRows)),
                         block, 0, st, x, ldx, rows, D, mod, ld_mod, shift_off, scale_off, map,
                         (bf16*)out, ldo, eps);
      return hipGetLastError();
    }
    if (D == 3072) T2I_LN(bf16, 768);
    else T2I_LN(bf16, 0);
  } else {
    T2I_LN(float, 0);
  }
#undef T2I_LN
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Patchify + patch embedding (+ 2D sin-cos position embedding).
// Token i*(w/p)+j of a request reads latent [c, i*p+a, j*p+b] as feature
// (a*p+b)*C+c.  Writes x0 (one copy, unless NULL) and `copies` copies into x
// (one per guidance branch, branch-major).
//
// The position table (launch_call_tables) holds (sin, cos)(pos * 10000^(-f/qd)),
// qd = D/4.  The first D/2 channels add the row's sin-cos embedding, the last
// D/2 the column's; within a half the first D/4 are sin, the next D/4 cos.

// embed_mfma_kernel (P a multiple of 16): a workgroup takes 16 tokens x 16 ET
// channels per wave on v_mfma_f32_16x16x4_f32 (fp32 patches, weights widened to
// fp32).  That instruction is a chain of four fused multiply-adds, lane group 0
// first, so with MFMA m of a 16-feature chunk taking features 4 m + g every
// channel is its bias plus the products in ascending order, bit for bit what
// embed_kernel computes.  The patches are gathered into LDS once and kept in
// registers as the token operand; with the weights as the row operand a lane
// ends with four consecutive channels of one token; the tile leaves along the
// rows.  Bound by the stores:
// 14 us at 4096 tokens x 2 branches of width 1152 (one channel per thread with
// the patches read from LDS: 16.6), 48 at 4096 tokens of width 3072 (53).
// embed_kernel: any other P <= 64, one channel per thread.

// Four consecutive values per lane -> o[m] of lane group g (lanes 16 g .. 16 g +
// 15) = value g of lane group m, in fp32: the two lane bits trade places with
// the two index bits (bf16: the upper index bit while two values share a
// register).
__device__ __forceinline__ void swap16(float& a, float& b) {
  const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  a = __uint_as_float(p[0]);
  b = __uint_as_float(p[1]);
}
__device__ __forceinline__ void transpose_groups(bf16x4 q, float (&o)[4]) {
  union {
    bf16x4 v;
    uint32_t u[2];
  } x = {q};
  const auto p = __builtin_amdgcn_permlane32_swap(x.u[0], x.u[1], false, false);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    o[2 * h] = __uint_as_float(p[h] << 16);
    o[2 * h + 1] = __uint_as_float(p[h] & 0xffff0000u);
    swap16(o[2 * h], o[2 * h + 1]);
  }
}
__device__ __forceinline__ void transpose_groups(f32x4 q, float (&o)[4]) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(q[h]), __float_as_uint(q[2 + h]),
                                                    false, false);
    o[h] = __uint_as_float(p[0]);
    o[2 + h] = __uint_as_float(p[1]);
  }
  swap16(o[0], o[1]);
  swap16(o[2], o[3]);
}

// the 16-token patch gather both kernels start with: patch[t][(a p + b) C + c],
// and each token's grid position
template <int TOK, int PITCH>
struct EmbedTokens {
  float patch[TOK][PITCH];
  long long base[TOK];
  int w[TOK], hw[TOK], pos[TOK][2];
};

template <int TOK, int PITCH>
__device__ __forceinline__ void gather_patches(EmbedTokens<TOK, PITCH>& e, const float* lat,
                                               const ReqMap& rm, int t0, int P, int C, int p) {
  // each token's patch origin in its request's latent, once
  if (threadIdx.x < TOK) {
    const int t = threadIdx.x, tok = t0 + t;
    long long base = -1;
    int W = 0, HW = 0, gi = 0, gj = 0;
    if (tok < rm.tokens_total) {
      const int r = req_of_token(rm, tok);
      const int lt = tok - rm.tok_off[r];
      W = rm.w[r];
      HW = rm.h[r] * W;
      const int gw = W / p;
      gi = lt / gw;
      gj = lt - gi * gw;
      base = rm.lat_off[r] + (long long)(gi * p) * W + gj * p;
    }
    e.pos[t][0] = gi;
    e.pos[t][1] = gj;
    e.base[t] = base;
    e.w[t] = W;
    e.hw[t] = HW;
  }
  __syncthreads();
  // element (t, k = (a p + b) C + c) in the order (c, a, t, b): the pixels of
  // neighbouring threads are neighbours in a latent row
  for (int i = threadIdx.x; i < TOK * P; i += 256) {
    const int b = i % p, rest = i / p;
    const int t = rest % TOK, ca = rest / TOK;
    const int a = ca % p, c = ca / p;
    float v = 0.f;
    if (e.base[t] >= 0) v = lat[e.base[t] + (long long)c * e.hw[t] + (long long)a * e.w[t] + b];
    e.patch[t][(a * p + b) * C + c] = v;
  }
  __syncthreads();
}

// KC: P / 16.  x0 may be NULL (no copy wanted besides x).
template <typename TW, int KC, int ET>
__global__ __launch_bounds__(256) void embed_mfma_kernel(const float* __restrict__ lat, ReqMap rm,
                                                         const TW* __restrict__ w_pe,
                                                         const TW* __restrict__ b_pe, int D, int C,
                                                         int p, const float2* __restrict__ pe,
                                                         float* __restrict__ x0,
                                                         float* __restrict__ x, int copies) {
  constexpr int P = 16 * KC;
  __shared__ __attribute__((aligned(16))) EmbedTokens<16, P + 4> es;
  const int lane = threadIdx.x & 63, fr = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // the workgroups of a token tile are neighbours, all in grid x (grid y ends at
  // 65535 workgroups, a million tokens)
  const int gy = (D + 64 * ET - 1) / (64 * ET), tile = blockIdx.x / gy;
  const int T = rm.tokens_total, t0 = tile * 16;
  const int qd = D / 4, d00 = (((int)blockIdx.x - tile * gy) * 4 + wave) * ET * 16;
  // the wave's weights and biases, fetched while the patches are gathered
  // (channel tiles past D repeat the last one and are not stored)
  typedef TW tw4 __attribute__((ext_vector_type(4)));
  tw4 w[ET][KC];
  float add[ET][4];
#pragma unroll
  for (int j = 0; j < ET; ++j) {
    const int d0 = min(d00 + j * 16, D - 16);
    const TW* wr = w_pe + (size_t)(d0 + fr) * P + 4 * g;
#pragma unroll
    for (int c = 0; c < KC; ++c) w[j][c] = *(const tw4*)(wr + 16 * c);
#pragma unroll
    for (int e = 0; e < 4; ++e) add[j][e] = to_f32(b_pe[d0 + 4 * g + e]);
  }
  gather_patches(es, lat, rm, t0, P, C, p);
  float pf[KC][4];
#pragma unroll
  for (int c = 0; c < KC; ++c)
#pragma unroll
    for (int m = 0; m < 4; ++m) pf[c][m] = es.patch[fr][16 * c + 4 * m + g];
  float pos[ET][4];
  if (pe) {
    // D / 4 is a multiple of 16: a lane's four channels lie in one of the four
    // parts (row sin, row cos, column sin, column cos)
#pragma unroll
    for (int j = 0; j < ET; ++j) {
      const int d = min(d00 + j * 16, D - 16) + 4 * g;
      const int part = d / qd, f = d - part * qd;
      const float4* sc = (const float4*)(pe + (size_t)es.pos[fr][part >> 1] * qd + f);
      const float4 s0 = sc[0], s1 = sc[1];
      pos[j][0] = part & 1 ? s0.y : s0.x;
      pos[j][1] = part & 1 ? s0.w : s0.z;
      pos[j][2] = part & 1 ? s1.y : s1.x;
      pos[j][3] = part & 1 ? s1.w : s1.z;
    }
  }
  // the wave's 16 tokens x 16 ET channels through its own part of LDS, so that
  // they go out along the rows (a fragment's store would write 16 rows x 64
  // bytes)
  constexpr int SP = 16 * ET + 4;
  __shared__ __attribute__((aligned(16))) float stage[4][16 * SP];
  float* const sw = stage[wave];
#pragma unroll
  for (int j = 0; j < ET; ++j) {
    f32x4 acc = f32x4{add[j][0], add[j][1], add[j][2], add[j][3]};
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      float wt[4];
      transpose_groups(w[j][c], wt);
#pragma unroll
      for (int m = 0; m < 4; ++m)
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wt[m], pf[c][m], acc, 0, 0, 0);
    }
    if (pe) {
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] += pos[j][e];
    }
    *(f32x4*)&sw[fr * SP + j * 16 + 4 * g] = acc;
  }
#pragma unroll
  for (int i = 0; i < ET; ++i) {
    const int idx = i * 64 + lane, t = idx / (4 * ET), c = 4 * (idx - t * 4 * ET);
    if (t0 + t < T && d00 + c < D) {
      const f32x4 y = *(const f32x4*)&sw[t * SP + c];
      const size_t o = (size_t)(t0 + t) * D + d00 + c;
      if (x0) *(f32x4*)(x0 + o) = y;
      for (int cp = 0; cp < copies; ++cp) *(f32x4*)(x + (size_t)cp * T * D + o) = y;
    }
  }
}

// 8 tokens per workgroup, one channel per thread, its weight row in registers
constexpr int kEmbTok = 8;

template <typename TW>
__global__ __launch_bounds__(256) void embed_kernel(const float* __restrict__ lat, ReqMap rm,
                                                    const TW* __restrict__ w_pe,
                                                    const TW* __restrict__ b_pe, int D, int C,
                                                    int p, const float2* __restrict__ pe,
                                                    float* __restrict__ x0, float* __restrict__ x,
                                                    int copies) {
  __shared__ __attribute__((aligned(16))) EmbedTokens<kEmbTok, 68> es;
  const int P = p * p * C;
  const int T = rm.tokens_total;
  const int t0 = blockIdx.x * kEmbTok, d = blockIdx.y * 256 + threadIdx.x;
  gather_patches(es, lat, rm, t0, P, C, p);
  if (d >= D) return;
  float w[64];
#pragma unroll
  for (int k = 0; k < 64; ++k) w[k] = k < P ? to_f32(w_pe[(size_t)d * P + k]) : 0.f;
  const float bias = to_f32(b_pe[d]);
  const int half = D / 2, qd = D / 4, kk = d % half, f = kk % qd;
  for (int t = 0; t < kEmbTok; ++t) {
    const int tok = t0 + t;
    if (tok >= T) break;
    float acc = bias;
#pragma unroll
    for (int k = 0; k < 64; ++k)
      if (k < P) acc = fmaf(w[k], es.patch[t][k], acc);
    if (pe) {
      const float2 sc = pe[es.pos[t][d < half ? 0 : 1] * qd + f];
      acc += kk < qd ? sc.x : sc.y;
    }
    if (x0) x0[(size_t)tok * D + d] = acc;
    for (int cp = 0; cp < copies; ++cp) x[((size_t)cp * T + tok) * D + d] = acc;
  }
}

hipError_t launch_embed(const float* lat, const ReqMap& rm, const void* w_pe, const void* b_pe,
                        bool w_bf16, int D, int C, int p, const float2* pe_table, float* x0,
                        float* x, int copies, hipStream_t st) {
  if (rm.tokens_total == 0) return hipSuccess;
  const int P = p * p * C, T = rm.tokens_total;
#define T2I_EMB(K_, TW_, GX_, GY_)                                                             \
  hipLaunchKernelGGL(K_, dim3(GX_, GY_), dim3(256), 0, st, lat, rm, (const TW_*)w_pe,          \
                     (const TW_*)b_pe, D, C, p, pe_table, x0, x, copies)
  // 6 channel tiles per wave (1152 channels: 3 workgroups per 16 tokens)
  constexpr int ET = 6;
  const int gx = (T + 15) / 16 * ((D + 64 * ET - 1) / (64 * ET));
  // (aligned weight rows, 16-byte vectors of the outputs)
  const bool mf = (uintptr_t)w_pe % 16 == 0 && (uintptr_t)x % 16 == 0 && (uintptr_t)x0 % 16 == 0;
#define T2I_EMB_ANY(TW_)                                                                       \
  if (P == 16 && mf) T2I_EMB((embed_mfma_kernel<TW_, 1, ET>), TW_, gx, 1);                     \
  else if (P == 64 && mf) T2I_EMB((embed_mfma_kernel<TW_, 4, ET>), TW_, gx, 1);                \
  else T2I_EMB((embed_kernel<TW_>), TW_, (T + kEmbTok - 1) / kEmbTok, (D + 255) / 256)
  if (w_bf16) {
    T2I_EMB_ANY(bf16);
  } else {
    T2I_EMB_ANY(float);
  }
#undef T2I_EMB_ANY
#undef T2I_EMB
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Per-call tables, in fp64 and one launch (they depend on the call's arguments
// only): the timestep sinusoid, row r with s = t_scale * t[r]: [cos(s f_k) |
// sin(s f_k)], f_k = exp(-ln(10000) k / half); and the position table of npos
// grid positions, tab[pos * q + f] from the angle pos * 10000^(-f/q): (sin,
// cos) for the additive embedding, (cos, sin) for RoPE (cos_first).

__global__ void call_tables_kernel(TVals tv, int freq_dim, double t_scale, float* __restrict__ out,
                                   float2* __restrict__ tab, int npos, int q, int cos_first) {
  const int nt = tv.n * freq_dim, half = freq_dim / 2;
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx < nt) {
    const int r = idx / freq_dim, k = idx - r * freq_dim;
    const int kk = k < half ? k : k - half;
    const double f = exp(-log(10000.0) * (double)kk / (double)half);
    const double a = t_scale * tv.t[r] * f;
    out[idx] = (float)(k < half ? cos(a) : sin(a));
  } else if (idx - nt < npos * q) {
    const int i = idx - nt, pos = i / q, f = i - pos * q;
    const double ang = (double)pos * pow(10000.0, -(double)f / (double)q);
    const float sn = (float)sin(ang), cs = (float)cos(ang);
    tab[i] = cos_first ? float2{cs, sn} : float2{sn, cs};
  }
}

hipError_t launch_call_tables(const double* t, int rows, int freq_dim, double t_scale, float* out,
                              float2* tab, int npos, int q, bool cos_first, hipStream_t st) {
  for (int r0 = 0; r0 < rows; r0 += kTValsChunk) {
    TVals tv;
    tv.n = std::min(kTValsChunk, rows - r0);
    for (int i = 0; i < tv.n; ++i) tv.t[i] = t[r0 + i];
    const int np = r0 == 0 ? npos : 0;   // the position table with the first chunk
    const int n = tv.n * freq_dim + np * q;
    hipLaunchKernelGGL(call_tables_kernel, dim3((n + 255) / 256), dim3(256), 0, st, tv, freq_dim,
                       t_scale, out + (size_t)r0 * freq_dim, tab, np, q, cos_first ? 1 : 0);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// dst[r][:] = src[:] (bf16 or fp32 rows of width D)
__global__ void broadcast_rows_kernel(const uint16_t* __restrict__ src16,
                                      const float* __restrict__ src32, int rows, int D,
                                      uint16_t* __restrict__ dst16, float* __restrict__ dst32) {
  const long n = (long)rows * D;
  for (long i = blockIdx.x * 256L + threadIdx.x; i < n; i += (long)gridDim.x * 256) {
    const int d = (int)(i % D);
    if (src16) dst16[i] = src16[d];
    else dst32[i] = src32[d];
  }
}

hipError_t launch_broadcast_rows(const void* src, bool bf16_io, int rows, int D, void* dst,
                                 hipStream_t st) {
  const long n = (long)rows * D;
  if (n == 0) return hipSuccess;
  const int grid = (int)std::min<long>((n + 255) / 256, 4096);
  hipLaunchKernelGGL(broadcast_rows_kernel, dim3(grid), dim3(256), 0, st,
                     bf16_io ? (const uint16_t*)src : nullptr, bf16_io ? nullptr : (const float*)src,
                     rows, D, bf16_io ? (uint16_t*)dst : nullptr, bf16_io ? nullptr : (float*)dst);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// 2D rotary position embedding of the image tokens (joint-attention model).

// one thread per (row, head, half, pair): rotates the q pair and the k pair
__global__ void rope_apply_kernel(bf16* __restrict__ qk, int ld, int row0, ReqMap rm, int heads,
                                  int hd, int patch, const float2* __restrict__ tab) {
  const int q = hd / 4;
  const long per_row = (long)heads * 2 * q;
  const long total = (long)rm.tokens_total * rm.branches * per_row;
  const int D = heads * hd;
  for (long i = blockIdx.x * 256L + threadIdx.x; i < total; i += (long)gridDim.x * 256) {
    const long row = i / per_row;
    int rem = (int)(i - row * per_row);
    const int h = rem / (2 * q);
    rem -= h * 2 * q;
    const int half = rem / q, j = rem - half * q;
    const int tok = (int)(row % rm.tokens_total);
    const int r = req_of_token(rm, tok);
    const int lt = tok - rm.tok_off[r];
    const int gw = rm.w[r] / patch;
    const int pos = half ? lt % gw : lt / gw;
    const float2 cs = tab[pos * q + j];
    bf16* base = qk + (size_t)(row0 + row) * ld + h * hd + half * (hd / 2) + 2 * j;
#pragma unroll
    for (int part = 0; part < 2; ++part) {   // q, then k (D columns further)
      bf16* pp = base + part * D;
      const float a = (float)pp[0], b = (float)pp[1];
      pp[0] = (bf16)(a * cs.x - b * cs.y);
      pp[1] = (bf16)(a * cs.y + b * cs.x);
    }
  }
}

// Head dims that are multiples of 16: one thread per (row, head, half, group
// of 4 pairs) moves 16 bytes of q and of k at a time, with 32-bit index math;
// each pair is rotated exactly as in rope_apply_kernel.
__global__ void rope_apply4_kernel(bf16* __restrict__ qk, int ld, int row0, ReqMap rm, int heads,
                                   int hd, int patch, const float2* __restrict__ tab) {
  const int q = hd / 4, g = q / 4;
  const int per_row = heads * 2 * g;
  const int T = rm.tokens_total;
  const int total = T * rm.branches * per_row;
  const int D = heads * hd;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < total; i += gridDim.x * 256) {
    const int row = i / per_row;
    int rem = i - row * per_row;
    const int h = rem / (2 * g);
    rem -= h * 2 * g;
    const int half = rem / g, jg = rem - half * g;
    const int tok = row >= T ? row - T : row;   // branch-major rows, two branches at most
    const int r = req_of_token(rm, tok);
    const int lt = tok - rm.tok_off[r];
    const int gw = rm.w[r] / patch;
    const int pos = half ? lt % gw : lt / gw;
    const float2* cs = tab + pos * q + 4 * jg;
    bf16* base = qk + (size_t)(row0 + row) * ld + h * hd + half * (hd / 2) + 8 * jg;
#pragma unroll
    for (int part = 0; part < 2; ++part) {   // q, then k (D columns further)
      bf16x8* pp = (bf16x8*)(base + part * D);
      const bf16x8 v = *pp;
      bf16x8 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float2 c = cs[e];
        const float a = (float)v[2 * e], b = (float)v[2 * e + 1];
        o[2 * e] = (bf16)(a * c.x - b * c.y);
        o[2 * e + 1] = (bf16)(a * c.y + b * c.x);
      }
      *pp = o;
    }
  }
}

hipError_t launch_rope_apply(bf16* qk, int ld, int row0, const ReqMap& rm, int heads, int head_dim,
                             int patch, const float2* table, hipStream_t st) {
  const long total = (long)rm.tokens_total * rm.branches * heads * (head_dim / 2);
  if (total == 0) return hipSuccess;
  if (head_dim % 16 == 0 && rm.branches <= 2 && ld % 8 == 0 && ((uintptr_t)qk % 16) == 0 &&
      total / 4 < (1L << 30)) {
    const int grid = (int)std::min<long>((total / 4 + 255) / 256, 16384);
    hipLaunchKernelGGL(rope_apply4_kernel, dim3(grid), dim3(256), 0, st, qk, ld, row0, rm, heads,
                       head_dim, patch, table);
    return hipGetLastError();
  }
  const int grid = (int)std::min<long>((total + 255) / 256, 16384);
  hipLaunchKernelGGL(rope_apply_kernel, dim3(grid), dim3(256), 0, st, qk, ld, row0, rm, heads,
                     head_dim, patch, table);
  return hipGetLastError();
}

// LoRA merge: a thread owns one input column i and keeps A[:, i] in
// registers; the workgroup walks kLoraRows output rows, B's rows staged in LDS.
// RK (16 / 32 / 64 / 128) is the rank rounded up; the padding is zero.
constexpr int kLoraRows = 64, kLoraMaxRank = 128;

template <typename T, int RK>
__global__ __launch_bounds__(256) void lora_merge_kernel(int n_out, int n_in, int rank, float alpha,
                                                         LoraGroup g, int ldw) {
  T* __restrict__ W = (T*)g.W[blockIdx.z];
  const T* __restrict__ A = (const T*)g.A[blockIdx.z];
  const T* __restrict__ B = (const T*)g.B[blockIdx.z];
  __shared__ float brow[kLoraRows][RK];
  const int i = blockIdx.x * 256 + threadIdx.x;
  const int o0 = blockIdx.y * kLoraRows;
  for (int e = threadIdx.x; e < kLoraRows * RK; e += 256) {
    const int r = e / RK, k = e - r * RK;
    brow[r][k] = (o0 + r < n_out && k < rank) ? to_f32(B[(size_t)(o0 + r) * rank + k]) : 0.f;
  }
  __syncthreads();
  if (i >= n_in) return;
  float a[RK];
#pragma unroll
  for (int k = 0; k < RK; ++k) a[k] = k < rank ? to_f32(A[(size_t)k * n_in + i]) : 0.f;
  const int rows = min(kLoraRows, n_out - o0);
  // 16 rows at a time: their W elements are loaded together (independent
  // loads in flight), updated, stored
  for (int r0 = 0; r0 < rows; r0 += 16) {
    float wv[16];
#pragma unroll
    for (int j = 0; j < 16; ++j)
      wv[j] = r0 + j < rows ? to_f32(W[(size_t)(o0 + r0 + j) * ldw + i]) : 0.f;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      float acc = 0.f;
#pragma unroll
      for (int k = 0; k < RK; ++k) acc = fmaf(brow[r0 + j][k], a[k], acc);
      if (r0 + j < rows) W[(size_t)(o0 + r0 + j) * ldw + i] = from_f32<T>(fmaf(alpha, acc, wv[j]));
    }
  }
}

// bf16 LoRA merge on MFMA, bound by reading and writing W.  A workgroup of 4
// waves owns TN columns of W and `steps` x 128 rows: it transposes its columns
// of A through LDS once, every wave keeps them as MFMA fragments in
// registers (k contiguous, zero past `rank`), and then walks its rows 32 at a
// time -- the rows of B straight from memory as the other operand, the product
// on v_mfma_f32_32x32x16_bf16 (fp32 accumulation over the rank), turned from
// the MFMA layout to row chunks in the wave's own part of LDS, added to W and
// rounded once.  The next rows' W and B are fetched before the current ones
// are finished.  Needs n_in % 8 == 0, ldw % 8 == 0 and 16-byte aligned W and A
// (the launcher checks).  28 weights of 3456 x 1152: 139 -> 91 us at rank 64
// (4.9 TB/s), 86 -> 72 at rank 16 (6.2 TB/s), 270 -> 116 at rank 128, against
// one 64 x 128 tile per workgroup with both operands transposed through LDS.

template <int RK, int TN>
__global__ __launch_bounds__(256) void lora_merge_mfma_kernel(int n_out, int n_in, int rank,
                                                              float alpha, LoraGroup g, int ldw,
                                                              int steps) {
  // weight blockIdx.z of the group
  bf16* __restrict__ W = (bf16*)g.W[blockIdx.z];
  const bf16* __restrict__ A = (const bf16*)g.A[blockIdx.z];
  const bf16* __restrict__ B = (const bf16*)g.B[blockIdx.z];
  constexpr int KP = RK + 8;        // LDS row pitch of A^T (bf16)
  constexpr int PP = TN + 4;   // LDS row pitch of the product (fp32)
  constexpr int ABYTES = TN * KP * 2, PBYTES = 4 * 32 * PP * 4;
  __shared__ __attribute__((aligned(16))) char smem[ABYTES > PBYTES ? ABYTES : PBYTES];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i0 = blockIdx.x * TN;
  const int l32 = lane & 31, hl = lane >> 5;
  const int o_begin = (blockIdx.y * 4 + wave) * 32 * steps, o_end = min(o_begin + 32 * steps, n_out);
  typedef bf16 bf16x8u __attribute__((ext_vector_type(8), aligned(2)));   // B's rows start anywhere

  // W of rows o .. o + 31: NC 16-byte chunks per lane, row RC c + lane / CR,
  // columns 8 (lane % CR) ..
  constexpr int CR = TN / 8, RC = 64 / CR, NC = 32 / RC, NT = TN / 32;
  const int wr = lane / CR, wc = i0 + (lane % CR) * 8;
  auto load_w = [&](int o, bf16x8 (&v)[NC]) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int r = o + RC * c + wr;
      v[c] = bf16x8{};
      if (r < o_end && wc < n_in) v[c] = *(const bf16x8*)(W + (size_t)r * ldw + wc);
    }
  };
  auto load_b = [&](int o, bf16x8 (&v)[RK / 16]) {
    const int row = min(o + l32, n_out - 1);
    const bf16* p = B + (size_t)row * rank + 8 * hl;
#pragma unroll
    for (int k = 0; k < RK / 16; ++k) {
      v[k] = bf16x8{};
      const int kk = 16 * k + 8 * hl;
      if (kk + 8 <= rank) {
        v[k] = *(const bf16x8u*)(p + 16 * k);
      } else if (RK == 16 && kk < rank && (long)(n_out - row) * rank >= kk + 8) {
        // a small rank would spend its time on single elements: one load that
        // runs on into the rows after this one, whose values are dropped
        v[k] = *(const bf16x8u*)(p + 16 * k);
#pragma unroll
        for (int j = 1; j < 8; ++j)
          if (kk + j >= rank) v[k][j] = (bf16)0.f;
      } else {
#pragma unroll
        for (int j = 0; j < 8; ++j)
          if (kk + j < rank) v[k][j] = p[16 * k + j];
      }
    }
  };
  bf16x8 wv[NC], bv[RK / 16];
  if (o_begin < o_end) {
    load_w(o_begin, wv);
    load_b(o_begin, bv);
  }
  // A^T [64][KP], zero past rank / the matrix edge: a thread takes 8 rows k of
  // one column chunk at a time, so that LDS is written 16 bytes of one column
  bf16* At = (bf16*)smem;
  for (int e = tid; e < (RK / 8) * (TN / 8); e += 256) {
    const int k = e / (TN / 8) * 8, c = (e % (TN / 8)) * 8;
    bf16x8 r[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      r[j] = bf16x8{};
      if (k + j < rank && i0 + c < n_in) r[j] = *(const bf16x8*)(A + (size_t)(k + j) * n_in + i0 + c);
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      bf16x8 t;
#pragma unroll
      for (int j = 0; j < 8; ++j) t[j] = r[j][q];
      *(bf16x8*)(At + (c + q) * KP + k) = t;
    }
  }
  __syncthreads();
  bf16x8 af[NT][RK / 16];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int k = 0; k < RK / 16; ++k)
      af[t][k] = *(const bf16x8*)(At + (32 * t + l32) * KP + 16 * k + 8 * hl);
  __syncthreads();   // the product takes A^T's place

  float* Ps = (float*)smem + wave * 32 * PP;
  for (int o = o_begin; o < o_end; o += 32) {
    f32x16 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = f32x16{};
#pragma unroll
    for (int k = 0; k < RK / 16; ++k)
#pragma unroll
      for (int t = 0; t < NT; ++t)
        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[t][k], bv[k], acc[t], 0, 0, 0);
    // lane: row l32, columns 32 t + 8 q + 4 hl .. + 3
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *(f32x4*)&Ps[l32 * PP + 32 * t + 8 * q + 4 * hl] =
            f32x4{acc[t][4 * q], acc[t][4 * q + 1], acc[t][4 * q + 2], acc[t][4 * q + 3]};
    bf16x8 wn[NC];
    if (o + 32 < o_end) {
      load_b(o + 32, bv);
      load_w(o + 32, wn);
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const float* pr = &Ps[(RC * c + wr) * PP + (lane % CR) * 8];
      const f32x4 p0 = *(const f32x4*)pr, p1 = *(const f32x4*)(pr + 4);
      bf16x8 y;
#pragma unroll
      for (int j = 0; j < 8; ++j) y[j] = (bf16)fmaf(alpha, j < 4 ? p0[j] : p1[j - 4], (float)wv[c][j]);
      const int r = o + RC * c + wr;
      if (r < o_end && wc < n_in) *(bf16x8*)(W + (size_t)r * ldw + wc) = y;
    }
    if (o + 32 < o_end)
#pragma unroll
      for (int c = 0; c < NC; ++c) wv[c] = wn[c];
  }
}

template <typename T>
static hipError_t lora_dispatch(int n, int n_out, int n_in, int rank, float alpha,
                                const LoraGroup& g, int ldw, hipStream_t st) {
  dim3 grid((n_in + 255) / 256, (n_out + kLoraRows - 1) / kLoraRows, n);
#define T2I_LORA(RK_)                                                                             \
  hipLaunchKernelGGL((lora_merge_kernel<T, RK_>), grid, dim3(256), 0, st, n_out, n_in, rank, alpha, \
                     g, ldw)
  if (rank <= 16) T2I_LORA(16);
  else if (rank <= 32) T2I_LORA(32);
  else if (rank <= 64) T2I_LORA(64);
  else T2I_LORA(128);
#undef T2I_LORA
  return hipGetLastError();
}

hipError_t launch_lora_merge(bool bf16_io, int n_out, int n_in, int rank, float alpha, void* W,
                             int ldw, const void* A, const void* B, hipStream_t st) {
  if (n_out <= 0 || n_in <= 0) return hipSuccess;
  if (rank < 1 || rank > kLoraMaxRank) return hipErrorInvalidValue;
  LoraGroup g;
  g.W[0] = W;
  g.A[0] = A;
  g.B[0] = B;
  return launch_lora_merge_group(bf16_io, 1, n_out, n_in, rank, alpha, g, ldw, st);
}

hipError_t launch_lora_merge_group(bool bf16_io, int n, int n_out, int n_in, int rank,
                                   float alpha, const LoraGroup& g, int ldw, hipStream_t st) {
  if (n <= 0 || n_out <= 0 || n_in <= 0) return hipSuccess;
  if (n > kMaxGroups || rank < 1 || rank > kLoraMaxRank) return hipErrorInvalidValue;
  bool vec = bf16_io && n_in % 8 == 0 && ldw % 8 == 0;
  for (int i = 0; i < n; ++i)
    vec = vec && (uintptr_t)g.W[i] % 16 == 0 && (uintptr_t)g.A[i] % 16 == 0;
  if (vec) {
    // 32-row steps per wave, which share the transposed A: two from 1024
    // workgroups of two steps on; four from 2048 workgroups of four where the
    // transposed A is large (28 x 3456 x 1152 at rank 128 136 us, 149 with two;
    // at rank 16 93 against 89 with two, from memory).
    const long tiles = (long)((n_in + 63) / 64) * ((n_out + 127) / 128) * n;
    const int steps = tiles >= 8192 && rank > 32 ? 4 : tiles >= 2048 ? 2 : 1;
    // Rows of 256 bytes instead of 128 per workgroup for large wide weights of
    // a small rank, whose time is W's alone (from memory at rank 8: 15 x 1152 x
    // 4096 64.6 us against 67, 8 x 12288 x 3072 244 against 262; 15 x 4608 x
    // 1152 67.2 against 65.8).
    const bool wide = rank <= 16 && n_in >= 2048 && tiles >= 8192;
    const int cols = wide ? 128 : 64;
    dim3 grid((n_in + cols - 1) / cols, (n_out + 128 * steps - 1) / (128 * steps), n);
#define T2I_LORA_MF(RK_, TN_)                                                                  \
  hipLaunchKernelGGL((lora_merge_mfma_kernel<RK_, TN_>), grid, dim3(256), 0, st, n_out, n_in,  \
                     rank, alpha, g, ldw, steps)
    if (wide) T2I_LORA_MF(16, 128);
    else if (rank <= 16) T2I_LORA_MF(16, 64);
    else if (rank <= 32) T2I_LORA_MF(32, 64);
    else if (rank <= 64) T2I_LORA_MF(64, 64);
    else T2I_LORA_MF(128, 64);
#undef T2I_LORA_MF
    return hipGetLastError();
  }
  return bf16_io ? lora_dispatch<bf16>(n, n_out, n_in, rank, alpha, g, ldw, st)
                 : lora_dispatch<float>(n, n_out, n_in, rank, alpha, g, ldw, st);
}

__global__ void add_inplace_kernel(float* __restrict__ x, const float* __restrict__ r, size_t n) {
  for (size_t i = blockIdx.x * 256ul + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) x[i] += r[i];
}

hipError_t launch_add_inplace(float* x, const float* r, size_t n, hipStream_t st) {
  if (n == 0) return hipSuccess;
  const int grid = (int)std::min<size_t>((n + 255) / 256, 8192);
  hipLaunchKernelGGL(add_inplace_kernel, dim3(grid), dim3(256), 0, st, x, r, n);
  return hipGetLastError();
}

// Segment i moves rows [src[i], src[i] + len[i]) of `from` to rows
// [dst[i], ...) of `to`, D floats per row; one grid-stride pass over all
// segments' float4s (segments never overlap).
__global__ void copy_rows_kernel(const float* __restrict__ from, float* __restrict__ to,
                                 RowCopyMap m, int D) {
  const int q = D / 4;
  const long total = (long)m.row_end[m.n - 1] * q;
  for (long i = blockIdx.x * 256L + threadIdx.x; i < total; i += (long)gridDim.x * 256) {
    const int row = (int)(i / q), c = (int)(i - (long)row * q);
    int s = 0;
#pragma unroll 1
    for (int k = 0; k + 1 < m.n; ++k) s += row >= m.row_end[k] ? 1 : 0;
    const int r = row - (s ? m.row_end[s - 1] : 0);
    ((float4*)to)[(long)(m.dst[s] + r) * q + c] = ((const float4*)from)[(long)(m.src[s] + r) * q + c];
  }
}

hipError_t launch_copy_rows(const float* from, float* to, const RowCopyMap& m, int D,
                            hipStream_t st) {
  if (m.n == 0) return hipSuccess;
  const long total = (long)m.row_end[m.n - 1] * (D / 4);
  if (total == 0) return hipSuccess;
  const int grid = (int)std::min<long>((total + 255) / 256, 8192);
  hipLaunchKernelGGL(copy_rows_kernel, dim3(grid), dim3(256), 0, st, from, to, m, D);
  return hipGetLastError();
}

__global__ void bias_rows_f32_kernel(const bf16* __restrict__ b16, const float* __restrict__ b32,
                                     int rows, int D, float* __restrict__ dst) {
  const long n = (long)rows * D;
  for (long i = blockIdx.x * 256L + threadIdx.x; i < n; i += (long)gridDim.x * 256) {
    const int d = (int)(i % D);
    dst[i] = b16 ? (float)b16[d] : b32[d];
  }
}

hipError_t launch_bias_rows_f32(const void* bias, bool bias_bf16, int rows, int D, float* dst,
                                hipStream_t st) {
  const long n = (long)rows * D;
  if (n == 0) return hipSuccess;
  const int grid = (int)std::min<long>((n + 255) / 256, 8192);
  hipLaunchKernelGGL(bias_rows_f32_kernel, dim3(grid), dim3(256), 0, st,
                     bias_bf16 ? (const bf16*)bias : nullptr,
                     bias_bf16 ? nullptr : (const float*)bias, rows, D, dst);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Final layer: per image token and guidance branch,
//   out = LNmod(x; shift, scale) W_out^T + b_out     (P = p*p*C outputs)
// then v = v_u + g (v_c - v_u), unpatchify, noise_pred = v, latent += dt v.
//
// final_mfma_kernel (P = 16 or 64): a workgroup of 8 waves takes 16 tokens in
// all NB guidance branches.  A wave holds 2 NB rows in registers (one
// coalesced read), takes their LayerNorm statistics in two passes, and writes
// the modulated rows to LDS, CH columns at a time; the contraction runs on
// v_mfma_f32_16x16x4_f32 (fp32 rows against the weights widened to fp32),
// which is a chain of four fused multiply-adds.  A lane loads
// eight consecutive weights of its output and trades them between the lane
// groups, so that an MFMA takes four consecutive columns, and the sums are
// those of final_kernel, bit for bit:
//  * CHAINS: columns 256 i + 4 l .. + 3 belong to chain l of 64, as to lane l
//    there; wave w runs the chains 8 w + n (n = 0 .. 7) side by side, MFMA n of
//    its 32 columns of every 256, and the 64 are added in the pairs of wave_sum.
//  * otherwise one chain over all columns, ascending (P = 64 in bf16, where a
//    wave per token would read the projection once per token): wave w takes
//    outputs 16 (w % 4) .. of branch w / 4, 32 columns a step, and the next
//    part of the rows is written to LDS before a part is contracted.
// Bound by reading the rows and, at P = 64, by the one chain (768 dependent
// MFMAs, 10 us) and the projection read once per 16 tokens from L2.  Against
// one wave per token (P = 16) or a 32-token register tile (P = 64) on vector
// FMAs: 28.4 -> 20.9 us at 4096 tokens x 2 branches and 37.4 -> 21.7 at 8168 x 1
// (width 1152), 220 -> 51 at 4096 tokens of width 3072; 13 us either way at 1024
// tokens.  Sums in an order of their own, without the exchange of the 64 chains
// or the one chain, took 20.0, 19.6 and 46 us.

// v = v_u + g (v_c - v_u) into output f of token `tok` (request r): unpatchify,
// noise_pred, Euler update
__device__ __forceinline__ void final_store(const ReqMap& rm, int tok, int r, int f, float vc,
                                            float vu, float guidance, int C, int p, float* lat,
                                            float* noise_pred) {
  const float vel = rm.branches == 2 ? vu + guidance * (vc - vu) : vc;
  const int a = f / (p * C), b = (f / C) % p, c = f % C;
  const int lt = tok - rm.tok_off[r];
  const int W = rm.w[r], H = rm.h[r], gw = W / p;
  const int gi = lt / gw, gj = lt - gi * gw;
  const size_t li = (size_t)rm.lat_off[r] + (size_t)c * H * W + (size_t)(gi * p + a) * W + gj * p + b;
  if (noise_pred) noise_pred[li] = vel;
  const float dt = rm.dt[r];
  if (dt != 0.f) lat[li] = lat[li] + dt * vel;
}

// NI: float4 per lane and row (D <= 256 NI); CH: columns in LDS at a time (a
// multiple of 256, or all of them)
template <typename TW, int NI, int CH, int NB, bool CHAINS>
__global__ __launch_bounds__(512) void final_mfma_kernel(const float* __restrict__ x, ReqMap rm,
                                                         const TW* __restrict__ w_out,
                                                         const TW* __restrict__ b_out,
                                                         const float* __restrict__ mod, int ld_mod,
                                                         int shift_off, int scale_off, int D, int C,
                                                         int p, float eps, float guidance,
                                                         float* __restrict__ lat,
                                                         float* __restrict__ noise_pred) {
  constexpr int NR = 2 * NB, P = CH + 4;   // rows per wave; LDS row pitch
  constexpr int BUFS = CHAINS ? 1 : 2;
  constexpr int ROWS = BUFS * NB * 16 * P * 4, PART = (CHAINS ? 64 : 4) * NB * 64 * 16;
  __shared__ __attribute__((aligned(16))) char smem[ROWS > PART ? ROWS : PART];
  float* const hs = (float*)smem;          // [BUFS][NB][16][P]
  f32x4* const part = (f32x4*)smem;        // [NB][chain or output tile][64], after the last columns
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int fr = lane & 15, g = lane >> 4;
  const int T = rm.tokens_total, tok0 = blockIdx.x * 16;
  const int nv = D >> 2;
  // rows: branch i / 2, token 2 wave + i % 2 of the group (past the end: the last token)
  float4 v[NR][NI];
  float mean[NR], rstd[NR];
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    const int t = min(tok0 + 2 * wave + (i & 1), T - 1);
    const float4* xr = (const float4*)(x + ((size_t)(i >> 1) * T + t) * D);
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const int c = lane + 64 * j;
      v[i][j] = float4{0.f, 0.f, 0.f, 0.f};
      if (c < nv) v[i][j] = xr[c];
    }
  }
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    float s = 0.f, q = 0.f;
#pragma unroll
    for (int j = 0; j < NI; ++j) s += (v[i][j].x + v[i][j].y) + (v[i][j].z + v[i][j].w);
    mean[i] = wave_sum(s) / (float)D;
#pragma unroll
    for (int j = 0; j < NI; ++j)
      if (lane + 64 * j < nv) {
        const float a = v[i][j].x - mean[i], b = v[i][j].y - mean[i], c = v[i][j].z - mean[i],
                    d = v[i][j].w - mean[i];
        q += (a * a + b * b) + (c * c + d * d);
      }
    rstd[i] = 1.0f / sqrtf(wave_sum(q) / (float)D + eps);
  }
  // the modulation rows of the wave's two tokens
  const float* md[2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
    md[i] = mod + (size_t)rm.modrow[req_of_token(rm, min(tok0 + 2 * wave + i, T - 1))] * ld_mod;

  constexpr int NCH = CH % 256 ? 1 : NI * 256 / CH;   // (whole rows when CH is no multiple of 256)
  // columns ch CH .. of the modulated rows into LDS
  auto stage = [&](int ch) {
    float* const to = hs + (BUFS > 1 ? ch % 2 : 0) * NB * 16 * P - ch * CH;
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      // (with several chunks CH is a multiple of 256: a float4 column lies in one)
      if (NCH > 1 && j / (CH / 256) != ch) continue;
      const int c = lane + 64 * j;
      if (c < nv) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const float4 a = *(const float4*)(md[t] + shift_off + 4 * c);
          const float4 b = *(const float4*)(md[t] + scale_off + 4 * c);
#pragma unroll
          for (int br = 0; br < NB; ++br) {
            const int i = 2 * br + t;
            float4 y;
            y.x = (v[i][j].x - mean[i]) * rstd[i] * (1.f + b.x) + a.x;
            y.y = (v[i][j].y - mean[i]) * rstd[i] * (1.f + b.y) + a.y;
            y.z = (v[i][j].z - mean[i]) * rstd[i] * (1.f + b.z) + a.z;
            y.w = (v[i][j].w - mean[i]) * rstd[i] * (1.f + b.w) + a.w;
            *(float4*)&to[(br * 16 + 2 * wave + t) * P + 4 * c] = y;
          }
        }
      }
    }
  };
  // a lane's eight weights: operand m of quad h is column 4 h + g of lane group m
  typedef TW tw4 __attribute__((ext_vector_type(4)));
  struct W8 {
    tw4 q[2];
  };
  auto ld8 = [&](const TW* w) { return W8{{*(const tw4*)w, *(const tw4*)(w + 4)}}; };
  // final sums of output tile j of both branches, in every lane: token fr,
  // outputs 16 j + 4 g .. + 3
  auto finish = [&](int j, f32x4 vc, f32x4 vu) {
    const int tok = tok0 + fr;
    if (tok >= T) return;
    const int r = req_of_token(rm, tok);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int f = 16 * j + 4 * g + e;
      const float bo = to_f32(b_out[f]);
      final_store(rm, tok, r, f, vc[e] + bo, vu[e] + bo, guidance, C, p, lat, noise_pred);
    }
  };

  if constexpr (CHAINS) {
    const int jt = blockIdx.y;   // output tile
    const TW* const wp = w_out + (size_t)(16 * jt + fr) * D + 32 * wave + 8 * g;
    f32x4 acc[NB][8];
#pragma unroll
    for (int br = 0; br < NB; ++br)
#pragma unroll
      for (int n = 0; n < 8; ++n) acc[br][n] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
      const int k0 = ch * CH;
      if (k0 >= D) break;
      constexpr int NS = (CH + 255) / 256;   // 32-column steps of a wave
      W8 wr[NS];
      auto load_w = [&](int s) {
        const int k = k0 + 256 * s;
        if (k + 32 * wave < D) wr[s] = ld8(wp + k);
      };
      // (narrow rows: while they load; wide ones leave no registers for that)
#pragma unroll
      for (int s = 0; NCH == 1 && s < NS; ++s) load_w(s);
      if (ch > 0) __syncthreads();
      stage(ch);
      __syncthreads();
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const int k = 256 * s + 32 * wave;
        if (k0 + k >= D) break;
        if (NCH > 1) {
          __builtin_amdgcn_sched_barrier(0);
          load_w(s);
        }
        float w[2][4];
        transpose_groups(wr[s].q[0], w[0]);
        transpose_groups(wr[s].q[1], w[1]);
#pragma unroll
        for (int br = 0; br < NB; ++br)
#pragma unroll
          for (int n = 0; n < 8; ++n)
            acc[br][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                w[n & 1][n >> 1], hs[(br * 16 + fr) * P + k + 4 * n + g], acc[br][n], 0, 0, 0);
      }
    }
    __syncthreads();
#pragma unroll
    for (int br = 0; br < NB; ++br)
#pragma unroll
      for (int n = 0; n < 8; ++n) part[(br * 64 + 8 * wave + n) * 64 + lane] = acc[br][n];
    __syncthreads();
    // the tree of wave_sum: chains 32, 16, 8 apart (wave n's share: chains 8 q + n) ...
    auto pairs = [&](int c0, int step) {
      f32x4 s[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) s[q] = part[(c0 + step * q) * 64 + lane];
      return ((s[0] + s[4]) + (s[2] + s[6])) + ((s[1] + s[5]) + (s[3] + s[7]));
    };
#pragma unroll
    for (int br = 0; br < NB; ++br) part[(br * 64 + wave) * 64 + lane] = pairs(br * 64 + wave, 8);
    __syncthreads();
    // ... then 4, 2, 1
    if (wave == 0) finish(jt, pairs(0, 1), NB == 2 ? pairs(64, 1) : f32x4{0.f, 0.f, 0.f, 0.f});
  } else {
    const int j = wave & 3, br = wave >> 2;
    const bool works = br < NB;
    const TW* const wp = w_out + (size_t)(16 * j + fr) * D + 8 * g;
    const int steps = D / 32;
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
    constexpr int PF = 4;   // weight loads in flight (CH / 32 is a multiple)
    static_assert(CH % (32 * PF) == 0, "steps of a part");
    W8 ring[PF];
    if (works)
#pragma unroll
      for (int s = 0; s < PF; ++s) ring[s] = ld8(wp + 32 * min(s, steps - 1));
    stage(0);
    __syncthreads();
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
      if (ch * CH >= D) break;
      if (ch + 1 < NCH) stage(ch + 1);
      if (works) {
        // MFMA 2 m + c of a step takes columns 4 (2 m + c) + g, read one step ahead
        const float* hp = hs + ((ch % 2 * NB + br) * 16 + fr) * P + g;
        const int n = min(steps - ch * CH / 32, CH / 32);
        float h[2][8];
#pragma unroll
        for (int q = 0; q < 8; ++q) h[0][q] = hp[4 * q];
        for (int s0 = 0; s0 < n; s0 += PF) {
#pragma unroll
          for (int s = 0; s < PF; ++s) {
            if (s0 + s >= n) break;
            float w[2][4];
            transpose_groups(ring[s].q[0], w[0]);
            transpose_groups(ring[s].q[1], w[1]);
            ring[s] = ld8(wp + 32 * min(ch * (CH / 32) + s0 + s + PF, steps - 1));
            const float* hn = hp + 32 * min(s0 + s + 1, n - 1);
#pragma unroll
            for (int q = 0; q < 8; ++q) h[(s + 1) & 1][q] = hn[4 * q];
#pragma unroll
            for (int q = 0; q < 8; ++q)
              acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w[q & 1][q >> 1], h[s & 1][q], acc, 0, 0, 0);
          }
        }
      }
      __syncthreads();
    }
    if constexpr (NB == 1) {
      if (works) finish(j, acc, acc);
    } else {
      if (br == 1) part[j * 64 + lane] = acc;
      __syncthreads();
      if (br == 0) finish(j, acc, part[j * 64 + lane]);
    }
  }
}

// Any other P (<= 64): one wave per token, each output summed over the wave.
template <typename TW>
__global__ __launch_bounds__(256) void final_kernel(const float* __restrict__ x, ReqMap rm,
                                                    const TW* __restrict__ w_out,
                                                    const TW* __restrict__ b_out,
                                                    const float* __restrict__ mod, int ld_mod,
                                                    int shift_off, int scale_off, int D, int C,
                                                    int p, float eps, float guidance,
                                                    float* __restrict__ lat,
                                                    float* __restrict__ noise_pred) {
  constexpr int NI = kMaxV4;
  const int lane = threadIdx.x & 63;
  const int tok = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (tok >= rm.tokens_total) return;
  const int r = req_of_token(rm, tok);
  const int P = p * p * C;
  const int nv = D >> 2;
  const float* md = mod + (size_t)rm.modrow[r] * ld_mod;
  const float4* sh = (const float4*)(md + shift_off);
  const float4* sc = (const float4*)(md + scale_off);
  const int nb = rm.branches;
  float mine[2] = {0.f, 0.f};
#pragma unroll
  for (int br = 0; br < 2; ++br) {
    if (br >= nb) continue;
    float4 v[NI];
    const float4* xr = (const float4*)(x + ((size_t)br * rm.tokens_total + tok) * D);
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = lane + 64 * i;
      if (c < nv) {
        v[i] = xr[c];
        s += (v[i].x + v[i].y) + (v[i].z + v[i].w);
      }
    }
    const float mean = wave_sum(s) / (float)D;
    float q = 0.f;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = lane + 64 * i;
      if (c < nv) {
        const float a = v[i].x - mean, b = v[i].y - mean, cc = v[i].z - mean, d = v[i].w - mean;
        q += (a * a + b * b) + (cc * cc + d * d);
      }
    }
    const float rstd = 1.0f / sqrtf(wave_sum(q) / (float)D + eps);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = lane + 64 * i;
      if (c < nv) {
        const float4 a = sh[c], b = sc[c];
        v[i].x = (v[i].x - mean) * rstd * (1.f + b.x) + a.x;
        v[i].y = (v[i].y - mean) * rstd * (1.f + b.y) + a.y;
        v[i].z = (v[i].z - mean) * rstd * (1.f + b.z) + a.z;
        v[i].w = (v[i].w - mean) * rstd * (1.f + b.w) + a.w;
      }
    }
    for (int f = 0; f < P; ++f) {
      const TW* wr = w_out + (size_t)f * D;
      float part = 0.f;
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int c = lane + 64 * i;
        if (c < nv) {
          part = fmaf(v[i].x, to_f32(wr[4 * c + 0]), part);
          part = fmaf(v[i].y, to_f32(wr[4 * c + 1]), part);
          part = fmaf(v[i].z, to_f32(wr[4 * c + 2]), part);
          part = fmaf(v[i].w, to_f32(wr[4 * c + 3]), part);
        }
      }
      const float tot = wave_sum(part) + to_f32(b_out[f]);
      if (lane == f) mine[br] = tot;
    }
  }
  if (lane < P) final_store(rm, tok, r, lane, mine[0], mine[1], guidance, C, p, lat, noise_pred);
}

hipError_t launch_final_layer(const float* x, const ReqMap& rm, const void* w_out,
                              const void* b_out, bool w_bf16, const float* mod, int ld_mod,
                              int shift_off, int scale_off, int D, int C, int p, float eps,
                              float guidance, float* latents, float* noise_pred, hipStream_t st) {
  if (rm.tokens_total == 0) return hipSuccess;
  const int P = p * p * C, T = rm.tokens_total;
#define T2I_FIN(K_, GX_, GY_, BLOCK_, TW_)                                                       \
  hipLaunchKernelGGL(K_, dim3(GX_, GY_), dim3(BLOCK_), 0, st, x, rm, (const TW_*)w_out,          \
                     (const TW_*)b_out, mod, ld_mod, shift_off, scale_off, D, C, p, eps, guidance, \
                     latents, noise_pred)
  // (16-byte weight loads)
  const bool al = (uintptr_t)w_out % 16 == 0, two = rm.branches == 2;
  const int gt = (T + 15) / 16;
#define T2I_FIN_NB(TW_, NI_, CH_, CHAINS_)                                                       \
  if (two) T2I_FIN((final_mfma_kernel<TW_, NI_, CH_, 2, CHAINS_>), gt, (CHAINS_ ? P / 16 : 1), 512, TW_); \
  else T2I_FIN((final_mfma_kernel<TW_, NI_, CH_, 1, CHAINS_>), gt, (CHAINS_ ? P / 16 : 1), 512, TW_)
  // rows of at most 1152 columns are staged whole, wider ones in parts
#define T2I_FIN_CHAINS(TW_)                                                                      \
  if (D <= 1152) {                                                                               \
    T2I_FIN_NB(TW_, 5, 1152, true);                                                              \
  } else {                                                                                       \
    T2I_FIN_NB(TW_, kMaxV4, 1024, true);                                                         \
  }
  if (P == 64 && al && w_bf16) {
    T2I_FIN_NB(bf16, kMaxV4, 512, false);
  } else if (P == 16 && al && w_bf16) {
    T2I_FIN_CHAINS(bf16);
  } else if ((P == 16 || P == 64) && al && !w_bf16) {
    T2I_FIN_CHAINS(float);
  } else if (w_bf16) {
    T2I_FIN((final_kernel<bf16>), (T + 3) / 4, 1, 256, bf16);
  } else {
    T2I_FIN((final_kernel<float>), (T + 3) / 4, 1, 256, float);
  }
#undef T2I_FIN_CHAINS
#undef T2I_FIN_NB
#undef T2I_FIN
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Step-skip cache.
//
// cache_signal_kernel: workgroup = 16 rows of one request, one wave each (a
// wave that took four rows in turn paid their memory latency four times: 24.0
// -> 7.4 us at 1408 rows).  m = LNmod(x0; block-0 shift_msa,
// scale_msa) in fp32; partial[blk] = (sum|m - m_prev|, sum|m_prev|) in fp64
// (lane order, butterfly, then waves 0..15); m_prev := m.
// cache_decide_kernel: one wave per request sums its partials (lane l the
// blocks l, l + 64, .. in order, then a butterfly), applies the rule and also
// writes the header to page-locked host memory for the caller, if given.

int cache_partial_blocks(const ReqMap& rm) {
  int n = 0;
  for (int r = 0; r < rm.n; ++r)
    n += (rm.tok_off[r + 1] - rm.tok_off[r] + kCacheRowsPerBlock - 1) / kCacheRowsPerBlock;
  return n;
}

// NI: float4 per lane (D <= 256 NI); NW: waves, each with 16 / NW rows in turn
// (16 waves leave a lane 128 registers: too few for two rows of 3072 columns,
// 36 us at 4096 of them; 8 waves 32)
template <int NI, int NW>
__global__ __launch_bounds__(64 * NW) void cache_signal_kernel(
    const float* __restrict__ x0, ReqMap rm, const float* __restrict__ mod, int ld_mod,
    int shift_off, int scale_off, int D, float eps, float* __restrict__ m_prev,
    const CacheHeader* __restrict__ hdr, int step, double* __restrict__ partial) {
  __shared__ double red[kCacheRowsPerBlock][2];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // block -> (request, row chunk)
  int r = 0, base = 0;
  for (;;) {
    const int nb = (rm.tok_off[r + 1] - rm.tok_off[r] + kCacheRowsPerBlock - 1) / kCacheRowsPerBlock;
    if ((int)blockIdx.x < base + nb || r == rm.n - 1) break;
    base += nb;
    ++r;
  }
  const int nv = D >> 2;
#pragma unroll 1
  for (int row = wave; row < kCacheRowsPerBlock; row += NW) {
    double num = 0.0, den = 0.0;
    const int tok = rm.tok_off[r] + ((int)blockIdx.x - base) * kCacheRowsPerBlock + row;
    if (tok < rm.tok_off[r + 1]) {
      const bool have_prev = step > 0 && hdr[r].has_m;
      const float* md = mod + (size_t)rm.modrow[r] * ld_mod;
      const float4* sh = (const float4*)(md + shift_off);
      const float4* sc = (const float4*)(md + scale_off);
      const float4* xr = (const float4*)(x0 + (size_t)tok * D);
      float4* mr = (float4*)(m_prev + (size_t)tok * D);
      float4 v[NI], o[NI];
      float s = 0.f;
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int c = lane + 64 * i;
        v[i] = o[i] = float4{0.f, 0.f, 0.f, 0.f};
        if (c < nv) v[i] = xr[c];
        if (c < nv && have_prev) o[i] = mr[c];
      }
#pragma unroll
      for (int i = 0; i < NI; ++i) s += (v[i].x + v[i].y) + (v[i].z + v[i].w);
      const float mean = wave_sum(s) / (float)D;
      float q = 0.f;
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int c = lane + 64 * i;
        if (c < nv) {
          const float a = v[i].x - mean, b = v[i].y - mean, cc = v[i].z - mean, d = v[i].w - mean;
          q += (a * a + b * b) + (cc * cc + d * d);
        }
      }
      const float rstd = 1.0f / sqrtf(wave_sum(q) / (float)D + eps);
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int c = lane + 64 * i;
        if (c < nv) {
          const float4 a = sh[c], b = sc[c];
          float4 m;
          m.x = (v[i].x - mean) * rstd * (1.f + b.x) + a.x;
          m.y = (v[i].y - mean) * rstd * (1.f + b.y) + a.y;
          m.z = (v[i].z - mean) * rstd * (1.f + b.z) + a.z;
          m.w = (v[i].w - mean) * rstd * (1.f + b.w) + a.w;
          if (have_prev) {
            num += (double)fabsf(m.x - o[i].x) + (double)fabsf(m.y - o[i].y) +
                   (double)fabsf(m.z - o[i].z) + (double)fabsf(m.w - o[i].w);
            den += (double)fabsf(o[i].x) + (double)fabsf(o[i].y) + (double)fabsf(o[i].z) +
                   (double)fabsf(o[i].w);
          }
          mr[c] = m;
        }
      }
    }
    num = wave_sum(num);
    den = wave_sum(den);
    if (lane == 0) {
      red[row][0] = num;
      red[row][1] = den;
    }
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    double t = 0.0;
    for (int w = 0; w < kCacheRowsPerBlock; ++w) t += red[w][threadIdx.x];
    partial[2 * blockIdx.x + threadIdx.x] = t;
  }
}

// one workgroup of one wave per request
__global__ void cache_decide_kernel(ReqMap rm, const double* __restrict__ partial,
                                    CacheHeader* __restrict__ hdr,
                                    CacheHeader* __restrict__ host, int step, int n_steps,
                                    double tau, int mode) {
  const int r = blockIdx.x, lane = threadIdx.x;
  int b0 = 0;
  for (int i = 0; i < r; ++i)
    b0 += (rm.tok_off[i + 1] - rm.tok_off[i] + kCacheRowsPerBlock - 1) / kCacheRowsPerBlock;
  const int nb = (rm.tok_off[r + 1] - rm.tok_off[r] + kCacheRowsPerBlock - 1) / kCacheRowsPerBlock;
  CacheHeader hd = hdr[r];
  double num = 0.0, den = 0.0;
  for (int b = lane; b < nb; b += 64) {
    num += partial[2 * (b0 + b) + 0];
    den += partial[2 * (b0 + b) + 1];
  }
  num = wave_sum(num);
  den = wave_sum(den);
  if (lane != 0) return;
  if (step == 0) {
    hd.acc = 0.0;
    hd.has_m = 0;
    hd.has_r = 0;
  }
  double d = __longlong_as_double(0x7ff8000000000000LL);   // NaN: no predecessor
  if (hd.has_m) d = num / den;
  int skip = 0;
  double acc = hd.acc;
  if (tau > 0.0 && step != 0 && step != n_steps - 1 && hd.has_r && hd.has_m) {
    if (mode == 0) {
      acc = acc + d;
      skip = acc < tau;
    } else {
      acc = d;
      skip = d < tau;
    }
  }
  if (!skip) acc = 0.0;
  hd.acc = acc;
  hd.d = d;
  hd.skip = skip;
  hd.has_m = 1;
  hdr[r] = hd;
  if (host) host[r] = hd;
}

hipError_t launch_cache_signal(const float* x0, const ReqMap& rm, const float* mod, int ld_mod,
                               int shift_off, int scale_off, int D, float eps, float* m_prev,
                               CacheHeader* hdr, int step, double* partial, hipStream_t st) {
  const int nb = cache_partial_blocks(rm);
  if (nb == 0) return hipSuccess;
#define T2I_SIG(NI_, NW_)                                                                     \
  hipLaunchKernelGGL((cache_signal_kernel<NI_, NW_>), dim3(nb), dim3(64 * NW_), 0, st, x0, rm, mod, \
                     ld_mod, shift_off, scale_off, D, eps, m_prev, hdr, step, partial)
  if (D <= 1280) T2I_SIG(5, 16);
  else T2I_SIG(kMaxV4, 8);
#undef T2I_SIG
  return hipGetLastError();
}

hipError_t launch_cache_decide(const ReqMap& rm, const double* partial, CacheHeader* hdr,
                               CacheHeader* host, int step, int n_steps, double tau, int mode, hipStream_t st) {
  hipLaunchKernelGGL(cache_decide_kernel, dim3(rm.n), dim3(64), 0, st, rm, partial, hdr, host,
                     step, n_steps, tau, mode);
  return hipGetLastError();
}

// x[b][tok] = x0[tok] + R[b][tok] (skip_mask) / R[b][tok] = x[b][tok] - x0[tok] (store_mask)
__global__ void residual_kernel(const float* __restrict__ x0, const float* __restrict__ R_in,
                                float* __restrict__ x, float* __restrict__ R_out, ReqMap rm,
                                uint32_t mask, int D, int store, CacheHeader* __restrict__ hdr) {
  const int nv = D >> 2;
  const long per_branch = (long)rm.tokens_total * nv;
  const long total = per_branch * rm.branches;
  if (store && blockIdx.x == 0 && threadIdx.x < (unsigned)rm.n && ((mask >> threadIdx.x) & 1u))
    hdr[threadIdx.x].has_r = 1;
  for (long i = blockIdx.x * 256L + threadIdx.x; i < total; i += (long)gridDim.x * 256) {
    const int br = (int)(i / per_branch);
    const long j = i - (long)br * per_branch;
    const int tok = (int)(j / nv);
    const int r = req_of_token(rm, tok);
    if (!((mask >> r) & 1u)) continue;
    const float4 a = ((const float4*)x0)[j];
    if (store) {
      const float4 b = ((const float4*)x)[i];
      ((float4*)R_out)[i] = float4{b.x - a.x, b.y - a.y, b.z - a.z, b.w - a.w};
    } else {
      const float4 b = ((const float4*)R_in)[i];
      ((float4*)x)[i] = float4{a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w};
    }
  }
}

hipError_t launch_apply_residual(const float* x0, const float* R, float* x, const ReqMap& rm,
                                 uint32_t skip_mask, int D, hipStream_t st) {
  const long total = (long)rm.tokens_total * (D / 4) * rm.branches;
  if (total == 0 || skip_mask == 0) return hipSuccess;
  const int grid = (int)std::min<long>((total + 255) / 256, 8192);
  hipLaunchKernelGGL(residual_kernel, dim3(grid), dim3(256), 0, st, x0, R, x, (float*)nullptr, rm,
                     skip_mask, D, 0, (CacheHeader*)nullptr);
  return hipGetLastError();
}

hipError_t launch_store_residual(const float* x0, const float* x, float* R, const ReqMap& rm,
                                 uint32_t store_mask, int D, CacheHeader* hdr, hipStream_t st) {
  const long total = (long)rm.tokens_total * (D / 4) * rm.branches;
  if (total == 0 || store_mask == 0) return hipSuccess;
  const int grid = (int)std::min<long>((total + 255) / 256, 8192);
  hipLaunchKernelGGL(residual_kernel, dim3(grid), dim3(256), 0, st, x0, (const float*)nullptr,
                     (float*)x, R, rm, store_mask, D, 1, hdr);
  return hipGetLastError();
}

}  // namespace t2i
