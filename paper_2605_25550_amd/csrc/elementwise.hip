// Memory-bound kernels of the DiT step on gfx950:
//   * LayerNorm + adaLN modulate: h = LN(x) * (1 + scale) + shift, fp32 in,
//     GEMM operand (bf16 or fp32) out; one wavefront per token row, 16-byte
//     loads, exact two-pass mean/variance from registers.
//   * adaLN modulation GEMV: m = SiLU(c) W_ada^T + b_ada for many (block,
//     stream) weight matrices in one launch; HBM-bound on the weights.
//   * timestep + class conditioning, patch embedding, 2-D sin-cos table.
#include <math.h>

#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace ditmi {

// ---------------------------------------------------------------- LayerNorm + modulate
template <typename OutT, int NV>
__global__ __launch_bounds__(256) void ln_mod_kernel(LnArgs a) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= a.total_rows) return;  // whole wavefront leaves together
  const int si = (a.nseg > 1 && row >= a.s[1].row_begin) ? 1 : 0;
  // select by value: indexing the by-value argument array with a runtime
  // index would copy it to scratch memory
  const LnSeg S = si ? a.s[1] : a.s[0];
  const int r = row - S.row_begin;
  const int b = r / S.rows_per_batch;
  const int D = a.D, nq = D >> 2;
  const f32x4* __restrict__ xr = (const f32x4*)(S.x + (long)r * D);

  // shift/scale are loaded with x, before the reductions, so that their
  // latency overlaps the row's.  Loads use a clamped (always valid) index and
  // the values are selected afterwards; vectors are clang ext_vector types
  // (HIP's float4/uint2 structs, kept in arrays, are placed in memory).
  const f32x4* __restrict__ sh = (const f32x4*)(S.shift + (long)b * S.mod_stride);
  const f32x4* __restrict__ sc = (const f32x4*)(S.scale + (long)b * S.mod_stride);
  f32x4 v[NV], s4[NV], c4[NV];
  float sum = 0.f;
  const f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int c = lane + 64 * i;
    const int cc = min(c, nq - 1);
    const bool in = c < nq;
    const f32x4 tx = xr[cc], ts = sh[cc], tc = sc[cc];
    v[i] = in ? tx : z;
    s4[i] = in ? ts : z;
    c4[i] = in ? tc : z;
    sum += (v[i][0] + v[i][1]) + (v[i][2] + v[i][3]);
  }
  const float mean = wave_sum(sum) / (float)D;
  float sq = 0.f;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int c = lane + 64 * i;
    const f32x4 d = v[i] - mean;
    const float q = (d[0] * d[0] + d[1] * d[1]) + (d[2] * d[2] + d[3] * d[3]);
    sq += c < nq ? q : 0.f;
  }
  const float var = wave_sum(sq) / (float)D;
  const float rstd = 1.0f / sqrtf(var + a.eps);
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int c = lane + 64 * i;
    if (c >= nq) continue;
    const f32x4 y = (v[i] - mean) * rstd * (1.f + c4[i]) + s4[i];
    if constexpr (sizeof(OutT) == 2) {
      ((u32x2*)S.out)[(long)r * nq + c] = u32x2{pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3])};
    } else {
      ((f32x4*)S.out)[(long)r * nq + c] = y;
    }
  }
}

template <typename OutT>
static hipError_t ln_dispatch(const LnArgs& a, hipStream_t st) {
  dim3 grid((a.total_rows + 3) / 4), block(256);
  const int nv = (a.D / 4 + 63) / 64;
  if (nv <= 2) hipLaunchKernelGGL((ln_mod_kernel<OutT, 2>), grid, block, 0, st, a);
  else if (nv <= 5) hipLaunchKernelGGL((ln_mod_kernel<OutT, 5>), grid, block, 0, st, a);
  else if (nv <= 8) hipLaunchKernelGGL((ln_mod_kernel<OutT, 8>), grid, block, 0, st, a);
  else if (nv <= 12) hipLaunchKernelGGL((ln_mod_kernel<OutT, 12>), grid, block, 0, st, a);
  else hipLaunchKernelGGL((ln_mod_kernel<OutT, 16>), grid, block, 0, st, a);
  return hipGetLastError();
}

hipError_t launch_ln_mod(const LnArgs& a, int dtype, hipStream_t st) {
  return dtype == 1 ? ln_dispatch<bf16_t>(a, st) : ln_dispatch<float>(a, st);
}

// Eight weights of either type as floats.
template <typename WT> struct W8;
template <> struct W8<bf16_t> {
  static __device__ __forceinline__ void load(const bf16_t* p, float* w) {
    uint4 u = *(const uint4*)p;
    uint32_t x[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      w[2 * i] = __uint_as_float(x[i] << 16);
      w[2 * i + 1] = __uint_as_float(x[i] & 0xFFFF0000u);
    }
  }
};
template <> struct W8<float> {
  static __device__ __forceinline__ void load(const float* p, float* w) {
    float4 u0 = *(const float4*)p, u1 = *(const float4*)(p + 4);
    w[0] = u0.x; w[1] = u0.y; w[2] = u0.z; w[3] = u0.w;
    w[4] = u1.x; w[5] = u1.y; w[6] = u1.z; w[7] = u1.w;
  }
};

// ---------------------------------------------------------------- split-K reduction + LayerNorm + modulate
// The reduction of a split residual GEMM (splitk_resid_kernel) and the
// LayerNorm-modulate of the rows it updates in one launch: x += gate (sum of
// the partials + bias), h = LN(x) (1 + scale) + shift.  A workgroup of four
// waves per row (NV 4-column groups per thread), so that 256 rows still are
// 256 workgroups; exact two-pass statistics as in ln_mod_kernel.  Bound by
// latency at the row counts that are split: 256 rows of 1152 in six ranges 5.1 us
// (6.1 with a loop over the ranges), against 4.2 + 3.8 for the two launches.
__device__ __forceinline__ float block_sum(float v, float* slot) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) slot[threadIdx.x >> 6] = v;
  __syncthreads();
  return (slot[0] + slot[1]) + (slot[2] + slot[3]);
}

template <typename WT, int NV, int MS>
__global__ __launch_bounds__(256) void splitk_resid_ln_kernel(const float* __restrict__ part, int S, long MN, int D,
                                                              const WT* __restrict__ bias,
                                                              const float* __restrict__ gate, int gate_stride,
                                                              float* __restrict__ resid, LnSeg seg, float eps) {
  __shared__ float slots[2][4];
  const int row = blockIdx.x, tid = threadIdx.x, nq = D >> 2;
  const int b = row / seg.rows_per_batch;  // uniform
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  f32x4 v[NV], s4[NV], c4[NV];
  float sum = 0.f;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int c = tid + 256 * i, n = min(c, nq - 1) * 4;  // clamped: always valid
    const long e = (long)row * D + n;
    const f32x4 y = sum_parts<MS>(part + e, S, MN);
    f32x4 bv;
    if constexpr (sizeof(WT) == 2) {
      const u32x2 w = *(const u32x2*)(bias + n);
      bv = f32x4{__uint_as_float(w[0] << 16), __uint_as_float(w[0] & 0xFFFF0000u), __uint_as_float(w[1] << 16),
                 __uint_as_float(w[1] & 0xFFFF0000u)};
    } else {
      bv = *(const f32x4*)(bias + n);
    }
    const f32x4 x = *(const f32x4*)(resid + e) + *(const f32x4*)(gate + (long)b * gate_stride + n) * (y + bv);
    s4[i] = *(const f32x4*)(seg.shift + (long)b * seg.mod_stride + n);
    c4[i] = *(const f32x4*)(seg.scale + (long)b * seg.mod_stride + n);
    v[i] = c < nq ? x : zero;
    if (c < nq) *(f32x4*)(resid + e) = x;
    sum += (v[i][0] + v[i][1]) + (v[i][2] + v[i][3]);
  }
  const float mean = block_sum(sum, slots[0]) / (float)D;
  float sq = 0.f;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const f32x4 d = v[i] - mean;
    sq += tid + 256 * i < nq ? (d[0] * d[0] + d[1] * d[1]) + (d[2] * d[2] + d[3] * d[3]) : 0.f;
  }
  const float rstd = 1.0f / sqrtf(block_sum(sq, slots[1]) / (float)D + eps);
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int c = tid + 256 * i;
    if (c >= nq) continue;
    const f32x4 y = (v[i] - mean) * rstd * (1.f + c4[i]) + s4[i];
    if constexpr (sizeof(WT) == 2)
      ((u32x2*)seg.out)[(long)row * nq + c] = u32x2{pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3])};
    else
      ((f32x4*)seg.out)[(long)row * nq + c] = y;
  }
}

template <typename WT>
static hipError_t resid_ln_dispatch(const float* part, int S, int M, int N, const WT* bias, const float* gate,
                                    int gate_stride, float* resid, const LnArgs& ln, hipStream_t st) {
  const long MN = (long)M * N;
  if (M == 0) return hipSuccess;
  const int nv = (N / 4 + 255) / 256;  // hidden <= 4096
  with_max_parts(S, [&](auto ms) {
    constexpr int MS = decltype(ms)::value;
    if (nv <= 1)
      hipLaunchKernelGGL((splitk_resid_ln_kernel<WT, 1, MS>), dim3(M), dim3(256), 0, st, part, S, MN, N, bias, gate,
                         gate_stride, resid, ln.s[0], ln.eps);
    else if (nv <= 2)
      hipLaunchKernelGGL((splitk_resid_ln_kernel<WT, 2, MS>), dim3(M), dim3(256), 0, st, part, S, MN, N, bias, gate,
                         gate_stride, resid, ln.s[0], ln.eps);
    else
      hipLaunchKernelGGL((splitk_resid_ln_kernel<WT, 4, MS>), dim3(M), dim3(256), 0, st, part, S, MN, N, bias, gate,
                         gate_stride, resid, ln.s[0], ln.eps);
  });
  return hipGetLastError();
}

hipError_t launch_splitk_resid_ln(const float* part, int S, int M, int N, const void* bias, const float* gate,
                                  int gate_stride, float* resid, const LnArgs& ln, int dtype, hipStream_t st) {
  return dtype == 1 ? resid_ln_dispatch(part, S, M, N, (const bf16_t*)bias, gate, gate_stride, resid, ln, st)
                    : resid_ln_dispatch(part, S, M, N, (const float*)bias, gate, gate_stride, resid, ln, st);
}

// ---------------------------------------------------------------- adaLN GEMV
// out^T [N, B] = W [N, K] * SiLU(c)^T [K, B] on 16-row MFMA tiles
// (v_mfma_f32_16x16x32_bf16; for fp32 weights four v_mfma_f32_16x16x4_f32,
// exact fp32 products).  A step of the k loop takes 64 bytes of each of the 16
// rows: lane (row r16 = lane % 16, quarter kq = lane / 16) reads the 16 bytes
// at 16 kq of its row's 64, and the B operand holds the same k positions of
// sample r16, so the assignment of k to MFMA lanes cancels.
//
// Bound by HBM reads of W, i.e. by how many loads are in flight.  A workgroup
// owns 16 RT rows of one matrix and its four waves take a quarter of k each,
// added through LDS in wave order; the loads of the next U steps are in
// flight while the current U are multiplied.  One block's matrix (6912 x 1152)
// is then 216 or 432 workgroups; as 27 workgroups whose waves each walked the
// whole of k it was a serial chain of loads.  Measured with SiLU's launch,
// before -> after: that matrix at 1 sample 22.8 -> 7.8 us, at 8 25 -> 10, the
// joint block's two (18432 x 3072, 226 MB) 83 -> 57 us, one of them at 8
// samples 77 -> 39 us; all 28 of DiT-XL/2 (450 MB) at 8 samples 109 -> 107, at
// 1 sample 94 -> 86 us.  16 loads in flight per lane instead of 8 leave too few
// waves (28 matrices: 167 us).
//
// SiLU(c): FUSED, every workgroup computes it into LDS for up to nbc samples
// at a time and one launch fewer is needed (adaln_fused).  In fp32 each further
// pass of what 64 KB hold reads the matrix again, from hidden 3072 on slower than
// the VALU kernel it replaced (8 samples: 120 -> 147 us; 4096 160 -> 230; one sample
// 58 -> 52, 90 -> 88); 132 KB helped only where it saved the one further pass
// (2048: 67 -> 48) and cost residency elsewhere (3072: 153).  Otherwise (bf16
// only) it comes from `act`, written once by silu_bf16_kernel and read through
// L2 with the weights.  Lanes of samples past the batch supply zeros.  D
// lanes hold sample lane % 16, rows 4 (lane / 16) + i.
__global__ void silu_bf16_kernel(int B, int D, int rows, const float* cond, bf16_t* act) {
  const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (long)rows * D) return;
  const int r = (int)(idx / D);
  act[idx] = r < B ? f2bf(silu(cond[idx])) : (bf16_t)0;
}

hipError_t launch_silu_bf16(int B, int D, const float* cond, void* act, hipStream_t st) {
  const int rows = (B + 15) / 16 * 16;
  const long n = (long)rows * D;
  hipLaunchKernelGGL(silu_bf16_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, B, D, rows, cond,
                     (bf16_t*)act);
  return hipGetLastError();
}

// Staged sample rows are padded by 16 bytes, which spreads the 16 rows of a
// fragment read over the LDS banks.
template <typename WT>
static constexpr int ada_row_elems(int K) { return K + 16 / (int)sizeof(WT); }

template <typename WT, int RT, bool FUSED, bool NT>
__global__ __launch_bounds__(256) void adaln_mfma_kernel(AdaArgs a) {
  constexpr int KE = 64 / sizeof(WT);  // k per step
  constexpr int LE = 16 / sizeof(WT);  // elements per lane and step
  constexpr int U = 8 / RT;            // steps per group of loads
  extern __shared__ __attribute__((aligned(16))) unsigned char ada_smem[];
  f32x4* const red = (f32x4*)ada_smem;                 // [4 waves][RT][64]
  WT* const act_s = (WT*)(ada_smem + 4 * RT * 64 * 16);  // FUSED: [nbc][ada_row_elems]
  // every matrix but the last (the final layer's) has the same row count
  const int wg = blockIdx.x;
  const int ei = min(wg / a.wg_per_entry, a.ne - 1);
  const AdaEntry E = a.e[ei];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int K = a.D, N = E.N;
  const int nbase = (wg - E.wg_begin) * (16 * RT);  // N is a multiple of 128
  const int r16 = lane & 15, kq = lane >> 4;
  // the wave's k range, in whole 128-byte lines (K is a multiple of 64)
  const int lines = K * (int)sizeof(WT) / 128;
  const int s0 = 2 * (lines * wave / 4), s1 = 2 * (lines * (wave + 1) / 4);
  const WT* wr[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) wr[t] = (const WT*)E.W + (long)(nbase + 16 * t + r16) * K + LE * kq;

  // weight fragments of U steps, and (not fused) SiLU(c) fragments with them
  u32x4 cur[RT][U], nxt[RT][U], cur_b[U], nxt_b[U];
  const WT* sp = nullptr;  // the lane's SiLU(c) row
  bool live = false;       // this lane's sample exists
  auto load = [&](u32x4 (&w)[RT][U], u32x4 (&b)[U], int s) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (s + u < s1) {
#pragma unroll
        for (int t = 0; t < RT; ++t) {
          const u32x4* p = (const u32x4*)(wr[t] + (s + u) * KE);
          w[t][u] = NT ? __builtin_nontemporal_load(p) : *p;
        }
        if (!FUSED) b[u] = live ? *(const u32x4*)(sp + (s + u) * KE) : u32x4{0u, 0u, 0u, 0u};
      }
  };
  const int step_b = FUSED ? a.nbc : 16;
  const int row_e = ada_row_elems<WT>(K);
  for (int b0 = 0; b0 < a.B; b0 += step_b) {
    const int nb = min(step_b, a.B - b0);
    live = r16 < nb;
    sp = FUSED ? act_s + r16 * row_e + LE * kq : (const WT*)a.act + (long)(b0 + r16) * K + LE * kq;
    load(cur, cur_b, s0);
    if (FUSED) {
      if (b0) __syncthreads();  // the previous samples' reads are done
      // four samples at a time, so that their loads overlap (cond is only
      // 4-byte aligned)
      for (int r = 0; r < nb; r += 4)
#pragma unroll 2
        for (int k = tid; k < K; k += 256) {
          float z[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) z[i] = a.cond[(long)(b0 + min(r + i, nb - 1)) * K + k];
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (r + i < nb) {
              if constexpr (sizeof(WT) == 2) act_s[(r + i) * row_e + k] = f2bf(silu(z[i]));
              else act_s[(r + i) * row_e + k] = z[i] / (1.0f + expf(-z[i]));
            }
        }
      __syncthreads();
    }
    f32x4 acc[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int s = s0; s < s1; s += U) {
      load(nxt, nxt_b, s + U);
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (s + u < s1) {
          const u32x4 bw = !FUSED ? cur_b[u] : live ? *(const u32x4*)(sp + (s + u) * KE) : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
          for (int t = 0; t < RT; ++t) {
            if constexpr (sizeof(WT) == 2) {
              acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, cur[t][u]),
                                                               __builtin_bit_cast(bf16x8, bw), acc[t], 0, 0, 0);
            } else {
              const f32x4 wf = __builtin_bit_cast(f32x4, cur[t][u]), bf = __builtin_bit_cast(f32x4, bw);
#pragma unroll
              for (int e = 0; e < 4; ++e)
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[e], bf[e], acc[t], 0, 0, 0);
            }
          }
        }
#pragma unroll
      for (int u = 0; u < U; ++u) {
#pragma unroll
        for (int t = 0; t < RT; ++t) cur[t][u] = nxt[t][u];
        cur_b[u] = nxt_b[u];
      }
    }
    if (b0) __syncthreads();  // the previous samples' sums have been read
#pragma unroll
    for (int t = 0; t < RT; ++t) red[(wave * RT + t) * 64 + lane] = acc[t];
    __syncthreads();
    if (wave < RT && live) {  // wave t adds row tile t
      f32x4 v = red[wave * 64 + lane];
#pragma unroll
      for (int w = 1; w < 4; ++w) v += red[(w * RT + wave) * 64 + lane];
      const int n = nbase + 16 * wave + 4 * kq;
      const WT* bias = (const WT*)E.bias + n;
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] += ld_as_float<WT>(bias, i);
      *(f32x4*)(E.out + (long)(b0 + r16) * N + n) = v;
    }
  }
}

// Whether the workgroups compute SiLU(c) themselves: always for fp32; for
// bf16 while matrices x samples is at most 4 (one block at four samples, a
// joint block at two), where repeating it in every workgroup costs less than
// a launch.  One 6912 x 1152 matrix at 1, 4, 8, 16 samples: 7.8, 9.5, 13.1,
// 19.7 us fused against 7.2-7.6 + 2.5 for SiLU's launch; 18432 x 3072 at 1, 4,
// 7 samples: 29, 37, 54 us against 31-34 + 4.7.
bool adaln_fused(int entries, int B, int dtype) { return dtype != 1 || entries * std::min(B, 16) <= 4; }

template <typename WT, int RT, bool FUSED, bool NT>
static hipError_t adaln_launch_t(AdaArgs& a, hipStream_t st) {
  int wg = 0;
  for (int j = 0; j < a.ne; ++j) {
    a.e[j].wg_begin = wg;
    wg += a.e[j].N / (16 * RT);
  }
  a.wg_per_entry = a.e[0].N / (16 * RT);
  const int row_bytes = ada_row_elems<WT>(a.D) * (int)sizeof(WT);
  // samples staged per pass: what 64 KB hold
  a.nbc = std::min(std::min(a.B, 16), std::max(1, 64 * 1024 / row_bytes));
  const size_t lds = 4 * RT * 64 * 16 + (FUSED ? (size_t)a.nbc * row_bytes : 0);
  if (lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute((const void*)adaln_mfma_kernel<WT, RT, FUSED, NT>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((adaln_mfma_kernel<WT, RT, FUSED, NT>), dim3(wg), dim3(256), lds, st, a);
  return hipGetLastError();
}

// Non-temporal weight loads (bf16) keep a matrix that is read once out of the
// way of the block's other weights and activations, which then stay cached from
// call to call: DiT-XL/2 block at 8 samples of 256 tokens 144.4 -> 138.9 us, joint
// block (226 MB of modulation weights) 1282 -> 1264; steps of 12 blocks at hidden
// 768 (85 MB) and 1 to 16 samples of 64 tokens 470-788 -> 429-715 (their adaLN
// launch alone 20-25 -> 25-30); of 384 (21 MB, all cached) the same within 0.7%;
// steps of 28 blocks unchanged.  Not where several passes over the samples read
// the matrix again, nor for fused launches below 64 MB: whole blocks with and
// without them at 16 MB 58.0 and 56.9 us, 28 MB 70.5 and 68.7, 57 MB 75.0 and
// 72.5, but 100 MB 103 and 126, 113 MB 102 and 121.
hipError_t launch_adaln(AdaArgs a, int dtype, bool fused, hipStream_t st) {
  if (dtype != 1) return adaln_launch_t<float, 1, true, false>(a, st);
  double bytes = 0;
  for (int j = 0; j < a.ne; ++j) bytes += 2.0 * a.e[j].N * a.D;
  if (fused)
    return bytes >= 64e6 ? adaln_launch_t<bf16_t, 1, true, true>(a, st) : adaln_launch_t<bf16_t, 1, true, false>(a, st);
  return a.B <= 16 ? adaln_launch_t<bf16_t, 2, false, true>(a, st) : adaln_launch_t<bf16_t, 2, false, false>(a, st);
}

// ---------------------------------------------------------------- conditioning
// e_b = [cos(t_b f_i), sin(t_b f_i)], f_i = exp(-ln(10000) i / 128), i < 128;
// h1 = SiLU(e W1^T + b1);  cond = h1 W2^T + b2 + class_table[y].  Two
// dependent launches, each bound by latency (3.3 MB at DiT-XL/2, 8 samples):
// what counts is that a wave's loads are all in flight at once, that samples
// are independent chains, and that their inputs sit in LDS.  Measured at 8
// samples, hidden 1152: three launches (features,
// and each layer a wave per row with a serial loop over the samples) 2.5 + 6.8 +
// 11.6 us, now 5.3 + 5.9; 16 samples 34.5 -> 18 us, 11 samples at hidden 3072 in
// fp32 42 -> 29 us
//
// Sum over the wavefront of v[i], i < NV (independent chains).
template <int NV>
__device__ __forceinline__ void wave_sums(float (&v)[NV]) {
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] += dpp_move<0xB1>(v[i]);
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] += dpp_move<0x4E>(v[i]);
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] += dpp_move<0x141>(v[i]);
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] += dpp_move<0x140>(v[i]);
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int b = __float_as_int(v[i]);
    v[i] = (__int_as_float(__builtin_amdgcn_readlane(b, 0)) + __int_as_float(__builtin_amdgcn_readlane(b, 16))) +
           (__int_as_float(__builtin_amdgcn_readlane(b, 32)) + __int_as_float(__builtin_amdgcn_readlane(b, 48)));
  }
}

// Four consecutive weights of either type as floats.
__device__ __forceinline__ f32x4 ld_w4(const float* p) { return *(const f32x4*)p; }
__device__ __forceinline__ f32x4 ld_w4(const bf16_t* p) {
  const u32x2 w = *(const u32x2*)p;
  return f32x4{__uint_as_float(w[0] << 16), __uint_as_float(w[0] & 0xFFFF0000u), __uint_as_float(w[1] << 16),
               __uint_as_float(w[1] & 0xFFFF0000u)};
}
__device__ __forceinline__ float dot4(const f32x4& a, const f32x4& b, float acc) {
  return fmaf(a[3], b[3], fmaf(a[2], b[2], fmaf(a[1], b[1], fmaf(a[0], b[0], acc))));
}

// Hidden layer: 16 waves, one row of W1 each; the features of up to CND_NB
// samples at a time are computed by every workgroup (in double, for the large
// arguments; one or two per thread) rather than by a launch of their own.
// t = NULL: every sample at t_val.  N is a multiple of 64.
constexpr int CND_NB = 16;
template <typename WT>
__global__ __launch_bounds__(1024) void cond_hidden_kernel(int B, int N, const float* t, float t_val, const WT* W,
                                                           const WT* bias, float* h1) {
  __shared__ __attribute__((aligned(16))) float feat[CND_NB][256];
  const int tid = threadIdx.x, lane = tid & 63, n = blockIdx.x * 16 + (tid >> 6);
  const f32x4 w = ld_w4(W + (long)n * 256 + lane * 4);
  const float bn = ld_as_float<WT>(bias, n);
  const double f = exp(-9.210340371976184 * (double)(tid & 127) / 128.0);  // ln(10000)
  for (int b0 = 0; b0 < B; b0 += CND_NB) {
    const int nb = min(CND_NB, B - b0);
    if (b0) __syncthreads();  // the previous samples' reads are done
    for (int b = tid >> 7; b < nb; b += 8) {
      double sn, cs;
      sincos((double)(t ? t[b0 + b] : t_val) * f, &sn, &cs);
      feat[b][tid & 127] = (float)cs;
      feat[b][128 + (tid & 127)] = (float)sn;
    }
    __syncthreads();
    for (int b = 0; b < nb; b += 4) {
      float acc[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[i] = dot4(w, *(const f32x4*)&feat[min(b + i, nb - 1)][lane * 4], 0.f);
      wave_sums(acc);
      const float z = (lane == 0 ? acc[0] : lane == 1 ? acc[1] : lane == 2 ? acc[2] : acc[3]) + bn;
      if (lane < 4 && b + lane < nb) h1[(long)(b0 + b + lane) * N + n] = z / (1.0f + expf(-z));
    }
  }
}

// Output layer: NW waves, one row of W2 each, held in registers (G groups of
// 4 E consecutive weights per lane, 256 E apart).  NS = 4: h1 of up to nbc
// samples at a time staged in LDS, four samples per pass, E = 1 (conflict-free
// reads); NS = 1 (one sample): read straight from global memory with the
// weights, E = 2 (16-byte loads of bf16 weights).  Lanes past a row's end
// must add nothing, whatever they read (zero weights would make NaN of an
// infinity): their sums are dropped.  They read on past a staged row, which costs
// less than a clamped address: hs has room for 256 G floats from its last row on.
template <typename WT, int G, int E, int NW, int NS>
__global__ __launch_bounds__(NW * 64) void cond_out_kernel(int B, int N, int K, int nbc, const float* h1, const WT* W,
                                                           const WT* bias, const WT* table, const int32_t* y,
                                                           float* cond) {
  extern __shared__ __attribute__((aligned(16))) float hs[];  // NS = 4: [nbc][K]
  const int tid = threadIdx.x, lane = tid & 63, n = blockIdx.x * NW + (tid >> 6);
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  f32x4 w[G][E];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const int k = (256 * g + lane * 4) * E;
    if (E == 2) {
      float t[8] = {};
      if (k < K) W8<WT>::load(W + (long)n * K + k, t);
#pragma unroll
      for (int e = 0; e < E; ++e) w[g][e] = f32x4{t[4 * e], t[4 * e + 1], t[4 * e + 2], t[4 * e + 3]};
    } else {
      w[g][0] = k < K ? ld_w4(W + (long)n * K + k) : zero;
    }
  }
  const float bn = ld_as_float<WT>(bias, n);
  for (int b0 = 0; b0 < B; b0 += nbc) {
    const int nb = min(nbc, B - b0);
    // lane i: class embedding of sample b0 + i
    const float emb = lane < nb ? ld_as_float<WT>(table, (long)y[b0 + lane] * N + n) : 0.f;
    if (NS > 1) {
      if (b0) __syncthreads();  // the previous samples' reads are done
#pragma unroll 4
      for (int i = tid; i < nb * K / 4; i += NW * 64) ((f32x4*)hs)[i] = ((const f32x4*)(h1 + (long)b0 * K))[i];
      __syncthreads();
    }
    const float* const in = NS > 1 ? hs : h1;
    for (int b = 0; b < nb; b += NS) {
      float acc[NS] = {};
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const int kl = (256 * g + lane * 4) * E, k = NS > 1 ? kl : min(kl, K - 4 * E);
#pragma unroll
        for (int i = 0; i < NS; ++i) {
          float s = acc[i];
#pragma unroll
          for (int e = 0; e < E; ++e) s = dot4(w[g][e], *(const f32x4*)&in[min(b + i, nb - 1) * K + k + 4 * e], s);
          acc[i] = kl < K ? s : acc[i];
        }
      }
      wave_sums(acc);
      float v = acc[0];
#pragma unroll
      for (int i = 1; i < NS; ++i) v = lane - b == i ? acc[i] : v;
      if (lane >= b && lane < b + NS && lane < nb) cond[(long)(b0 + lane) * N + n] = v + bn + emb;
    }
  }
}

template <typename WT>
static hipError_t cond_launch_t(int B, int D, const float* t, float t_val, const int32_t* y, const WT* w1,
                                const WT* b1, const WT* w2, const WT* b2, const WT* table, float* h1, float* cond,
                                hipStream_t st) {
  hipLaunchKernelGGL((cond_hidden_kernel<WT>), dim3(D / 16), dim3(1024), 0, st, B, D, t, t_val, w1, b1, h1);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // h1 of as many samples as 64 KB hold (at least 4: hidden <= 4096), one lane
  // each at most, and what the lanes past the last row's end read (at most 11 KB).
  // 4 rows per workgroup fill the GPU soonest; 16 where staging the samples for
  // every 4 rows would be the larger part of the work (11 samples at hidden 3072,
  // fp32: 34 us with 4 rows, 23 with 16).
  const int past = ((D <= 1280 ? 5 : 16) * 256 - D) * 4;
  const int nbc = std::min(std::min(B, 64), 64 * 1024 / (D * 4));
  const size_t lds = B > 1 ? (size_t)nbc * D * 4 + past : 0;
#define COND_OUT(G, E, NW, NS)                                                                                       \
  do {                                                                                                               \
    if (lds > 64 * 1024 &&                                                                                           \
        (e = hipFuncSetAttribute((const void*)cond_out_kernel<WT, G, E, NW, NS>,                                     \
                                 hipFuncAttributeMaxDynamicSharedMemorySize, 76 * 1024)) != hipSuccess)              \
      return e;                                                                                                      \
    hipLaunchKernelGGL((cond_out_kernel<WT, G, E, NW, NS>), dim3(D / NW), dim3(NW * 64), lds, st, B, D, D, nbc, h1,  \
                       w2, b2, table, y, cond);                                                                      \
  } while (0)
  const bool wide = (size_t)B * D * 4 > 40 * 1024;
  if (D <= 1280) {  // 5 x 256 weights per row
    if (B == 1) COND_OUT(3, 2, 4, 1);
    else if (wide) COND_OUT(5, 1, 16, 4);
    else COND_OUT(5, 1, 4, 4);
  } else {
    if (B == 1) COND_OUT(8, 2, 4, 1);
    else if (wide) COND_OUT(16, 1, 16, 4);
    else COND_OUT(16, 1, 4, 4);
  }
#undef COND_OUT
  return hipGetLastError();
}

hipError_t launch_cond_embed(int B, int D, const float* t, float t_val, const int32_t* y, const void* w1,
                             const void* b1, const void* w2, const void* b2, const void* table, float* h1,
                             float* cond, int dtype, hipStream_t st) {
  if (dtype == 1)
    return cond_launch_t(B, D, t, t_val, y, (const bf16_t*)w1, (const bf16_t*)b1, (const bf16_t*)w2,
                         (const bf16_t*)b2, (const bf16_t*)table, h1, cond, st);
  return cond_launch_t(B, D, t, t_val, y, (const float*)w1, (const float*)b1, (const float*)w2, (const float*)b2,
                       (const float*)table, h1, cond, st);
}

// Patch embedding x = z W^T + b (+ pos), fp32 accumulation from b on over the
// channels (in order, but for the matrix cores' order within four), then pos.
//
// Up to 16 channels (patch_row_kernel): one workgroup per token row, the
// patch vector in LDS, each lane a column.
template <typename WT>
__global__ __launch_bounds__(256) void patch_row_kernel(int T, int P, int D, const float* __restrict__ z,
                                                        const WT* __restrict__ w, const WT* __restrict__ bias,
                                                        const float* __restrict__ pos, float* __restrict__ x) {
  __shared__ float zs[16];
  const int row = blockIdx.x, tid = threadIdx.x;
  if (tid < P) zs[tid] = z[(long)row * P + tid];
  __syncthreads();
  const int t = row % T;
  for (int n = tid; n < D; n += 256) {
    float acc = ld_as_float<WT>(bias, n);
    const WT* wr = w + (long)n * P;
    for (int p = 0; p < P; ++p) acc = fmaf(ld_as_float<WT>(wr, p), zs[p], acc);
    if (pos) acc += pos[(long)t * D + n];
    x[(long)row * D + n] = acc;
  }
}

// More channels (patch_tile_kernel): a workgroup owns 256 consecutive
// columns and PT_ROWS rows.  Per chunk of 64 channels, the rows' latent
// values are staged in LDS (read back as one broadcast 16-byte read per four
// channels) and each lane holds its column's 64 weights in registers, so
// every weight element is read once per workgroup instead of once per row.
constexpr int PT_ROWS = 32, PT_CHUNK = 64;

template <typename WT>
__global__ __launch_bounds__(256) void patch_tile_kernel(int rows, int T, int P, int D, const float* __restrict__ z,
                                                         const WT* __restrict__ w, const WT* __restrict__ bias,
                                                         const float* __restrict__ pos, float* __restrict__ x) {
  __shared__ __attribute__((aligned(16))) float zs[PT_ROWS][PT_CHUNK];
  const int tid = threadIdx.x;
  const int n = blockIdx.x * 256 + tid;
  const int r0 = blockIdx.y * PT_ROWS;
  const int nr = min(PT_ROWS, rows - r0);
  const bool col = n < D;
  const float b = col ? ld_as_float<WT>(bias, n) : 0.f;
  float acc[PT_ROWS];
#pragma unroll
  for (int r = 0; r < PT_ROWS; ++r) acc[r] = b;
  for (int p0 = 0; p0 < P; p0 += PT_CHUNK) {
    const int pc = min(PT_CHUNK, P - p0);
    __syncthreads();  // the previous chunk's reads are done
    for (int e = tid; e < PT_ROWS * PT_CHUNK; e += 256) {
      const int r = e / PT_CHUNK, c = e % PT_CHUNK;
      zs[r][c] = r < nr && c < pc ? z[(long)(r0 + r) * P + p0 + c] : 0.f;
    }
    float wv[PT_CHUNK];
    if (col && pc == PT_CHUNK && P % 8 == 0) {
      // the lane's 64 weights as 16-byte loads (8 elements each, aligned:
      // n P + p0 + c is a multiple of 8)
#pragma unroll
      for (int c = 0; c < PT_CHUNK; c += 8) W8<WT>::load(w + (long)n * P + p0 + c, &wv[c]);
    } else {
#pragma unroll
      for (int c = 0; c < PT_CHUNK; ++c) wv[c] = col && c < pc ? ld_as_float<WT>(w, (long)n * P + p0 + c) : 0.f;
    }
    __syncthreads();
    if (pc == PT_CHUNK) {
#pragma unroll
      for (int r = 0; r < PT_ROWS; ++r)
#pragma unroll
        for (int c = 0; c < PT_CHUNK; c += 4) {
          const f32x4 zv = *(const f32x4*)&zs[r][c];
          acc[r] = fmaf(wv[c], zv[0], acc[r]);
          acc[r] = fmaf(wv[c + 1], zv[1], acc[r]);
          acc[r] = fmaf(wv[c + 2], zv[2], acc[r]);
          acc[r] = fmaf(wv[c + 3], zv[3], acc[r]);
        }
    } else {  // last, partial chunk (static register indices, channels c < pc only)
#pragma unroll
      for (int r = 0; r < PT_ROWS; ++r)
#pragma unroll
        for (int c = 0; c < PT_CHUNK; ++c)
          if (c < pc) acc[r] = fmaf(wv[c], zs[r][c], acc[r]);
    }
  }
  if (!col) return;
#pragma unroll
  for (int r = 0; r < PT_ROWS; ++r) {
    if (r >= nr) break;
    const int row = r0 + r;
    float v = acc[r];
    if (pos) v += pos[(long)(row % T) * D + n];
    x[(long)row * D + n] = v;
  }
}

// Channels in whole 16s (patch_mfma_kernel): v_mfma_f32_16x16x4_f32 (exact fp32
// products, fp32 accumulation from the bias on).  A wave owns 64 columns and
// PM_ROWS rows: A = the weights (converted to fp32 once per 64 channels, kept
// in registers for all its rows), B = the latent rows, both 16 bytes of fp32 per
// lane and 16 channels straight from global memory.  Column n = 16 kq + 4 j + e
// of the 64 is row 4 kq + e of tile j, so a lane ends with 16 consecutive
// columns of one row and a row is stored as 256 contiguous bytes.  Bound by
// the stores (x is 4 D bytes a row).  64 channels, 2000 rows of 1536: 21.4 us (the
// tile kernel above) -> 16.4; 16 channels, 4096 rows of 3072: 33.7 us (a
// workgroup per row) -> 26.1, 256 rows of 1152: 6.8 -> 4.9.
constexpr int PM_ROWS = 32;

template <typename WT>
__global__ __launch_bounds__(256) void patch_mfma_kernel(int rows, int T, int P, int D, const float* __restrict__ z,
                                                         const WT* __restrict__ w, const WT* __restrict__ bias,
                                                         const float* __restrict__ pos, float* __restrict__ x) {
  constexpr int RT = PM_ROWS / 16;
  const int lane = threadIdx.x & 63, r16 = lane & 15, kq = lane >> 4;
  // column blocks fastest, in one dimension: the row blocks can exceed the 65536 of a grid's second
  const int cb = D >> 6, rb = blockIdx.x / cb;
  const int n0 = (blockIdx.x - rb * cb) * 64, row0 = (rb * 4 + (threadIdx.x >> 6)) * PM_ROWS;
  if (row0 >= rows) return;
  const WT* wr = w + (long)(n0 + 16 * (r16 >> 2) + (r16 & 3)) * P + 4 * kq;  // tile j: + 4 j rows
  const float* zr[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) zr[t] = z + (long)min(row0 + 16 * t + r16, rows - 1) * P + 4 * kq;
  f32x4 acc[RT][4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    f32x4 b;
#pragma unroll
    for (int e = 0; e < 4; ++e) b[e] = ld_as_float<WT>(bias, n0 + 16 * kq + 4 * j + e);
#pragma unroll
    for (int t = 0; t < RT; ++t) acc[t][j] = b;
  }
  for (int p0 = 0; p0 < P; p0 += 64) {
    f32x4 wv[4][4], zv[RT][4];  // [16-channel step][column tile], [row tile][step]
#pragma unroll
    for (int s = 0; s < 4; ++s)
      if (p0 + 16 * s < P) {
#pragma unroll
        for (int j = 0; j < 4; ++j) wv[s][j] = ld_w4(wr + (long)4 * j * P + p0 + 16 * s);
#pragma unroll
        for (int t = 0; t < RT; ++t) zv[t][s] = *(const f32x4*)(zr[t] + p0 + 16 * s);
      }
#pragma unroll
    for (int s = 0; s < 4; ++s)
      if (p0 + 16 * s < P)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j)
              acc[t][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[s][j][e], zv[t][s][e], acc[t][j], 0, 0, 0);
  }
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    const int row = row0 + 16 * t + r16, n = n0 + 16 * kq;
    if (row >= rows) continue;
    const float* pr = pos ? pos + (long)(row % T) * D + n : nullptr;  // 4-byte aligned
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      f32x4 v = acc[t][j];
      if (pos)
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] += pr[4 * j + e];
      *(f32x4*)(x + (long)row * D + n + 4 * j) = v;
    }
  }
}

template <typename WT>
static void launch_patch_embed_t(int rows, int T, int P, int D, const float* z, const WT* w, const WT* b,
                                 const float* pos, float* x, hipStream_t st) {
  // the MFMA kernel's loads are 4 consecutive channels: whole 16s of channels
  // and latents and weights aligned for it (the entry points ask for 4 bytes only)
  const bool mfma = P % 16 == 0 && (uintptr_t)z % 16 == 0 && (uintptr_t)w % (4 * sizeof(WT)) == 0;
  if (mfma)
    hipLaunchKernelGGL((patch_mfma_kernel<WT>), dim3(D / 64 * ((rows + 4 * PM_ROWS - 1) / (4 * PM_ROWS))), dim3(256),
                       0, st, rows, T, P, D, z, w, b, pos, x);
  else if (P <= 16)
    hipLaunchKernelGGL((patch_row_kernel<WT>), dim3(rows), dim3(256), 0, st, T, P, D, z, w, b, pos, x);
  else
    hipLaunchKernelGGL((patch_tile_kernel<WT>), dim3((D + 255) / 256, (rows + PT_ROWS - 1) / PT_ROWS), dim3(256), 0,
                       st, rows, T, P, D, z, w, b, pos, x);
}

hipError_t launch_patch_embed(int rows, int T, int P, int D, const float* z, const void* w, const void* b,
                              const float* pos, float* x, int dtype, hipStream_t st) {
  if (rows <= 0) return hipSuccess;
  if (dtype == 1)
    launch_patch_embed_t<bf16_t>(rows, T, P, D, z, (const bf16_t*)w, (const bf16_t*)b, pos, x, st);
  else
    launch_patch_embed_t<float>(rows, T, P, D, z, (const float*)w, (const float*)b, pos, x, st);
  return hipGetLastError();
}

// ---------------------------------------------------------------- 2-D sin-cos table
__global__ void pos_embed_2d_kernel(int gh, int gw, int D, float* pos) {
  const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const long total = (long)gh * gw * D;
  if (idx >= total) return;
  const int n = (int)(idx / D), dd = (int)(idx - (long)n * D);
  const int r = n / gw, c = n - r * gw;
  const int half = D / 2, q = D / 4;
  const int p = dd < half ? c : r;
  const int e = dd < half ? dd : dd - half;
  const int i = e < q ? e : e - q;
  const double omega = exp(-9.210340371976184 * (double)i / (double)q);  // 10000^(-i/q)
  const double arg = (double)p * omega;
  pos[idx] = (float)(e < q ? sin(arg) : cos(arg));
}

hipError_t launch_pos_embed_2d(int gh, int gw, int D, float* pos, hipStream_t st) {
  const long total = (long)gh * gw * D;
  hipLaunchKernelGGL(pos_embed_2d_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, gh, gw, D, pos);
  return hipGetLastError();
}

// ---------------------------------------------------------------- sampler loop
// Euler update z += a * v over n floats (n a multiple of 4, 16-byte aligned).
__global__ void axpy_f32_kernel(f32x4* z, const f32x4* v, float a, long n4) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n4) z[i] += a * v[i];
}

hipError_t launch_axpy_f32(float* z, const float* v, float a, long n, hipStream_t st) {
  const long n4 = n / 4;
  if (n4 <= 0) return hipSuccess;
  hipLaunchKernelGGL(axpy_f32_kernel, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, st, (f32x4*)z,
                     (const f32x4*)v, a, n4);
  return hipGetLastError();
}


}  // namespace ditmi
