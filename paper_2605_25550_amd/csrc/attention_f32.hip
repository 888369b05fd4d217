// Multi-head attention for the fp32 DiT path: O = softmax(q k^T / sqrt(dh)) v
// with fp32 products on the matrix cores (v_mfma_f32_16x16x4_f32), fp32 exp and
// fp32 accumulation (online softmax).
//
// A workgroup of four waves owns 16 QT queries of one (sample, head).  The
// waves split the keys: wave w takes the 32-key groups w, w + 4, ... with a
// softmax state of its own, and the four states are merged through LDS at the
// end, so a short sequence still gives four waves per query block and a chain
// of a quarter of its keys.  K and V fragments come straight from global
// memory (L2) as 16-byte loads: no two waves of a workgroup read the same
// key, so staging them in LDS would share nothing.
//
// S^T = K Q^T: A = 16 keys (lane row r16 = lane % 16, four consecutive d at
// 4 kq, kq = lane / 16), B = Q^T held in registers (column r16), MFMA e of a
// 16-wide d step takes element e of both.  A lane then holds, of query r16,
// keys 4 kq + e: MFMA e of O^T = V^T P^T uses keys 4 kq + e as its k, so P is
// its B operand as it is.  The rows of O^T tile t are d = 64 (t / 4) + 4 i +
// t % 4, so that one 16-byte load of V row (4 kq + e) at d = 4 r16 feeds four
// tiles; head_dim 72's last eight columns are a tile of single loads.  Lane
// rows 4 kq + e of the four tiles are again four consecutive d of O.
//
// Bound by the serial chain of a wave (small calls) or the matrix pipe and
// L2; measured (before: four lanes per query on the VALU, 64 queries per
// workgroup over all keys): 6 heads of 64 over 256 tokens 74 -> 8.3 us, 2 x 16
// heads of 72 over 333 tokens 184 -> 25 us, 16 heads of 72 over 2048 tokens
// 274 us (71 TFLOP/s of the 155 the pipe gives).
#include "common.h"
#include "kernels.h"

namespace ditmi {

template <int DH, int QT>
__global__ __launch_bounds__(256) void attn_f32_kernel(AttnArgs a) {
  constexpr int KS = (DH + 15) / 16;      // 16-wide steps of QK^T; the last of head_dim 72 is half empty
  constexpr int VB = DH / 64;             // 64-column blocks of V (16-byte loads) ...
  constexpr int VX = DH % 64 ? 1 : 0;     // ... and a tile of the last DH % 64 columns (head_dim 72)
  constexpr int TV = 4 * VB + VX;         // O^T tiles
  constexpr int OS = DH + 4;              // row stride of a wave's O in LDS
  __shared__ __attribute__((aligned(16))) float os[4][16 * QT][OS];
  __shared__ float ml[4][2][16 * QT];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, kq = lane >> 4;
  const int b = blockIdx.z, h = blockIdx.y, q0 = blockIdx.x * (16 * QT);
  const int Tj = a.Tj;
  const long bh = (long)b * a.H + h;
  const float* __restrict__ qp = (const float*)a.q + bh * Tj * DH;
  const float* __restrict__ kp = (const float*)a.k + bh * Tj * DH;
  const float* __restrict__ vp = (const float*)a.v + bh * Tj * DH;

  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  const bool dlast = 16 * (KS - 1) + 4 * kq < DH;  // the lane's columns of the last step exist
  f32x4 qf[QT][KS], o[QT][TV];
  float m_run[QT], l_run[QT];
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    const float* qr = qp + (long)min(q0 + 16 * t + r16, Tj - 1) * DH + 4 * kq;
#pragma unroll
    for (int s = 0; s < KS; ++s) qf[t][s] = s < KS - 1 || dlast ? *(const f32x4*)(qr + 16 * s) : zero;
#pragma unroll
    for (int v = 0; v < TV; ++v) o[t][v] = zero;
    m_run[t] = -INFINITY;
    l_run[t] = 0.f;
  }

  const int ng = (Tj + 31) / 32;
  f32x4 kf[2][KS];
  auto load_k = [&](int g) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const float* kr = kp + (long)min(g * 32 + 16 * c + r16, Tj - 1) * DH + 4 * kq;  // past the end: masked
#pragma unroll
      for (int s = 0; s < KS; ++s) kf[c][s] = s < KS - 1 || dlast ? *(const f32x4*)(kr + 16 * s) : zero;
    }
  };
  if (wave < ng) load_k(wave);
  for (int g = wave; g < ng; g += 4) {
    const int kv0 = g * 32;
    // V rows 4 kq + e of both 16-key halves, requested before the scores
    f32x4 vf[2][4][VB];
    float vx[2][4];
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float* vr = vp + (long)min(kv0 + 16 * c + 4 * kq + e, Tj - 1) * DH;
#pragma unroll
        for (int v = 0; v < VB; ++v) vf[c][e][v] = *(const f32x4*)(vr + 64 * v + 4 * r16);
        if (VX) vx[c][e] = r16 < DH % 64 ? vr[64 * VB + r16] : 0.f;
      }
    if (kv0 + 32 > Tj) {  // keys past the end: a zero probability must not meet an infinite value
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (kv0 + 16 * c + 4 * kq + e >= Tj) {
#pragma unroll
            for (int v = 0; v < VB; ++v) vf[c][e][v] = zero;
            vx[c][e] = 0.f;
          }
    }
    f32x4 s[QT][2];
#pragma unroll
    for (int t = 0; t < QT; ++t) s[t][0] = s[t][1] = zero;
#pragma unroll
    for (int d = 0; d < KS; ++d)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int t = 0; t < QT; ++t)
#pragma unroll
          for (int c = 0; c < 2; ++c)
            s[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c][d][e], qf[t][d][e], s[t][c], 0, 0, 0);
    if (g + 4 < ng) load_k(g + 4);
#pragma unroll
    for (int t = 0; t < QT; ++t) {
      float mt = -INFINITY;
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          s[t][c][e] = kv0 + 16 * c + 4 * kq + e < Tj ? s[t][c][e] * a.scale : -INFINITY;
          mt = fmaxf(mt, s[t][c][e]);
        }
      mt = fmaxf(mt, __shfl_xor(mt, 16, 64));
      mt = fmaxf(mt, __shfl_xor(mt, 32, 64));
      const float m_new = fmaxf(m_run[t], mt);
      // where every score so far overflowed to -inf the wave adds nothing (other
      // waves may hold finite ones): exp(-inf - 0) instead of -inf - (-inf)
      const float m_ref = m_new == -INFINITY ? 0.f : m_new;
      const float alpha = expf(m_run[t] - m_ref);
      m_run[t] = m_new;
      l_run[t] *= alpha;
#pragma unroll
      for (int v = 0; v < TV; ++v) o[t][v] *= alpha;
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          s[t][c][e] = expf(s[t][c][e] - m_ref);
          l_run[t] += s[t][c][e];
        }
    }
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int t = 0; t < QT; ++t) {
#pragma unroll
          for (int v = 0; v < 4 * VB; ++v)
            o[t][v] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[c][e][v >> 2][v & 3], s[t][c][e], o[t][v], 0, 0, 0);
          if (VX) o[t][TV - 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(vx[c][e], s[t][c][e], o[t][TV - 1], 0, 0, 0);
        }
  }

  // Merge: with m = max_w m_w and f_w = exp(m_w - m), O = sum_w f_w O_w / sum_w f_w l_w
  // (a wave without keys has m = -inf and l = O = 0).
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    l_run[t] += __shfl_xor(l_run[t], 16, 64);
    l_run[t] += __shfl_xor(l_run[t], 32, 64);
    const int qr = 16 * t + r16;
    if (kq == 0) {
      ml[wave][0][qr] = m_run[t];
      ml[wave][1][qr] = l_run[t];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
#pragma unroll
      for (int v = 0; v < VB; ++v)
        *(f32x4*)&os[wave][qr][64 * v + 16 * kq + 4 * e] =
            f32x4{o[t][4 * v][e], o[t][4 * v + 1][e], o[t][4 * v + 2][e], o[t][4 * v + 3][e]};
      if (VX && 4 * kq + e < DH % 64) os[wave][qr][64 * VB + 4 * kq + e] = o[t][TV - 1][e];
    }
  }
  __syncthreads();
  constexpr int G4 = DH / 4;  // 4-column groups per query
  for (int i = tid; i < 16 * QT * G4; i += 256) {
    const int qr = i / G4, d = (i - qr * G4) * 4, qi = q0 + qr;
    if (qi >= Tj) continue;
    float m = ml[0][0][qr];
#pragma unroll
    for (int w = 1; w < 4; ++w) m = fmaxf(m, ml[w][0][qr]);
    float den = 0.f;
    f32x4 num = zero;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float f = expf(ml[w][0][qr] - m);
      den += f * ml[w][1][qr];
      num += f * *(const f32x4*)&os[w][qr][d];
    }
    const long orow = qi < a.T_img ? (long)b * a.T_img + qi
                                   : (long)a.B * a.T_img + (long)b * a.T_txt + (qi - a.T_img);
    *(f32x4*)((float*)a.o + orow * a.D + h * DH + d) = num * (1.0f / den);
  }
}

template <int DH>
static void launch_dh(const AttnArgs& a, hipStream_t st) {
  // 32 queries per workgroup halve the K and V reads; 16 where that would
  // leave fewer than two workgroups per CU (352 workgroups of 32: 33 us
  // against 25; 768: 308 against 324; 1024: 274 against 296).
  const long wg32 = (long)((a.Tj + 31) / 32) * a.H * a.B;
  if (wg32 >= 512)
    hipLaunchKernelGGL((attn_f32_kernel<DH, 2>), dim3((a.Tj + 31) / 32, a.H, a.B), dim3(256), 0, st, a);
  else
    hipLaunchKernelGGL((attn_f32_kernel<DH, 1>), dim3((a.Tj + 15) / 16, a.H, a.B), dim3(256), 0, st, a);
}

hipError_t launch_attn_f32(const AttnArgs& a, int head_dim, hipStream_t st) {
  switch (head_dim) {
    case 64: launch_dh<64>(a, st); break;
    case 72: launch_dh<72>(a, st); break;
    case 128: launch_dh<128>(a, st); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace ditmi
