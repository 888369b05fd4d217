// bf16 GEMM for grids that cannot fill the GPU with the large tiles of
// gemm_bf16.hip: y[M, N] = A[M, K] * W[N, K]^T + bias with the same epilogues.
//
// A workgroup owns a BM x BN tile; its waves form KG k-groups of WGM x WGN
// waves, each wave holding TM x TN accumulators of 16 x 16
// (v_mfma_f32_16x16x32_bf16).  K is consumed in 64-wide slices (128 bytes per
// row, one cache line); k-group g takes slices g, g + KG, ... and keeps a ring
// of ST slice buffers of its own, filled by the global_load_lds_dwordx4 DMA
// path.  So a tile's serial chain is KG times shorter and KG ST slices are in
// flight per workgroup, which is what bounds these calls: a chain of dependent
// slice loads, not the matrix pipe.  Slice format and swizzle as in
// gemm_bf16.hip.  Measured per launch (weights from HBM), 64 x 128 tiles of
// gemm_bf16.hip -> here, 256 x 1152 x 1152: 9.9 -> 6.2 us (64 x 32; with three
// k-ranges and their reduction before 6.4 + 3.6), 256 x 3456 x 1152: 9.4 -> 7.5
// (64 x 64), 256 x 4608 x 1152: 9.6 -> 8.7 (64 x 96), 64 x 3456 x 1152: 12.2 ->
// 6.1 (64 x 32).  One wave per k-group, four k-groups of four waves and rings
// of four slices were no faster.
#include "common.h"
#include "kernels.h"

namespace ditmi {

template <int WGM, int WGN, int KG, int TM, int TN, int ST>
struct KgCfg {
  static constexpr int NW = WGM * WGN;          // waves per k-group
  static constexpr int BM = WGM * TM * 16, BN = WGN * TN * 16;
  static constexpr int ROWS = BM + BN;          // A rows then W rows in a slice buffer
  static constexpr int SLICE = ROWS * 128;
  static constexpr int IPW = ROWS / (8 * NW);   // DMA instructions per wave per slice
  static constexpr int CST = BN + 4;            // row stride of a k-group's partial tile in LDS
  static constexpr int LDS_MAIN = KG * ST * SLICE;
  static constexpr int LDS_RED = KG * BM * CST * 4;
  static constexpr int LDS = LDS_MAIN > LDS_RED ? LDS_MAIN : LDS_RED;
  static constexpr int THREADS = NW * KG * 64;
  static constexpr int GROUPS = BM * BN / 4;    // 4-column groups of the tile
  static constexpr int GPT = (GROUPS + THREADS - 1) / THREADS;
  static_assert(ROWS % (8 * NW) == 0 && BM % 8 == 0, "uniform DMA split");
  static_assert(ST >= 2 && (ST - 1) * IPW < 64, "vmcnt range");
  static_assert(LDS <= 160 * 1024, "LDS per CU");
};

template <int WGM, int WGN, int KG, int TM, int TN, int ST, int EPI>
__global__ __launch_bounds__(WGM * WGN * KG * 64) void gemm_bf16_kg_kernel(GemmArgs args) {
  using C = KgCfg<WGM, WGN, KG, TM, TN, ST>;
  constexpr bool RES = EPI == EPI_RESID || EPI == EPI_RESID2;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[C::LDS];

  const int tile = xcd_remap(blockIdx.x, args.total_tiles);
  // by value: indexing the by-value argument array with a runtime index would copy it to scratch memory
  const bool second = args.nprob > 1 && tile >= args.p[1].tile_begin;
  const GemmProb P = second ? args.p[1] : args.p[0];
  int local = tile - P.tile_begin;
  const int M = P.M, N = P.N, K = P.K;
  // slices kb .. kb + KT - 1; with split K unit u is range u / tiles of tile u % tiles
  int kb = 0, KT = K / 64;
  const bool raw = (RES || EPI == EPI_GELU) && P.ksplit > 1;
  float* part = P.part;
  if (raw) {
    const int per = P.tiles_m * P.tiles_n, s = local / per;
    local -= s * per;
    kb = KT * s / P.ksplit;
    KT = KT * (s + 1) / P.ksplit - kb;
    part += (long)s * M * N;
  }
  // groups of group_m M-tiles x all N-tiles, M fastest
  const int GM = max(P.group_m, 1);
  const int group = local / (GM * P.tiles_n);
  const int gm = min(P.tiles_m - group * GM, GM);
  const int in_group = local - group * GM * P.tiles_n;
  const int m0 = (group * GM + in_group % gm) * C::BM, n0 = (in_group / gm) * C::BN;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave_id = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave_id / C::NW, wave = wave_id - kg * C::NW;
  const int wm = wave / WGN, wn = wave - wm * WGN;
  const int r16 = lane & 15, kq = lane >> 4;
  const int nk = (KT - kg + KG - 1) / KG;      // slices of this k-group
  const unsigned ring = (unsigned)(kg * ST * C::SLICE);
  const unsigned lds0 = __builtin_amdgcn_readfirstlane(lds_address(smem)) + ring;

  // DMA instruction t of this wave fills slice rows 8q .. 8q+7, q = wave + NW t
  unsigned voff[C::IPW];
#pragma unroll
  for (int t = 0; t < C::IPW; ++t) {
    const int q = wave + C::NW * t, row = 8 * q + (lane >> 3);
    const int grow = q < C::BM / 8 ? min(m0 + row, M - 1) : min(n0 + row - C::BM, N - 1);  // clamped: ragged tiles
    voff[t] = (unsigned)grow * (unsigned)K * 2u + (unsigned)(((lane & 7) ^ (lane >> 3) ^ (q & 1)) * 16);
  }
  auto issue = [&](int i, int t) __attribute__((always_inline)) {  // instruction t of slice i of this k-group
    const long k0 = (long)(kb + kg + i * KG) * 64;
    const int q = wave + C::NW * t;
    dma_16s((q < C::BM / 8 ? (const bf16_t*)P.A : (const bf16_t*)P.W) + k0, voff[t],
            lds0 + (unsigned)((i % ST) * C::SLICE + q * 1024));
  };

  // LDS offsets of this lane's fragments: rows are r16 plus multiples of 16
  const int a_row = (wm * TM * 16 + r16) * 128, b_row = (C::BM + wn * TN * 16 + r16) * 128;
  const int swz = (r16 & 7) ^ (r16 >> 3);
  const int pos[2] = {(kq ^ swz) << 4, ((4 + kq) ^ swz) << 4};  // of the slice's two 32-wide halves

  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Software pipeline over half slices, as in the fp32 GEMM: Y (second half)
  // is read while X (first half) is multiplied; after the barrier the next
  // slice's X is read and this slice's buffer refilled while Y is multiplied.
  // A k-group of one wave has its buffers to itself and needs no barrier.
  bf16x8 xa[TM], xb[TN], ya[TM], yb[TN];
  auto read = [&](bf16x8 (&fa)[TM], bf16x8 (&fb)[TN], int it, int s) __attribute__((always_inline)) {
    const unsigned char* sl = smem + ring + (it % ST) * C::SLICE;
#pragma unroll
    for (int i = 0; i < TM; ++i) fa[i] = *(const bf16x8*)(sl + a_row + i * 2048 + pos[s]);
#pragma unroll
    for (int j = 0; j < TN; ++j) fb[j] = *(const bf16x8*)(sl + b_row + j * 2048 + pos[s]);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto multiply = [&](const bf16x8 (&fa)[TM], const bf16x8 (&fb)[TN], bool dma, int it) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int j = 0; j < TN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if (dma)
#pragma unroll
        for (int t = i * C::IPW / TM; t < (i + 1) * C::IPW / TM; ++t) issue(it, t);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
#pragma unroll
  for (int i = 0; i < ST; ++i)
    if (i < nk)
#pragma unroll
      for (int t = 0; t < C::IPW; ++t) issue(i, t);
  if (nk >= ST) wait_vmcnt<(ST - 1) * C::IPW>();
  else wait_vmcnt<0>();
  if (C::NW > 1) __syncthreads();
  read(xa, xb, 0, 0);
  auto slice = [&](int it, bool refill, bool ahead) __attribute__((always_inline)) {
    read(ya, yb, it, 1);
    multiply(xa, xb, false, 0);
    if (ahead) wait_vmcnt<(ST - 2) * C::IPW>();  // this wave's DMA of slice it + 1
    else wait_vmcnt<0>();
    if (C::NW > 1) __syncthreads();
    read(xa, xb, it + 1, 0);  // past the last slice: stale, unused
    multiply(ya, yb, refill, it + ST);
  };
  // The slices every k-group has, without a branch around the MFMAs (which
  // would move the accumulators every slice); then the one some have.
  const int full = KT / KG;
  int it = 0;
  for (; it + ST < full; ++it) slice(it, true, true);
  for (; it < full; ++it) slice(it, it + ST < nk, it + ST - 1 < nk);
  if (KG > 1 && full < nk) {
    read(ya, yb, full, 1);
    multiply(xa, xb, false, 0);
    multiply(ya, yb, false, 0);
  }

  // Epilogue: the k-groups' partial tiles go through LDS; a thread then adds
  // them in group order, four consecutive columns at a time (v columns of the
  // QKV projection: four consecutive rows of one column).  Residual rows and
  // bias are requested before.
  const bool vcols = EPI == EPI_QKV && n0 >= 2 * P.hidden;  // tiles never straddle k|v (2D % BN == 0)
  constexpr int CPR = C::BN / 4, RPC = C::BM / 4;
  f32x4 x[RES ? C::GPT : 1], bias[C::GPT];
  const bf16_t* const bp = (const bf16_t*)P.bias;
  if (!raw) {
#pragma unroll
    for (int t = 0; t < C::GPT; ++t) {
      const int c = tid + t * C::THREADS, m = m0 + c / CPR, n = n0 + c % CPR * 4;
      if (c >= C::GROUPS) continue;
      if (vcols) {
        const float b = bf2f(bp[min(n0 + c / RPC, N - 1)]);
        bias[t] = f32x4{b, b, b, b};
      } else {
        const u32x2 w = *(const u32x2*)(bp + min(n, N - 4));
        bias[t] = f32x4{__uint_as_float(w[0] << 16), __uint_as_float(w[0] & 0xFFFF0000u),
                        __uint_as_float(w[1] << 16), __uint_as_float(w[1] & 0xFFFF0000u)};
      }
      if (RES && m < M && n < N) x[t] = *(const f32x4*)(P.resid + (long)m * N + n);
    }
  }
  float* const red = (float*)smem;
  __syncthreads();  // every wave is done with the slices
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        red[(kg * C::BM + (wm * TM + i) * 16 + 4 * kq + e) * C::CST + (wn * TN + j) * 16 + r16] = acc[i][j][e];
  __syncthreads();
  const int rpb = P.rows_per_batch;
  const float inv_rpb = 1.0f / (float)rpb, inv_dh = EPI == EPI_QKV ? 1.0f / (float)P.head_dim : 0.f;
#pragma unroll
  for (int t = 0; t < C::GPT; ++t) {
    const int c = tid + t * C::THREADS;
    if (c >= C::GROUPS) continue;
    if (vcols) {
      // v^T[b][h][d][j]: element (b D + n - 2D) Tj_pad + v_key_pos(j)
      const int nr = c / RPC, mr = c % RPC * 4, m = m0 + mr, n = n0 + nr;
      if (m >= M || n >= N) continue;
      f32x4 y;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        y[e] = red[(mr + e) * C::CST + nr];
#pragma unroll
        for (int q = 1; q < KG; ++q) y[e] += red[(q * C::BM + mr + e) * C::CST + nr];
      }
      y += bias[t];
      const int b = div_exact(m, rpb, inv_rpb), j = m - b * rpb, jp = j + P.seq_off;
      bf16_t* const vt = (bf16_t*)P.v;
      const long vrow = (long)n - 2 * P.hidden;
      if (m + 3 < M && j + 3 < rpb && (jp & 3) == 0) {  // 4 keys stay contiguous under v_key_pos
        *(u32x2*)(vt + ((long)b * P.hidden + vrow) * P.Tj_pad + v_key_pos(jp)) =
            u32x2{pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3])};
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (m + e < M) {
            const int be = div_exact(m + e, rpb, inv_rpb), je = m + e - be * rpb + P.seq_off;
            vt[((long)be * P.hidden + vrow) * P.Tj_pad + v_key_pos(je)] = f2bf(y[e]);
          }
      }
      continue;
    }
    const int mr = c / CPR, nr = c % CPR * 4, m = m0 + mr, n = n0 + nr;
    if (m >= M || n >= N) continue;  // N is a multiple of 4
    f32x4 y = *(const f32x4*)&red[mr * C::CST + nr];
#pragma unroll
    for (int q = 1; q < KG; ++q) y += *(const f32x4*)&red[(q * C::BM + mr) * C::CST + nr];
    const long off = (long)m * N + n;
    if (raw) {
      *(f32x4*)(part + off) = y;
      continue;
    }
    y += bias[t];
    if (RES) {
      const int b = div_exact(m, rpb, inv_rpb);
      *(f32x4*)(P.resid + off) = x[t] + *(const f32x4*)(P.gate + (long)b * P.gate_stride + n) * y;
    } else if (EPI == EPI_GELU) {
      *(u32x2*)((bf16_t*)P.out + off) =
          u32x2{pack_bf16x2(gelu_tanh(y[0]), gelu_tanh(y[1])), pack_bf16x2(gelu_tanh(y[2]), gelu_tanh(y[3]))};
    } else if (EPI == EPI_STORE) {
      *(f32x4*)((float*)P.out + off) = y;
    } else {  // q and k columns: four consecutive d of one head; k in the softmax's exp2 domain
      const int sel = n >= P.hidden ? 1 : 0, rem = n - sel * P.hidden;
      const int h = div_exact(rem, P.head_dim, inv_dh), d = rem - h * P.head_dim;
      const int b = div_exact(m, rpb, inv_rpb), jp = m - b * rpb + P.seq_off;
      bf16_t* dst = (bf16_t*)(sel ? P.k : P.q) + (((long)b * P.heads + h) * P.Tj + jp) * P.qk_stride + d;
      if (sel) y *= P.k_scale;
      *(u32x2*)dst = u32x2{pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3])};
      // padding columns after the head's last group: zero, but 1 in k's column head_dim
      if (d + 4 == P.head_dim)
        for (int z = 4; z < P.qk_stride - P.head_dim + 4; z += 4)
          *(u32x2*)(dst + z) = u32x2{sel && z == 4 ? 0x3F80u : 0u, 0u};
    }
  }
}

template <int WGM, int WGN, int KG, int TM, int TN, int ST>
static hipError_t launch_cfg(const GemmArgs& a, int epi, hipStream_t st) {
  dim3 grid(a.total_tiles), block(WGM * WGN * KG * 64);
#define KG_EPI_CASE(E) hipLaunchKernelGGL((gemm_bf16_kg_kernel<WGM, WGN, KG, TM, TN, ST, E>), grid, block, 0, st, a)
  switch (epi) {
    case EPI_QKV: KG_EPI_CASE(EPI_QKV); break;
    case EPI_GELU: KG_EPI_CASE(EPI_GELU); break;
    case EPI_RESID: KG_EPI_CASE(EPI_RESID); break;
    case EPI_RESID2: KG_EPI_CASE(EPI_RESID2); break;
    default: KG_EPI_CASE(EPI_STORE); break;
  }
#undef KG_EPI_CASE
  return hipGetLastError();
}

hipError_t launch_gemm_bf16_kg(const GemmArgs& a, int epi, int tile_cfg, hipStream_t st) {
  switch (tile_cfg) {
    case TILE_64x32: return launch_cfg<2, 1, 4, 2, 2, 3>(a, epi, st);
    case TILE_64x64: return launch_cfg<2, 2, 2, 2, 2, 3>(a, epi, st);
    case TILE_64x96: return launch_cfg<2, 2, 2, 2, 3, 3>(a, epi, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace ditmi
