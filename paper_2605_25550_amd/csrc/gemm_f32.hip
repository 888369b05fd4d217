// fp32 GEMM for the fp32 DiT path: y[M, N] = A[M, K] * W[N, K]^T + bias with
// true fp32 products and fp32 accumulation on the matrix cores
// (v_mfma_f32_16x16x4_f32), followed by the same fused epilogues as the bf16
// GEMM.
//
// A workgroup owns a BM x BN tile; its waves form KG k-groups of WGM x WGN
// waves, each wave holding TM x TN accumulators of 16 x 16.  K is consumed in
// 32-wide slices (128 bytes per row, one cache line); k-group g takes slices
// g, g + KG, ... and keeps a ring of ST slice buffers of its own, filled
// by the global_load_lds_dwordx4 DMA path.  A DMA
// instruction moves 8 rows x 128 bytes; the 16-byte chunk c of row r is stored
// at position c ^ f(r), f(r) = (r & 7) ^ ((r >> 3) & 1), which keeps the
// fragment reads off each other's banks.  A fragment is one 16-byte read per
// lane (row lane % 16, four consecutive k at 4 (lane / 16)) and feeds four
// MFMAs: MFMA e takes element e of both operands.
//
// What bounds it: the matrix pipe (155 TFLOP/s) and, for the small tiles, the
// L2 traffic of (BM + BN) rows of K per tile.  Deeper rings and more k-groups
// were no faster; the fragment reads of all waves at once after a barrier cost
// 5-20% until they were taken half a slice ahead.  Measured per launch, VALU
// kernel of 64 x 64 tiles before -> now, DiT-XL/2 widths at 666 rows: QKV
// 120 -> 53 us, output projection 74 -> 22, fc1 136 -> 63, fc2 274 -> 68 (with
// its reduction; 104 TFLOP/s); 256 rows at hidden 384: 31, 29, 27, 94 -> 7.4,
// 5.6, 7.4, 10.9 us; 2048 rows at hidden 1152: fc1 177 us (123 TFLOP/s).
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace ditmi {

template <int WGM, int WGN, int KG, int TM, int TN, int ST>
struct F32Cfg {
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
  static_assert(LDS <= 160 * 1024, "LDS per CU");
};

template <int WGM, int WGN, int KG, int TM, int TN, int ST, int EPI>
__global__ __launch_bounds__(WGM * WGN * KG * 64) void gemm_f32_kernel(GemmArgs args) {
  using C = F32Cfg<WGM, WGN, KG, TM, TN, ST>;
  constexpr bool RES = EPI == EPI_RESID || EPI == EPI_RESID2;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[C::LDS];

  const int tile = xcd_remap(blockIdx.x, args.total_tiles);
  // by value: indexing the by-value argument array with a runtime index would copy it to scratch memory
  const bool second = args.nprob > 1 && tile >= args.p[1].tile_begin;
  const GemmProb P = second ? args.p[1] : args.p[0];
  int local = tile - P.tile_begin;
  const int M = P.M, N = P.N, K = P.K;
  // slices kb .. kb + KT - 1 (K is a multiple of 64); with split K unit u is
  // range u / tiles of tile u % tiles
  int kb = 0, KT = K / 32;
  float* part = P.part;
  if (RES && P.ksplit > 1) {
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

  // DMA instruction t of this wave fills slice rows 8q .. 8q+7, q = wave + NW t.
  // Lane offsets are 32 bits and an fp32 operand may hold up to 8 GiB (2^31
  // elements), so they count from the tile's first row, which is part of the
  // 64-bit base (gemm_f32_tile_fits: such offsets fit).
  const long a_tile = (unsigned)m0 * (unsigned)K, w_tile = (unsigned)n0 * (unsigned)K;
  unsigned voff[C::IPW];
#pragma unroll
  for (int t = 0; t < C::IPW; ++t) {
    const int q = wave + C::NW * t, row = 8 * q + (lane >> 3);
    const int trow = q < C::BM / 8 ? min(row, M - 1 - m0) : min(row - C::BM, N - 1 - n0);  // clamped: ragged tiles
    voff[t] = (unsigned)trow * (unsigned)K * 4u + (unsigned)(((lane & 7) ^ (lane >> 3) ^ (q & 1)) * 16);
  }
  auto issue = [&](int i, int t) __attribute__((always_inline)) {  // instruction t of slice i of this k-group
    const long k0 = (long)(kb + kg + i * KG) * 32;
    const int q = wave + C::NW * t;
    dma_16s(q < C::BM / 8 ? (const float*)P.A + (a_tile + k0) : (const float*)P.W + (w_tile + k0), voff[t],
            lds0 + (unsigned)((i % ST) * C::SLICE + q * 1024));
  };

  // LDS offsets of this lane's fragments: rows are r16 plus multiples of 16
  const int a_row = (wm * TM * 16 + r16) * 128, b_row = (C::BM + wn * TN * 16 + r16) * 128;
  const int swz = (r16 & 7) ^ (r16 >> 3);
  const int pos[2] = {(kq ^ swz) << 4, ((4 + kq) ^ swz) << 4};  // of the slice's two 16-wide halves

  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Software pipeline over half slices: fragments X of a slice's first half,
  // Y of its second.  Y is read while X is multiplied; then the wave waits for
  // its DMA of the next slice, and after the barrier every wave's has landed
  // and every read of this slice is done: the next slice's X is read and this
  // slice's buffer refilled while Y is multiplied.  So a matrix instruction
  // is ready on both sides of the barrier and the fragment reads of all waves
  // (80 KB per slice pair at 96 x 64) do not hold it up.  A k-group of one
  // wave has its buffers to itself and needs no barrier (Y's reads are waited
  // for by its first MFMA, before the refill).
  f32x4 xa[TM], xb[TN], ya[TM], yb[TN];
  auto read = [&](f32x4 (&fa)[TM], f32x4 (&fb)[TN], int it, int s) __attribute__((always_inline)) {
    const unsigned char* sl = smem + ring + (it % ST) * C::SLICE;
#pragma unroll
    for (int i = 0; i < TM; ++i) fa[i] = *(const f32x4*)(sl + a_row + i * 2048 + pos[s]);
#pragma unroll
    for (int j = 0; j < TN; ++j) fb[j] = *(const f32x4*)(sl + b_row + j * 2048 + pos[s]);
    __builtin_amdgcn_sched_barrier(0);
  };
  // DMA: the instructions of slice `it` go between the MFMAs
  auto multiply = [&](const f32x4 (&fa)[TM], const f32x4 (&fb)[TN], bool dma, int it) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[i][e], fb[j][e], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if (dma)
#pragma unroll
        for (int t = e * C::IPW / 4; t < (e + 1) * C::IPW / 4; ++t) issue(it, t);
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
  // them in group order for four consecutive columns at a time (residual rows
  // requested before).  D lanes hold column r16, rows 4 kq + e.
  f32x4 x[RES ? C::GPT : 1];
  const bool raw = RES && P.ksplit > 1;
  if (RES && !raw) {
#pragma unroll
    for (int t = 0; t < C::GPT; ++t) {
      const int c = tid + t * C::THREADS, m = m0 + c / (C::BN / 4), n = n0 + c % (C::BN / 4) * 4;
      if (c < C::GROUPS && m < M && n < N) x[t] = *(const f32x4*)(P.resid + (long)m * N + n);
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
  const float inv_rpb = 1.0f / (float)rpb;
#pragma unroll
  for (int t = 0; t < C::GPT; ++t) {
    const int c = tid + t * C::THREADS, mr = c / (C::BN / 4), nr = c % (C::BN / 4) * 4;
    const int m = m0 + mr, n = n0 + nr;
    if (c >= C::GROUPS || m >= M || n >= N) continue;  // N is a multiple of 4
    f32x4 y = *(const f32x4*)&red[mr * C::CST + nr];
#pragma unroll
    for (int q = 1; q < KG; ++q) y += *(const f32x4*)&red[(q * C::BM + mr) * C::CST + nr];
    const long off = (long)m * N + n;
    if (raw) {
      *(f32x4*)(part + off) = y;
      continue;
    }
    y += *(const f32x4*)((const float*)P.bias + n);
    if (RES) {
      const int b = div_exact(m, rpb, inv_rpb);
      *(f32x4*)(P.resid + off) = x[t] + *(const f32x4*)(P.gate + (long)b * P.gate_stride + n) * y;
    } else if (EPI == EPI_GELU) {
      *(f32x4*)((float*)P.out + off) = f32x4{gelu_tanh(y[0]), gelu_tanh(y[1]), gelu_tanh(y[2]), gelu_tanh(y[3])};
    } else if (EPI == EPI_STORE) {
      *(f32x4*)((float*)P.out + off) = y;
    } else {  // four consecutive d of one head of q, k or v
      const int s = n / P.hidden, rem = n - s * P.hidden, h = rem / P.head_dim, d = rem - h * P.head_dim;
      const int b = div_exact(m, rpb, inv_rpb), jpos = m - b * rpb + P.seq_off;
      float* dst = (float*)(s == 0 ? P.q : (s == 1 ? P.k : P.v));
      *(f32x4*)(dst + (((long)b * P.heads + h) * P.Tj + jpos) * P.head_dim + d) = y;
    }
  }
}

void gemm_f32_tile_dims(int tile_cfg, int* bm, int* bn) {
  const int dims[F32_COUNT][2] = {{32, 32}, {64, 64}, {96, 64}, {96, 48}};
  *bm = dims[tile_cfg][0];
  *bn = dims[tile_cfg][1];
}

bool gemm_f32_tile_fits(int tile_cfg, int K) {
  int bm = 0, bn = 0;
  gemm_f32_tile_dims(tile_cfg, &bm, &bn);
  return (uint64_t)(std::max(bm, bn) - 1) * K * 4 + 128 <= UINT32_MAX;
}

template <int WGM, int WGN, int KG, int TM, int TN, int ST>
static hipError_t launch_cfg(const GemmArgs& a, int epi, hipStream_t st) {
  dim3 grid(a.total_tiles), block(WGM * WGN * KG * 64);
#define F32_EPI_CASE(E) hipLaunchKernelGGL((gemm_f32_kernel<WGM, WGN, KG, TM, TN, ST, E>), grid, block, 0, st, a)
  switch (epi) {
    case EPI_QKV: F32_EPI_CASE(EPI_QKV); break;
    case EPI_GELU: F32_EPI_CASE(EPI_GELU); break;
    case EPI_RESID: F32_EPI_CASE(EPI_RESID); break;
    case EPI_RESID2: F32_EPI_CASE(EPI_RESID2); break;
    default: F32_EPI_CASE(EPI_STORE); break;
  }
#undef F32_EPI_CASE
  return hipGetLastError();
}

hipError_t launch_gemm_f32(const GemmArgs& a, int epi, int tile_cfg, hipStream_t st) {
  switch (tile_cfg) {
    case F32_32x32: return launch_cfg<1, 1, 4, 2, 2, 2>(a, epi, st);
    case F32_64x64: return launch_cfg<2, 2, 2, 2, 2, 2>(a, epi, st);
    case F32_96x64: return launch_cfg<2, 2, 2, 3, 2, 2>(a, epi, st);
    default: return launch_cfg<2, 1, 2, 3, 3, 2>(a, epi, st);
  }
}

}  // namespace ditmi
