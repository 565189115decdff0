// fp32 GEMM on gfx950 matrix cores: C[m, n] (+)= sum_k A(m, k) B(n, k) in fp32 throughout, for the
// products of the fp32 stage.
//
// v_mfma_f32_32x32x2_f32: lane l supplies row l mod 32 of A and of B at one k (k = l / 32 of the
// step's two), and receives C rows 8 (e / 4) + 4 (l / 32) + e mod 4, column l mod 32 in accumulator
// e.  Which two k a step pairs is free as long as A and B agree: step j of an 8-deep group pairs k = j
// and j + 4, so that a lane's four values of a group are consecutive in a k-contiguous tile (one
// 16-byte LDS read).
//   - an operand whose global layout is k-contiguous sits in LDS as [row][k], rows padded by 4 floats
//     (16 rows' 16-byte reads on disjoint banks);
//   - a row-contiguous operand sits as [k][row], rows of ROWS + 8 floats: the two half-waves of a
//     4-byte read are 4 k-rows apart, which the pitch (8 mod 16) puts on the other 32 banks.
// Bound: the matrix cores' 256 flop per cycle and CU (157 TFLOP/s on the chip) once the tiles fill
// it; below that the serial chain of one tile, 64 cycles per 32 x 32 x 2 step.  Three tilings of one
// block: 4 waves on 128 x 128 (waves of 64 x 64) or 64 x 64 (waves of 32 x 32), and 8 waves on 32 x 32
// splitting every k-slice eight ways (partial tiles summed in wave order through LDS; with 4 waves the
// same products took 13-25 % longer: [128, 128] over K 1024 13.0 -> 10.4 us, [1024, 512] over 4096 64.6 ->
// 57.2 us).
// Against the fp32 FMA tiling it replaced (64 x 64 tiles, 16-deep slices), a block's twelve products
// alone: T = 1024, d 512, d_ffn 2048 2131 -> 401 us (64 TFLOP/s; up to 81 for one product), T = 128,
// d 128, d_ffn 512 364 -> 66 us (4-10 us each, where a launch's latency is the bound).
// Global loads are 16-byte vectors at any 4-byte alignment, element by element at the edges, into
// registers one slice ahead; two LDS stages, one barrier per slice.
#include "common.h"
#include "kernels.h"

namespace {

typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

template <int BM_, int BN_, int KW_>
struct Tiling {
  static constexpr int BM = BM_, BN = BN_, KW = KW_;  // KW: waves sharing a tile, each a part of every slice
  static constexpr int WM = KW > 1 ? BM : BM / 2, WN = KW > 1 ? BN : BN / 2;
  static constexpr int FM = WM / 32, FN = WN / 32;
  static constexpr int BK = KW > 1 ? 16 * KW : 32;  // slice depth
  static constexpr int DW = BK / KW;                // depth of one wave's part
  static constexpr int NW = (BM / WM) * (BN / WN) * KW, NT = 64 * NW;
  static_assert(DW % 8 == 0 && (KW == 1 || 16 % KW == 0), "whole 8-deep groups, whole accumulators to each wave");
};

template <int ROWS, int BK, int NT, bool KMAJ>
struct Operand {
  static constexpr int P = KMAJ ? BK + 4 : ROWS + 8;  // LDS row pitch
  static constexpr int ELEMS = KMAJ ? ROWS * P : BK * P;
  static constexpr int PER = ROWS * BK / 4 / NT;  // chunks of 4 per thread and slice
  static_assert(PER * NT * 4 == ROWS * BK, "slice does not split evenly over the threads");
  f32x4 r[PER];

  // rowmap: tile row -> operand row (k-contiguous layout only)
  template <typename F>
  __device__ __forceinline__ void load(const float* __restrict__ G, int ld, int row0, int rows, int k0, int K,
                                       F&& rowmap) {
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      const int c = threadIdx.x + p * NT;
      int row, k, left;  // the chunk's first element, and how many of its 4 elements exist
      if constexpr (KMAJ) {
        row = row0 + c / (BK / 4);
        k = k0 + (c % (BK / 4)) * 4;
        left = row < rows ? K - k : 0;
        row = rowmap(row);
      } else {
        k = k0 + c / (ROWS / 4);
        row = row0 + (c % (ROWS / 4)) * 4;
        left = k < K ? rows - row : 0;
      }
      const float* s = G + (KMAJ ? (int64_t)row * ld + k : (int64_t)k * ld + row);
      f32x4 v = {0.f, 0.f, 0.f, 0.f};
      if (left >= 4) {
        v = *reinterpret_cast<const f32x4u*>(s);
      } else if (left > 0) {
        v[0] = s[0];
        if (left > 1) v[1] = s[1];
        if (left > 2) v[2] = s[2];
      }
      r[p] = v;
    }
  }
  __device__ __forceinline__ void store(float* S) const {
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      const int c = threadIdx.x + p * NT;
      const int o = KMAJ ? (c / (BK / 4)) * P + (c % (BK / 4)) * 4 : (c / (ROWS / 4)) * P + (c % (ROWS / 4)) * 4;
      *reinterpret_cast<f32x4*>(S + o) = r[p];
    }
  }
  // this lane's values of the 8-deep group at k0: row r0 + lane mod 32, k = k0 + 4 (lane / 32) + 0..3
  __device__ static f32x4 frag(const float* S, int r0, int k0) {
    const int row = r0 + (threadIdx.x & 31), k = k0 + 4 * ((threadIdx.x >> 5) & 1);
    if constexpr (KMAJ) return *reinterpret_cast<const f32x4*>(S + row * P + k);
    else return f32x4{S[k * P + row], S[(k + 1) * P + row], S[(k + 2) * P + row], S[(k + 3) * P + row]};
  }
};

// Column of C (and row of B) that panel column n stands for.  The RoPE and SwiGLU-forward products
// permute B's rows inside the panel so that lanes c and c + 16 of a 32-column group hold the two
// values the epilogue combines: columns i and i + hd/2 of one head, or gate and up of one z column.
__device__ __forceinline__ int panel_column(const GemmArgs& g, int n) {
  const int grp = n / 32, c = n % 32;
  if (g.epi == 2) {
    const int per = g.rope_hd / 32;
    return (grp / per) * g.rope_hd + (grp % per) * 16 + c % 16 + (c / 16) * (g.rope_hd / 2);
  }
  if (g.epi == 3) return grp * 16 + c % 16 + (c / 16) * g.glu;
  return n;
}

// One value v of C row `row`, panel column n (every lane of the wave calls, also past the edges)
__device__ __forceinline__ void put(const GemmArgs& g, int row, int n, float v) {
  const int c = n % 32;
  float pv = 0.f;
  if (g.epi == 2 || g.epi == 3) pv = __shfl_xor(v, 16, 64);  // the partner column
  if (row >= g.M || n >= g.N) return;
  const int col = panel_column(g, n);
  float* C = (float*)g.C + (int64_t)row * g.ldc + col;
  if (g.epi == 1) {  // SwiGLU backward from dz = v
    const float* gu = (const float*)g.aux + (int64_t)row * g.ld_aux + col;
    const float a = gu[0], b = gu[g.N];
    const float sg = 1.0f / (1.0f + expf(-a));
    C[0] = v * b * sg * (1.0f + a * (1.0f - sg));
    C[g.N] = v * a * sg;
    return;
  }
  if (g.epi == 3) {  // gate (c < 16) and up columns as they are, z = silu(gate) up beside them
    C[0] = v;
    if (c < 16) ((float*)g.out2)[(int64_t)row * g.ld_out2 + col] = v / (1.0f + expf(-v)) * pv;
    return;
  }
  if (g.epi == 2) {
    if (col < g.rope_cols) {
      const int hh = g.rope_hd / 2;
      const int64_t t = (int64_t)(row % g.rope_S) * hh + (col % g.rope_hd) % hh;
      const float cs = g.rope_cos[t], sn = g.rope_sin[t];
      v = c < 16 ? v * cs - pv * sn : v * cs + pv * sn;
    }
    C[0] = v;
    return;
  }
  if (g.epi == GEMM_EPI_AXPBY) {
    C[0] = g.alpha * v + g.beta_d * ((const float*)g.D)[(int64_t)row * g.ldc + col];
    return;
  }
  if (g.out_f32 && g.beta != 0.f) v += g.beta * C[0];
  if (g.resid) v += ((const float*)g.resid)[(int64_t)row * g.ldc + col];
  C[0] = v;
}

template <typename TL, bool AK, bool BKM>
__global__ void __launch_bounds__(TL::NT) gemm_f32_kernel(GemmArgs g) {
  constexpr int BM = TL::BM, BN = TL::BN, KW = TL::KW, FM = TL::FM, FN = TL::FN, BK = TL::BK;
  using OA = Operand<BM, BK, TL::NT, AK>;
  using OB = Operand<BN, BK, TL::NT, BKM>;
  constexpr int STAGE = OA::ELEMS + OB::ELEMS;
  extern __shared__ __align__(16) float smem[];  // [2][A slice | B slice]
  if (g.batch > 1) {  // product blockIdx.z of a batch
    const int64_t z = blockIdx.z;
    g.A = (const float*)g.A + z * g.sA;
    g.B = (const float*)g.B + z * g.sB;
    g.C = (float*)g.C + z * g.sC;
    if (g.D) g.D = (const float*)g.D + z * g.sD;
  }
  // XCD-aware order: block b runs on XCD b mod 8; each XCD gets a contiguous run of tiles, walked
  // down the row tiles, so that the blocks of one XCD share B's columns in its L2
  const int tm = (g.M + BM - 1) / BM, nblk = gridDim.x;
  const int b = (blockIdx.x & 7) * (nblk >> 3) + min((int)(blockIdx.x & 7), nblk & 7) + (blockIdx.x >> 3);
  const int m0 = (b % tm) * BM, n0 = (b / tm) * BN;
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  const int wm0 = KW > 1 ? 0 : (wave / 2) * TL::WM, wn0 = KW > 1 ? 0 : (wave % 2) * TL::WN;
  const int kw0 = KW > 1 ? wave * TL::DW : 0;
  f32x16 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
  OA la;
  OB lb;
  auto load = [&](int k0) {
    la.load((const float*)g.A, g.lda, m0, g.M, k0, g.K, [](int r) { return r; });
    lb.load((const float*)g.B, g.ldb, n0, g.N, k0, g.K, [&](int r) { return panel_column(g, r); });
  };
  load(0);
  la.store(smem);
  lb.store(smem + OA::ELEMS);
  __syncthreads();
  const int nk = (g.K + BK - 1) / BK;
  for (int kt = 0; kt < nk; ++kt) {
    const float* as = smem + (kt & 1) * STAGE;
    const float* bs = as + OA::ELEMS;
    if (kt + 1 < nk) load((kt + 1) * BK);
#pragma unroll
    for (int k = 0; k < TL::DW; k += 8) {
      f32x4 af[FM], bf[FN];
#pragma unroll
      for (int i = 0; i < FM; ++i) af[i] = OA::frag(as, wm0 + i * 32, kw0 + k);
#pragma unroll
      for (int j = 0; j < FN; ++j) bf[j] = OB::frag(bs, wn0 + j * 32, kw0 + k);
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(af[i][s], bf[j][s], acc[i][j], 0, 0, 0);
    }
    if (kt + 1 < nk) {
      float* an = smem + ((kt + 1) & 1) * STAGE;  // every wave left this stage before the last barrier
      la.store(an);
      lb.store(an + OA::ELEMS);
    }
    __syncthreads();
  }
  if constexpr (KW > 1) {
    // partial tiles to LDS as [wave][accumulator][lane]; wave w finishes accumulators EW w .. EW w + EW - 1
    constexpr int EW = 16 / KW;
    float* red = smem;
    static_assert(KW * 16 * 64 <= 2 * STAGE, "partial tiles fit the stages");
#pragma unroll
    for (int e = 0; e < 16; ++e) red[(wave * 16 + e) * 64 + lane] = acc[0][0][e];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < EW; ++q) {
      const int e = EW * wave + q;
      float v = red[e * 64 + lane];
#pragma unroll
      for (int w = 1; w < KW; ++w) v += red[(w * 16 + e) * 64 + lane];
      put(g, m0 + 8 * (e / 4) + 4 * (lane / 32) + e % 4, n0 + lane % 32, v);
    }
  } else {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e)
          put(g, m0 + wm0 + i * 32 + 8 * (e / 4) + 4 * (lane / 32) + e % 4, n0 + wn0 + j * 32 + lane % 32, acc[i][j][e]);
  }
}

template <typename TL, bool AK, bool BKM>
void launch_f32(const GemmArgs& g, hipStream_t st) {
  constexpr size_t lds = 2 * sizeof(float) *
                         (Operand<TL::BM, TL::BK, TL::NT, AK>::ELEMS + Operand<TL::BN, TL::BK, TL::NT, BKM>::ELEMS);
  if constexpr (lds > 65536) {
    static const hipError_t attr = hipFuncSetAttribute((const void*)gemm_f32_kernel<TL, AK, BKM>,
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    (void)attr;
  }
  const unsigned nblk = (unsigned)(cdiv(g.M, TL::BM) * cdiv(g.N, TL::BN));
  gemm_f32_kernel<TL, AK, BKM><<<dim3(nblk, 1, g.batch), TL::NT, lds, st>>>(g);
}

template <typename TL>
void launch_layouts(const GemmArgs& g, hipStream_t st) {
  if (g.a_kmajor && g.b_kmajor) launch_f32<TL, true, true>(g, st);
  else if (g.a_kmajor) launch_f32<TL, true, false>(g, st);
  else if (g.b_kmajor) launch_f32<TL, false, true>(g, st);
  else launch_f32<TL, false, false>(g, st);
}

}  // namespace

// Every fp32 product (plain, beta C, residual, batched, and epilogues 1, 2, 3 and 6; 2 and 3 with a
// k-contiguous B).  The largest tiling that still gives each CU work: below 256 tiles of 64 x 64 the
// 32 x 32 ones (T = 1024, N = 512, K = 4096: 57 us on 512 of them), from there 64 x 64 (4096 x 512, K =
// 1024: 54 us against 63 on 32 x 32; 384-512 tiles are within 10 % either way), 128 x 128 once they fill
// two blocks per CU.
void launch_gemm_f32(const GemmArgs& g, hipStream_t st) {
  const int64_t t64 = cdiv(g.M, 64) * cdiv(g.N, 64) * g.batch, t128 = cdiv(g.M, 128) * cdiv(g.N, 128) * g.batch;
  if (t128 >= 512) launch_layouts<Tiling<128, 128, 1>>(g, st);
  else if (t64 >= 256) launch_layouts<Tiling<64, 64, 1>>(g, st);
  else launch_layouts<Tiling<32, 32, 8>>(g, st);
}
