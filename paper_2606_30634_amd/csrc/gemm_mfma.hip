// bf16 GEMM on gfx950 matrix cores: C[m, n] (+)= sum_k A(m, k) B(n, k), fp32 accumulation.
//
// v_mfma_f32_32x32x16_bf16: lane l supplies row (l mod 32) of A and of B with the 8 consecutive k
// values 8*(l/32)..+7, and receives C rows 8*(i/4) + 4*(l/32) + (i mod 4), column l mod 32 in
// accumulator i.  Both operands therefore sit in LDS as [row][k], k contiguous.
//   - an operand whose global layout is k-contiguous (x W^T's x and W, dy W's dy) is copied in
//     16-byte chunks;
//   - an operand whose global layout is row-contiguous (W in dy W, both operands of dy^T x) is
//     staged as it sits in memory ([k][row], 16-byte chunks) and its fragments are read with
//     gfx950's transposing LDS read ds_read_b64_tr_b16.
// Block tiles are 128 x 128 (4 waves of 64 x 64), 256 x 256 (8 waves of 64 x 128) or, for weight
// gradients, 128 x 192 (4 waves of 64 x 96), with 64-deep k-slices that go straight from global memory
// to LDS.  Inside a k-slice the fragments of the next
// 16-deep step are read from LDS while the MFMAs of the current one run.  The epilogue stages each
// wave's tile through LDS and writes 16-byte rows.  Block order is remapped so that consecutive
// tiles of one output row band land on one XCD (one L2).  Deterministic split-K for underfilled
// fp32-output products.
#include "common.h"
#include "kernels.h"
#include <algorithm>

namespace {

constexpr int BKT = 64;  // depth of a k-slice

// XCD-aware tile order: hardware places block b on XCD b mod 8; give each XCD a contiguous run
// of tiles, walked in groups of GM row tiles (down a group's rows, then to its next column), so
// the blocks resident on one XCD at a time cover a compact patch of C and share their A and B
// slices in that XCD's L2.
template <int BM, int BN>
__device__ __forceinline__ void tile_origin(const GemmArgs& g, int b, int& m0, int& n0) {
  constexpr int GM = 8;
  const int tiles_n = (g.N + BN - 1) / BN;
  const int tiles_m = (g.M + BM - 1) / BM;
  const int nblk = tiles_m * tiles_n;
  b = (b & 7) * (nblk >> 3) + min(b & 7, nblk & 7) + (b >> 3);
  const int first_m = (b / (GM * tiles_n)) * GM;
  const int gsz = min(tiles_m - first_m, GM);
  m0 = (first_m + (b % (GM * tiles_n)) % gsz) * BM;
  n0 = ((b % (GM * tiles_n)) / gsz) * BN;
}

// Tile b of a symmetric product (M == N, square tiles): the b-th tile (i, j) with i <= j, counted
// row by row (T (T + 1) / 2 tiles for T tile rows).
template <int BM, int BN>
__device__ __forceinline__ void tri_origin(const GemmArgs& g, int b, int& m0, int& n0) {
  static_assert(BM == BN, "square tiles");
  const int T = g.M / BM;
  int i = 0, first = 0;
  while (i + 1 < T && b >= first + (T - i)) {
    first += T - i;
    ++i;
  }
  m0 = i * BM;
  n0 = (i + b - first) * BN;
}

// Epilogue kinds of the direct-to-LDS kernels (compile-time; the numbers of the first five are
// GemmArgs::epi): bf16 output as is, SwiGLU backward, RoPE, SwiGLU forward, attention delta, plus
// a residual row added, alpha (A B) + beta D.
enum { EPI_PLAIN = 0, EPI_SWIGLU_BWD = 1, EPI_ROPE = 2, EPI_SWIGLU_FWD = 3, EPI_DELTA = 4, EPI_RESID = 5,
       EPI_AXPBY = GEMM_EPI_AXPBY, EPI_AXPBY_DUP = GEMM_EPI_AXPBY_DUP, EPI_NS_SPLIT = GEMM_EPI_NS_SPLIT };

// Output chunks leave with non-temporal stores and read-once epilogue operands arrive with
// non-temporal loads: a product streams 10-150 MB of them through the 4 MB L2 of each XCD, which
// would otherwise evict the operand panels that the tiles resident on the XCD share.
template <typename V>
__device__ __forceinline__ void st_nt(void* p, const V& v) {
  static_assert(sizeof(V) == 16, "16-byte chunk");
  u32x4 u;
  __builtin_memcpy(&u, &v, 16);
  __builtin_nontemporal_store(u, reinterpret_cast<u32x4*>(p));
}
template <typename V>
__device__ __forceinline__ V ld_nt(const void* p) {
  static_assert(sizeof(V) == 16, "16-byte chunk");
  const u32x4 u = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
  V v;
  __builtin_memcpy(&v, &u, 16);
  return v;
}

// Global operands of one 16-byte output chunk (8 bf16 columns) that an epilogue reads.
template <int EPI> struct EpiIn { static constexpr bool loads = false; };
template <> struct EpiIn<EPI_RESID> { static constexpr bool loads = true; bf16x8 r; };
template <> struct EpiIn<EPI_AXPBY> { static constexpr bool loads = true; bf16x8 r; };
template <> struct EpiIn<EPI_AXPBY_DUP> { static constexpr bool loads = true; bf16x8 r; };
template <> struct EpiIn<EPI_NS_SPLIT> { static constexpr bool loads = true; bf16x8 a, b; };
template <> struct EpiIn<EPI_SWIGLU_BWD> { static constexpr bool loads = true; bf16x8 a, b; };
template <> struct EpiIn<EPI_DELTA> { static constexpr bool loads = true; f32x4 o0, o1; };
template <> struct EpiIn<EPI_ROPE> { static constexpr bool loads = true; f32x4 c0, c1, s0, s1; };

template <int EPI>
__device__ __forceinline__ void epi_load(EpiIn<EPI>& in, const GemmArgs& g, int row, int col) {
  if constexpr (EPI == EPI_RESID) {
    in.r = ld_nt<bf16x8>((const bf16*)g.resid + (int64_t)row * g.ldc + col);
  } else if constexpr (EPI == EPI_AXPBY) {
    in.r = ld_nt<bf16x8>((const bf16*)g.D + (int64_t)row * g.ldc + col);
  } else if constexpr (EPI == EPI_AXPBY_DUP) {
    in.r = ld_nt<bf16x8>((const bf16*)g.D + (int64_t)row * g.ld_aux + col);
  } else if constexpr (EPI == EPI_NS_SPLIT) {  // hi and lo of the previous x
    const bf16* dp = (const bf16*)g.D + (int64_t)row * g.ldc + col;
    in.a = ld_nt<bf16x8>(dp);
    in.b = ld_nt<bf16x8>(dp + g.N);
  } else if constexpr (EPI == EPI_SWIGLU_BWD) {
    const bf16* gu = (const bf16*)g.aux + (int64_t)row * g.ld_aux + col;
    in.a = ld_nt<bf16x8>(gu);
    in.b = ld_nt<bf16x8>(gu + g.N);
  } else if constexpr (EPI == EPI_DELTA) {
    const float* op = (const float*)g.aux + (int64_t)row * g.ld_aux + col;
    in.o0 = ld_nt<f32x4>(op);
    in.o1 = ld_nt<f32x4>(op + 4);
  } else if constexpr (EPI == EPI_ROPE) {
    if (col < g.rope_cols) {
      const int hh = g.rope_hd / 2, i0 = (col % g.rope_hd) % hh;
      const int64_t tb = (int64_t)(row % g.rope_S) * hh + i0;
      in.c0 = *reinterpret_cast<const f32x4*>(g.rope_cos + tb);
      in.c1 = *reinterpret_cast<const f32x4*>(g.rope_cos + tb + 4);
      in.s0 = *reinterpret_cast<const f32x4*>(g.rope_sin + tb);
      in.s1 = *reinterpret_cast<const f32x4*>(g.rope_sin + tb + 4);
    }
  }
}

// RAG: the library's exponential and divide, which the fp32 tiling these products came from used: some
// calls had them, and the rest of their time is the latency of few tiles
template <bool RAG>
__device__ __forceinline__ float sigmoid(float a) {
  if constexpr (RAG) return 1.0f / (1.0f + expf(-a));
  else return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * a));
}

// Epilogue of the direct-to-LDS kernels (RAG: the tile may reach past C; only chunks inside it are
// read and written, and fp32 rows that do not start on 16 bytes leave element by element).  Per RP-row part of each 32-row fragment
// row of the wave tile: the accumulators go through the wave's own LDS staging area and leave as
// 16-byte rows.  The global operands the epilogue kind reads are all requested before the first
// part is written (or one part ahead, where the registers for all of them would not fit), so their
// latency is paid about once per tile instead of once per part.  A wave reads back only what it wrote and
// its LDS operations complete in issue order: no barrier between parts, and the stores are never
// waited for here.  The staging area (waves x RP x (WN + 4) floats) must be free.
template <int BM, int BN, int WM, int WN, typename OutT, int EPI, int RP, bool RAG>
__device__ __forceinline__ void dma_epilogue(const GemmArgs& g, f32x16 (&acc)[WM / 32][WN / 32],
                                             float* stage, int m0, int n0, int wm0, int wn0, int tail) {
  static_assert(RP == 16 || RP == 8, "staging part of 8 or 16 rows");
  static_assert(sizeof(OutT) == 2 || EPI == EPI_PLAIN, "fp32 output has no fused epilogue");
  constexpr int FM = WM / 32, FN = WN / 32;
  constexpr int EP = WN + 4;  // staging pitch (fp32 elements)
  constexpr int NP = 32 / RP, EPP = 16 / NP;  // parts per fragment row, accumulators per part
  constexpr int VEC = sizeof(OutT) == 2 ? 8 : 4;  // elements per 16-byte chunk
  constexpr int CPR = WN / VEC;                   // chunks per staged row
  constexpr int CPL = RP * CPR / 64;              // chunks per lane and part
  constexpr int NPART = FM * NP;
  static_assert(CPL * 64 == RP * CPR, "every lane writes the same number of chunks per part");
  // Parts requested ahead of the one being written, within a per-lane register budget for the
  // requested operands (the wider wave tile holds more accumulators): all of them, one, or none.
  constexpr int PART_BYTES = EpiIn<EPI>::loads ? CPL * (int)sizeof(EpiIn<EPI>) : 0;
  constexpr int BUDGET = WN <= 64 ? 256 : 128;
  constexpr int PD = PART_BYTES == 0 ? 0
                     : PART_BYTES * NPART <= BUDGET ? NPART
                     : 2 * PART_BYTES <= BUDGET ? 1 : 0;
  constexpr int RS = PD >= NPART ? NPART : PD + 1;  // ring of requested parts
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  float* stg = stage + wave * RP * EP;
  const bool split = sizeof(OutT) == 4 && g.ksplit > 1;
  // partial sums: whole [M, N] arrays, or BM x BN tiles when only a range of tiles is split (W and ldw
  // such that C's row and column index both)
  const bool range = split && g.tile_n > 0;
  const int ldw = range ? BN : g.N;
  float* W = !split ? nullptr
             : range ? g.ws + ((int64_t)blockIdx.y * g.tile_n + tail) * BM * BN - ((int64_t)m0 * BN + n0)
                     : g.ws + (int64_t)blockIdx.y * g.M * g.N;
  // output chunk j of part p of this lane: staged row r, column cc; C row, column
  auto chunk = [&](int p, int j, int& r, int& cc, int& row, int& col) {
    const int c = lane + 64 * j;
    r = c / CPR;
    cc = (c % CPR) * VEC;
    row = m0 + wm0 + (p / NP) * 32 + RP * (p % NP) + r;
    col = n0 + wn0 + cc;
  };
  EpiIn<EPI> in[RS][CPL];
  auto request = [&](auto P) {
    constexpr int p = P;
#pragma unroll
    for (int j = 0; j < CPL; ++j) {
      int r, cc, row, col;
      chunk(p, j, r, cc, row, col);
      if (!RAG || (row < g.M && col < g.N)) epi_load<EPI>(in[p % RS][j], g, row, col);
      else in[p % RS][j] = EpiIn<EPI>{};
    }
  };
  if constexpr (PD > 0) static_for<(PD < NPART ? PD : NPART)>(request);
  static_for<NPART>([&](auto P) {
    constexpr int p = P, i = p / NP, h = p % NP;
    if constexpr (EpiIn<EPI>::loads && p + PD < NPART) request(std::integral_constant<int, p + PD>{});
    // accumulator e of lane l holds fragment row 8 (e / 4) + 4 (l / 32) + e mod 4: rows
    // RP h .. RP h + RP - 1 are e = EPP h .. EPP h + EPP - 1
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int e = EPP * h; e < EPP * h + EPP; ++e)
        stg[(8 * (e / 4) - RP * h + 4 * (lane / 32) + (e % 4)) * EP + j * 32 + lane % 32] = acc[i][j][e];
    asm volatile("" ::: "memory");
#pragma unroll
    for (int j = 0; j < CPL; ++j) {
      int r, cc, row, col;
      chunk(p, j, r, cc, row, col);
      const EpiIn<EPI>& x = in[p % RS][j];
      if (RAG && (row >= g.M || col >= g.N)) continue;  // bf16 output: N is a multiple of 8
      float v[VEC];
#pragma unroll
      for (int q = 0; q < VEC; ++q) v[q] = stg[r * EP + cc + q];
      if constexpr (sizeof(OutT) == 4) {
        if (RAG && (g.N | (split ? 0 : g.ldc)) % 4 != 0) {
          for (int q = 0; q < 4 && col + q < g.N; ++q) {
            if (split) {
              W[(int64_t)row * ldw + col + q] = v[q];
            } else {
              float* c = (float*)g.C + (int64_t)row * g.ldc + col + q;
              *c = g.beta != 0.f ? v[q] + g.beta * *c : v[q];
            }
          }
        } else if (split) {
          st_nt(W + (int64_t)row * ldw + col, make_float4(v[0], v[1], v[2], v[3]));
        } else {
          float* Cf = (float*)g.C + (int64_t)row * g.ldc + col;
          if (g.beta != 0.f) {
            const float4 old = *reinterpret_cast<const float4*>(Cf);
            v[0] += g.beta * old.x; v[1] += g.beta * old.y; v[2] += g.beta * old.z; v[3] += g.beta * old.w;
          }
          st_nt(Cf, make_float4(v[0], v[1], v[2], v[3]));
        }
      } else {
        bf16* Cb = (bf16*)g.C;
        const int64_t o = (int64_t)row * g.ldc + col;
        if constexpr (EPI == EPI_SWIGLU_BWD) {  // dz = v -> dgate | dup
          bf16x8 da, db;
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            const float a = (float)x.a[q], bb = (float)x.b[q];
            const float sg = sigmoid<RAG>(a);
            da[q] = (bf16)(v[q] * bb * sg * (1.0f + a * (1.0f - sg)));
            db[q] = (bf16)(v[q] * a * sg);
          }
          st_nt(Cb + o, da);
          st_nt(Cb + o + g.N, db);
        } else if constexpr (EPI == EPI_DELTA) {  // dO, plus delta = rowsum(dO O) per head
          bf16x8 ov;
#pragma unroll
          for (int q = 0; q < 8; ++q) ov[q] = (bf16)v[q];
          st_nt(Cb + o, ov);
          float dot = 0.f;
#pragma unroll
          for (int q = 0; q < 8; ++q) dot += (float)ov[q] * (q < 4 ? x.o0[q] : x.o1[q - 4]);
          // the head's delta_hd / 8 chunks sit in consecutive lanes (aligned groups)
          for (int m = 1; m < g.delta_hd / 8; m <<= 1) dot += __shfl_xor(dot, m, 64);
          if (col % g.delta_hd == 0) {
            const int bb = row / g.delta_S, ii = row % g.delta_S, hh = col / g.delta_hd;
            g.delta[((int64_t)bb * (g.N / g.delta_hd) + hh) * g.delta_S + ii] = dot;
          }
        } else if constexpr (EPI == EPI_SWIGLU_FWD) {  // panel column col: gate or up of z column zc
          const int grp = col / 32, zc = (grp / 2) * 32 + col % 32;
          bf16x8 ov;
#pragma unroll
          for (int q = 0; q < 8; ++q) ov[q] = (bf16)v[q];
          bf16* Crow = Cb + (int64_t)row * g.ldc;
          if ((grp & 1) == 0) {
            st_nt(Crow + zc, ov);
            const float* up = stg + r * EP + cc + 32;  // the up values of the same z columns
            bf16x8 zv;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
              // RAG: z of the stored gate and up, as the SwiGLU kernel makes it
              if constexpr (RAG) {
                const float gt = (float)ov[q];
                zv[q] = (bf16)(gt * (1.0f / (1.0f + expf(-gt))) * (float)(bf16)up[q]);
              } else {
                zv[q] = (bf16)(v[q] * sigmoid<RAG>(v[q]) * up[q]);
              }
            }
            st_nt((bf16*)g.out2 + (int64_t)row * g.ld_out2 + zc, zv);
          } else {
            st_nt(Crow + g.glu + zc, ov);
          }
        } else if constexpr (EPI == EPI_ROPE) {  // rotate pairs (i, i + hd/2) of each head
          bf16x8 ov;
          if (col < g.rope_cols) {
            const int hh = g.rope_hd / 2;
            const bool first = (col % g.rope_hd) < hh;
            const float* xp = stg + r * EP + (first ? cc + hh : cc - hh);  // partner columns
            const float cs[8] = {x.c0[0], x.c0[1], x.c0[2], x.c0[3], x.c1[0], x.c1[1], x.c1[2], x.c1[3]};
            const float sn[8] = {x.s0[0], x.s0[1], x.s0[2], x.s0[3], x.s1[0], x.s1[1], x.s1[2], x.s1[3]};
#pragma unroll
            for (int q = 0; q < 8; ++q)
              ov[q] = (bf16)(first ? v[q] * cs[q] - xp[q] * sn[q] : v[q] * cs[q] + xp[q] * sn[q]);
          } else {
#pragma unroll
            for (int q = 0; q < 8; ++q) ov[q] = (bf16)v[q];
          }
          st_nt(Cb + o, ov);
        } else if constexpr (EPI == EPI_AXPBY_DUP) {  // each value into two adjacent columns
          bf16x8 d0, d1;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const bf16 u0 = (bf16)(g.alpha * v[q] + g.beta_d * (float)x.r[q]);
            const bf16 u1 = (bf16)(g.alpha * v[q + 4] + g.beta_d * (float)x.r[q + 4]);
            d0[2 * q] = u0; d0[2 * q + 1] = u0;
            d1[2 * q] = u1; d1[2 * q + 1] = u1;
          }
          bf16* Cd = Cb + (int64_t)row * g.ldc + 2 * col;
          st_nt(Cd, d0);
          st_nt(Cd + 8, d1);
        } else if constexpr (EPI == EPI_NS_SPLIT) {  // x = v + beta_d (hi + lo), then its hi/lo form
          bf16x8 h8, l8;
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            const float xv = v[q] + g.beta_d * ((float)x.a[q] + (float)x.b[q]);
            const bf16 hq = (bf16)xv;
            h8[q] = hq;
            l8[q] = (bf16)(xv - (float)hq);
          }
          st_nt(Cb + o, h8);
          st_nt(Cb + o + g.N, l8);
        } else {
          if constexpr (EPI == EPI_RESID) {
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] += (float)x.r[q];
          } else if constexpr (EPI == EPI_AXPBY) {
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = g.alpha * v[q] + g.beta_d * (float)x.r[q];
          }
          bf16x8 ov;
#pragma unroll
          for (int q = 0; q < 8; ++q) ov[q] = (bf16)v[q];
          st_nt(Cb + o, ov);
        }
      }
    }
    if constexpr (EPI == EPI_PLAIN && sizeof(OutT) == 2) {
      if (!RAG && g.sym && m0 != n0) {
        // symmetric product, a tile above the diagonal: the part again at C[col, row], as 8-row
        // column segments of the staged rows
        constexpr int CT = WN * (RP / 8) / 64;  // segments per lane
        static_assert(CT * 64 == WN * (RP / 8), "every lane writes the same number of segments");
        bf16* Cb = (bf16*)g.C;
#pragma unroll
        for (int j = 0; j < CT; ++j) {
          const int c = lane + 64 * j, cc = c % WN, rg = c / WN;
          bf16x8 tv;
#pragma unroll
          for (int q = 0; q < 8; ++q) tv[q] = (bf16)stg[(rg * 8 + q) * EP + cc];
          const int row = m0 + wm0 + (p / NP) * 32 + RP * (p % NP) + rg * 8, col = n0 + wn0 + cc;
          st_nt(Cb + (int64_t)col * g.ldc + row, tv);
        }
      }
    }
    asm volatile("" ::: "memory");
  });
}

// ---------------------------------------------------------------------------------------------
// Kernel with direct-to-LDS operand loads (gfx950 global_load_lds_dwordx4): each lane's
// 16 bytes land at the wave's LDS base + 16 * lane, so a tile is written in lane order and the
// bank spreading is an XOR swizzle of 16-byte chunks instead of padding:
//   k-contiguous tile [ROWS][BKT]: chunk kc of row r sits at r * BKT/8 + (kc ^ ((r / (128/BKT)) mod
//     BKT/8)), so the 16 rows one 16-lane group reads for a fragment cover all 64 banks;
//   row-contiguous tile [BKT][ROWS]: chunk rc of k-row k sits at k * ROWS/8 + (rc ^ 4 (k mod 4)), so
//     the 4 k-rows x 32 rows of one half-wave transposing read fall in 4 different 64-byte bank
//     groups (ROWS 128 or 256: whole 256-byte bank periods per k-row; ROWS 192: 4 (k / 2 mod 2)).
// RAG: any M, N, K (the same pipeline; whole products keep the kernels without ranges and predicates,
// whose epilogue stores need not be waited for).  It replaced a register-staged kernel (M, N, K
// multiples of 8) and, for the rest, an fp32 FMA tiling: T = 2331 tokens, d 1024, d_ffn 2816, a
// block's twelve products 5.2 ms -> 0.39 ms (405 TFLOP/s; latency of 152-tile grids); T = 999,
// vocabulary 32001, the head's three 9.5 -> 0.54 ms.  The loads are buffer loads whose range ends with the operand, so rows past it
// land in LDS as zeros, and so do the k chunks of a k-contiguous operand past K (their lanes get an
// offset no range holds); columns past a row-contiguous operand's edge bring its next row, which
// only reaches outputs outside C.
// NS stages: the loads of slice kt + NS - 1 are issued while slice kt is consumed, so a load has
// NS - 1 slices of MFMAs to land; one barrier per slice, after each thread has seen its own loads
// of the slice complete (vmcnt), makes every thread's loads of it visible.
template <int ROWS, int BKT, bool KMAJ, int NT>
struct DmaTile {
  static constexpr int CHUNKS = ROWS * BKT / 8;
  static constexpr int PER = CHUNKS / NT;  // loads per thread and slice
  static constexpr int ELEMS = ROWS * BKT;
  static_assert(CHUNKS % NT == 0, "tile does not split evenly over the threads");
  static_assert(KMAJ || ROWS == 128 || ROWS == 192 || ROWS == 256, "row-contiguous swizzle");
  // row-contiguous tile: the XOR of k-row k's chunks (k-rows of an odd number of 128 bytes alternate
  // between the bank halves by themselves)
  __device__ static int swz(int k) { return ROWS % 128 == 0 ? 4 * (k & 3) : 4 * ((k >> 1) & 1); }
  // k-contiguous tile: the row and the 8-element k chunk whose data LDS chunk p holds
  __device__ static void row_chunk(int p, int& r, int& kc) {
    constexpr int CPR = BKT / 8, RPB = 128 / BKT;
    r = p / CPR;
    kc = (p % CPR) ^ ((r / RPB) % CPR);
  }
  // element offset, from the tile origin in global memory, of the data for LDS chunk p
  __device__ static int64_t src(int p, int ld) {
    if constexpr (KMAJ) {
      constexpr int CPR = BKT / 8, RPB = 128 / BKT;
      const int r = p / CPR, kc = (p % CPR) ^ ((r / RPB) % CPR);
      return (int64_t)r * ld + kc * 8;
    } else {
      constexpr int CPK = ROWS / 8;
      const int k = p / CPK, rc = (p % CPK) ^ swz(k);
      return (int64_t)k * ld + rc * 8;
    }
  }
  // MFMA fragment: row r0 + lane mod 32, k = k0 + 8 (lane / 32) .. +7
  __device__ static bf16x8 frag(const bf16* T, int r0, int k0) {
    const int l = threadIdx.x % 64;
    if constexpr (KMAJ) {
      constexpr int CPR = BKT / 8, RPB = 128 / BKT;
      const int r = r0 + l % 32, kc = k0 / 8 + l / 32;
      return *reinterpret_cast<const bf16x8*>(T + r * BKT + ((kc ^ ((r / RPB) % CPR)) << 3));
    } else {
      const int gq = l / 16, i = l % 16;
      const int r = r0 + 16 * (gq & 1) + 4 * (i & 3);
      const int k = k0 + 8 * (gq >> 1) + (i >> 2);  // k and k + 4 share k mod 4
      const int col = (((r >> 3) ^ swz(k)) << 3) + (r & 7);
      typedef __attribute__((address_space(3))) v4i16_t lds_v4i16;
      const v4i16_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16*)(T + k * ROWS + col));
      const v4i16_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16*)(T + (k + 4) * ROWS + col));
      bf16x8 f;
      __builtin_memcpy(&f, &lo, 8);
      __builtin_memcpy(reinterpret_cast<char*>(&f) + 8, &hi, 8);
      return f;
    }
  }
};

template <int BM, int BN, int WM, int WN, bool AK, bool BKM, int BKT, int NS>
struct DmaCfg {
  static constexpr int NW = (BM / WM) * (BN / WN);
  static constexpr int NT = NW * 64;
  using TA = DmaTile<BM, BKT, AK, NT>;
  using TB = DmaTile<BN, BKT, BKM, NT>;
  // one stage: the A tile, then the B tile (bf16 elements)
  static constexpr int STAGE = TA::ELEMS + TB::ELEMS;
  // epilogue staging rows per part: 16 when that fits in one stage, else 8
  static constexpr int RP = (size_t)NW * 16 * (WN + 4) * sizeof(float) <= (size_t)STAGE * sizeof(bf16) ? 16 : 8;
  static constexpr size_t epi_lds = (size_t)NW * RP * (WN + 4) * sizeof(float);
  // A block walks several tiles when the epilogue's staging fits in one stage: the stage of a
  // tile's last slice is then free for it while the next tile's first slices land in the others.
  static constexpr bool persist = epi_lds <= (size_t)STAGE * sizeof(bf16);
  static constexpr size_t main_lds = (size_t)NS * STAGE * sizeof(bf16);
  static constexpr size_t lds = main_lds > epi_lds ? main_lds : epi_lds;
};

// waves per SIMD: the block's waves over the 4 SIMDs times the blocks the LDS lets a CU hold
template <int BM, int BN, int WM, int WN, bool AK, bool BKM, int BKT, int NS>
constexpr int dma_waves_per_simd() {
  using C_ = DmaCfg<BM, BN, WM, WN, AK, BKM, BKT, NS>;
  const int blocks = (int)(163840 / C_::lds);
  const int w = (C_::NW / 4) * (blocks > 0 ? blocks : 1);
  return w > 8 ? 8 : (w < 1 ? 1 : w);
}

// Block b takes tiles b, b + gridDim.x, ... of the launch's range (tile0 a multiple of 8, gridDim.x a multiple of 8 when it is below the tile
// count, so that every tile of a block maps to the block's XCD).  The slices of all its tiles form
// one sequence: the loads of slice G + NS - 1 of that sequence (the next tile's first slices near
// the end of a tile) are issued while slice G is consumed, into stage (G + NS - 1) mod NS.
template <int BM, int BN, int WM, int WN, bool AK, bool BKM, typename OutT, int BKT, int NS, int EPI, bool RAG>
__global__ void __launch_bounds__((BM / WM) * (BN / WN) * 64)
__attribute__((amdgpu_waves_per_eu(dma_waves_per_simd<BM, BN, WM, WN, AK, BKM, BKT, NS>(),
                                   dma_waves_per_simd<BM, BN, WM, WN, AK, BKM, BKT, NS>())))
gemm_dma_kernel(GemmArgs g) {
  if (g.batch > 1) {  // product blockIdx.z of a batch
    const int64_t z = blockIdx.z;
    g.A = (const bf16*)g.A + z * g.sA;
    g.B = (const bf16*)g.B + z * g.sB;
    g.C = (char*)g.C + z * g.sC * (int64_t)sizeof(OutT);
    if (g.D) g.D = (const OutT*)g.D + z * g.sD;
  }
  using C_ = DmaCfg<BM, BN, WM, WN, AK, BKM, BKT, NS>;
  using TA = typename C_::TA;
  using TB = typename C_::TB;
  constexpr int WAVES_N = BN / WN, NW = C_::NW, STAGE = C_::STAGE;
  constexpr int FM = WM / 32, FN = WN / 32;
  constexpr int PA = TA::PER, PB = TB::PER;
  // vector-memory operations one thread's epilogue issues at least: one per 16-byte output chunk
  constexpr int RP = C_::RP, CPP = RP * WN / (sizeof(OutT) == 2 ? 8 : 4);  // 16-byte chunks per part
  static_assert(CPP % 64 == 0, "every lane stores the same number of chunks per part");
  // (RAG: a wave outside C issues none)
  constexpr int EPI_OPS = RAG ? 0 : FM * (32 / RP) * (CPP / 64);
  static_assert((NS - 2) * (PA + PB) + EPI_OPS < 64, "vmcnt range");
  extern __shared__ __align__(16) unsigned char smem[];
  bf16* S = reinterpret_cast<bf16*>(smem);  // [NS][A tile | B tile]

  const bool sym = !RAG && BM == BN && g.sym;
  const int tiles = sym ? (g.M / BM) * (g.M / BM + 1) / 2 : ((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN);
  auto origin = [&](int b, int& m0_, int& n0_) {
    if constexpr (BM == BN) {
      if (sym) return tri_origin<BM, BN>(g, b, m0_, n0_);
    }
    tile_origin<BM, BN>(g, b, m0_, n0_);
  };
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
  const int wm0 = (wave / WAVES_N) * WM, wn0 = (wave % WAVES_N) * WN;
  // split-K: this block covers slices [s0, s0 + nk) of every tile
  const int slices = (g.K + BKT - 1) / BKT, per = (slices + g.ksplit - 1) / g.ksplit, s0 = blockIdx.y * per;
  const int nk = min(per, slices - s0);  // at least 1: the launcher leaves no split empty
  const bool glu = BKM && EPI == EPI_SWIGLU_FWD;
  // this thread's byte offsets from a tile's slice origin
  uint32_t oa[PA], ob[PB];
#pragma unroll
  for (int q = 0; q < PA; ++q) oa[q] = 2u * (uint32_t)TA::src((q * NW + wave) * 64 + lane, g.lda);
#pragma unroll
  for (int q = 0; q < PB; ++q) {
    const int p = (q * NW + wave) * 64 + lane;
    if (glu) {
      // epilogue 3: panel row n0 + r is gate row (or, in odd 32-row groups, up row) n0/2 + ...
      int r, kc;
      TB::row_chunk(p, r, kc);
      ob[q] = 2u * (uint32_t)((((r / 32) & 1) * g.glu + (r / 64) * 32 + r % 32) * g.ldb + kc * 8);
    } else {
      ob[q] = 2u * (uint32_t)TB::src(p, g.ldb);
    }
  }
  // slice 0 (of this split) of the tiles at row m0 / column n0
  auto a_tile = [&](int m0) {
    return (const bf16*)g.A + (AK ? (int64_t)m0 * g.lda + (int64_t)s0 * BKT : (int64_t)s0 * BKT * g.lda + m0);
  };
  auto b_tile = [&](int n0) {
    if (glu) return (const bf16*)g.B + (int64_t)(n0 / 2) * g.ldb + (int64_t)s0 * BKT;
    return (const bf16*)g.B + (BKM ? (int64_t)n0 * g.ldb + (int64_t)s0 * BKT : (int64_t)s0 * BKT * g.ldb + n0);
  };
  const int64_t step_a = AK ? BKT : (int64_t)BKT * g.lda;
  const int64_t step_b = BKM ? BKT : (int64_t)BKT * g.ldb;
  // LDS byte addresses of this wave's first chunk of the A and B tiles of stage 0
  typedef __attribute__((address_space(3))) bf16 lds_bf16;
  const uint32_t la0 = (uint32_t)(uintptr_t)(lds_bf16*)(S + wave * 512);
  const uint32_t lb0 = la0 + TA::ELEMS * 2;
  // RAG: the ends of the operands, and this thread's k chunk within a slice (the same for all its
  // loads: NW waves' loads are whole periods of the swizzle apart)
  const bf16* ea = (const bf16*)g.A + (AK ? (int64_t)(g.M - 1) * g.lda + (g.a_padded ? g.lda : g.K)
                                          : (int64_t)(g.K - 1) * g.lda + (g.a_padded ? g.lda : g.M));
  const bf16* eb = (const bf16*)g.B + (BKM ? (int64_t)(glu ? 2 * g.glu - 1 : g.N - 1) * g.ldb + g.K
                                           : (int64_t)(g.K - 1) * g.ldb + g.N);
  int kca, kcb, r_;
  static_assert(BKT == 64 && NW % 4 == 0, "one k chunk per thread");
  TA::row_chunk(wave * 64 + lane, r_, kca);
  TB::row_chunk(wave * 64 + lane, r_, kcb);
  auto issue = [&](const bf16* at, const bf16* bt, int s, int stage) {
    const bf16* as = at + s * step_a;
    const bf16* bs = bt + s * step_b;
    const uint32_t ta = la0 + stage * STAGE * 2, tb = lb0 + stage * STAGE * 2;
    if constexpr (RAG) {
      const u32x4 ra = buffer_range(as, ea), rb = buffer_range(bs, eb);
      const int krem = g.K - (s0 + s) * BKT;
      const bool outa = AK && 8 * kca >= krem, outb = BKM && 8 * kcb >= krem;
#pragma unroll
      for (int q = 0; q < PA; ++q) dma16_range(ra, outa ? BUFFER_OUT : oa[q], ta + q * NW * 1024);
#pragma unroll
      for (int q = 0; q < PB; ++q) dma16_range(rb, outb ? BUFFER_OUT : ob[q], tb + q * NW * 1024);
    } else {
#pragma unroll
      for (int q = 0; q < PA; ++q) dma16(as, oa[q], ta + q * NW * 1024);
#pragma unroll
      for (int q = 0; q < PB; ++q) dma16(bs, ob[q], tb + q * NW * 1024);
    }
  };

  const int tile_end = g.tile_n > 0 ? g.tile0 + g.tile_n : tiles;
  int t = g.tile0 + blockIdx.x;
  int m0, n0;
  origin(t, m0, n0);
  const bf16* at = a_tile(m0);
  const bf16* bt = b_tile(n0);
  // slices NS - 1 and later ahead come from the next tile only when a tile has that many
  const bool chain = C_::persist && nk >= NS - 1;
#pragma unroll
  for (int s = 0; s < NS - 1; ++s) issue(at, bt, min(s, nk - 1), s);
  int G = 0;  // position in the block's slice sequence
  for (bool first = true;; first = false) {
    const int tn = t + gridDim.x;
    const bool next = chain && tn < tile_end;
    int m1 = m0, n1 = n0;
    if (next) origin(tn, m1, n1);
    const bf16* atn = a_tile(m1);
    const bf16* btn = b_tile(n1);

    f32x16 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    for (int kt = 0; kt < nk; ++kt, ++G) {
      // this thread's loads of slice G are in LDS: issued after them are the loads of the NS - 2
      // following slices and, in a tile's first slices, the previous tile's epilogue
      if (!first && kt < NS - 1) wait_vm_lds<(NS - 2) * (PA + PB) + EPI_OPS>();
      else wait_vm_lds<(NS - 2) * (PA + PB)>();
      block_barrier();  // ... and every thread's; the stage of slice G - 1 is free
      {
        const int x = kt + NS - 1, stage = (G + NS - 1) % NS;
        if (x < nk) issue(at, bt, x, stage);
        else if (next) issue(atn, btn, x - nk, stage);
        else issue(at, bt, nk - 1, stage);  // a reload into a stage nobody reads again
      }
      const bf16* as = S + (G % NS) * STAGE;
      const bf16* bs = as + TA::ELEMS;
      bf16x8 af[2][FM], bfr[2][FN];
#pragma unroll
      for (int i = 0; i < FM; ++i) af[0][i] = TA::frag(as, wm0 + i * 32, 0);
#pragma unroll
      for (int j = 0; j < FN; ++j) bfr[0][j] = TB::frag(bs, wn0 + j * 32, 0);
      // the next k-step's fragment reads go out between this step's MFMAs (one read after each
      // MFMA; they write the other fragment buffer), so the LDS and matrix pipes work together
      static_for<BKT / 16>([&](auto KS) {
        constexpr int ks = KS, c = ks & 1;
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (ks + 1 < BKT / 16) {
#pragma unroll
          for (int i = 0; i < FM; ++i) af[c ^ 1][i] = TA::frag(as, wm0 + i * 32, (ks + 1) * 16);
#pragma unroll
          for (int j = 0; j < FN; ++j) bfr[c ^ 1][j] = TB::frag(bs, wn0 + j * 32, (ks + 1) * 16);
        }
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[c][i], bfr[c][j], acc[i][j], 0, 0, 0);
        if constexpr (ks + 1 < BKT / 16) {
          static_assert(FM * FN >= FM + FN, "one MFMA ahead of every fragment read");
          static_for<FM + FN>([&](auto) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // one MFMA
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // one LDS read
          });
          __builtin_amdgcn_sched_group_barrier(0x008, FM * FN - (FM + FN), 0);
        }
        __builtin_amdgcn_sched_barrier(0);
      });
    }
    float* stg;
    if constexpr (C_::persist) {
      // the stage of the tile's last slice, once every wave is past its fragment reads
      stg = reinterpret_cast<float*>(S + ((G - 1) % NS) * STAGE);
    } else {
      wait_vm_lds<0>();  // the whole LDS: the reloads too
      stg = reinterpret_cast<float*>(smem);
    }
    wait_vm_lds<63>();
    block_barrier();
    dma_epilogue<BM, BN, WM, WN, OutT, EPI, C_::RP, RAG>(g, acc, stg, m0, n0, wm0, wn0, t - g.tile0);
    if (!next) break;
    t = tn; m0 = m1; n0 = n1; at = atn; bt = btn;
  }
  wait_vm_lds<0>();  // no load may land in the LDS after the block ends
}

// C = beta C + sum over splits of the partial tiles, in split order (fp32 output, ldc == N)
__global__ void __launch_bounds__(256) splitk_reduce(const float* __restrict__ ws, int splits, int64_t mn,
                                                     float* __restrict__ C, float beta) {
  const int64_t i = 4 * ((int64_t)blockIdx.x * blockDim.x + threadIdx.x);
  if (i >= mn) return;
  if (i + 3 < mn) {
    float4 acc = ld_nt<float4>(ws + i);
    for (int s = 1; s < splits; ++s) {
      const float4 v = ld_nt<float4>(ws + (int64_t)s * mn + i);
      acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
    }
    if (beta != 0.f) {
      const float4 c = *reinterpret_cast<const float4*>(C + i);
      acc.x += beta * c.x; acc.y += beta * c.y; acc.z += beta * c.z; acc.w += beta * c.w;
    }
    *reinterpret_cast<float4*>(C + i) = acc;
  } else {
    for (int64_t k = i; k < mn; ++k) {
      float acc = 0.f;
      for (int s = 0; s < splits; ++s) acc += ws[(int64_t)s * mn + k];
      C[k] = beta != 0.f ? acc + beta * C[k] : acc;
    }
  }
}

// The same for the BM x BN partial tiles of the products' tiles tile0 .. tile0 + tile_n - 1, one block row
// per tile (whole tiles)
template <int BM, int BN>
__global__ void __launch_bounds__(256) splitk_reduce_tiles(GemmArgs g) {
  int m0, n0;
  tile_origin<BM, BN>(g, g.tile0 + blockIdx.y, m0, n0);
  const int e = 4 * (blockIdx.x * 256 + threadIdx.x);
  const float* w = g.ws + (int64_t)blockIdx.y * BM * BN + e;
  float4 acc = ld_nt<float4>(w);
  for (int s = 1; s < g.ksplit; ++s) {
    const float4 v = ld_nt<float4>(w + (int64_t)s * g.tile_n * BM * BN);
    acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
  }
  float* c = (float*)g.C + (int64_t)(m0 + e / BN) * g.ldc + n0 + e % BN;
  if (g.beta != 0.f) {
    const float4 o = *reinterpret_cast<const float4*>(c);
    acc.x += g.beta * o.x; acc.y += g.beta * o.y; acc.z += g.beta * o.z; acc.w += g.beta * o.w;
  }
  *reinterpret_cast<float4*>(c) = acc;
}

// C = bf16 of the sum over splits of the partial tiles, in split order, plus resid (all rows of N)
__global__ void __launch_bounds__(256) splitk_reduce_bf16(const float* __restrict__ ws, int splits, int64_t mn,
                                                          const bf16* __restrict__ resid, bf16* __restrict__ C) {
  const int64_t i = 8 * ((int64_t)blockIdx.x * blockDim.x + threadIdx.x);  // N, so mn, is a multiple of 8
  if (i >= mn) return;
  f32x4 lo = ld_nt<f32x4>(ws + i), hi = ld_nt<f32x4>(ws + i + 4);
  for (int s = 1; s < splits; ++s) {
    lo += ld_nt<f32x4>(ws + (int64_t)s * mn + i);
    hi += ld_nt<f32x4>(ws + (int64_t)s * mn + i + 4);
  }
  bf16x8 o;
  if (resid) {
    const bf16x8 r = *reinterpret_cast<const bf16x8*>(resid + i);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      lo[q] += (float)r[q];
      hi[q] += (float)r[q + 4];
    }
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    o[q] = (bf16)lo[q];
    o[q + 4] = (bf16)hi[q];
  }
  *reinterpret_cast<bf16x8*>(C + i) = o;
}

template <int BM, int BN, int WM, int WN, bool AK, bool BKM, typename OutT, int BKT, int NS, int EPI, bool RAG>
void launch_dma_one(const GemmArgs& g, int nblk, hipStream_t st) {
  using C_ = DmaCfg<BM, BN, WM, WN, AK, BKM, BKT, NS>;
  static bool attr_set = false;
  if (!attr_set) {
    (void)hipFuncSetAttribute((const void*)gemm_dma_kernel<BM, BN, WM, WN, AK, BKM, OutT, BKT, NS, EPI, RAG>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)C_::lds);
    attr_set = true;
  }
  // more tiles than the chip holds blocks at once: one block per slot, each walking its tiles
  int grid = nblk;
  if (C_::persist && g.batch == 1 && cdiv(g.K, BKT) / g.ksplit >= NS - 1) {
    const int per_cu = (int)(163840 / C_::lds);
    const int slots = (per_cu * device_cu_count() / g.ksplit) / 8 * 8;
    if (slots >= 8 && nblk > slots) grid = slots;
  }
  gemm_dma_kernel<BM, BN, WM, WN, AK, BKM, OutT, BKT, NS, EPI, RAG>
      <<<dim3(grid, g.ksplit, g.batch), C_::NT, C_::lds, st>>>(g);
}

// Direct-to-LDS product of block tiles BM x BN; false if the kernels do not take the operand layouts
// and the epilogue.  fp32 output: every operand layout, no fused epilogue; bf16 output: a
// k-contiguous A (every bf16-output product of the stage has one) with each epilogue kind.
template <int BM, int BN, int WM, int WN, typename OutT, int BKT, int NS, bool RAG>
bool launch_dma_cfg(const GemmArgs& g, hipStream_t st) {
  const int nblk = g.tile_n > 0 ? g.tile_n
                   : !RAG && g.sym ? (g.M / BM) * (g.M / BM + 1) / 2 : (int)(cdiv(g.M, BM) * cdiv(g.N, BN));
#define L_(AK, BKM, E) launch_dma_one<BM, BN, WM, WN, AK, BKM, OutT, BKT, NS, E, RAG>(g, nblk, st)
  if constexpr (sizeof(OutT) == 4) {
    if (g.a_kmajor && g.b_kmajor) L_(true, true, EPI_PLAIN);
    else if (g.a_kmajor) L_(true, false, EPI_PLAIN);
    else if (g.b_kmajor) L_(false, true, EPI_PLAIN);
    else L_(false, false, EPI_PLAIN);
  } else {
    if (!g.a_kmajor) return false;
    const int kind = g.epi != 0 ? g.epi : (g.resid ? EPI_RESID : EPI_PLAIN);
#define K_(E)                     \
  case E:                         \
    if (g.b_kmajor) L_(true, true, E); \
    else L_(true, false, E);      \
    break;
    switch (kind) {
      K_(EPI_PLAIN) K_(EPI_SWIGLU_BWD) K_(EPI_ROPE) K_(EPI_SWIGLU_FWD) K_(EPI_DELTA) K_(EPI_RESID) K_(EPI_AXPBY)
      default:
        if constexpr (!RAG) {  // the forms of whole tiles only
          switch (kind) {
            K_(EPI_AXPBY_DUP) K_(EPI_NS_SPLIT)
            default: return false;
          }
        } else {
          return false;
        }
    }
#undef K_
  }
#undef L_
  return true;
}

template <int BM, int BN, int WM, int WN, bool RAG>
bool launch_dma(const GemmArgs& g, hipStream_t st) {
  return g.out_f32 ? launch_dma_cfg<BM, BN, WM, WN, float, BKT, 2, RAG>(g, st)
                   : launch_dma_cfg<BM, BN, WM, WN, bf16, BKT, 2, RAG>(g, st);
}

// Whether the chip holds all blocks of `tiles` 128 x 128 tiles in s splits at once (two per CU; the launcher
// gives every split a multiple of 8 of them).  One block more takes a second round: K 4104, 2304 x 768, 108
// tiles, 5 splits 39 us, 4 splits 28; K 8200, 2688 x 512, 84 tiles, 6 splits (80 blocks each) 53, 5 splits 36.
bool one_round(int64_t tiles, int s) { return s == 1 || tiles <= 512 / s / 8 * 8; }

// Tile choice: 256 x 256 (8 waves of 64 x 128, 64-deep slices in 2 stages, one block per CU) when the
// product has enough of them, is deep enough and fills their rounds of 256, else 128 x 128 (two blocks per
// CU, rounds of 512).  Measured 128 x 128 against 256 x 256:
//   - from K = 1536 on enough tiles decide;
//   - from K = 768 to there C has to fill 92 % of the rounds (M 8192, K 768, N 6144, 3 rounds: 92 : 81 us; M
//     20480, N 5632, K 1024, 6.9 of 7: 257 : 233; M 8192 there, 2.75 of 3: 99.6 : 102.7); 97 %, whole columns
//     and K 1280 for the SwiGLU backward, whose two outputs and reads one block per CU hides less (M 16384:
//     N 3072, K 768 121 : 126; N 2816, K 1024 123 : 138; N 5120, K 1280 279 : 265); 85 % where RoPE or delta
//     of 128-wide heads ride in the epilogue of the larger tile only (M 16384, N 2688, K 896: 125 : 97);
//   - a C of whole 128 x 128 but not 256 x 256 tiles takes the larger ones, partial at its edge, when they
//     need half the rounds (0.6 of them in fp32, or with those heads) and lie to a tenth outside C at most:
//     K 5120, 8192 x 1920, 1 : 2 rounds 148 : 142; K 5888, 8192 x 2176, 2 : 3 rounds 217 : 280; K 2432, 32768 x
//     896, an eighth outside, 137 : 149; fp32 over K 4096: 17408 x 3200, 4 : 7 rounds, 465 : 412, 10240 x 1920,
//     2 : 3, 154 : 194.
bool use_big(const GemmArgs& g) {
  const int64_t t256 = cdiv(g.M, 256) * cdiv(g.N, 256), rounds = cdiv(t256, 256), mn = (int64_t)g.M * g.N;
  // fp32 products of 129-255 tiles: one round, where 128 x 128 tiles take two (K 8192: 2048 x 6144 201 -> 176
  // us, 2048 x 5632 182 -> 163; where one round of 128 x 192 tiles holds it, that measures 166 for the first)
  if (g.out_f32 && g.K >= 2048 && g.M % 256 == 0 && g.N % 256 == 0 && t256 > 128 && t256 < 256) return true;
  const bool heads = (g.epi == 2 && g.rope_hd == 128) || (g.epi == 4 && g.delta_hd == 128);
  if (g.M % 128 == 0 && g.N % 128 == 0 && g.K % BKT == 0 && (g.M % 256 || g.N % 256) &&
      (10 * rounds > (g.out_f32 || heads ? 6 : 5) * cdiv(mn, 512 * 128 * 128) || 10 * 65536 * t256 > 11 * mn))
    return false;
  if (g.K >= 1536) return t256 >= 512 || (t256 >= 256 && g.K >= 2048);
  if (g.K < 768 || t256 < 512 || (g.epi == 1 && (g.K < 1280 || g.N % 256))) return false;
  return 100 * mn >= (g.epi == 1 ? 97 : heads ? 85 : 92) * 65536 * 256 * rounds;
}

// Weight-gradient products (fp32, row-contiguous operands) whose 128 x 128 blocks just miss a round of
// the 512 the chip holds: 128 x 192 tiles (4 waves of 64 x 96, two blocks per CU) when they need fewer
// rounds by more than their size (8 % more work per unit of time by fewer operand bytes).  K 8192, 768 x
// 3072 in 4 splits, 576 -> 384 blocks: 71 -> 53 us; 6144 x 768 in 2: 121 -> 85 us; 768 x 768 in 8, one
// round either way: 26.3 against 27.0 us.
bool use_wide(const GemmArgs& g) {
  if (!g.out_f32 || g.a_kmajor || g.b_kmajor || g.M % 128 || g.N % 192 || g.K % BKT) return false;
  const int64_t r128 = cdiv(cdiv(g.M, 128) * cdiv(g.N, 128) * g.ksplit, 512);
  const int64_t r192 = cdiv((int64_t)(g.M / 128) * (g.N / 192) * g.ksplit, 512);
  return 138 * r192 < 100 * r128;
}

// Splits of a deep bf16-output product of few tiles (plain or with a residual): up to one round of the
// 512 blocks the chip holds, at least 512 of K each.  M 999, N 768: K 32001 379 -> 92 us, K 6144
// 67 -> 27 us, the sum over the splits included.  That sum costs 8-14 us with the partial tiles' traffic,
// and the more tiles there are, the less a split gains: K above 640 + 11 tiles.  Unsplit against split,
// NT and NN: 96 tiles K 2048 23 : 19 us; 128 tiles K 2048 21 : 22.5, K 2816 31 : 26; 160 tiles K 2048
// 24 : 26.5, K 2816 31 : 30; 192 tiles K 2048 23.5 : 25.5, K 2816 31 : 29.5, K 4096 42 : 37; 256 tiles K 2048
// 26 : 31, K 2816 34 : 36.5, K 4096 47 : 44.5, K 5632 62 : 56.
int activation_splits(const GemmArgs& g) {
  if (g.out_f32 || !g.ws || g.epi != 0 || g.batch > 1 || g.sym || g.ldc != g.N || !g.a_kmajor || g.K < 2048) return 1;
  if ((uintptr_t)g.resid % 16) return 1;
  const int64_t tiles = cdiv(g.M, 128) * cdiv(g.N, 128), slices = cdiv(g.K, BKT), mn = (int64_t)g.M * g.N;
  if (g.K <= 640 + 11 * tiles) return 1;
  int s = (int)std::min<int64_t>(8, 512 / tiles);
  while (s > 1 && (s * mn > g.ws_elems || g.K / s < 512 || !one_round(tiles, s) || (s - 1) * cdiv(slices, s) >= slices))
    --s;
  return s;
}

// fp32 products of whole 256 x 256 tiles over more than one round of 256: the tiles past the last full
// round would take a round to themselves at a half or less of the blocks, so they are split over K as far
// as a round holds them.  K 8192: 4096 x 14336, 768 + 128 tiles, 824 -> 777 us; 49152 x 768, 512 + 64, 624 ->
// 576 us.  (128 x 128 tiles gain nothing: 2048 x 6144, 512 + 256 tiles, 195 -> 202 us.)
// s splits save 1 - 1/s of the tail's round, in proportion to K, and write and sum s tail partial tiles:
// they break even at K (s - 1) = 8 s^2 tail.  Whole against split: tail 128, s 2: K 2048 107 : 121 us, 3072
// 151 : 157, 4096 195 : 193, 6144 279 : 265; tail 96, s 2: K 2048 104 : 110, 3072 147 : 145, 4096 189 : 178;
// tail 64, s 4: K 2048 104.5 : 109, 3072 147 : 140; tail 14, s 4: K 2048 101 : 83.
bool launch_tail_split(const GemmArgs& g, hipStream_t st) {
  constexpr int B = 256, WM = 64, WN = 128, slots = 256;
  const int tiles = (g.M / B) * (g.N / B), tail = tiles % slots, slices = g.K / BKT;
  if (!g.out_f32 || g.ksplit > 1 || !g.ws || tiles < slots || tail == 0 || tail > slots / 2) return false;
  int s = std::min(8, slots / tail);
  while (s > 1 && (slices % s || g.K / s < 512 || tail > slots / s / 8 * 8 || (int64_t)s * tail * B * B > g.ws_elems)) --s;
  if (s < 2 || (int64_t)g.K * (s - 1) < (int64_t)8 * s * s * tail) return false;
  GemmArgs p = g;
  p.tile_n = tiles - tail;
  if (!launch_dma<B, B, WM, WN, false>(p, st)) return false;
  p.tile0 = tiles - tail;
  p.tile_n = tail;
  p.ksplit = s;
  if (!launch_dma<B, B, WM, WN, false>(p, st)) return false;
  splitk_reduce_tiles<B, B><<<dim3(B * B / 1024, tail), 256, 0, st>>>(p);
  return true;
}

// What every direct-to-LDS kernel needs: 16-byte aligned operand rows (a k-contiguous operand of
// whole 8-element chunks, or zero-padded rows; a row-contiguous one of whole chunks of rows), 16-byte
// output rows for bf16 output, and tile offsets below 2^31 bytes.
bool dma_operands(const GemmArgs& g) {
  if (g.K <= 0 || g.lda % 8 || g.ldb % 8) return false;
  if ((uintptr_t)g.A % 16 || (uintptr_t)g.B % 16 || (uintptr_t)g.C % 16) return false;
  if (!g.a_padded && (g.a_kmajor ? g.K : g.M) % 8) return false;
  if ((g.b_kmajor ? g.K : g.N) % 8) return false;
  if (!g.out_f32 && (g.N % 8 || g.ldc % 8)) return false;
  return 256 * (int64_t)std::max(g.lda, g.ldb) < ((int64_t)1 << 30);
}

}  // namespace

int device_cu_count() {
  static int cus[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (cus[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    cus[dev] = n;
  }
  return cus[dev];
}

bool gemm_mfma_try(const GemmArgs& g0, hipStream_t st) {
  if (!dma_operands(g0)) return false;
  if (const int s = activation_splits(g0); s > 1) {
    GemmArgs p = g0;  // fp32 partial tiles, then their sum in split order with the residual
    p.out_f32 = true;
    p.resid = nullptr;
    p.ksplit = s;
    const bool whole = g0.M % 128 == 0 && g0.N % 128 == 0 && g0.K % BKT == 0 && (g0.K / BKT) % s == 0;
    if (!(whole ? launch_dma<128, 128, 64, 64, false>(p, st) : launch_dma<128, 128, 64, 64, true>(p, st))) return false;
    const int64_t mn = (int64_t)g0.M * g0.N;
    splitk_reduce_bf16<<<(unsigned)cdiv(mn / 8, 256), 256, 0, st>>>(g0.ws, s, mn, (const bf16*)g0.resid, (bf16*)g0.C);
    return true;
  }
  GemmArgs g = g0;
  g.ksplit = 1;
  if (g.batch > 1 || g.sym || g.epi == EPI_AXPBY || g.epi == EPI_AXPBY_DUP || g.epi == EPI_NS_SPLIT) {
    // batched, symmetric and AXPBY products (a k-contiguous A; AXPBY with bf16 output, fp32 output
    // plain or accumulating beta C; 16-byte aligned batch strides)
    if (!g.a_kmajor || g.resid || (g.epi != 0 && (g.epi < EPI_AXPBY || g.out_f32)) || (uintptr_t)g.D % 16 ||
        (g.sA | g.sB | g.sC | g.sD) % 8 || (g.out_f32 && (g.N | g.ldc) % 4))
      return false;
    if (g.sym && (g.M != g.N || g.epi != 0 || g.out_f32)) return false;
    if (gemm_batched_tiles(g.M, g.N, g.K)) return launch_dma<128, 128, 64, 64, false>(g, st);
    return launch_dma<128, 128, 64, 64, true>(g, st);  // every tile of a symmetric product
  }
  if (g.epi == 3) {
    // the SwiGLU forward rides in the epilogue (the B loader gathers gate and up rows) when the
    // panels are whole and the up rows within a tile offset of the gate rows; any other shape runs the
    // product, then the SwiGLU kernel
    const bool fused = !g.out_f32 && g.b_kmajor && g.N == 2 * g.glu && g.glu % 64 == 0 && g.ld_out2 % 8 == 0 &&
                       (uintptr_t)g.out2 % 16 == 0 && (256 + (int64_t)g.glu) * g.ldb < ((int64_t)1 << 30);
    if (!fused) {
      GemmArgs p = g;
      p.epi = 0;
      p.glu = 0;
      if (!gemm_mfma_try(p, st)) return false;
      launch_swiglu_fwd(true, g.C, g.out2, g.M, g.glu, st);
      return true;
    }
  }
  if (g.epi == 1 && (g.out_f32 || g.ld_aux % 8 || (uintptr_t)g.aux % 16)) return false;
  if ((uintptr_t)g.resid % 16) return false;
  const bool big = use_big(g);
  const int wn = big ? 128 : 64;  // columns of one wave
  // delta rides in the epilogue when a wave's columns hold whole heads; otherwise the caller
  // computes it separately
  if (g.epi == 4 && (g.out_f32 || g.delta_hd < 8 || wn % g.delta_hd || g.N % g.delta_hd || g.ld_aux % 8 ||
                     (uintptr_t)g.aux % 16))
    return false;
  const int64_t mn = (int64_t)g.M * g.N;
  const int64_t tiles = big ? cdiv(g.M, 256) * cdiv(g.N, 256) : cdiv(g.M, 128) * cdiv(g.N, 128);
  const int64_t slices = cdiv(g.K, BKT);
  if (g.out_f32 && g.ws && g.ldc == g.N && tiles < 512 && g.K >= 2048) {
    // deterministic split-K for underfilled fp32-output products: whole slices per split, equal
    // splits where K is a whole number of slices, otherwise none empty and all in one round
    int s = big && tiles < 256 ? 1 : (int)std::min<int64_t>(8, cdiv(512, tiles));
    while (s > 1 && (s * mn > g.ws_elems || g.K / s < 512 ||
                     (g.K % BKT == 0 ? slices % s != 0 : !one_round(tiles, s) || (s - 1) * cdiv(slices, s) >= slices)))
      --s;
    g.ksplit = s;
  }
  // RoPE in the epilogue needs every head whole inside one wave's columns
  const bool rope_after = g.epi == 2 && (g.out_f32 || wn % g.rope_hd != 0);
  if (rope_after) g.epi = 0;
  // whole tiles and slices (and equal splits): the loads and stores need no range
  const int bm = big ? 256 : 128;
  const bool whole = g.M % bm == 0 && g.N % bm == 0 && g.K % BKT == 0 && slices % g.ksplit == 0 &&
                     (g.N | g.ldc) % 4 == 0;
  const bool wide = whole && !big && use_wide(g);
  bool done;
  if (whole && big && launch_tail_split(g, st)) return true;
  if (big) done = whole ? launch_dma<256, 256, 64, 128, false>(g, st) : launch_dma<256, 256, 64, 128, true>(g, st);
  else if (wide) {
    launch_dma_one<128, 192, 64, 96, false, false, float, BKT, 2, EPI_PLAIN, false>(g, (g.M / 128) * (g.N / 192), st);
    done = true;
  } else done = whole ? launch_dma<128, 128, 64, 64, false>(g, st) : launch_dma<128, 128, 64, 64, true>(g, st);
  if (!done) return false;
  if (g.ksplit > 1)
    splitk_reduce<<<(unsigned)cdiv(cdiv(mn, 4), 256), 256, 0, st>>>(g.ws, g.ksplit, mn, (float*)g.C, g.beta);
  if (rope_after)
    launch_rope(!g.out_f32, g.C, g.M, g.rope_S, g.rope_cols / g.rope_hd, g.rope_hd, g.ldc, g.rope_cos,
                g.rope_sin, false, st);
  return true;
}
