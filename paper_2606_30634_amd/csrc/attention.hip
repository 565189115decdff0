// Causal grouped-query attention (App. E.2) in fp32 on the matrix cores, for the fp32 stage and for
// the bf16 stage's head dimensions that attention_mfma.hip does not take (bf16 in and out there).
//
//   S = q k^T / sqrt(hd) on j <= i;  P = softmax(S);  o = P v;  lse_i = log sum_j exp(S_ij)
//   delta_i = sum_c dO_ic O_ic;  dP = dO v^T;  dS = P (dP - delta);  dq = dS k / sqrt(hd)
//   dk = dS^T q / sqrt(hd) and dv = P^T dO, summed over the query heads of a key/value head.
// Query head h reads key/value head h / (Hq / Hkv).
//
// v_mfma_f32_32x32x2_f32 throughout (lane l: operand row l mod 32 at k = l / 32; accumulator e of
// lane l: row 8 (e / 4) + 4 (l / 32) + e mod 4, column l mod 32).  A block of 4 waves owns 32 rows
// (queries for o and dq, keys for dk and dv) of one head; its waves take every fourth 32-row tile of
// the other side and their sums meet in LDS, in wave order, at the end: the sequences here are short,
// so it is the serial chain of one row block, not the chip's rate, that bounds a launch.  Scores are
// formed with the block's rows as columns (S^T = K Q^T; S = Q K^T for dk, dv), so accumulator e of a
// lane pair holds two rows 4 apart of the other side and is itself the k = 2 operand of the next
// product: no value moves between lanes.  Operands come from global memory (L2) straight into
// registers: an MFMA takes 64 cycles, a lane's loads for it at most 2.
// At 4 sequences of 256, 8 heads of 64: forward 211 -> 11 us, backward 632 -> 41 us (delta, rotation,
// dq, dk and dv; one thread per row in five launches before).
#include "common.h"
#include "kernels.h"

bool attention_mfma_fwd_try(const AttnArgs& a, hipStream_t st);  // attention_mfma.hip
bool attention_mfma_bwd_try(const AttnArgs& a, hipStream_t st);
bool attention_mfma_delta_try(const AttnArgs& a, hipStream_t st);

namespace {

constexpr int TR = 32;  // rows of a block and of a tile
constexpr int NW = 4;   // waves of a block

__device__ __forceinline__ f32x16 mfma2(float a, float b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// Orders one lane's LDS accesses before another lane's of the same wave
__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Four consecutive elements as fp32 (rows start on 4 elements: head_dim and every width are
// multiples of 32)
__device__ __forceinline__ f32x4 ld4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }
__device__ __forceinline__ f32x4 ld4(const bf16* p) {
  const bf16x4 v = *reinterpret_cast<const bf16x4*>(p);
  return f32x4{(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
}
__device__ __forceinline__ void st4(float* p, const f32x4& v) { *reinterpret_cast<f32x4*>(p) = v; }
__device__ __forceinline__ void st4(bf16* p, const f32x4& v) {
  *reinterpret_cast<bf16x4*>(p) = bf16x4{(bf16)v[0], (bf16)v[1], (bf16)v[2], (bf16)v[3]};
}

// Row operand: this lane's half of row `row` (stride ld) for a contraction over the head dimension:
// group q holds elements 8 q + 4 (lane / 32) .. + 3, so that step (q, j) pairs 8 q + j with 8 q + 4 + j.
template <int HD>
struct RowFrag {
  f32x4 v[HD / 8];
  template <typename T>
  __device__ __forceinline__ void load(const T* p, int64_t row, int ld) {
    const T* r = p + row * ld + 4 * (threadIdx.x % 64 / 32);
#pragma unroll
    for (int q = 0; q < HD / 8; ++q) v[q] = ld4(r + 8 * q);
  }
  // whether every value of the wave's rows is finite (the sum stays 0 as long as they are)
  __device__ __forceinline__ bool finite() const {
    float z = 0.f;
#pragma unroll
    for (int q = 0; q < HD / 8; ++q)
#pragma unroll
      for (int j = 0; j < 4; ++j) z = __builtin_fmaf(v[q][j], 0.f, z);
    return __all(z == 0.f);
  }
};
// S (+)= A B^T over the head dimension: accumulator rows are A's rows, columns B's
template <int HD>
__device__ __forceinline__ f32x16 rows_product(const RowFrag<HD>& a, const RowFrag<HD>& b) {
  f32x16 s;
#pragma unroll
  for (int e = 0; e < 16; ++e) s[e] = 0.f;
#pragma unroll
  for (int q = 0; q < HD / 8; ++q)
#pragma unroll
    for (int j = 0; j < 4; ++j) s = mfma2(a.v[q][j], b.v[q][j], s);
  return s;
}

// acc[dt] (rows 32 dt .. of X^T, columns the block's rows) += X^T W over the 32 tile rows of X, whose
// weights w sit in an accumulator (rows: tile rows).  Tile row r is row min(row0 + r, last) of X.
template <int HD, typename T>
__device__ __forceinline__ void cols_product(f32x16 (&acc)[HD / 32], const T* x, int row0, int last, int ld,
                                             const f32x16& w) {
  const int lane = threadIdx.x % 64;
  float f[HD / 32][16];
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const T* r = x + (int64_t)min(row0 + 8 * (e / 4) + 4 * (lane / 32) + e % 4, last) * ld + lane % 32;
#pragma unroll
    for (int dt = 0; dt < HD / 32; ++dt) f[dt][e] = to_f32(r[32 * dt]);
  }
#pragma unroll
  for (int e = 0; e < 16; ++e)
#pragma unroll
    for (int dt = 0; dt < HD / 32; ++dt) acc[dt] = mfma2(f[dt][e], w[e], acc[dt]);
}

// The same sum where some column does not see every tile row and a row holds an infinity or a NaN: its
// weights there are 0, and 0 times such a value would be a NaN.  Row by row, each column the rows that
// it sees (seen(r) for this lane's); tile: 32 x 32 floats of this wave's LDS.
template <int HD, typename T, typename F>
__device__ __forceinline__ void cols_product_seen(f32x16 (&acc)[HD / 32], const T* x, int row0, int ld,
                                                  const f32x16& w, float* tile, F&& seen) {
  const int lane = threadIdx.x % 64;
#pragma unroll
  for (int e = 0; e < 16; ++e) tile[(8 * (e / 4) + 4 * (lane / 32) + e % 4) * TR + lane % 32] = w[e];
  wave_fence();
#pragma unroll
  for (int dt = 0; dt < HD / 32; ++dt)
#pragma unroll 1
    for (int r = 0; r < TR; ++r) {
      if (!seen(r)) continue;
      const float wr = tile[r * TR + lane % 32];
      const T* xr = x + (int64_t)(row0 + r) * ld + 32 * dt + 4 * (lane / 32);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4 v = ld4(xr + 8 * q);
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[dt][4 * q + j] += wr * v[j];
      }
    }
  wave_fence();
}

// LDS of one wave (floats): its partial sums, [dt][e][lane]
template <int HD>
constexpr int WAVE_LDS = (HD / 32) * 16 * 64;

// Sum of the waves' accumulators over red ([wave][dt][e][lane]), in wave order.
template <int HD>
__device__ __forceinline__ void put_partial(float* red, const f32x16 (&acc)[HD / 32], float scale) {
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
#pragma unroll
  for (int dt = 0; dt < HD / 32; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) red[((wave * (HD / 32) + dt) * 16 + e) * 64 + lane] = acc[dt][e] * scale;
}
template <int HD>
__device__ __forceinline__ float get_sum(const float* red, int dt, int e) {
  const int lane = threadIdx.x % 64;
  float v = red[(dt * 16 + e) * 64 + lane];
#pragma unroll
  for (int w = 1; w < NW; ++w) v += red[((w * (HD / 32) + dt) * 16 + e) * 64 + lane];
  return v;
}

// The summed rows leave as rows of out (row row0 + lane mod 32, elements 32 dt + 8 (e / 4) + 4 (lane /
// 32) ..+ 3: 16-byte chunks): wave w writes the chunks e / 4 = w.  With RoPE tables the rows are
// rotated back by -angle(position) first: element c < hd/2 pairs with c + hd/2, which the same lane
// holds (another dt, or for head dimension 32 e + 8).
template <int HD, typename T>
__device__ __forceinline__ void store_rows(const float* red, float scale, T* out, int ld, int row0, int S,
                                           const float* cos_t, const float* sin_t, float* out32 = nullptr) {
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  const int row = row0 + lane % 32;
#pragma unroll
  for (int dt = 0; dt < HD / 32; ++dt) {
    const int c = 32 * dt + 8 * wave + 4 * (lane / 32);
    f32x4 v;
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = get_sum<HD>(red, dt, 4 * wave + j) * scale;
    if (cos_t) {
      constexpr int HH = HD / 2;
      const bool first = c < HH;
      const int pd = HD == 32 ? dt : (first ? dt + HD / 64 : dt - HD / 64), pe = HD == 32 ? (4 * wave) ^ 8 : 4 * wave;
      const int64_t t = (int64_t)min(row, S - 1) * HH + c % HH;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float p = get_sum<HD>(red, pd, pe + j) * scale, cs = cos_t[t + j], sn = sin_t[t + j];
        v[j] = first ? v[j] * cs + p * sn : v[j] * cs - p * sn;
      }
    }
    if (row < S) {
      st4(out + (int64_t)row * ld + c, v);
      if (out32) st4(out32 + (int64_t)row * ld + c, v);
    }
  }
}

struct Geo {
  int ld, koff, voff, group;
  __device__ explicit Geo(const AttnArgs& a) {
    ld = (a.Hq + 2 * a.Hkv) * a.hd;
    koff = a.Hq * a.hd;
    voff = (a.Hq + a.Hkv) * a.hd;
    group = a.Hq / a.Hkv;
  }
};

__device__ __forceinline__ float pair_max(float v) { return fmaxf(v, __shfl_xor(v, 32, WAVE)); }
__device__ __forceinline__ float pair_sum(float v) { return v + __shfl_xor(v, 32, WAVE); }

// Waves per SIMD the kernels are built for: within these bounds the accumulators stay in vector registers
// and nothing spills.  Left to itself the compiler keeps them in accumulator registers, copies them for the
// row-by-row sums of a tile with non-finite rows, and fits one wave less (16 sequences of 512, 8 heads of
// 64: forward 122 us against 99, backward 469 against 423).
constexpr int fwd_waves(int hd) { return hd == 128 ? 1 : hd == 64 ? 3 : 4; }
constexpr int bwd_waves(int hd) { return hd == 128 ? 1 : 2; }

// One block per (32 queries, query head, sequence); longest causal ranges first.
template <typename T, int HD>
__global__ void __launch_bounds__(NW * 64, fwd_waves(HD)) attn_fwd(AttnArgs a) {
  __shared__ float red[NW * WAVE_LDS<HD>];
  const Geo g(a);
  const int b = blockIdx.z, h = blockIdx.y, kvh = h / g.group;
  const int q0 = (gridDim.x - 1 - blockIdx.x) * TR;
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, q = q0 + lane % 32;
  float* mine = red + wave * WAVE_LDS<HD>;  // this wave's part
  const T* qkv = (const T*)a.qkv + (int64_t)b * a.S * g.ld;
  const T* kp = qkv + g.koff + kvh * HD;
  const T* vp = qkv + g.voff + kvh * HD;
  const float scale = 1.0f / sqrtf((float)HD);
  RowFrag<HD> qf;
  qf.load(qkv + h * HD, min(q, a.S - 1), g.ld);
#pragma unroll
  for (int i = 0; i < HD / 8; ++i) qf.v[i] *= scale;
  f32x16 o[HD / 32];
#pragma unroll
  for (int dt = 0; dt < HD / 32; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) o[dt][e] = 0.f;
  float m = -INFINITY, l = 0.f;
  // one tile of keys; edge: the last, whose keys some queries do not see
  auto tile = [&](int k0, auto edge) {
    RowFrag<HD> kf;
    kf.load(kp, min(k0 + lane % 32, a.S - 1), g.ld);
    f32x16 s = rows_product<HD>(kf, qf);  // rows: keys; column: this lane's query
    float mt = -INFINITY;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      if (edge && k0 + 8 * (e / 4) + 4 * (lane / 32) + e % 4 > q) s[e] = -INFINITY;
      mt = fmaxf(mt, s[e]);
    }
    const float mn = fmaxf(m, pair_max(mt));
    const float base = mn == -INFINITY ? 0.f : mn;  // no score above -inf yet: every weight 0
    const float corr = expf(m - base);              // 0 for the first tile
    float rs = 0.f;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      s[e] = expf(s[e] - base);
      rs += s[e];
    }
    l = l * corr + pair_sum(rs);
    m = mn;
#pragma unroll
    for (int dt = 0; dt < HD / 32; ++dt) o[dt] *= corr;
    if constexpr (edge) {
      kf.load(vp, min(k0 + lane % 32, a.S - 1), g.ld);
      if (!kf.finite()) {
        cols_product_seen<HD>(o, vp, k0, g.ld, s, mine, [&](int r) { return k0 + r <= q && k0 + r < a.S; });
        return;
      }
    }
    cols_product<HD>(o, vp, k0, a.S - 1, g.ld, s);
  };
  int k0 = wave * TR;
  for (; k0 < q0; k0 += NW * TR) tile(k0, std::false_type{});
  if (k0 == q0) tile(k0, std::true_type{});
  // the waves' statistics: o = sum_w e^(m_w - M) o_w / sum_w e^(m_w - M) l_w (wave 0 always has a tile)
  if (lane < TR) {
    mine[lane] = m;
    mine[TR + lane] = l;
  }
  __syncthreads();
  float M = -INFINITY, L = 0.f;
#pragma unroll
  for (int w = 0; w < NW; ++w) M = fmaxf(M, red[w * WAVE_LDS<HD> + lane % 32]);
#pragma unroll
  for (int w = 0; w < NW; ++w)
    L += expf(red[w * WAVE_LDS<HD> + lane % 32] - M) * red[w * WAVE_LDS<HD> + TR + lane % 32];
  __syncthreads();
  put_partial<HD>(red, o, expf(m - M) / L);
  __syncthreads();
  store_rows<HD>(red, 1.0f, (T*)a.o + (int64_t)b * a.S * a.Hq * HD + h * HD, a.Hq * HD, q0, a.S, nullptr, nullptr,
                 sizeof(T) == 2 && a.o32 ? a.o32 + (int64_t)b * a.S * a.Hq * HD + h * HD : nullptr);
  if (wave == 0 && lane < TR && q < a.S) a.lse[((int64_t)b * a.Hq + h) * a.S + q] = M + logf(L);
}

// delta_i = sum_c dO_ic O_ic per (batch, head, query): HD / 4 lanes per row
template <typename T, int HD>
__global__ void __launch_bounds__(256) attn_delta(AttnArgs a) {
  constexpr int LR = HD / 4;
  const int64_t r = ((int64_t)blockIdx.x * 256 + threadIdx.x) / LR;  // (b, i, h) in memory order
  const int c = (threadIdx.x % LR) * 4;
  float s = 0.f;
  const bool in = r < (int64_t)a.B * a.S * a.Hq;
  if (in) {
    const f32x4 d = ld4((const T*)a.dout + r * HD + c);
    const f32x4 o = sizeof(T) == 2 && a.o32 ? ld4(a.o32 + r * HD + c) : ld4((const T*)a.o + r * HD + c);
    s = (o[0] * d[0] + o[1] * d[1]) + (o[2] * d[2] + o[3] * d[3]);
  }
#pragma unroll
  for (int k = 1; k < LR; k <<= 1) s += __shfl_xor(s, k, WAVE);
  if (in && c == 0) {
    const int h = r % a.Hq;
    const int64_t row = r / a.Hq, b = row / a.S, i = row % a.S;
    a.delta[(b * a.Hq + h) * a.S + i] = s;
  }
}

// dq of 32 queries of head h
template <typename T, int HD>
__device__ __forceinline__ void bwd_dq(const AttnArgs& a, int qb, int h, int b, float* red) {
  const Geo g(a);
  const int kvh = h / g.group, q0 = qb * TR;
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, q = q0 + lane % 32, qc = min(q, a.S - 1);
  const T* qkv = (const T*)a.qkv + (int64_t)b * a.S * g.ld;
  const T* kp = qkv + g.koff + kvh * HD;
  const T* vp = qkv + g.voff + kvh * HD;
  const float scale = 1.0f / sqrtf((float)HD);
  RowFrag<HD> qf, df;
  qf.load(qkv + h * HD, qc, g.ld);
  df.load((const T*)a.dout + (int64_t)b * a.S * a.Hq * HD + h * HD, qc, a.Hq * HD);
#pragma unroll
  for (int i = 0; i < HD / 8; ++i) qf.v[i] *= scale;
  const int64_t sidx = ((int64_t)b * a.Hq + h) * a.S + qc;
  const float lse = a.lse[sidx], dl = a.delta[sidx];
  f32x16 dq[HD / 32];
#pragma unroll
  for (int dt = 0; dt < HD / 32; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) dq[dt][e] = 0.f;
  auto tile = [&](int k0, auto edge) {  // as in the forward
    const int kr = min(k0 + lane % 32, a.S - 1);
    RowFrag<HD> f;
    f.load(kp, kr, g.ld);
    const bool plain = !edge || f.finite();
    f32x16 s = rows_product<HD>(f, qf);
    f.load(vp, kr, g.ld);
    const f32x16 dp = rows_product<HD>(f, df);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const bool seen = !edge || k0 + 8 * (e / 4) + 4 * (lane / 32) + e % 4 <= q;
      s[e] = seen ? expf(s[e] - lse) * (dp[e] - dl) : 0.f;
    }
    if (plain) cols_product<HD>(dq, kp, k0, a.S - 1, g.ld, s);
    else cols_product_seen<HD>(dq, kp, k0, g.ld, s, red + wave * WAVE_LDS<HD>, [&](int r) { return k0 + r <= q && k0 + r < a.S; });
  };
  int k0 = wave * TR;
  for (; k0 < q0; k0 += NW * TR) tile(k0, std::false_type{});
  if (k0 == q0) tile(k0, std::true_type{});
  put_partial<HD>(red, dq, 1.0f);
  __syncthreads();
  store_rows<HD>(red, scale, (T*)a.dqkv + (int64_t)b * a.S * g.ld + h * HD, g.ld, q0, a.S, a.rope_cos, a.rope_sin);
}

// dk and dv of 32 keys of key/value head kvh, summed over its query heads
template <typename T, int HD>
__device__ __forceinline__ void bwd_dkv(const AttnArgs& a, int kb, int kvh, int b, float* red) {
  const Geo g(a);
  const int k0 = kb * TR;
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, key = k0 + lane % 32, kc = min(key, a.S - 1);
  const T* qkv = (const T*)a.qkv + (int64_t)b * a.S * g.ld;
  const float scale = 1.0f / sqrtf((float)HD);
  RowFrag<HD> kf, vf;
  kf.load(qkv + g.koff + kvh * HD, kc, g.ld);
  vf.load(qkv + g.voff + kvh * HD, kc, g.ld);
#pragma unroll
  for (int i = 0; i < HD / 8; ++i) kf.v[i] *= scale;
  f32x16 dk[HD / 32], dv[HD / 32];
#pragma unroll
  for (int dt = 0; dt < HD / 32; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) { dk[dt][e] = 0.f; dv[dt][e] = 0.f; }
  // tiles: every query tile at or after the keys, of every query head of the group
  const int nt = (a.S + TR - 1) / TR - kb;
  for (int it = wave; it < g.group * nt; it += NW) {
    const int h = kvh * g.group + it / nt, q0 = k0 + (it % nt) * TR;
    const T* qp = qkv + h * HD;
    const T* dp_ = (const T*)a.dout + (int64_t)b * a.S * a.Hq * HD + h * HD;
    const int64_t sb = ((int64_t)b * a.Hq + h) * a.S;
    const int qr = min(q0 + lane % 32, a.S - 1);
    const bool whole = q0 != k0 && q0 + TR <= a.S;  // every key sees every query of the tile
    RowFrag<HD> f;
    f.load(qp, qr, g.ld);
    const bool plain_q = whole || f.finite();
    f32x16 p = rows_product<HD>(f, kf);  // rows: queries; column: this lane's key
    f.load(dp_, qr, a.Hq * HD);
    const bool plain_d = whole || f.finite();
    f32x16 ds = rows_product<HD>(f, vf);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int q = q0 + 8 * (e / 4) + 4 * (lane / 32) + e % 4, qc = min(q, a.S - 1);
      const bool sees = q >= key && q < a.S;
      p[e] = sees ? expf(p[e] - a.lse[sb + qc]) : 0.f;
      ds[e] = sees ? p[e] * (ds[e] - a.delta[sb + qc]) : 0.f;
    }
    auto seen = [&](int r) { return q0 + r >= key && q0 + r < a.S; };
    if (plain_d) cols_product<HD>(dv, dp_, q0, a.S - 1, a.Hq * HD, p);
    else cols_product_seen<HD>(dv, dp_, q0, a.Hq * HD, p, red + wave * WAVE_LDS<HD>, seen);
    if (plain_q) cols_product<HD>(dk, qp, q0, a.S - 1, g.ld, ds);
    else cols_product_seen<HD>(dk, qp, q0, g.ld, ds, red + wave * WAVE_LDS<HD>, seen);
  }
  T* out = (T*)a.dqkv + (int64_t)b * a.S * g.ld;
  put_partial<HD>(red, dk, 1.0f);
  __syncthreads();
  store_rows<HD>(red, scale, out + g.koff + kvh * HD, g.ld, k0, a.S, a.rope_cos, a.rope_sin);
  __syncthreads();
  put_partial<HD>(red, dv, 1.0f);
  __syncthreads();
  store_rows<HD>(red, 1.0f, out + g.voff + kvh * HD, g.ld, k0, a.S, nullptr, nullptr);
}

// dk/dv blocks (first, low keys see the most queries) and dq blocks (longest ranges first) in one
// launch: independent given delta, and together they fill more of the chip.
template <typename T, int HD>
__global__ void __launch_bounds__(NW * 64, bwd_waves(HD)) attn_bwd(AttnArgs a) {
  __shared__ float red[NW * WAVE_LDS<HD>];
  const int h = blockIdx.y, b = blockIdx.z;
  if (h < a.Hkv) bwd_dkv<T, HD>(a, blockIdx.x, h, b, red);
  else bwd_dq<T, HD>(a, gridDim.x - 1 - blockIdx.x, h - a.Hkv, b, red);
}

template <typename T, int HD>
void fwd_t(const AttnArgs& a, hipStream_t st) {
  attn_fwd<T, HD><<<dim3((unsigned)cdiv(a.S, TR), a.Hq, a.B), NW * 64, 0, st>>>(a);
}
template <typename T, int HD>
void delta_t(const AttnArgs& a, hipStream_t st) {
  attn_delta<T, HD><<<(unsigned)cdiv((int64_t)a.B * a.Hq * a.S * (HD / 4), 256), 256, 0, st>>>(a);
}
template <typename T, int HD>
void bwd_t(const AttnArgs& a, hipStream_t st) {
  if (!a.delta_ready) delta_t<T, HD>(a, st);
  attn_bwd<T, HD><<<dim3((unsigned)cdiv(a.S, TR), a.Hkv + a.Hq, a.B), NW * 64, 0, st>>>(a);
}

template <typename T, typename F>
void dispatch_hd(int hd, F&& run) {
  if (hd == 32) run(T{}, std::integral_constant<int, 32>{});
  else if (hd == 64) run(T{}, std::integral_constant<int, 64>{});
  else run(T{}, std::integral_constant<int, 128>{});
}
template <typename F>
void dispatch(bool bf, int hd, F&& run) {  // run(type tag, head dimension)
  if (bf) dispatch_hd<bf16>(hd, run);
  else dispatch_hd<float>(hd, run);
}

}  // namespace

void launch_attention_fwd(bool bf, const AttnArgs& a, hipStream_t st) {
  if (bf && attention_mfma_fwd_try(a, st)) return;
  dispatch(bf, a.hd, [&](auto t, auto hd) { fwd_t<decltype(t), decltype(hd)::value>(a, st); });
}
void launch_attention_delta(bool bf, const AttnArgs& a, hipStream_t st) {
  if (bf && attention_mfma_delta_try(a, st)) return;
  dispatch(bf, a.hd, [&](auto t, auto hd) { delta_t<decltype(t), decltype(hd)::value>(a, st); });
}
void launch_attention_bwd(bool bf, const AttnArgs& a, hipStream_t st) {
  if (bf && attention_mfma_bwd_try(a, st)) return;
  dispatch(bf, a.hd, [&](auto t, auto hd) { bwd_t<decltype(t), decltype(hd)::value>(a, st); });
}
