// kernels_f32.hip -- fp32 mode of the co-batched multi-LoRA layer, with the same
// semantics and layouts as the bf16 path and fixed summation orders.  Every
// contraction runs on v_mfma_f32_16x16x4_f32 (fp32 products and sums, as exact
// as scalar fused multiply-adds).
//
// One workgroup computes 32 rows x 32 NCT columns of one contraction, 4 waves
// of 16 rows x 16 NCT columns.  The contraction runs in chunks of 64: a
// thread loads 8 values of each operand two chunks ahead into registers, one
// of two LDS buffers takes a chunk, one barrier per chunk.  These batches are
// small (a few hundred rows), so the tile is small to spread them over the CUs
// and the loads are deep because each chunk's latency is what bounds it.
// At T = 256 (64 training rows), K = N = 512, rank 8 a forward and backward take
// 33 us in four launches (shrink 8.0, y 7.6, g and dB 9.4, dA and dX 7.7: latency,
// not the 0.17 GFLOP), against 317 us in six launches of one thread per element
// (58 + 138, 40 + 13, 16 + 53), each a serial chain over the whole contraction.
#include <hip/hip_runtime.h>

#include "kernels.h"
#include "plan.h"

namespace dsv {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int CK = 64;        // contraction per chunk
constexpr int LS = CK + 4;    // LDS row stride (floats): 16-byte reads of 16 rows on distinct banks
constexpr int MR = 32;        // rows per workgroup

// Dropout: is element k of compact training row i kept?
__device__ __forceinline__ bool kept(const F32Args& g, int i, int k) {
  return (g.keep[(int64_t)i * g.keep_words + (k >> 5)] >> (k & 31)) & 1u;
}

struct V8 {
  f32x4 a, b;
};
__device__ __forceinline__ V8 zero8() { return V8{f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}}; }
// 8 floats at a 16-byte aligned address
__device__ __forceinline__ V8 ld8v(const float* p) {
  return V8{*reinterpret_cast<const f32x4*>(p), *reinterpret_cast<const f32x4*>(p + 4)};
}
// n < 8 (or unaligned) floats, the rest zero
__device__ __forceinline__ V8 ld8s(const float* p, int n) {
  V8 v = zero8();
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if (e < n) v.a[e] = p[e];
    if (e + 4 < n) v.b[e] = p[e + 4];
  }
  return v;
}

// Operand whose contraction is contiguous: a thread's 8 values of row t / 8 are
// contraction entries 8 (t % 8) .. +7 of the chunk.
__device__ __forceinline__ void put_rows(float (*s)[LS], const V8& v) {
  float* d = &s[threadIdx.x >> 3][8 * (threadIdx.x & 7)];
  *reinterpret_cast<f32x4*>(d) = v.a;
  *reinterpret_cast<f32x4*>(d + 4) = v.b;
}
// Operand whose rows are contiguous: a thread's 8 values of contraction entry
// t / 4 are rows 8 (t % 4) .. +7; they go into LDS transposed.
__device__ __forceinline__ void put_cols(float (*s)[LS], const V8& v) {
  const int i = threadIdx.x >> 2, m = 8 * (threadIdx.x & 3);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    s[m + e][i] = v.a[e];
    s[m + 4 + e][i] = v.b[e];
  }
}

// acc[ct][v] += the chunk's product over the contraction entries 4 i + v (four
// sums instead of one: their chains round a quarter as often, so the result is
// closer to 64 bits than one chain's): lane (l15 = lane % 16, g4 = lane / 16) ends with
// row 16 (wave % 2) + l15, columns 16 (wave / 2 + 2 ct) + 4 g4 .. +3 of the tile.
template <int NCT>
__device__ __forceinline__ void chunk_mm(const float (*sa)[LS], const float (*sb)[LS], f32x4 (&acc)[NCT][4]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l15 = lane & 15, g4 = lane >> 4;
  const float* pa = &sa[16 * (wave & 1) + l15][4 * g4];
#pragma unroll
  for (int h = 0; h < CK / 16; ++h) {
    const f32x4 a = *reinterpret_cast<const f32x4*>(pa + 16 * h);
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) {
      const f32x4 b = *reinterpret_cast<const f32x4*>(&sb[16 * (wave >> 1) + 32 * ct + l15][16 * h + 4 * g4]);
#pragma unroll
      for (int v = 0; v < 4; ++v)
        acc[ct][v] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[v], a[v], acc[ct][v], 0, 0, 0);
    }
  }
}

template <int NCT>
struct TileLds {
  float a[2][MR][LS];
  float b[2][MR * NCT][LS];
};

// The contraction of one tile over chunks [0, n).  la(c) / lb(c, ct) load a
// thread's 8 values of chunk c (column tile pair ct), pa / pb store them.
template <int NCT, class LA, class LB, class PA, class PB>
__device__ __forceinline__ void tile_mm(TileLds<NCT>& L, int n, LA la, LB lb, PA pa, PB pb, f32x4 (&out)[NCT]) {
  f32x4 acc[NCT][4];
  V8 a[2], b[2][NCT];
  auto load = [&](int c, int s) {
    a[s] = la(c);
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) b[s][ct] = lb(c, ct);
  };
  auto step = [&](int c, int s) {
    pa(L.a[s], a[s]);
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) pb(&L.b[s][MR * ct], b[s][ct]);
    if (c + 2 < n) load(c + 2, s);
    // buffer s is complete; every wave is past chunk c - 1, so the other buffer
    // may be rewritten in the next step
    __syncthreads();
    chunk_mm<NCT>(L.a[s], L.b[s], acc);
  };
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[ct][v] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (n > 0) load(0, 0);
  if (n > 1) load(1, 1);
  for (int c = 0; c < n; c += 2) {
    step(c, 0);
    if (c + 1 < n) step(c + 1, 1);
  }
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct) out[ct] = (acc[ct][0] + acc[ct][1]) + (acc[ct][2] + acc[ct][3]);
}

// h = x A_a^T of one item (<= 32 rows of one adapter).  rows: item element ->
// token row (forward) / the training rows (REC: the backward's h again, the same
// sums).  Dropout on a training row's low-rank input.
template <int NCT, bool REC>
__device__ __forceinline__ void shrink_tile(const F32Args& g, TileLds<NCT>& L, int item) {
  const int32_t* it = (REC ? g.train_items : g.shrink_items) + (int64_t)item * kItemWords;
  const int a = it[0], begin = it[1], cnt = it[2], r = g.ranks[a];
  const int tr8 = threadIdx.x >> 3, k8 = 8 * (threadIdx.x & 7);
  const int e = begin + min(tr8, cnt - 1);
  const int t = REC ? g.train_rows[e] : g.shrink_rows[e];
  const int tr = REC ? e : g.row_train[t];
  const bool in = tr8 < cnt, drop = g.keep && tr >= 0;
  const float* x = g.X + (int64_t)t * g.ldx;
  const float* A = g.A + (int64_t)a * g.r_max * g.K;
  f32x4 acc[NCT];
  tile_mm<NCT>(
      L, (g.K + CK - 1) / CK,
      [&](int c) {
        const int k = c * CK + k8;
        V8 v = (in && k < g.K) ? ld8v(x + k) : zero8();
        if (drop && k < g.K) {  // 8 columns share a mask word
          const uint32_t m = g.keep[(int64_t)tr * g.keep_words + (k >> 5)] >> (k & 31);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            v.a[i] = (m >> i) & 1u ? v.a[i] : 0.f;
            v.b[i] = (m >> (i + 4)) & 1u ? v.b[i] : 0.f;
          }
        }
        return v;
      },
      [&](int c, int ct) {
        const int k = c * CK + k8, j = tr8 + MR * ct;
        return (j < r && k < g.K) ? ld8v(A + (int64_t)j * g.K + k) : zero8();
      },
      [](float (*s)[LS], const V8& v) { put_rows(s, v); }, [](float (*s)[LS], const V8& v) { put_rows(s, v); }, acc);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row = 16 * (wave & 1) + (lane & 15);
  if (row >= cnt) return;
  const int ro = REC ? begin + row : g.shrink_rows[begin + row];
  const int ro_tr = REC ? ro : g.row_train[ro];
  const bool scaled = g.keep && ro_tr >= 0;
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int j = 16 * (wave >> 1) + 32 * ct + 4 * (lane >> 4) + v;
      if (j >= r) continue;
      const float h = scaled ? acc[ct][v] * g.drop_scale : acc[ct][v];
      if (REC) {
        g.Hrec[(int64_t)ro * g.r_max + j] = h;
      } else {
        g.Hall[(int64_t)ro * g.r_max + j] = h;
        if (ro_tr >= 0 && g.Hsave) g.Hsave[(int64_t)ro_tr * g.r_max + j] = h;
      }
    }
}

template <int NCT, bool REC>
__global__ __launch_bounds__(256) void f32_shrink(F32Args g) {
  __shared__ TileLds<NCT> L;
  shrink_tile<NCT, REC>(g, L, blockIdx.x);
}

// y = x W^T + s_a h B_a^T: 32 token rows x 32 columns.
__global__ __launch_bounds__(256) void f32_out(F32Args g) {
  __shared__ TileLds<1> L;
  const int n_nt = (g.N + 31) / 32;
  const int t0 = (int)(blockIdx.x / n_nt) * MR, n0 = (int)(blockIdx.x % n_nt) * 32;
  const int r8 = threadIdx.x >> 3, k8 = 8 * (threadIdx.x & 7);
  const float* x = g.X + (int64_t)min(t0 + r8, g.T - 1) * g.ldx;
  const float* w = g.W + (int64_t)min(n0 + r8, g.N - 1) * g.ldw;
  f32x4 acc[1];
  tile_mm<1>(
      L, (g.K + CK - 1) / CK, [&](int c) { return c * CK + k8 < g.K ? ld8v(x + c * CK + k8) : zero8(); },
      [&](int c, int) { return c * CK + k8 < g.K ? ld8v(w + c * CK + k8) : zero8(); },
      [](float (*s)[LS], const V8& v) { put_rows(s, v); }, [](float (*s)[LS], const V8& v) { put_rows(s, v); }, acc);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int t = t0 + 16 * (wave & 1) + (lane & 15), n = n0 + 16 * (wave >> 1) + 4 * (lane >> 4);
  if (t >= g.T || n >= g.N) return;
  const int a = g.row_adapter[t], r = g.ranks[a];
  const float* h = g.Hall + (int64_t)t * g.r_max;
  const float* b = g.B + ((int64_t)a * g.N + n) * g.r_max;
  f32x4 low = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int j = 0; j < r; ++j) {
    const float hj = h[j];
#pragma unroll
    for (int v = 0; v < 4; ++v) low[v] = fmaf(hj, b[(int64_t)v * g.r_max + j], low[v]);
  }
  f32x4 y;
  const float s = g.scales[a];
#pragma unroll
  for (int v = 0; v < 4; ++v) y[v] = fmaf(s, low[v], acc[0][v]);
  *reinterpret_cast<f32x4*>(g.Y + (int64_t)t * g.ldy + n) = y;
}

// g = s_a dy B_a of one item (<= 16 compact training rows of one adapter).
template <int NCT>
__device__ __forceinline__ void gmat_tile(const F32Args& g, TileLds<NCT>& L, int item) {
  const int32_t* it = g.train_items + (int64_t)item * kItemWords;
  const int a = it[0], begin = it[1], cnt = it[2], r = g.ranks[a];
  const int r8 = threadIdx.x >> 3, k8 = 8 * (threadIdx.x & 7);
  const int i4 = threadIdx.x >> 2, m8 = 8 * (threadIdx.x & 3);
  const bool vec = (g.r_max & 3) == 0;
  const float* dy = g.dY + (int64_t)(begin + min(r8, cnt - 1)) * g.lddy;
  const float* B = g.B + (int64_t)a * g.N * g.r_max;
  f32x4 acc[NCT];
  tile_mm<NCT>(
      L, (g.N + CK - 1) / CK,
      [&](int c) { return (r8 < cnt && c * CK + k8 < g.N) ? ld8v(dy + c * CK + k8) : zero8(); },
      [&](int c, int ct) {
        const int n = c * CK + i4, j = m8 + 32 * ct, nv = n < g.N ? min(8, r - j) : 0;
        const float* p = B + (int64_t)n * g.r_max + j;
        return nv >= 8 && vec ? ld8v(p) : ld8s(p, nv);
      },
      [](float (*s)[LS], const V8& v) { put_rows(s, v); }, [](float (*s)[LS], const V8& v) { put_cols(s, v); }, acc);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row = 16 * (wave & 1) + (lane & 15);
  if (row >= cnt) return;
  const float s = g.scales[a];
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int j = 16 * (wave >> 1) + 32 * ct + 4 * (lane >> 4) + v;
      if (j < r) g.G[(int64_t)(begin + row) * g.r_max + j] = s * acc[ct][v];
    }
}

// Sums over an adapter's training rows in compact order, 64 of them per step: rows of one
// chunk (a run of up to 256 rows) while it has that many left, else of up to 64 chunks, one
// to a lane, packed by a prefix sum of their lengths.  (719 rows alternating between two
// adapters, K = 136, N = 64, rank 33: the backward takes 38 us; 1147 with a step per chunk.)
struct TokenSteps {
  const F32Args& g;
  int p, end, off = 0, n;  // the next chunk of the list, its rows taken already; steps
  int i = 0;               // compact row of this thread's entry (thread / 4) of the current step ...
  bool in = false;         // ... if it has one
  __device__ const int32_t* chunk(int q) const { return g.chunks + (int64_t)g.tad_chunks[q] * kItemWords; }
  __device__ TokenSteps(const F32Args& g_, int slot) : g(g_), p(g_.tad_ptr[slot]), end(g_.tad_ptr[slot + 1]) {
    int rows = 0;
    if (end - p <= 8) {
      for (int q = p; q < end; ++q) rows += chunk(q)[2];
    } else {
      for (int q = p + (int)(threadIdx.x & 63); q < end; q += 64) rows += chunk(q)[2];
#pragma unroll
      for (int d = 32; d > 0; d >>= 1) rows += __shfl_xor(rows, d);
      rows = __builtin_amdgcn_readfirstlane(rows);
    }
    n = (rows + CK - 1) / CK;
  }
  __device__ void next() {  // called n times, by every thread of the workgroup
    const int slot = threadIdx.x >> 2, lane = threadIdx.x & 63;
    const int32_t* ck = chunk(p);
    const int left = ck[2] - off;
    if (left >= CK || p + 1 == end) {
      in = slot < left;
      i = ck[1] + off + slot;
      off = left > CK ? off + CK : 0;
      p += left > CK ? 0 : 1;
      return;
    }
    int begin = 0, sum = 0;
    if (p + lane < end) {
      const int32_t* c = chunk(p + lane);
      const int taken = lane == 0 ? off : 0;
      begin = c[1] + taken;
      sum = min(c[2] - taken, CK + 1);
    }
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int v = __shfl_up(sum, d);
      sum += lane >= d ? v : 0;
    }
    int l = 0;  // the chunk of this thread's row: the first whose sum exceeds it
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) l += __shfl(sum, l + d - 1) <= slot ? d : 0;
    const int before = __shfl(sum, max(l - 1, 0));
    in = slot < __shfl(sum, 63);
    i = __shfl(begin, l) + slot - (l > 0 ? before : 0);
    // chunks used up (the first at least), and the rows of the next one taken
    const int used = __popcll(__ballot(p + lane < end && sum <= CK));
    p += used;
    off = p < end && used < 64 ? CK - __builtin_amdgcn_readlane(sum, used - 1) : 0;
  }
};

// Rank operand of a token sum: 8 ranks of compact row `i` of M ([T_t][r_max]).
__device__ __forceinline__ V8 rank8(const float* M, int r_max, int i, int j, int r, bool in) {
  const int nv = in ? min(8, r - j) : 0;
  const float* p = M + (int64_t)i * r_max + j;
  return nv >= 8 && (r_max & 3) == 0 ? ld8v(p) : ld8s(p, nv);
}

// dB[a][n][j] (+)= s_a sum_i dy[i][n] H_save[i][j]: 32 columns n of one training adapter.
template <int NCT>
__device__ __forceinline__ void db_tile(const F32Args& g, TileLds<NCT>& L, int nb, int slot) {
  const int a = g.train_ads[slot], r = g.ranks[a], n0 = nb * MR;
  const int m8 = 8 * (threadIdx.x & 3);
  TokenSteps ts(g, slot);
  f32x4 acc[NCT];
  tile_mm<NCT>(
      L, ts.n,
      [&](int) {  // steps are loaded in order, this operand first
        ts.next();
        return (ts.in && n0 + m8 < g.N) ? ld8v(g.dY + (int64_t)ts.i * g.lddy + n0 + m8) : zero8();
      },
      [&](int, int ct) { return rank8(g.Hs, g.r_max, ts.i, m8 + 32 * ct, r, ts.in); },
      [](float (*s)[LS], const V8& v) { put_cols(s, v); }, [](float (*s)[LS], const V8& v) { put_cols(s, v); }, acc);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n = n0 + 16 * (wave & 1) + (lane & 15);
  if (n >= g.N) return;
  const float s = g.scales[a];
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int j = 16 * (wave >> 1) + 32 * ct + 4 * (lane >> 4) + v;
      if (j >= r) continue;
      float* o = g.dB + ((int64_t)a * g.N + n) * g.r_max + j;
      const float x = s * acc[ct][v];
      *o = g.accumulate ? *o + x : x;
    }
}

// dA[a][j][k] (+)= sum_i g[i][j] x[t_i][k] (x through the dropout mask): 32 columns k.
template <int NCT>
__device__ __forceinline__ void da_tile(const F32Args& g, TileLds<NCT>& L, int kb, int slot) {
  const int a = g.train_ads[slot], r = g.ranks[a], k0 = kb * MR;
  const int m8 = 8 * (threadIdx.x & 3);
  TokenSteps ts(g, slot);
  f32x4 acc[NCT];
  tile_mm<NCT>(
      L, ts.n,
      [&](int) {
        ts.next();
        const int i = ts.i, k = k0 + m8;
        if (!ts.in || k >= g.K) return zero8();
        V8 v = ld8v(g.X + (int64_t)g.train_rows[i] * g.ldx + k);
        if (g.keep) {
          const uint32_t m = g.keep[(int64_t)i * g.keep_words + (k >> 5)] >> (k & 31);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            v.a[e] = (m >> e) & 1u ? v.a[e] : 0.f;
            v.b[e] = (m >> (e + 4)) & 1u ? v.b[e] : 0.f;
          }
        }
        return v;
      },
      [&](int, int ct) { return rank8(g.G, g.r_max, ts.i, m8 + 32 * ct, r, ts.in); },
      [](float (*s)[LS], const V8& v) { put_cols(s, v); }, [](float (*s)[LS], const V8& v) { put_cols(s, v); }, acc);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int k = k0 + 16 * (wave & 1) + (lane & 15);
  if (k >= g.K) return;
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int j = 16 * (wave >> 1) + 32 * ct + 4 * (lane >> 4) + v;
      if (j >= r) continue;
      float* o = g.dA + ((int64_t)a * g.r_max + j) * g.K + k;
      const float x = g.keep ? acc[ct][v] * g.drop_scale : acc[ct][v];
      *o = g.accumulate ? *o + x : x;
    }
}

// dx = dy W + g A_a: 32 compact training rows x 32 columns.
__device__ __forceinline__ void dx_tile(const F32Args& g, TileLds<1>& L, int b) {
  const int n_kt = (g.K + 31) / 32;
  const int i0 = (b / n_kt) * MR, k0 = (b % n_kt) * 32;
  const int r8 = threadIdx.x >> 3, k8 = 8 * (threadIdx.x & 7);
  const int i4 = threadIdx.x >> 2, m8 = 8 * (threadIdx.x & 3);
  const float* dy = g.dY + (int64_t)min(i0 + r8, g.Tt - 1) * g.lddy;
  f32x4 acc[1];
  tile_mm<1>(
      L, (g.N + CK - 1) / CK, [&](int c) { return c * CK + k8 < g.N ? ld8v(dy + c * CK + k8) : zero8(); },
      [&](int c, int) {
        const int n = c * CK + i4;
        return (n < g.N && k0 + m8 < g.K) ? ld8v(g.W + (int64_t)n * g.ldw + k0 + m8) : zero8();
      },
      [](float (*s)[LS], const V8& v) { put_rows(s, v); }, [](float (*s)[LS], const V8& v) { put_cols(s, v); }, acc);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i = i0 + 16 * (wave & 1) + (lane & 15), k = k0 + 16 * (wave >> 1) + 4 * (lane >> 4);
  if (i >= g.Tt || k >= g.K) return;
  const int a = g.train_adapter[i], r = g.ranks[a];
  const float* gi = g.G + (int64_t)i * g.r_max;
  const float* Aa = g.A + (int64_t)a * g.r_max * g.K + k;
  f32x4 low = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int j = 0; j < r; ++j) {
    const f32x4 aj = *reinterpret_cast<const f32x4*>(Aa + (int64_t)j * g.K);
    const float gj = gi[j];
#pragma unroll
    for (int v = 0; v < 4; ++v) low[v] = fmaf(gj, aj[v], low[v]);
  }
  if (g.keep) {  // through the dropout mask
#pragma unroll
    for (int v = 0; v < 4; ++v) low[v] = kept(g, i, k + v) ? low[v] * g.drop_scale : 0.f;
  }
  *reinterpret_cast<f32x4*>(g.dX + (int64_t)i * g.lddx + k) = acc[0] + low;
}

// g (the first n_titems workgroups) and dB, which need nothing of each other.
template <int NCT>
__global__ __launch_bounds__(256) void f32_g_db(F32Args g) {
  __shared__ TileLds<NCT> L;
  const int b = blockIdx.x, nb = (g.N + MR - 1) / MR;
  if (b < g.n_titems) gmat_tile<NCT>(g, L, b);
  else db_tile<NCT>(g, L, (b - g.n_titems) % nb, (b - g.n_titems) / nb);
}

// dA (the first n_tads ceil(K / 32) workgroups) and dX, which need g only.
template <int NCT>
__global__ __launch_bounds__(256) void f32_da_dx(F32Args g) {
  __shared__ union {
    TileLds<NCT> a;
    TileLds<1> x;
  } L;
  const int b = blockIdx.x, nb = (g.K + MR - 1) / MR, n_da = nb * g.n_tads;
  if (b < n_da) da_tile<NCT>(g, L.a, b % nb, b / nb);
  else dx_tile(g, L.x, b - n_da);
}

}  // namespace

hipError_t launch_f32_fwd(const F32Args& a, hipStream_t s) {
  if (a.T <= 0) return hipSuccess;
  if (a.r_used < 1 || a.r_used > 64 || a.n_shrink < 1) return hipErrorInvalidValue;
  if (a.r_used <= 32) hipLaunchKernelGGL((f32_shrink<1, false>), dim3(a.n_shrink), dim3(256), 0, s, a);
  else hipLaunchKernelGGL((f32_shrink<2, false>), dim3(a.n_shrink), dim3(256), 0, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int64_t tiles = (int64_t)((a.T + MR - 1) / MR) * ((a.N + 31) / 32);
  if (tiles > INT32_MAX) return hipErrorInvalidValue;
  hipLaunchKernelGGL(f32_out, dim3((unsigned)tiles), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_f32_bwd(const F32Args& a0, hipStream_t s) {
  if (a0.Tt <= 0) return hipSuccess;
  F32Args a = a0;
  if (a.r_train < 1 || a.r_train > 64 || a.n_titems < 1 || a.n_tads < 1) return hipErrorInvalidValue;
  const bool wide = a.r_train > 32;
  hipError_t e;
  if (!a.Hs) {
    if (wide) hipLaunchKernelGGL((f32_shrink<2, true>), dim3(a.n_titems), dim3(256), 0, s, a);
    else hipLaunchKernelGGL((f32_shrink<1, true>), dim3(a.n_titems), dim3(256), 0, s, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    a.Hs = a.Hrec;
  }
  const int64_t n1 = a.n_titems + (int64_t)((a.N + MR - 1) / MR) * a.n_tads;
  const int64_t n2 = (int64_t)((a.K + MR - 1) / MR) * a.n_tads +
                     (a.dX ? (int64_t)((a.Tt + MR - 1) / MR) * ((a.K + 31) / 32) : 0);
  if (n1 > INT32_MAX || n2 > INT32_MAX) return hipErrorInvalidValue;
  if (wide) hipLaunchKernelGGL((f32_g_db<2>), dim3((unsigned)n1), dim3(256), 0, s, a);
  else hipLaunchKernelGGL((f32_g_db<1>), dim3((unsigned)n1), dim3(256), 0, s, a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (wide) hipLaunchKernelGGL((f32_da_dx<2>), dim3((unsigned)n2), dim3(256), 0, s, a);
  else hipLaunchKernelGGL((f32_da_dx<1>), dim3((unsigned)n2), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace dsv
