// gemm_part.hip -- CDNA4 (gfx950) GEMMs of batches whose 256 x 256 tiles leave
// most of the chip idle (decode steps, prefill chunks, the backward of a few
// hundred training rows): the contraction is cut into pieces, so that small
// batches still run on every CU, and a second kernel sums the pieces.
//
//   part_gemm    fp32 partial products of P Q^T (or P Q) over one piece of the
//                contraction each; no low-rank work, so it does not wait for h or g.
//   part_finish  per (rows of one adapter, 256 columns): the pieces summed in
//                order, plus the adapter's low-rank term on the matrix cores,
//                one rounding to bf16.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "device_common.h"
#include "kernels.h"
#include "plan.h"

namespace dsv {
namespace {

extern "C" __device__ void llvm_amdgcn_raw_buffer_load_lds_p(i32x4 rsrc, lds_u32* lds, int size, int voffset,
                                                             int soffset, int offset,
                                                             int aux) __asm("llvm.amdgcn.raw.buffer.load.lds");

// Buffer descriptor over `bytes` bytes from base (reads past them return zeros).
__device__ __forceinline__ i32x4 part_rsrc(const void* base, int64_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(base);
  const int64_t rg = bytes < 0 ? 0 : (bytes > 0x7FFFFFF0ll ? 0x7FFFFFF0ll : bytes);
  i32x4 r;
  r.x = __builtin_amdgcn_readfirstlane((int)(uint32_t)a);
  r.y = __builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32));
  r.z = __builtin_amdgcn_readfirstlane((int)rg);
  r.w = 0x00020000;
  return r;
}

template <int V>
struct stage_c {  // a compile-time number passed as a value
  static constexpr int value = V;
};

// ---------------------------------------------------------------------------
// Shrink of one item (<= 32 rows of one adapter) over one piece of the
// contraction, in the workgroups behind the pieces of the base product: it
// needs X and A only, so it hides behind the stream of W instead of being a
// launch (and a second one for its own pieces) before it.  They are dispatched
// last: the tiles seldom fill the last CUs (365 rows, K = N = 4096: 26.8 us with
// the shrink first, 22.6 last, 22.4 without any, and 10 us for the two launches).  Fragments go from
// global memory straight into registers, U chunks of 256 columns at a time; the
// sums are skinny_kernel's to the bit (columns [32w, 32w + 32) of every chunk in
// one accumulator, w = 0 .. 7, added in order), so the backward's recomputed h
// and this one agree.  red: LDS for one 16 x 16 tile of 8 partials.
// ---------------------------------------------------------------------------
constexpr int kRedBytes = 8 * 16 * 17 * 4;

template <int NW, int NJ>
__device__ __forceinline__ void shrink_piece(const PartShrink& g, const PartGroup& G, int item, int piece, char* red_) {
  constexpr int SL = 8 / NW;  // 32-column slices per wave
  constexpr int U = NJ == 4 ? 2 : 4;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l15 = lane & 15, g4 = lane >> 4;
  const int32_t* it = G.items + (int64_t)item * kItemWords;
  const int a = it[0], begin = it[1], cnt = it[2], r = G.ranks[a];
  const int nch = (g.C + 255) / 256;
  const int c0 = piece * g.cpp, c1 = min(nch, c0 + g.cpp);
  const uint16_t* x[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) x[t] = g.X + (int64_t)G.rows[begin + min(16 * t + l15, cnt - 1)] * g.ldx;
  const uint16_t* q[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) q[j] = g.A + ((int64_t)a * G.r_max + min(16 * j + l15, r - 1)) * g.C;
  const bool two = cnt > 16;
  f32x4 acc[SL][2][NJ];
#pragma unroll
  for (int s = 0; s < SL; ++s)
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int j = 0; j < NJ; ++j) acc[s][t][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < SL; ++s) {
    const int w = wave + NW * s;
    for (int c = c0; c < c1; c += U) {
      u32x4 xv[U][2], qv[U][NJ];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        // chunks past the piece and columns past C read column 0 and count as zeros
        const int k = (c + u) * 256 + 32 * w + 8 * g4;
        const int kc = (c + u < c1 && k < g.C) ? k : 0;
        xv[u][0] = ld16(x[0] + kc);
        if (two) xv[u][1] = ld16(x[1] + kc);
#pragma unroll
        for (int j = 0; j < NJ; ++j) qv[u][j] = ld16(q[j] + kc);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (c + u >= c1) break;
        const bool in = (c + u) * 256 + 32 * w + 8 * g4 < g.C;
#pragma unroll
        for (int j = 0; j < NJ; ++j) qv[u][j] = in ? qv[u][j] : zero4();
        xv[u][0] = in ? xv[u][0] : zero4();
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          acc[s][0][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf(xv[u][0]), as_bf(qv[u][j]), acc[s][0][j], 0, 0, 0);
        if (two) {
          xv[u][1] = in ? xv[u][1] : zero4();
#pragma unroll
          for (int j = 0; j < NJ; ++j)
            acc[s][1][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf(xv[u][1]), as_bf(qv[u][j]), acc[s][1][j], 0, 0, 0);
        }
      }
    }
  }
  float* red = reinterpret_cast<float*>(red_);  // [8][16][17]
  float* part = g.part + (int64_t)piece * G.T * G.r_max;
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    if (16 * t >= cnt) break;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      if (16 * j >= r) break;
#pragma unroll
      for (int s = 0; s < SL; ++s)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[((wave + NW * s) * 16 + 4 * g4 + v) * 17 + l15] = acc[s][t][j][v];
      __syncthreads();
      if (tid < 256) {
        const int row = tid >> 4, jj = tid & 15;
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < 8; ++w) sum += red[(w * 16 + row) * 17 + jj];
        if (16 * t + row < cnt && 16 * j + jj < r)
          part[(int64_t)(begin + 16 * t + row) * G.r_max + 16 * j + jj] = sum;
      }
      __syncthreads();
    }
  }
}

// ---------------------------------------------------------------------------
// One workgroup: a TM x TN tile over K-steps [kb, ke) of 64, 4 waves in a
// WGM x WGN grid, v_mfma_f32_16x16x32_bf16.  Operand tiles go from global
// memory straight into LDS, NS buffers deep: NS - 1 K-steps are in flight
// while one is multiplied, one barrier per K-step.  Every K-step issues the
// same number of loads (past the piece they read nothing and write zeros), so
// the wait at its top is a constant count.  The buffers are separate arrays
// picked by a compile-time number: a read of one then never waits for the
// direct loads into the others.
//   LDS image, contraction-contiguous tiles (128-byte rows): 16-byte chunk c
//   of row r in slot c ^ (r ^ r/8) % 8; NN weight tile ([64][TN]): chunk c of
//   row n in slot c ^ 2(n % 4), read back with ds_read_b64_tr_b16.
// Decode is bound by the stream of W: the tiles keep about 12 MB of it in flight
// over the chip (T = 64, 4096 x 28672: 41 us, 5.7 TB/s; with 256 x 256 tiles 101).
// A few hundred rows are bound by the latency of a K-step, hence the buffers: a
// 128 x 128 workgroup takes 0.98 us per K-step with two, 0.41 with four (365 rows,
// 4096 x 4096: 22 us, before 45); 128 x 256 reads a quarter less per product.
// Accumulators: weight fragment first, so acc[i][j][v] is output row
// 16i + lane%16, column 16j + 4(lane/16) + v of the wave's part.
// ---------------------------------------------------------------------------
// NJ: 16-rank tiles of the shrink beside the pieces (0: no shrink in the launch).
template <bool NN, int NJ, int TM, int TN, int WGM, int WGN, int NS>
__global__ __launch_bounds__(64 * WGM * WGN) __attribute__((amdgpu_waves_per_eu(2))) void part_gemm_kernel(PartGroup G) {
  constexpr int TK = 64, NW = WGM * WGN;
  constexpr int WM = TM / WGM, WN = TN / WGN, FM = WM / 16, FN = WN / 16;
  constexpr int A_BYTES = TM * TK * 2, B_BYTES = TN * TK * 2, STAGE = A_BYTES + B_BYTES;
  constexpr int LA = A_BYTES / 1024 / NW, LB = B_BYTES / 1024 / NW, L = LA + LB;
  static_assert(LA * 1024 * NW == A_BYTES && LB * 1024 * NW == B_BYTES, "loads per wave");
  static_assert(NS >= 2 && NS <= 4, "stages");
  __shared__ __attribute__((aligned(1024))) char st0[STAGE];
  __shared__ __attribute__((aligned(1024))) char st1[STAGE];
  __shared__ __attribute__((aligned(1024))) char st2[NS > 2 ? STAGE : 16];
  __shared__ __attribute__((aligned(1024))) char st3[NS > 3 ? STAGE : 16];
  auto buf = [&](auto sel) -> char* {
    constexpr int b = decltype(sel)::value;
    if constexpr (b == 0) return st0;
    else if constexpr (b == 1) return st1;
    else if constexpr (b == 2) return st2;
    else return st3;
  };
  int bx = blockIdx.x;
  if constexpr (NJ > 0) {
    static_assert(STAGE >= kRedBytes, "the shrink's sums fit one buffer");
    const int sx = bx - G.off[G.n];
    if (sx >= 0) {
      int p = 0;
#pragma unroll
      for (int i = 1; i < kMaxGroup; ++i) p += (i < G.n && sx >= G.sh_off[i]) ? 1 : 0;
      const int local = sx - G.sh_off[p];
      shrink_piece<NW, NJ>(G.sh[p], G, local % G.n_items, local / G.n_items, st0);
      return;
    }
  }
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WGN, wn = wave % WGN;
  const int l15 = lane & 15, g4 = lane >> 4;

  // workgroup -> (projection, piece, column tile, row tile): the row tiles of
  // one weight tile are neighbours on one XCD, then the columns, then the pieces
  int pj = 0;
#pragma unroll
  for (int p = 1; p < kMaxGroup; ++p) pj += (p < G.n && bx >= G.off[p]) ? 1 : 0;
  const PartArgs g = G.a[pj];
  const int nwg = G.off[pj + 1] - G.off[pj];
  const int bid = bx - G.off[pj];
  const int per = nwg >> 3, rem = nwg & 7, xcd = bid & 7;
  const int lin = xcd * per + min(xcd, rem) + (bid >> 3);
  const int mt = lin % g.n_m, rest = lin / g.n_m;
  const int nt = rest % g.n_n, piece = rest / g.n_n;
  const int nk = (g.C + TK - 1) / TK;
  const int kb = (int)(((int64_t)piece * nk) / g.split), ke = (int)(((int64_t)(piece + 1) * nk) / g.split);
  const int m0 = mt * TM, n0 = nt * TN;
  const int kend = min(g.C, ke * TK);  // the piece's contraction range ends here

  const int64_t a_rows = min(TM, g.M - m0), b_cols = min(TN, g.Nout - n0);
  const i32x4 ra = part_rsrc(g.P + (int64_t)m0 * g.ldp, ((a_rows - 1) * g.ldp + g.C) * 2);
  const uint16_t* b_base = NN ? g.Q + n0 : g.Q + (int64_t)n0 * g.ldq;

  // Lane offsets of the loads: load q = wave * LA + i fills LDS rows 8q .. 8q+7,
  // lane ln taking row 8q + ln/8, slot ln%8.  Offsets stay within 2^29
  // bytes (at most 256 rows of 2^20 elements), so the out-of-range value exceeds them all.
  const int lr = lane >> 3;
  int off_la[LA], ch_a[LA], off_lb[LB], ch_b[LB];
#pragma unroll
  for (int i = 0; i < LA; ++i) {
    const int row = 8 * (wave * LA + i) + lr;
    ch_a[i] = 8 * ((lane & 7) ^ ((row ^ (row >> 3)) & 7));
    off_la[i] = (row * (int)g.ldp + ch_a[i]) * 2;
  }
#pragma unroll
  for (int i = 0; i < LB; ++i) {
    const int q = wave * LB + i;
    if constexpr (!NN) {
      const int row = 8 * q + lr;
      ch_b[i] = 8 * ((lane & 7) ^ ((row ^ (row >> 3)) & 7));
      off_lb[i] = (row * (int)g.ldq + ch_b[i]) * 2;
    } else {
      const int byte = q * 1024 + 16 * lane;
      const int n = byte / (TN * 2), slot = (byte % (TN * 2)) / 16;
      ch_b[i] = n;
      off_lb[i] = (n * (int)g.ldq + 8 * (slot ^ (2 * (n & 3)))) * 2;
    }
  }
  const i32x4 rb_nt = part_rsrc(b_base, NN ? 0 : ((b_cols - 1) * g.ldq + g.C) * 2);
  // Neighbouring column tiles start one K-step apart (and wrap around): rows of
  // W are a power of two apart, so tiles in lockstep would all read the same few
  // memory channels (W of 4096 x 28672 at T = 64: 57.6 us in step, 49.1 us apart).
  const int nsteps = ke - kb, rot = nt % nsteps;
  auto issue = [&](int ki, char* st) {
    const int kt = ki >= ke ? ke : (ki + rot >= ke ? ki + rot - nsteps : ki + rot);
    const int k0 = kt * TK, kby = k0 * 2;
    const bool whole = k0 + TK <= kend;
    // NN: the descriptor moves with the K-step (weights may exceed 2^31 bytes)
    const i32x4 rb = NN ? part_rsrc(b_base + (int64_t)min(k0, g.C - 1) * g.ldq,
                                    k0 < kend ? ((int64_t)(min(TK, kend - k0) - 1) * g.ldq + g.Nout - n0) * 2 : 0)
                        : rb_nt;
#pragma unroll
    for (int i = 0; i < LA; ++i) {
      const int vo = (whole || k0 + ch_a[i] < kend) ? off_la[i] + kby : 0x7FFFFFF0;
      llvm_amdgcn_raw_buffer_load_lds_p(ra, (lds_u32*)(st + (wave * LA + i) * 1024), 16, vo, 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
      const int vo = NN ? ((whole || k0 + ch_b[i] < kend) ? off_lb[i] : 0x7FFFFFF0)
                        : ((whole || k0 + ch_b[i] < kend) ? off_lb[i] + kby : 0x7FFFFFF0);
      llvm_amdgcn_raw_buffer_load_lds_p(rb, (lds_u32*)(st + A_BYTES + (wave * LB + i) * 1024), 16, vo, 0, 0, 0);
    }
  };

  // Byte offsets of the fragment reads: 32-wide step s of the K-step, chunk 4s + lane/16.
  int fa[2][FM], fb[2][FN];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      const int row = wm * WM + 16 * i + l15;
      fa[s][i] = row * 128 + 16 * ((4 * s + g4) ^ ((row ^ (row >> 3)) & 7));
    }
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      if constexpr (!NN) {
        const int row = wn * WN + 16 * j + l15;
        fb[s][j] = A_BYTES + row * 128 + 16 * ((4 * s + g4) ^ ((row ^ (row >> 3)) & 7));
      } else {
        const int n = 32 * s + 8 * g4 + (l15 >> 2), c = wn * WN + 16 * j + 4 * (l15 & 3);
        fb[s][j] = A_BYTES + n * (TN * 2) + 16 * ((c >> 3) ^ (2 * (n & 3))) + 2 * (c & 7);
      }
    }
  }
  f32x4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  issue(kb, st0);
  if constexpr (NS > 2) issue(kb + 1, st1);
  if constexpr (NS > 3) issue(kb + 2, st2);

  auto step = [&](int kt, auto sel) {
    constexpr int b = decltype(sel)::value, bn = (b + NS - 1) % NS;
    __builtin_amdgcn_s_waitcnt(vmcnt_imm((NS - 2) * L));  // this wave's loads of kt are in
    // everyone's part of kt is in and everyone has read buffer bn (a plain
    // barrier: a fence would also wait for the loads in flight)
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    issue(kt + NS - 1, buf(stage_c<bn>{}));
    const char* st = buf(stage_c<b>{});
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      bf16x8 af[FM], bq[FN];
#pragma unroll
      for (int i = 0; i < FM; ++i) af[i] = as_bf(*reinterpret_cast<const u32x4*>(st + fa[s][i]));
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        if constexpr (!NN) {
          bq[j] = as_bf(*reinterpret_cast<const u32x4*>(st + fb[s][j]));
        } else {
          const s16x4 h0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(st + fb[s][j]));
          const s16x4 h1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(st + (fb[s][j] + 4 * (TN * 2))));
          typedef uint32_t u32x2p __attribute__((ext_vector_type(2)));
          const u32x2p a0 = __builtin_bit_cast(u32x2p, h0), a1 = __builtin_bit_cast(u32x2p, h1);
          bq[j] = as_bf(u32x4{a0[0], a0[1], a1[0], a1[1]});
        }
      }
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int i = 0; i < FM; ++i)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bq[j], af[i], acc[i][j], 0, 0, 0);
    }
  };
  // whole rounds of NS steps, then the rest: every path into a step has the
  // other buffers' loads issued after this buffer's
  int kt = kb;
  for (; kt + NS <= ke; kt += NS) {
    step(kt, stage_c<0>{});
    step(kt + 1, stage_c<1>{});
    if constexpr (NS > 2) step(kt + 2, stage_c<2>{});
    if constexpr (NS > 3) step(kt + 3, stage_c<3>{});
  }
  if (kt < ke) {
    step(kt, stage_c<0>{});
    if (NS > 2 && kt + 1 < ke) {
      step(kt + 1, stage_c<1>{});
      if constexpr (NS > 3)
        if (kt + 2 < ke) step(kt + 2, stage_c<2>{});
    }
  }
  vmem_wait_all();  // the loads past the piece are in before the LDS is released

  float* part = g.part + (int64_t)piece * g.M * g.Nout;
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    const int row = m0 + wm * WM + 16 * i + l15;
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int col = n0 + wn * WN + 16 * j + 4 * g4;
      if (row < g.M && col < g.Nout) *reinterpret_cast<f32x4*>(part + (int64_t)row * g.Nout + col) = acc[i][j];
    }
  }
}

// ---------------------------------------------------------------------------
// Sum of the pieces plus the low-rank term: one workgroup per (16 rows of one
// item, `iters` blocks of 256 columns), each wave 64 columns of a block.
//   forward: rows are token rows (rows[begin + i]), low = s_a h B_a^T; items of
//            up to 32 rows take two workgroups
//   BWD:     rows are compact training rows (begin + i), low = g A_a through
//            the dropout mask when there is one
// Few rows per item make this a stream of B (and of the pieces): the next
// block's operands load while the current one is finished.
// ---------------------------------------------------------------------------
// NR: 32-rank steps (every rank <= 32 NR); Q16: Q rows of 16-byte aligned rank
// octets; HP: h comes as pieces; PF: more than one block per workgroup.
template <bool BWD, int NR, bool Q16, bool HP, bool PF>
__global__ __launch_bounds__(256) void part_finish_kernel(FinishGroup G) {
  int pj = 0;
#pragma unroll
  for (int p = 1; p < kMaxGroup; ++p) pj += (p < G.n && (int)blockIdx.x >= G.yoff[p]) ? 1 : 0;
  const FinishArgs g = G.a[pj];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l15 = lane & 15, g4 = lane >> 4;
  const int32_t* it = G.items + (int64_t)(BWD ? blockIdx.y : blockIdx.y >> 1) * kItemWords;
  const int a = it[0], begin = it[1] + (BWD ? 0 : 16 * ((int)blockIdx.y & 1));
  const int cnt = it[2] - (begin - it[1]);
  if (cnt <= 0) return;
  const int nb0 = ((int)blockIdx.x - G.yoff[pj]) * 256 * g.iters + wave * 64;
  const int nb_end = min(g.Nout, nb0 + 256 * g.iters);
  if (nb0 >= nb_end) return;
  const int r = G.ranks[a];
  const float sc = G.scales ? G.scales[a] : 1.f;
  const int e = begin + min(l15, cnt - 1);
  const int pr = G.rows ? G.rows[e] : e;
  const int64_t ps = (int64_t)g.M * g.Nout;
  const float* src = g.part + (int64_t)pr * g.Nout;
  uint16_t* out = g.out + (int64_t)pr * g.ldo;
  // Ranks of the lane in each step: straight-line 16-byte loads from clamped
  // addresses, entries past the rank masked to zero (rows whose stride is not
  // a multiple of 8 entries are read entry by entry).
  int jc[NR], nv[NR];
  u32x4 mk[NR], lv[NR];
#pragma unroll
  for (int s = 0; s < NR; ++s) {
    const int jb = 32 * s + 8 * g4;
    nv[s] = max(0, min(8, r - jb));
    jc[s] = nv[s] > 0 ? jb : 0;
#pragma unroll
    for (int d = 0; d < 4; ++d)
      mk[s][d] = (2 * d < nv[s] ? 0x0000ffffu : 0u) | (2 * d + 1 < nv[s] ? 0xffff0000u : 0u);
    if constexpr (!HP) lv[s] = ld16(g.L + (int64_t)pr * g.ldl + jc[s]) & mk[s];  // rows padded to 8 entries
  }
  struct Set {
    u32x4 q[NR][4];
    f32x4 p0[4];
  };
  auto load_q = [&](int nb, Set& S) {
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) {
      const int n = min(nb + 16 * ct + l15, g.Nout - 1);
#pragma unroll
      for (int s = 0; s < NR; ++s) {
        if constexpr (BWD) {
          S.q[s][ct] = ld8_sel(g.Q + ((int64_t)a * G.r_max + jc[s]) * g.Nout + n, g.Nout, max(nv[s], 1));
        } else {
          const uint16_t* p = g.Q + ((int64_t)a * g.Nout + n) * G.r_max + jc[s];
          if constexpr (Q16) S.q[s][ct] = ld16(p);
          else S.q[s][ct] = ld8_sel(p, 1, max(nv[s], 1));
        }
      }
    }
  };
  auto load_p = [&](int nb, Set& S) {
#pragma unroll
    for (int ct = 0; ct < 4; ++ct)
      S.p0[ct] = *reinterpret_cast<const f32x4*>(src + min(nb + 16 * ct + 4 * g4, g.Nout - 4));
  };
  auto finish = [&](int nb, Set& S) {
    f32x4 acc[4];
    int col[4];
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) {
      acc[ct] = S.p0[ct];
      col[ct] = nb + 16 * ct + 4 * g4;
    }
    // the other pieces in order, PB in flight
    constexpr int PB = 4;
    for (int p = 1; p < g.split; p += PB) {
      f32x4 v[PB][4];
#pragma unroll
      for (int u = 0; u < PB; ++u)
#pragma unroll
        for (int ct = 0; ct < 4; ++ct)
          v[u][ct] = *reinterpret_cast<const f32x4*>(src + min(p + u, g.split - 1) * ps + min(col[ct], g.Nout - 4));
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < PB; ++u)
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) acc[ct] += p + u < g.split ? v[u][ct] : f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) {
      f32x4 low = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < NR; ++s)
        low = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf(S.q[s][ct] & mk[s]), as_bf(lv[s]), low, 0, 0, 0);
      if (BWD && g.keep != nullptr && col[ct] < g.Nout) {
        // the lane's 4 columns share one mask word
        const uint32_t mw = g.keep[(int64_t)pr * g.keep_words + (col[ct] >> 5)] >> (col[ct] & 31);
#pragma unroll
        for (int v = 0; v < 4; ++v) low[v] = ((mw >> v) & 1u) ? low[v] * g.keep_scale : 0.f;
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[ct][v] = fmaf(sc, low[v], acc[ct][v]);
      if (l15 < cnt && col[ct] < g.Nout)
        *reinterpret_cast<uint2*>(out + col[ct]) =
            make_uint2(f2bf2(acc[ct][0], acc[ct][1]), f2bf2(acc[ct][2], acc[ct][3]));
    }
  };
  auto load = [&](int nb, Set& S) {
    load_q(nb, S);
    load_p(nb, S);
  };
  Set s0, s1;
  load_q(nb0, s0);
  if constexpr (HP) {
    // the pieces of the lane's ranks, in piece order, rounded once
    const float* hp = g.h_part + (int64_t)e * G.r_max;
    const int64_t hs = (int64_t)g.M * G.r_max;
    float h[NR][8];
#pragma unroll
    for (int s = 0; s < NR; ++s)
#pragma unroll
      for (int u = 0; u < 8; ++u) h[s][u] = 0.f;
    for (int q = 0; q < g.h_pieces; q += 4) {
      f32x4 v[4][NR][2];
#pragma unroll
      for (int w = 0; w < 4; ++w)
#pragma unroll
        for (int s = 0; s < NR; ++s) {
          const float* p = hp + min(q + w, g.h_pieces - 1) * hs;
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            if constexpr (Q16) {  // entries past the rank are read and masked below
              v[w][s][u] = *reinterpret_cast<const f32x4*>(p + jc[s] + 4 * u);
            } else {
#pragma unroll
              for (int x = 0; x < 4; ++x) v[w][s][u][x] = p[min(jc[s] + 4 * u + x, r - 1)];
            }
          }
        }
      __builtin_amdgcn_sched_barrier(0);
      if (q == 0) load_p(nb0, s0);
#pragma unroll
      for (int w = 0; w < 4; ++w)
#pragma unroll
        for (int s = 0; s < NR; ++s)
#pragma unroll
          for (int u = 0; u < 8; ++u) h[s][u] += q + w < g.h_pieces ? v[w][s][u >> 2][u & 3] : 0.f;
    }
#pragma unroll
    for (int s = 0; s < NR; ++s) {
#pragma unroll
      for (int d = 0; d < 4; ++d) lv[s][d] = f2bf2(h[s][2 * d], h[s][2 * d + 1]) & mk[s][d];
      if (blockIdx.x == (unsigned)G.yoff[pj] && wave == 0 && g.h_save != nullptr && l15 < cnt) {
        const int tr = G.row_train[pr];
        if (tr >= 0)
#pragma unroll
          for (int u = 0; u < 8; ++u)
            if (u < nv[s]) g.h_save[(int64_t)tr * G.r_max + jc[s] + u] = (uint16_t)(lv[s][u >> 1] >> (16 * (u & 1)));
      }
    }
  } else {
    load_p(nb0, s0);
  }
  if constexpr (!PF) {
    finish(nb0, s0);
    return;
  }
  for (int nb = nb0; nb < nb_end; nb += 512) {
    if (nb + 256 < nb_end) load(nb + 256, s1);
    finish(nb, s0);
    if (nb + 256 >= nb_end) break;
    if (nb + 512 < nb_end) load(nb + 512, s0);
    finish(nb + 256, s1);
  }
}

template <bool NN, int NJ>
hipError_t launch_part(const PartGroup& g, int cfg, hipStream_t s, hipEvent_t start) {
  const dim3 grid((unsigned)(g.sh_off[g.n] + g.off[g.n])), block((unsigned)kPartCfg[cfg].threads);
  auto go = [&](auto kernel) {
    if (start) hipExtLaunchKernelGGL(kernel, grid, block, 0, s, start, nullptr, 0, g);
    else hipLaunchKernelGGL(kernel, grid, block, 0, s, g);
  };
  switch (cfg) {
    case 0: go(part_gemm_kernel<NN, NJ, 32, 64, 1, 4, 4>); break;
    case 1: go(part_gemm_kernel<NN, NJ, 64, 128, 2, 4, 4>); break;
    case 2: go(part_gemm_kernel<NN, NJ, 128, 128, 2, 4, 4>); break;
    case 3: go(part_gemm_kernel<NN, NJ, 128, 256, 2, 4, 3>); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_part_gemm(const PartGroup& g, int cfg, int32_t r_sel, bool nn, hipStream_t s) {
  if (g.n <= 0 || g.n > kMaxGroup || g.off[0] != 0 || cfg < 0 || cfg >= kPartCfgs) return hipErrorInvalidValue;
  const PartCfg& pc = kPartCfg[cfg];
  const bool shrink = g.sh_off[g.n] > 0;
  for (int p = 0; p < g.n; ++p) {
    const PartArgs& a = g.a[p];
    const int64_t nk = (a.C + 63) / 64;
    if (a.M < 1 || a.Nout < 8 || a.C < 8 || a.split < 1 || a.split > nk || !a.part) return hipErrorInvalidValue;
    if (a.n_m != (a.M + pc.tm - 1) / pc.tm || a.n_n != (a.Nout + pc.tn - 1) / pc.tn) return hipErrorInvalidValue;
    if ((int64_t)a.n_m * a.n_n * a.split != g.off[p + 1] - g.off[p]) return hipErrorInvalidValue;
    if (!shrink) continue;
    const PartShrink& h = g.sh[p];
    if (h.C != a.C || h.pieces < 1 || h.cpp < 1 || !h.part || g.sh_off[0] != 0 ||
        (int64_t)g.n_items * h.pieces != g.sh_off[p + 1] - g.sh_off[p])
      return hipErrorInvalidValue;
  }
  if (shrink && (nn || r_sel < 1 || r_sel > 64 || g.T != g.a[0].M)) return hipErrorInvalidValue;
  if ((int64_t)g.sh_off[g.n] + g.off[g.n] > INT32_MAX) return hipErrorInvalidValue;
  hipEvent_t start = take_launch_start();
  if (nn) return launch_part<true, 0>(g, cfg, s, start);
  if (!shrink) return launch_part<false, 0>(g, cfg, s, start);
  if (r_sel <= 16) return launch_part<false, 1>(g, cfg, s, start);
  if (r_sel <= 32) return launch_part<false, 2>(g, cfg, s, start);
  return launch_part<false, 4>(g, cfg, s, start);
}

hipError_t launch_part_finish(FinishGroup g, int32_t n_items, int32_t r_sel, bool bwd, hipStream_t s) {
  if (g.n <= 0 || g.n > kMaxGroup || n_items <= 0 || r_sel < 1 || r_sel > 64) return hipErrorInvalidValue;
  const int64_t xs = bwd ? n_items : 2 * (int64_t)n_items;
  if (xs > 65535) return hipErrorInvalidValue;
  int64_t blocks = 0;
  for (int p = 0; p < g.n; ++p) blocks += (g.a[p].Nout + 255) / 256;
  // Several blocks per workgroup once single ones would give every CU four
  // workgroups or more: the next block's operands then load during the current
  // one (B of 64 adapters at N = 2 x 14336, 147 MB: 49 us with one block per
  // workgroup, 40 with four).  With fewer workgroups one block each is faster, in
  // the form without a second register set (365 rows, N = 4096: 12 against 14 us).
  const int32_t iters = bwd ? 1 : (int32_t)std::max<int64_t>(1, std::min<int64_t>(4, n_items * blocks / 1024));
  g.yoff[0] = 0;
  for (int p = 0; p < g.n; ++p) {
    g.a[p].iters = iters;
    g.yoff[p + 1] = g.yoff[p] + ((g.a[p].Nout + 255) / 256 + iters - 1) / iters;
  }
  const dim3 grid((unsigned)g.yoff[g.n], (unsigned)xs);
  hipEvent_t e1 = take_launch_stop();
  auto go = [&](auto kernel) {
    if (e1) hipExtLaunchKernelGGL(kernel, grid, dim3(256), 0, s, nullptr, e1, 0, g);
    else hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, g);
  };
  const bool hp = !bwd && g.a[0].h_part != nullptr, q16 = (g.r_max & 7) == 0, wide = r_sel > 32;
  for (int p = 1; p < g.n; ++p)
    if ((g.a[p].h_part != nullptr) != hp) return hipErrorInvalidValue;
  const bool pf = iters > 1;
  auto fwd = [&](auto nr, auto q, auto h) {
    constexpr int NR = decltype(nr)::value;
    constexpr bool Q16 = decltype(q)::value != 0, HP = decltype(h)::value != 0;
    if (pf) go(part_finish_kernel<false, NR, Q16, HP, true>);
    else go(part_finish_kernel<false, NR, Q16, HP, false>);
  };
  auto fwd_h = [&](auto nr, auto q) {
    if (hp) fwd(nr, q, stage_c<1>{});
    else fwd(nr, q, stage_c<0>{});
  };
  if (bwd && wide) go(part_finish_kernel<true, 2, false, false, false>);
  else if (bwd) go(part_finish_kernel<true, 1, false, false, false>);
  else if (wide && q16) fwd_h(stage_c<2>{}, stage_c<1>{});
  else if (wide) fwd_h(stage_c<2>{}, stage_c<0>{});
  else if (q16) fwd_h(stage_c<1>{}, stage_c<1>{});
  else fwd_h(stage_c<1>{}, stage_c<0>{});
  return hipGetLastError();
}

}  // namespace dsv
