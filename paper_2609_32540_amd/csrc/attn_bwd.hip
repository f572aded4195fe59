// Backward pass of the packed block-causal attention (bf16 in and out, float32
// accumulation), the gradient of the packed training forward through its KV
// edges.  With c = scale * log2(e) and the forward's base-2 log-sum-exp L_i:
//   P_ij  = 2^(c q_i.k_j - L_i)                 (visible pairs only)
//   D_i   = dO_i . O_i
//   dV_j  = sum_i P_ij dO_i
//   dS_ij = P_ij (dO_i . v_j - D_i)
//   dQ_i  = scale sum_j dS_ij k_j
//   dK_j  = scale sum_i dS_ij q_i
// Three launches: D; dQ (query-stationary: a workgroup holds 256 queries of
// one chunk and head and streams the 64-key tiles of their read set, like the
// forward); dK and dV together (key-stationary: a workgroup holds 256 keys of
// one chunk or anchor frame and head and streams the query tiles of every
// chunk that sees them).  Every output element is written by exactly one
// workgroup: no atomics.  Launches too small to fill the GPU with these run the
// kernels of attn_bwd_split.hip (choose_split).
//
// Both kernels are bound by the matrix cores and the power they draw.  Products
// on v_mfma_f32_16x16x32_bf16 (the bf16 shape with the least register traffic
// per FLOP) with the forward's operand layouts: the stationary side sits in
// registers as the B operand (V of the dK/dV kernel, where they run out, in
// LDS), tiles of the streamed side are copied HBM -> LDS (global_load_lds) into
// a ring of five slots and read as the A operand by rows (16 bytes) or
// transposed (ds_read_b64_tr_b16); P and dS go from the accumulators to the B
// operand of the next product as bf16 (nearest even).  Against the 32x32x16
// kernels before them, at 12 heads x 128, 27 chunks of 4680 tokens (one box,
// whole training step 86.2 ms -> 77.9 ms): dQ with dO in LDS, products and VALU
// work in sequence 28.8 ms -> 25.2 ms; dK and dV 38.5 ms -> 34.0 ms.  Of the step's
// time, reading dK/dV's operands one region ahead saves 1.6 ms, waves without rows
// skipping the products of a ragged last tile 1.2 ms.

#include <hip/hip_runtime.h>

#include <math.h>

#include <cstring>
#include <utility>

#include "attn_tile.h"
#include "ff_internal.h"

namespace ff {
namespace {

constexpr int kWaves = 8;
constexpr int kThreads = 64 * kWaves;
constexpr int kBlockN = 32 * kWaves;   // stationary columns (queries or keys) per workgroup
constexpr int kBT = 64;                // streamed rows per tile (32 in the dK/dV kernel at d = 128)
constexpr int kXcds = 8;
constexpr int kMaxRuns = 2 * FF_MAX_ANCHOR_FRAMES + 1;   // segments of one streamed set

template <int D, int kRows>
struct Tile {
  static constexpr int KS = D / 32;                // 32-wide d slices
  static constexpr int DT = D / 16;                // 16-row d tiles of a gradient
  static constexpr int ROWB = 2 * D;
  static constexpr int TILE = kRows * ROWB;
  static constexpr int SLOT = 2 * TILE;            // the tiles of the two streamed tensors
  // Waves w and w + 4 share a SIMD and the older one (w < 4) is favoured by the
  // issue arbiter: waves 0-3 make the tile copies.
  static constexpr int kCopyWaves = kWaves / 2;
  static constexpr int N = TILE / 1024 / kCopyWaves;   // 1 KB copies per copying wave and tensor
  static constexpr int VGB = D / 64;               // 1 KB blocks per 8-row group
};

// Streamed tiles are read by rows and transposed: a tile is d-blocked per 8 rows
// (one 256-byte line per 16-wide d tile holds its 8 rows x 32 bytes), with the
// two 16-byte chunks of a line's rows swapped in odd 8-row groups; then a
// quarter-wave's row read (16 rows, one chunk) and a half-wave's transposing
// read (8 rows, both chunks) each touch every bank once, and d slices, d tiles
// and 16-row halves are immediate offsets.

// Copy of a tile of each tensor into LDS by waves 0 .. kCopyWaves-1: 1 KB copies
// of 16 bytes per lane, lane l at 16 l.  Block (G, H) = the lines of d tiles 4 H ..
// 4 H + 3 of 8-row group G: lane l carries row 8 G + (l % 16) / 2, chunk 8 H +
// 2 (l / 16) + (l % 2 ^ G % 2).  Rows past `last` re-read it.
template <int D, int kRows>
__device__ __attribute__((always_inline)) inline void copy_tiles(char* dst, uint64_t a, uint64_t b,
                                                                 uint32_t row_bytes, int last,
                                                                 int wave, int lane) {
  using C = Tile<D, kRows>;
  constexpr uint32_t kSpan = 1024u * (C::N - 1);
  int ln = lane;   // (keeps the per-lane offsets out of loop-invariant registers)
  asm volatile("" : "+v"(ln));
  uint32_t off[C::N];
#pragma unroll
  for (int i = 0; i < C::N; ++i) {
    const int blk = wave * C::N + i;
    const int G = blk / C::VGB;
    const int r = 8 * G + ((ln & 15) >> 1);
    const int ch = 8 * (blk % C::VGB) + 2 * (ln >> 4) + ((ln ^ G) & 1);
    off[i] = uint32_t(min(r, last)) * row_bytes + (16u * ch + kSpan - 1024u * i);
  }
  const uint32_t d = uint32_t(size_t(LDS_PTR(char, dst))) + wave * C::N * 1024;
  lds_copy_blocks<C::N>(d, reinterpret_cast<const char*>(a - kSpan), off);
  lds_copy_blocks<C::N>(d + C::TILE, reinterpret_cast<const char*>(b - kSpan), off);
}

// 4 bytes per lane from src (a lane's own address) into LDS at dst + 4 lane
__device__ inline void lds_copy_dwords(uint32_t dst, uint64_t src) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off"
               :: "s"(dst), "v"(src) : "memory");
}

// Lane offsets of the two reads of a tile, and the products fed by them.
template <int D>
struct TileLanes {
  using C = Tile<D, kBT>;
  int row, col;
  __device__ TileLanes(int l16, int grp) {
    // rows: lane (l16, grp) reads row 16 h + l16, chunk 4 s + grp at row + 512 s + 16 ROWB h
    row = (l16 >> 3) * (8 * C::ROWB) + 256 * (grp >> 1) + 32 * (l16 & 7) + 16 * ((grp ^ (l16 >> 3)) & 1);
    // transposed: rows 4 grp .. +3 and 16 + those, d tile dt at col + 256 dt (+ 16 ROWB)
    const int r = 4 * grp + (l16 >> 2);
    col = (r >> 3) * (8 * C::ROWB) + 32 * (r & 7) + 16 * (((l16 >> 1) ^ (r >> 3)) & 1) + 8 * (l16 & 1);
  }
  // rows of block kb, d slice s
  __device__ __attribute__((always_inline)) void read_slice(const char* t, int kb, int s, bf16x8 (&x)[2]) const {
#pragma unroll
    for (int h = 0; h < 2; ++h)
      x[h] = *reinterpret_cast<const bf16x8*>(t + (2 * kb + h) * 16 * C::ROWB + row + 512 * s);
  }
  __device__ __attribute__((always_inline)) void read_rows(const char* t, int kb, bf16x8 (&x)[C::KS][2]) const {
#pragma unroll
    for (int s = 0; s < C::KS; ++s) read_slice(t, kb, s, x[s]);
  }
  __device__ __attribute__((always_inline)) void read_cols(const char* t, int kb, bf16x8 (&x)[C::DT], int d0 = 0, int d1 = C::DT) const {
#pragma unroll
    for (int dt = d0; dt < d1; ++dt) {
      const char* p = t + kb * 32 * C::ROWB + col + 256 * dt;
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, p));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, p + 16 * C::ROWB));
      const u32x2 lo2 = __builtin_bit_cast(u32x2, lo), hi2 = __builtin_bit_cast(u32x2, hi);
      const u32x4 u = {lo2[0], lo2[1], hi2[0], hi2[1]};
      x[dt] = __builtin_bit_cast(bf16x8, u);
    }
  }
  // acc[dt][t] += x^T p (p packed bf16: a lane's rows 4 grp .. +3 of both halves)
  template <int T>
  __device__ __attribute__((always_inline)) void product(const bf16x8 (&x)[C::DT], const uint32_t (&p)[T][4],
                                                         f32x4 (&acc)[C::DT][T]) const {
#pragma unroll
    for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const u32x4 u = {p[t][0], p[t][1], p[t][2], p[t][3]};
        acc[dt][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[dt], __builtin_bit_cast(bf16x8, u),
                                                             acc[dt][t], 0, 0, 0);
      }
  }
};

// Cursor over the tiles of the runs: tile = (run, first row).
struct Cursor {
  int sg, k0;
};

// NM products, each followed by its share of NR LDS reads, NV plain VALU and NT
// transcendentals (sched_group_barrier classes 0x008, 0x100, 0x002, 0x400), after
// NRF reads ahead of the first one
template <int NM, int NR, int NRF, int NV, int NT, int... I>
__device__ __forceinline__ void interleave_seq(std::integer_sequence<int, I...>) {
  auto one = [](auto ic) __attribute__((always_inline)) {
    constexpr int i = decltype(ic)::value;
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    constexpr int r = ((NR - NRF) * (i + 1)) / NM - ((NR - NRF) * i) / NM;
    if constexpr (r > 0) __builtin_amdgcn_sched_group_barrier(0x100, r, 0);
    constexpr int v = (NV * (i + 1)) / NM - (NV * i) / NM;
    if constexpr (v > 0) __builtin_amdgcn_sched_group_barrier(0x002, v, 0);
    constexpr int t = (NT * (i + 1)) / NM - (NT * i) / NM;
    if constexpr (t > 0) __builtin_amdgcn_sched_group_barrier(0x400, t, 0);
  };
  (one(std::integral_constant<int, I>{}), ...);
}
template <int NM, int NR, int NRF, int NV, int NT>
__device__ __forceinline__ void interleave() {
  if constexpr (NRF > 0) __builtin_amdgcn_sched_group_barrier(0x100, NRF, 0);
  interleave_seq<NM, NR, NRF, NV, NT>(std::make_integer_sequence<int, NM>{});
}

__device__ inline int xcd_logical(int b, int n_wg) {
  const int xcd = b % kXcds, idx = b / kXcds;
  const int per = n_wg / kXcds, rem = n_wg % kXcds;
  return xcd * per + min(xcd, rem) + idx;
}

// Groups of `group` consecutive logical units that share a read set (the q
// tiles of one (chunk, head)) but cost differently from group to group: XCD x
// takes the groups x, x + 8, .. so every XCD gets the same mix; the last
// n_groups % 8 groups run in order.
__device__ inline int xcd_interleaved(int b, int n_wg, int group) {
  const int n_groups = n_wg / group;
  const int n_even = n_groups - n_groups % kXcds;
  if (b >= n_even * group) return b;
  const int xcd = b % kXcds, idx = b / kXcds;
  return (xcd + kXcds * (idx / group)) * group + idx % group;
}

// ---- D_i = dO_i . O_i ---------------------------------------------------------------
// L = d / 8 consecutive lanes per row (16 bytes of O and of dO each, so a wave
// reads contiguous memory), partial sums combined across the L lanes.
template <int L>
__global__ __launch_bounds__(256) void bwd_delta_kernel(const __bf16* __restrict__ o,
                                                        const __bf16* __restrict__ dout,
                                                        float* __restrict__ delta, int64_t rows) {
  const int64_t t = int64_t(blockIdx.x) * 256 + threadIdx.x;
  const int64_t r = t / L;
  float acc = 0.0f;
  if (r < rows) {
    const u32x4 a = reinterpret_cast<const u32x4*>(o)[t];
    const u32x4 b = reinterpret_cast<const u32x4*>(dout)[t];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      acc = fmaf(__uint_as_float(a[j] << 16), __uint_as_float(b[j] << 16), acc);
      acc = fmaf(__uint_as_float(a[j] & 0xffff0000u), __uint_as_float(b[j] & 0xffff0000u), acc);
    }
  }
#pragma unroll
  for (int off = L / 2; off > 0; off >>= 1) acc += __shfl_xor(acc, off, L);
  if (r < rows && (t % L) == 0) delta[r] = acc;
}

// ---- dQ: query-stationary ---------------------------------------------------------------
// A workgroup holds 256 queries of one chunk and head (32 per wave, Q and dO in
// registers) and streams the 64-key tiles of their read set through a ring of
// five slots (K tile, V tile), as the forward kernel does: waves 0-3 copy three
// tiles ahead, one barrier per tile.  Products on v_mfma_f32_16x16x32_bf16 (the
// least register traffic per FLOP).  One step per 32-key block b, in three
// scheduling regions of 16 products each:
//   S^T(b) = K Q^T              with dS of block b-1 (P (dP - D), bf16 packs) between its products
//   dP^T(b) = V dO^T            with P(b) = 2^(c S - L) between its products
//   dQ^T += K(b-1)^T dS(b-1)^T
// so the VALU work of a block never waits for products of its own region, and
// each region reads the LDS operands of the next one.
template <int D>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void bwd_dq_kernel(const __bf16* __restrict__ q, const __bf16* __restrict__ dout,
                   const float* __restrict__ lse, const float* __restrict__ delta,
                   __bf16* __restrict__ dq, int heads, float c_log2, float scale, PackedPlan plan,
                   int n_qtiles) {
  using C = Tile<D, kBT>;
  __shared__ __attribute__((aligned(1024))) char lds[5 * C::SLOT];
  const int nq = plan.chunk_tokens;
  const int logical = xcd_interleaved(blockIdx.x, gridDim.x, n_qtiles);
  const int nth = logical / (heads * n_qtiles);
  const int chunk = plan.n_chunks - 1 - nth;   // the first chunks' short read sets run last
  const int rest = logical - nth * heads * n_qtiles;
  const int head = rest / n_qtiles, qt = rest % n_qtiles;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, l16 = lane & 15, grp = lane >> 4;
  const int64_t tok0 = int64_t(chunk) * nq;
  const int64_t row_elems = int64_t(heads) * D;
  const int q0 = qt * kBlockN + wave * 32;
  const bool idle = q0 >= nq;   // no queries for this wave: it only copies and keeps the barriers

  // lane (l16, grp) holds query q0 + 16 qh + l16, elements 32 s + 8 grp .. +7
  bf16x8 qreg[2][C::KS], greg[2][C::KS];
  float L[2], Dq_[2];
#pragma unroll
  for (int qh = 0; qh < 2; ++qh) {
    const int64_t t = tok0 + min(q0 + 16 * qh + l16, nq - 1);
    const __bf16* qp = q + t * row_elems + head * D + 8 * grp;
    const __bf16* gp = dout + t * row_elems + head * D + 8 * grp;
#pragma unroll
    for (int s = 0; s < C::KS; ++s) {
      qreg[qh][s] = *reinterpret_cast<const bf16x8*>(qp + 32 * s);
      greg[qh][s] = *reinterpret_cast<const bf16x8*>(gp + 32 * s);
    }
    L[qh] = lse[t * heads + head];
    Dq_[qh] = delta[t * heads + head];
  }
  f32x4 acc[C::DT][2];
#pragma unroll
  for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
    for (int qh = 0; qh < 2; ++qh) acc[dt][qh] = f32x4{};

  // runs of the read set, one per lane (read with v_readlane)
  const int n_runs = packed_num_segments(plan, chunk);
  int sg_len = 0;
  uint64_t sg_k = 0, sg_v = 0;
  const uint32_t row_bytes = uint32_t(2 * row_elems);
#pragma unroll
  for (int i = 0; i < kMaxRuns; ++i)
    if (lane == i && i < n_runs) {
      const KvSegment sg = packed_segment(plan, chunk, i, heads, D, 2);
      sg_len = sg.len;
      sg_k = reinterpret_cast<uint64_t>(sg.k) + 2ull * uint64_t(head) * D;
      sg_v = reinterpret_cast<uint64_t>(sg.v) + 2ull * uint64_t(head) * D;
    }
  auto run_len = [&](int i) { return __builtin_amdgcn_readlane(sg_len, i); };
  int n_tiles = 0;
  for (int i = 0; i < n_runs; ++i) n_tiles += (run_len(i) + kBT - 1) / kBT;
  auto advance = [&](Cursor c) __attribute__((always_inline)) {
    c.k0 += kBT;
    if (c.k0 >= run_len(c.sg)) {
      ++c.sg;
      c.k0 = 0;
    }
    return c;
  };
  auto slot = [&](int i) __attribute__((always_inline)) { return lds + i * C::SLOT; };

  auto issue_tile = [&](char* base, Cursor c) __attribute__((always_inline)) {
    if (wave >= C::kCopyWaves) return;
    const uint64_t off = uint64_t(c.k0) * row_bytes;
    copy_tiles<D, kBT>(base, readlane_u64(sg_k, c.sg) + off, readlane_u64(sg_v, c.sg) + off, row_bytes,
                  run_len(c.sg) - 1 - c.k0, wave, lane);
  };
  const TileLanes<D> ln(l16, grp);
  auto rows_product = [&](const bf16x8 (&x)[C::KS][2], const bf16x8 (&st)[2][C::KS], f32x4 (&r)[2][2])
      __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < C::KS; ++s)
#pragma unroll
      for (int kh = 0; kh < 2; ++kh)
#pragma unroll
        for (int qh = 0; qh < 2; ++qh)
          r[kh][qh] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[s][kh], st[qh][s],
                                                              s == 0 ? f32x4{} : r[kh][qh], 0, 0, 0);
  };

  // p and dp: P and dP^T of the previous block
  f32x4 p[2][2], dp[2][2];
#pragma unroll
  for (int kh = 0; kh < 2; ++kh)
#pragma unroll
    for (int qh = 0; qh < 2; ++qh) {
      p[kh][qh] = f32x4{};
      dp[kh][qh] = f32x4{};
    }
  // dS of the previous block, packed as the B operand of dQ^T
  auto ds_pack = [&](uint32_t (&pk)[2][4]) __attribute__((always_inline)) {
#pragma unroll
    for (int qh = 0; qh < 2; ++qh)
#pragma unroll
      for (int kh = 0; kh < 2; ++kh)
#pragma unroll
        for (int j = 0; j < 4; j += 2)
          pk[qh][2 * kh + (j >> 1)] = pack_bf16(p[kh][qh][j] * (dp[kh][qh][j] - Dq_[qh]),
                                                p[kh][qh][j + 1] * (dp[kh][qh][j + 1] - Dq_[qh]));
  };
  // One step: block kb of the tile in st, whose K rows are in kx; (pt, pkb): the
  // previous block's tile and index, (nt, nkb): the next one's.  Each region reads
  // the operands of the next one.
  auto step = [&](bf16x8 (&kx)[C::KS][2], const char* st, int kb, const char* pt, int pkb,
                  const char* nt, int nkb, int nv) __attribute__((always_inline)) {
    uint32_t pk[2][4];
    f32x4 s[2][2];
    bf16x8 vx[C::KS][2], cx[C::DT];
    ln.read_rows(st + C::TILE, kb, vx);
    ds_pack(pk);
    rows_product(kx, qreg, s);
    interleave<4 * C::KS, 2 * C::KS, 0, 44, 0>();
    asm volatile("" ::"v"(pk[0][0]), "v"(pk[0][1]), "v"(pk[0][2]), "v"(pk[0][3]), "v"(pk[1][0]),
                 "v"(pk[1][1]), "v"(pk[1][2]), "v"(pk[1][3]));
    __builtin_amdgcn_sched_barrier(0);
    ln.read_cols(pt, pkb, cx);
#pragma unroll
    for (int kh = 0; kh < 2; ++kh)
#pragma unroll
      for (int qh = 0; qh < 2; ++qh)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          p[kh][qh][j] = __builtin_amdgcn_exp2f(fmaf(s[kh][qh][j], c_log2, -L[qh]));
    rows_product(vx, greg, dp);
    interleave<4 * C::KS, 2 * C::DT, 0, 20, 16>();
    __builtin_amdgcn_sched_barrier(0);
    ln.read_rows(nt, nkb, kx);
    ln.template product<2>(cx, pk, acc);
    interleave<2 * C::DT, 2 * C::KS, 0, 0, 0>();
    __builtin_amdgcn_sched_barrier(0);
    if (nv < kBT)   // keys past a run's end
#pragma unroll
      for (int kh = 0; kh < 2; ++kh)
#pragma unroll
        for (int qh = 0; qh < 2; ++qh)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            p[kh][qh][j] = 4 * grp >= nv - 32 * kb - 16 * kh - j ? 0.0f : p[kh][qh][j];
  };

  Cursor c_t = {0, 0}, c_dma = {0, 0};
#pragma unroll
  for (int i = 0; i < 3; ++i)
    if (i < n_tiles) {
      issue_tile(slot(i), c_dma);
      c_dma = advance(c_dma);
    }
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (idle) {   // only the copies and the barriers of the loop below
    int i3 = 3;
#pragma unroll 1
    for (int t = 0; t < n_tiles; ++t) {
      if (wave < C::kCopyWaves) {
        if (t + 2 < n_tiles)
          __builtin_amdgcn_s_waitcnt(waitcnt_vm(2 * C::N));
        else
          __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
      }
      asm volatile("s_barrier" ::: "memory");
      if (t + 3 < n_tiles) {
        issue_tile(slot(i3), c_dma);
        c_dma = advance(c_dma);
      }
      i3 = i3 == 4 ? 0 : i3 + 1;
    }
    return;
  }
  bf16x8 kx[C::KS][2];
  ln.read_rows(slot(0), 0, kx);
  // barrier t: tile t+1 has landed (each copying wave waits for its own copies)
  // and tile t-2 is no longer read; then tile t+3 is copied into its slot
  int i0 = 0;   // slot of tile t
#pragma unroll 1
  for (int t = 0; t < n_tiles; ++t) {
    const int i1 = i0 == 4 ? 0 : i0 + 1;
    const int i4 = i0 == 0 ? 4 : i0 - 1;        // slot of tile t-1
    const int i3 = i0 >= 2 ? i0 - 2 : i0 + 3;   // slot of tile t-2 (and of tile t+3)
    if (wave < C::kCopyWaves) {
      if (t + 2 < n_tiles)
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(2 * C::N));
      else
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    }
    asm volatile("s_barrier" ::: "memory");
    if (t + 3 < n_tiles) {
      issue_tile(slot(i3), c_dma);
      c_dma = advance(c_dma);
    }
    const int nv = min(kBT, run_len(c_t.sg) - c_t.k0);
    c_t = advance(c_t);
    char* st = slot(i0);
    // (the first step adds dS = 0 times tile 0's K; after the last tile the next
    // block's K rows come from a stale slot and are not used)
    step(kx, st, 0, t == 0 ? st : slot(i4), 1, st, 1, nv);
    step(kx, st, 1, st, 0, slot(i1), 0, nv);
    i0 = i1;
  }
  {
    // the last block
    uint32_t pk[2][4];
    ds_pack(pk);
    bf16x8 x[C::DT];
    ln.read_cols(slot(i0 == 0 ? 4 : i0 - 1), 1, x);
    ln.template product<2>(x, pk, acc);
  }

#pragma unroll
  for (int qh = 0; qh < 2; ++qh) {
    const int qi = q0 + 16 * qh + l16;
    if (qi < nq) {
      __bf16* op = dq + (tok0 + qi) * row_elems + head * D + 4 * grp;
#pragma unroll
      for (int dt = 0; dt < C::DT; ++dt) {
        u32x2 w;
        w.x = pack_bf16(acc[dt][qh][0] * scale, acc[dt][qh][1] * scale);
        w.y = pack_bf16(acc[dt][qh][2] * scale, acc[dt][qh][3] * scale);
        *reinterpret_cast<u32x2*>(op + 16 * dt) = w;
      }
    }
  }
}

// ---- dK and dV: key-stationary ----------------------------------------------------------
// Key units: the first n_frames * kpf units are anchor frames, kpf units of 256 keys
// each, the rest are keys [256 k, 256 k + 256) of a chunk, kpc units per chunk.  Each unit
// streams the query runs that see it (the chunk runs listed for the anchor
// frame, or chunks c .. c + window of the packed clip).  Frames come first: they
// are seen by the most chunks, and the longest streams should not start last.
struct KeyUnits {
  int32_t kpc, kpf, n_frames;
  uint8_t frame_runs[FF_MAX_ANCHOR_FRAMES * 8][16];   // per anchor frame: (first chunk, count) pairs
};

// A workgroup holds 256 keys (32 per wave: K in registers, V in LDS, where the
// registers run out beside both accumulators) and streams tiles of 32 queries (64
// at d = 64, where a tile of 32 is worked on for less time than a copy takes; Q, dO,
// the log-sum-exp and D) through a ring of five slots, with one barrier per two
// tiles: at the barrier of tiles t and t+1, tile t+2 has landed too (its Q rows are
// read ahead) and tiles t+3 and t+4 go into the slots of t-2 and t-1.  A block of 32
// queries in four scheduling regions of 16 products, each reading ahead what the registers
// allow of the next one's LDS operands:
//   S = Q K^T - L / c    (L / c enters as the accumulator's initial value)
//   dP = dO V^T          with P = 2^(c S) between its products
//   dV^T += dO^T P       with dS = P (dP - D) and the bf16 packs between its products
//   dK^T += Q^T dS
template <int D>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void bwd_dkv_kernel(const __bf16* __restrict__ q, const __bf16* __restrict__ dout,
                    const float* __restrict__ lse, const float* __restrict__ delta,
                    __bf16* __restrict__ dk_chunks, __bf16* __restrict__ dk_anchor,
                    __bf16* __restrict__ dv_chunks, __bf16* __restrict__ dv_anchor, int heads,
                    float c_log2, float scale, PackedPlan plan, KeyUnits ku) {
  constexpr int kRows = D == 128 ? 32 : 64;        // queries per tile
  constexpr int kBlocks = kRows / 32;
  using C = Tile<D, kRows>;
  constexpr int kSlot = C::SLOT + 2 * kRows * 4;   // Q tile, dO tile, L, D
  __shared__ __attribute__((aligned(1024))) char stash[kBlockN * C::ROWB];
  __shared__ __attribute__((aligned(1024))) char lds[5 * kSlot];
  const int nq = plan.chunk_tokens, G = plan.frame_tokens;
  const int n_frame_units = ku.n_frames * ku.kpf;
  const int n_units = n_frame_units + plan.n_chunks * ku.kpc;
  const int logical = xcd_logical(blockIdx.x, gridDim.x);
  const int head = logical / n_units;
  const int unit = logical - head * n_units;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, l16 = lane & 15, grp = lane >> 4;
  const int64_t row_elems = int64_t(heads) * D;
  const bool is_chunk = unit >= n_frame_units;
  int owner, k_first, n_keys;
  const __bf16 *kbase, *vbase;
  __bf16 *obase_k, *obase_v;
  if (is_chunk) {
    const int u = unit - n_frame_units;
    owner = u / ku.kpc;
    k_first = (u % ku.kpc) * kBlockN;
    n_keys = nq;
    const int64_t o = int64_t(owner) * nq * row_elems + head * D;
    kbase = static_cast<const __bf16*>(plan.k) + o;
    vbase = static_cast<const __bf16*>(plan.v) + o;
    obase_k = dk_chunks + o;
    obase_v = dv_chunks + o;
  } else {
    owner = unit / ku.kpf;
    k_first = (unit % ku.kpf) * kBlockN;
    n_keys = G;
    const int64_t o = int64_t(owner) * G * row_elems + head * D;
    kbase = static_cast<const __bf16*>(plan.ak) + o;
    vbase = static_cast<const __bf16*>(plan.av) + o;
    obase_k = dk_anchor + o;
    obase_v = dv_anchor + o;
  }
  const int k0 = k_first + wave * 32;
  const bool idle = k0 >= n_keys;   // no keys for this wave: it only copies and keeps the barriers

  // lane (l16, grp) holds key k0 + 16 t + l16, elements 32 s + 8 grp .. +7
  bf16x8 kreg[2][C::KS];
  char* stash_w = stash + 32 * wave * C::ROWB;
  const TileLanes<D> ln(l16, grp);
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int64_t r = min(k0 + 16 * t + l16, n_keys - 1);
    const __bf16* kp = kbase + r * row_elems + 8 * grp;
    const __bf16* vp = vbase + r * row_elems + 8 * grp;
#pragma unroll
    for (int s = 0; s < C::KS; ++s) {
      kreg[t][s] = *reinterpret_cast<const bf16x8*>(kp + 32 * s);
      *reinterpret_cast<bf16x8*>(stash_w + 16 * t * C::ROWB + ln.row + 512 * s) =
          *reinterpret_cast<const bf16x8*>(vp + 32 * s);
    }
  }
  f32x4 acc_k[C::DT][2], acc_v[C::DT][2];   // dK^T, dV^T
#pragma unroll
  for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      acc_k[dt][t] = f32x4{};
      acc_v[dt][t] = f32x4{};
    }

  // query runs of this unit, one per lane
  int rn_len = 0, n_runs = 0;
  uint64_t rn_q = 0, rn_g = 0, rn_l = 0, rn_d = 0;
  auto set_run = [&](int i, int c0, int c1) {   // chunks c0 .. c1 - 1
    if (lane == i) {
      const int64_t t0 = int64_t(c0) * nq;
      rn_len = (c1 - c0) * nq;
      rn_q = reinterpret_cast<uint64_t>(q + t0 * row_elems + head * D);
      rn_g = reinterpret_cast<uint64_t>(dout + t0 * row_elems + head * D);
      rn_l = reinterpret_cast<uint64_t>(lse + t0 * heads + head);
      rn_d = reinterpret_cast<uint64_t>(delta + t0 * heads + head);
    }
  };
  if (is_chunk) {
    set_run(0, owner, min(owner + min(plan.window, plan.n_chunks) + 1, plan.n_chunks));
    n_runs = 1;
  } else {
    while (n_runs < 8 && ku.frame_runs[owner][2 * n_runs + 1] != 0) {
      const int c0 = ku.frame_runs[owner][2 * n_runs];
      set_run(n_runs, c0, c0 + ku.frame_runs[owner][2 * n_runs + 1]);
      ++n_runs;
    }
  }
  auto run_len = [&](int i) { return __builtin_amdgcn_readlane(rn_len, i); };
  int n_tiles = 0;
  for (int i = 0; i < n_runs; ++i) n_tiles += (run_len(i) + kRows - 1) / kRows;
  Cursor c_t = {0, 0}, c_dma = {0, 0};
  auto advance = [&](Cursor c) __attribute__((always_inline)) {
    c.k0 += kRows;
    if (c.k0 >= run_len(c.sg)) {
      ++c.sg;
      c.k0 = 0;
    }
    return c;
  };
  const uint32_t row_bytes = uint32_t(2 * row_elems);
  auto issue_tile = [&](char* base, Cursor c) __attribute__((always_inline)) {
    if (wave >= C::kCopyWaves) return;
    const int last = run_len(c.sg) - 1 - c.k0;
    const uint64_t off = uint64_t(c.k0) * row_bytes;
    copy_tiles<D, kRows>(base, readlane_u64(rn_q, c.sg) + off, readlane_u64(rn_g, c.sg) + off, row_bytes,
                         last, wave, lane);
    // L, then D of the rows, 4 bytes per lane (one copy holds both of a 32-row tile)
    if (wave < 2 * kRows / 64) {
      const int i = 64 * wave + lane;
      const uint64_t v = i < kRows ? readlane_u64(rn_l, c.sg) : readlane_u64(rn_d, c.sg);
      lds_copy_dwords(uint32_t(size_t(LDS_PTR(char, base))) + C::SLOT + 256 * wave,
                      v + uint64_t(c.k0 + min(i & (kRows - 1), last)) * uint32_t(4 * heads));
    }
  };

  const float neg_inv_c = -1.0f / c_log2;
  bf16x8 xq[C::KS][2];   // Q rows of the next tile
  f32x4 p[2][2];         // [16-row half of the tile][16-key tile]: - L / c, S - L / c, then P
  auto read_ahead = [&](const char* st, int kb) __attribute__((always_inline)) {
    ln.read_rows(st, kb, xq);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const f32x4 Lr = *reinterpret_cast<const f32x4*>(st + C::SLOT + 4 * (32 * kb + 16 * h + 4 * grp)) * neg_inv_c;
#pragma unroll
      for (int t = 0; t < 2; ++t) p[h][t] = Lr;
    }
  };
  // block kb of the tile in st, whose Q rows have been read; (next, nkb): the block
  // after it (in a stale slot after the last one: not used); nv: the block's rows
  auto block = [&](const char* st, int kb, const char* next, int nkb, int nv) __attribute__((always_inline)) {
    constexpr int kHalf = C::KS / 2;
    f32x4 dp[2][2];
    bf16x8 xg[C::KS][2], xv[C::KS][2];
#pragma unroll
    for (int s = 0; s < kHalf; ++s) {
      ln.read_slice(st + C::TILE, kb, s, xg[s]);
      ln.read_slice(stash_w, 0, s, xv[s]);
    }
#pragma unroll
    for (int s = 0; s < C::KS; ++s)
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int t = 0; t < 2; ++t)
          p[h][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xq[s][h], kreg[t][s], p[h][t], 0, 0, 0);
    interleave<4 * C::KS, 4 * kHalf, 0, 0, 0>();
    __builtin_amdgcn_sched_barrier(0);
    if (nv < 32)   // rows past a run's end
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int j = 0; j < 4; ++j) p[h][t][j] = 4 * grp >= nv - 16 * h - j ? -INFINITY : p[h][t][j];
#pragma unroll
    for (int s = kHalf; s < C::KS; ++s) {
      ln.read_slice(st + C::TILE, kb, s, xg[s]);
      ln.read_slice(stash_w, 0, s, xv[s]);
    }
#pragma unroll
    for (int s = 0; s < C::KS; ++s)
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int t = 0; t < 2; ++t)
          dp[h][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xg[s][h], xv[s][t], s == 0 ? f32x4{} : dp[h][t], 0, 0, 0);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) p[h][t][j] = __builtin_amdgcn_exp2f(p[h][t][j] * c_log2);
    uint32_t pv[2][4], pk[2][4];
    bf16x8 xc[C::DT], xk[C::DT];
    ln.read_cols(st + C::TILE, kb, xc, 0, C::DT / 4);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < 4; j += 2) pv[t][2 * h + (j >> 1)] = pack_bf16(p[h][t][j], p[h][t][j + 1]);
    interleave<4 * C::KS, 4 * (C::KS - kHalf) + C::DT / 2, 0, 24, 16>();
    asm volatile("" ::"v"(pv[0][0]), "v"(pv[0][1]), "v"(pv[0][2]), "v"(pv[0][3]), "v"(pv[1][0]),
                 "v"(pv[1][1]), "v"(pv[1][2]), "v"(pv[1][3]));
    __builtin_amdgcn_sched_barrier(0);
    {
      ln.read_cols(st + C::TILE, kb, xc, C::DT / 4, C::DT);
      ln.read_cols(st, kb, xk, 0, C::DT / 4);
      ln.template product<2>(xc, pv, acc_v);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const f32x4 Dr = *reinterpret_cast<const f32x4*>(st + C::SLOT + 4 * (kRows + 32 * kb + 16 * h + 4 * grp));
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int j = 0; j < 4; j += 2)
            pk[t][2 * h + (j >> 1)] = pack_bf16(p[h][t][j] * (dp[h][t][j] - Dr[j]),
                                                p[h][t][j + 1] * (dp[h][t][j + 1] - Dr[j + 1]));
      }
      interleave<2 * C::DT, 2 * C::DT + 2, 0, 40, 0>();
      asm volatile("" ::"v"(pk[0][0]), "v"(pk[0][1]), "v"(pk[0][2]), "v"(pk[0][3]), "v"(pk[1][0]),
                   "v"(pk[1][1]), "v"(pk[1][2]), "v"(pk[1][3]));
      __builtin_amdgcn_sched_barrier(0);
    }
    {
      ln.read_cols(st, kb, xk, C::DT / 4, C::DT);
      ln.template product<2>(xk, pk, acc_k);
      read_ahead(next, nkb);
      interleave<2 * C::DT, 2 * C::DT - C::DT / 2 + 2 * C::KS + 2, 0, 16, 0>();
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  auto slot = [&](int i) __attribute__((always_inline)) { return lds + i * kSlot; };
  for (int i = 0; i < 3; ++i)
    if (i < n_tiles) {
      issue_tile(slot(i), c_dma);
      c_dma = advance(c_dma);
    }
  __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
  __syncthreads();
  if (idle) {   // only the copies and the barriers of the loop below
    int i3 = 3;
#pragma unroll 1
    for (int t = 0; t < n_tiles; t += 2) {
      __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
      asm volatile("s_barrier" ::: "memory");
      for (int i = 3; i < 5; ++i) {
        if (t + i < n_tiles) {
          issue_tile(slot(i3), c_dma);
          c_dma = advance(c_dma);
        }
        i3 = i3 == 4 ? 0 : i3 + 1;
      }
    }
    return;
  }
  read_ahead(slot(0), 0);
  int i0 = 0;   // slot of tile t
#pragma unroll 1
  for (int t = 0; t < n_tiles; t += 2) {
    const auto ahead = [&](int n) { return i0 + n >= 5 ? i0 + n - 5 : i0 + n; };
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    asm volatile("s_barrier" ::: "memory");
#pragma unroll
    for (int i = 3; i < 5; ++i)
      if (t + i < n_tiles) {
        issue_tile(slot(ahead(i)), c_dma);
        c_dma = advance(c_dma);
      }
    auto tile = [&](const char* st, const char* next) __attribute__((always_inline)) {
      const int nv = min(kRows, run_len(c_t.sg) - c_t.k0);
      c_t = advance(c_t);
      if constexpr (kBlocks == 2) block(st, 0, st, 1, nv);
      block(st, kBlocks - 1, next, 0, nv - 32 * (kBlocks - 1));
    };
    tile(slot(i0), slot(ahead(1)));
    if (t + 1 < n_tiles) tile(slot(ahead(1)), slot(ahead(2)));
    i0 = ahead(2);
  }

#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int key = k0 + 16 * t + l16;
    if (key < n_keys) {
      __bf16* pk = obase_k + key * row_elems + 4 * grp;
      __bf16* pv = obase_v + key * row_elems + 4 * grp;
#pragma unroll
      for (int dt = 0; dt < C::DT; ++dt) {
        u32x2 w;
        w.x = pack_bf16(acc_k[dt][t][0] * scale, acc_k[dt][t][1] * scale);
        w.y = pack_bf16(acc_k[dt][t][2] * scale, acc_k[dt][t][3] * scale);
        *reinterpret_cast<u32x2*>(pk + 16 * dt) = w;
        w.x = pack_bf16(acc_v[dt][t][0], acc_v[dt][t][1]);
        w.y = pack_bf16(acc_v[dt][t][2], acc_v[dt][t][3]);
        *reinterpret_cast<u32x2*>(pv + 16 * dt) = w;
      }
    }
  }
}

// Stationary 16-row tiles per workgroup of the split kernels (attn_bwd_split.hip),
// or 0 where the 256-row kernels of this file are the better ones: the shortest
// estimate, per pass, of a fixed part plus the 64-row tiles that the busiest CU
// streams (an even share of all and a third of the longest stream, at least the
// longest one) times the time of one.  The constants are fits to 45 launches of
// 1 to 40 heads, 3 to 27 chunks of 63 to 2016 tokens, each form forced (us of
// the whole backward, 256-row kernels / split dQ / split dK and dV: 6 heads x 64,
// 7 chunks of 351 tokens 104 / 96 / 74; 24 heads x 128, 11 x 1056, which fills the
// GPU, 2020 / 2220 / 2290).
struct SplitChoice {
  int q, k;   // dQ; dK and dV
};

SplitChoice choose_split(const PackedPlan& plan, int heads, int head_dim, const KeyUnits& ku) {
  struct Cost { double fixed, tile; };   // us, us per 64-row tile
  struct Load {
    double sum = 0.0, most = 0.0;        // tiles of all workgroups, of the longest
    void add(double tiles, double workgroups) {
      sum += tiles * workgroups;
      most = fmax(most, tiles);
    }
    double us(const Cost& c, int cus) const { return c.fixed + c.tile * fmax(most, sum / cus + 0.35 * most); }
  };
  constexpr double kMargin = 0.92;   // near a tie the 256-row kernels, which read less
  const bool wide = head_dim == 128;
  const int cus = device_cus();
  const Cost cost_q[3] = {wide ? Cost{4.0, 2.40} : Cost{4.0, 1.60}, wide ? Cost{6.0, 0.43} : Cost{7.0, 0.22},
                          wide ? Cost{7.0, 0.59} : Cost{6.0, 0.32}};
  const Cost cost_k[3] = {wide ? Cost{4.0, 2.70} : Cost{6.0, 1.75}, wide ? Cost{8.0, 0.46} : Cost{8.0, 0.27},
                          Cost{8.0, 0.32}};   // (two tiles: d = 64 only)
  const int nq = plan.chunk_tokens, n = plan.n_chunks;
  const int window = plan.window < n ? plan.window : n;
  const auto groups = [](int rows, int per) { return double((rows + per - 1) / per); };
  SplitChoice choice = {0, 0};
  double best_q = 0.0, best_k = 0.0;
  for (int t = 0; t <= 2; ++t) {
    const int per = t == 0 ? kBlockN : 16 * t;
    Load lq, lk;
    for (int c = 0; c < n; ++c) {
      double tiles = 0.0;
      for (int i = 0; i < packed_num_segments(plan, c); ++i)
        tiles += groups(packed_segment(plan, c, i, heads, head_dim, 2).len, kBT);
      lq.add(tiles, groups(nq, per) * heads);
      lk.add(groups(((c + window < n - 1 ? c + window : n - 1) - c + 1) * nq, kBT),
             groups(nq, per) * heads);
    }
    for (int f = 0; f < ku.n_frames; ++f) {
      double tiles = 0.0;
      for (int r = 0; r < 8; ++r) tiles += groups(ku.frame_runs[f][2 * r + 1] * nq, kBT);
      lk.add(tiles, groups(plan.frame_tokens, per) * heads);
    }
    const double margin = t == 0 ? kMargin : 1.0;
    const double us_q = margin * lq.us(cost_q[t], cus), us_k = margin * lk.us(cost_k[t], cus);
    if (t == 0 || us_q < best_q) {
      best_q = us_q;
      choice.q = t;
    }
    if (wide && t == 2) continue;   // dK and dV take one tile at d = 128
    if (t == 0 || us_k < best_k) {
      best_k = us_k;
      choice.k = t;
    }
  }
  return choice;
}

}  // namespace

hipError_t launch_attention_bwd_bf16(const void* q, const void* out, const void* dout,
                                     const float* lse, float* delta, void* dq, void* dk, void* dv,
                                     void* dak, void* dav, int heads, int head_dim,
                                     float softmax_scale, const PackedPlan& plan,
                                     const uint8_t (*frame_runs)[16], int n_frames,
                                     hipStream_t stream) {
  const int nq = plan.chunk_tokens;
  const int64_t rows = int64_t(plan.n_chunks) * nq * heads;
  if (rows == 0) return hipSuccess;
  {
    const int64_t threads = rows * (head_dim / 8);   // the last block may run past the rows
    const dim3 g(unsigned((threads + 255) / 256));
    if (head_dim == 128)
      hipLaunchKernelGGL(bwd_delta_kernel<16>, g, dim3(256), 0, stream,
                         static_cast<const __bf16*>(out), static_cast<const __bf16*>(dout), delta, rows);
    else
      hipLaunchKernelGGL(bwd_delta_kernel<8>, g, dim3(256), 0, stream,
                         static_cast<const __bf16*>(out), static_cast<const __bf16*>(dout), delta, rows);
  }
  const float c_log2 = float(double(softmax_scale) * 1.4426950408889634);
  const int n_qtiles = (nq + kBlockN - 1) / kBlockN;
  KeyUnits ku;
  std::memset(&ku, 0, sizeof(ku));
  ku.kpc = n_qtiles;
  ku.kpf = (plan.frame_tokens + kBlockN - 1) / kBlockN;
  ku.n_frames = n_frames;
  for (int f = 0; f < n_frames; ++f) std::memcpy(ku.frame_runs[f], frame_runs[f], 16);
  const int n_units = plan.n_chunks * ku.kpc + n_frames * ku.kpf;
  const dim3 g_q(unsigned(plan.n_chunks * heads * n_qtiles)), g_k(unsigned(n_units * heads));
  const __bf16* qp = static_cast<const __bf16*>(q);
  const __bf16* dp = static_cast<const __bf16*>(dout);
  __bf16 *dkp = static_cast<__bf16*>(dk), *dvp = static_cast<__bf16*>(dv);
  __bf16 *dakp = static_cast<__bf16*>(dak), *davp = static_cast<__bf16*>(dav);
  const SplitChoice split = choose_split(plan, heads, head_dim, ku);
  last_launch.bwd_q_tiles = split.q;
  last_launch.bwd_k_tiles = split.k;
  // Rings (LDS: 160 KB per workgroup): five slots each.  dQ: 64-row tiles of K and V, 32 KB a
  // slot at d = 128 (all of the LDS; Q and dO are in registers), 16 KB at d = 64.  dK and dV:
  // 64 KB of V beside slots of 16.25 KB at d = 128 (32-row tiles of Q and dO with their L and
  // D, which also keeps the per-block registers within two waves per SIMD beside both
  // accumulators), 32 KB beside 16.5 KB at d = 64 (64-row tiles).
  if (split.q) {
    const hipError_t e = launch_bwd_split_dq(split.q, q, dout, lse, delta, dq, heads, head_dim,
                                             softmax_scale, plan, stream);
    if (e != hipSuccess) return e;
  } else if (head_dim == 128) {
    hipLaunchKernelGGL((bwd_dq_kernel<128>), g_q, dim3(kThreads), 0, stream, qp, dp, lse, delta,
                       static_cast<__bf16*>(dq), heads, c_log2, softmax_scale, plan, n_qtiles);
  } else {
    hipLaunchKernelGGL((bwd_dq_kernel<64>), g_q, dim3(kThreads), 0, stream, qp, dp, lse, delta,
                       static_cast<__bf16*>(dq), heads, c_log2, softmax_scale, plan, n_qtiles);
  }
  if (split.k) {
    const hipError_t e = launch_bwd_split_dkv(split.k, q, dout, lse, delta, dk, dv, dak, dav, heads,
                                              head_dim, softmax_scale, plan, frame_runs, n_frames, stream);
    if (e != hipSuccess) return e;
  } else if (head_dim == 128) {
    hipLaunchKernelGGL((bwd_dkv_kernel<128>), g_k, dim3(kThreads), 0, stream, qp, dp, lse,
                       delta, dkp, dakp, dvp, davp, heads, c_log2, softmax_scale, plan, ku);
  } else {
    hipLaunchKernelGGL((bwd_dkv_kernel<64>), g_k, dim3(kThreads), 0, stream, qp, dp, lse,
                       delta, dkp, dakp, dvp, davp, heads, c_log2, softmax_scale, plan, ku);
  }
  return hipGetLastError();
}

}  // namespace ff
