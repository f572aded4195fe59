// Backward of the packed attention for launches too small to fill the GPU with
// the 256-row workgroups of attn_bwd.hip (same gradients, same D_i pass before
// it): as in attn_bf16_split.hip, a workgroup = 8 waves that share T tiles of 16
// stationary rows (queries for dQ, keys for dK and dV) and split the streamed
// rows, 32-row blocks dealt round robin.  The partial sums are added through LDS
// at the end, in wave order: every gradient element is still written by one
// workgroup and is the same on every run.
//
// Each wave copies its own blocks of the two streamed tensors (K and V for dQ, Q
// and dO for dK and dV) HBM -> LDS, in whole rows, and no wave waits for
// another inside the stream.  A block is read as the row operand of S and dP and,
// transposed (ds_read_b64_tr_b16), as that of the gradient products, so its
// layout has to serve both: row-major, the 16-byte chunks of row r permuted by
// an XOR with swz(r), under which 16 rows at one chunk (a quarter-wave of a row
// read) and 8 rows at one pair of chunks (a half-wave of a transposing read)
// fall on distinct banks.
//
// Products on v_mfma_f32_16x16x32_bf16, operand layouts as in attn_bf16.hip:
// S^T (or S) and dP^T (or dP) of a block come out with lane (l16, g) holding
// stationary row l16 and streamed rows 4 g .. 4 g + 3 of each 16, which is the B
// operand of the gradient products once P and dS are rounded to bf16.

#include <hip/hip_runtime.h>

#include <math.h>

#include <cstring>

#include "attn_tile.h"
#include "ff_internal.h"

namespace ff {
namespace {

constexpr int kWaves = 8;
constexpr int kThreads = 64 * kWaves;
constexpr int kBR = 32;                       // streamed rows per block
constexpr int kXcds = 8;
constexpr int kMaxFrameRuns = 8;              // chunk runs that may see one anchor frame

template <int D, int T>
struct BwdCfg {
  static constexpr int KS = D / 32;           // 32-wide d slices
  static constexpr int DT = D / 16;           // 16-row d tiles of a gradient
  static constexpr int ROWB = 2 * D;
  static constexpr int BLOCK = kBR * ROWB;    // bytes of one tensor's block
  static constexpr int COPIES = BLOCK / 1024;
  static constexpr int kRows = 16 * T;
  static constexpr int kPitch = D + 4;        // padded row of the merge buffer (floats)
  static constexpr int kPart = kWaves * kRows * kPitch * 4;
  static constexpr int kBlocks = kWaves * 2 * BLOCK;
  static constexpr int kLds = kBlocks > kPart ? kBlocks : kPart;
};

// chunk permutation of row r (see above); r + 16 gives the same value
template <int D>
__device__ inline int swz(int r) {
  if constexpr (D == 128) return ((r & 7) << 1) | ((r >> 3) & 1);
  else return (((r >> 1) & 3) << 1) | ((r >> 3) & 1);
}

// One wave's view of its streamed rows: runs of rows of two token-major tensors
// (row r of the current run at a + r * row_bytes and b + r * row_bytes), blocks
// wave, wave + 8, .. of them.
template <int D>
struct Blocks {
  const char* a;
  const char* b;
  uint32_t row_bytes;
  int len;        // rows of the current run
  int blk;        // next block of the current run

  // copy block blk to LDS at dst (a, then b).  Rows past the run's end re-read
  // its last row.  Returns the block's valid rows.
  template <int T>
  __device__ __attribute__((always_inline)) int fetch(uint32_t dst, int lane) const {
    using C = BwdCfg<D, T>;
    constexpr uint32_t kSpan = 3072;
    constexpr int RPB = 1024 / C::ROWB, CPR = D / 8;   // rows per copy, chunks per row
    const int r0 = blk * kBR, last = len - 1 - r0;
    const int64_t off = int64_t(r0) * row_bytes - kSpan;
    int ln = lane;   // (keeps the per-lane offsets out of loop-invariant registers)
    asm volatile("" : "+v"(ln));
#pragma unroll
    for (int c = 0; c < C::COPIES; c += 4) {
      uint32_t o[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = (c + i) * RPB + ln / CPR;
        const int ch = (ln % CPR) ^ swz<D>(r);
        o[i] = uint32_t(min(r, last)) * row_bytes + (16u * ch + kSpan - 1024u * i);
      }
      lds_copy_blocks<4>(dst + 1024 * c, a + off, o);
      lds_copy_blocks<4>(dst + C::BLOCK + 1024 * c, b + off, o);
    }
    return last + 1;
  }
};

// row operand: rows 16 h + l16 (h = 0, 1), elements 32 s + 8 grp .. +7
template <int D, int T>
__device__ inline void read_rows(const char* t, int l16, int grp, bf16x8 (&x)[2][D / 32]) {
#pragma unroll
  for (int s = 0; s < D / 32; ++s) {
    const char* p = t + l16 * (2 * D) + (((4 * s + grp) ^ swz<D>(l16)) << 4);
#pragma unroll
    for (int h = 0; h < 2; ++h) x[h][s] = *reinterpret_cast<const bf16x8*>(p + h * 16 * 2 * D);
  }
}

// transposed operand: d tile dt (16 rows of d) x the 32 rows in the order the B
// operand holds them (4 grp .. +3, 16 + 4 grp .. +3)
template <int D>
__device__ inline void read_cols(const char* t, int l16, int grp, bf16x8 (&x)[D / 16]) {
  const int r = 4 * grp + (l16 >> 2);
#pragma unroll
  for (int dt = 0; dt < D / 16; ++dt) {
    const int ch = 2 * dt + ((l16 >> 1) & 1);
    const char* p = t + r * (2 * D) + ((ch ^ swz<D>(r)) << 4) + 8 * (l16 & 1);
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, p));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, p + 16 * 2 * D));
    const u32x2 lo2 = __builtin_bit_cast(u32x2, lo), hi2 = __builtin_bit_cast(u32x2, hi);
    const u32x4 u = {lo2[0], lo2[1], hi2[0], hi2[1]};
    x[dt] = __builtin_bit_cast(bf16x8, u);
  }
}

// r[h][t] = rows (h) x stationary tile t, summed over d
template <int D, int T>
__device__ inline void rows_product(const bf16x8 (&rows)[2][D / 32], const bf16x8 (&st)[T][D / 32],
                                    f32x4 (&r)[2][T]) {
#pragma unroll
  for (int s = 0; s < D / 32; ++s)
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int t = 0; t < T; ++t)
        r[h][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(rows[h][s], st[t][s],
                                                          s == 0 ? f32x4{} : r[h][t], 0, 0, 0);
}

// acc[dt][t] += cols^T x p (p packed: lane's rows 4 grp .. +3 of both halves)
template <int D, int T>
__device__ inline void cols_product(const bf16x8 (&cols)[D / 16], const uint32_t (&p)[T][4],
                                    f32x4 (&acc)[D / 16][T]) {
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const u32x4 u = {p[t][0], p[t][1], p[t][2], p[t][3]};
    const bf16x8 pb = __builtin_bit_cast(bf16x8, u);
#pragma unroll
    for (int dt = 0; dt < D / 16; ++dt)
      acc[dt][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(cols[dt], pb, acc[dt][t], 0, 0, 0);
  }
}

// stationary operand: rows row0 + 16 t + l16 (clamped to n - 1) of a token-major tensor
template <int D, int T>
__device__ inline void load_stationary(const __bf16* base, int64_t row_elems, int row0, int n,
                                       int l16, int grp, bf16x8 (&x)[T][D / 32]) {
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const __bf16* p = base + int64_t(min(row0 + 16 * t + l16, n - 1)) * row_elems + 8 * grp;
#pragma unroll
    for (int s = 0; s < D / 32; ++s) x[t][s] = *reinterpret_cast<const bf16x8*>(p + 32 * s);
  }
}

// Sum of the waves' acc over LDS, times scale, rounded to rows row0 .. of out.
// Every wave of the workgroup calls it; the LDS is free again afterwards.
template <int D, int T>
__device__ inline void merge_store(char* lds, const f32x4 (&acc)[D / 16][T], int wave, int l16,
                                   int grp, __bf16* out, int64_t row_elems, int row0, int n,
                                   float scale) {
  using C = BwdCfg<D, T>;
  float* part = reinterpret_cast<float*>(lds);
  __syncthreads();
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int dt = 0; dt < C::DT; ++dt)
      *reinterpret_cast<f32x4*>(part + (wave * C::kRows + 16 * t + l16) * C::kPitch + 16 * dt + 4 * grp) =
          acc[dt][t];
  __syncthreads();
  for (int i = threadIdx.x; i < C::kRows * (D / 8); i += kThreads) {
    const int r = i / (D / 8), c = i % (D / 8);
    if (row0 + r >= n) continue;
    f32x4 s[2] = {};
#pragma unroll
    for (int w = 0; w < kWaves; ++w)
#pragma unroll
      for (int x = 0; x < 2; ++x)
        s[x] += *reinterpret_cast<const f32x4*>(part + (w * C::kRows + r) * C::kPitch + 8 * c + 4 * x);
    u32x4 w4;
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      w4[2 * x] = pack_bf16(s[x][0] * scale, s[x][1] * scale);
      w4[2 * x + 1] = pack_bf16(s[x][2] * scale, s[x][3] * scale);
    }
    *reinterpret_cast<u32x4*>(out + int64_t(row0 + r) * row_elems + 8 * c) = w4;
  }
}

// groups of `group` workgroups that stream the same rows, dealt to the XCDs
// round robin; the last n % 8 groups in order
__device__ inline int xcd_groups(int b, int n_wg, int group) {
  const int n_groups = n_wg / group, n_even = n_groups - n_groups % kXcds;
  if (b >= n_even * group) return b;
  return (b % kXcds + kXcds * (b / kXcds / group)) * group + b / kXcds % group;
}

// ---- dQ ----------------------------------------------------------------------------------
template <int D, int T>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void bwd_split_dq_kernel(const __bf16* __restrict__ q, const __bf16* __restrict__ dout,
                         const float* __restrict__ lse, const float* __restrict__ delta,
                         __bf16* __restrict__ dq, int heads, float c_log2, float scale,
                         PackedPlan plan, int n_qtiles) {
  using C = BwdCfg<D, T>;
  __shared__ __attribute__((aligned(1024))) char lds[C::kLds];
  const int nq = plan.chunk_tokens;
  const int logical = xcd_groups(blockIdx.x, gridDim.x, n_qtiles);
  const int chunk = logical / (heads * n_qtiles);
  const int rest = logical - chunk * heads * n_qtiles;
  const int head = rest / n_qtiles, q0 = (rest % n_qtiles) * C::kRows;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, l16 = lane & 15, grp = lane >> 4;
  const int64_t row_elems = int64_t(heads) * D;
  const int64_t tok0 = int64_t(chunk) * nq;

  bf16x8 qs[T][C::KS], gs[T][C::KS];   // Q and dO
  load_stationary<D, T>(q + tok0 * row_elems + head * D, row_elems, q0, nq, l16, grp, qs);
  load_stationary<D, T>(dout + tok0 * row_elems + head * D, row_elems, q0, nq, l16, grp, gs);
  float L[T], Dq[T];
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const int64_t i = (tok0 + min(q0 + 16 * t + l16, nq - 1)) * heads + head;
    L[t] = lse[i];
    Dq[t] = delta[i];
  }
  f32x4 acc[C::DT][T];
#pragma unroll
  for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
    for (int t = 0; t < T; ++t) acc[dt][t] = f32x4{};

  const int n_segs = packed_num_segments(plan, chunk);
  Blocks<D> bl;
  bl.row_bytes = uint32_t(2 * row_elems);
  bl.blk = wave;
  int sg = -1;
  auto next_run = [&]() __attribute__((always_inline)) {
    if (++sg >= n_segs) return false;
    const KvSegment s = packed_segment(plan, chunk, sg, heads, D, 2);
    bl.a = static_cast<const char*>(s.k) + 2 * int64_t(head) * D;
    bl.b = static_cast<const char*>(s.v) + 2 * int64_t(head) * D;
    bl.len = s.len;
    return true;
  };
  auto settle = [&]() __attribute__((always_inline)) {   // into the run that holds blk
    while (sg < n_segs) {
      const int n = (bl.len + kBR - 1) / kBR;
      if (bl.blk < n) return true;
      bl.blk -= n;
      if (!next_run()) break;
    }
    return false;
  };
  char* kt = lds + wave * 2 * C::BLOCK;
  char* vt = kt + C::BLOCK;
  const uint32_t dst = uint32_t(size_t(LDS_PTR(char, kt)));
  auto fetch = [&]() __attribute__((always_inline)) {
    if (!settle()) return 0;
    const int nv = bl.template fetch<T>(dst, lane);
    bl.blk += kWaves;
    return nv;
  };
  next_run();
  for (int nv = fetch(); nv > 0;) {
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    asm volatile("" ::: "memory");
    f32x4 s[2][T], dp[2][T];
    {
      bf16x8 rows[2][C::KS];
      read_rows<D, T>(kt, l16, grp, rows);
      rows_product<D, T>(rows, qs, s);             // S^T = K Q^T
    }
    {
      bf16x8 rows[2][C::KS];
      read_rows<D, T>(vt, l16, grp, rows);
      rows_product<D, T>(rows, gs, dp);            // dP^T = V dO^T
    }
    bf16x8 cols[C::DT];
    read_cols<D>(kt, l16, grp, cols);
    __builtin_amdgcn_s_waitcnt(0xc07f);            // lgkmcnt(0): the block is read
    __builtin_amdgcn_sched_barrier(0);
    const int nv_next = fetch();
    __builtin_amdgcn_sched_barrier(0);
    uint32_t pk[T][4];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        float ds[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float p = __builtin_amdgcn_exp2f(fmaf(s[h][t][j], c_log2, -L[t]));
          ds[j] = 16 * h + 4 * grp + j < nv ? p * (dp[h][t][j] - Dq[t]) : 0.0f;
        }
        pk[t][2 * h] = pack_bf16(ds[0], ds[1]);
        pk[t][2 * h + 1] = pack_bf16(ds[2], ds[3]);
      }
    cols_product<D, T>(cols, pk, acc);             // dQ^T += K^T dS^T
    nv = nv_next;
  }
  merge_store<D, T>(lds, acc, wave, l16, grp, dq + tok0 * row_elems + head * D, row_elems, q0, nq, scale);
}

// ---- dK and dV ---------------------------------------------------------------------------
// Units of 16 T keys: upc per chunk, then upf per anchor frame.
struct SplitKeyUnits {
  int32_t upc, upf, n_frames;
  uint8_t frame_runs[64][2 * kMaxFrameRuns];   // per anchor frame: (first chunk, count) pairs
};

template <int D, int T>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void bwd_split_dkv_kernel(const __bf16* __restrict__ q, const __bf16* __restrict__ dout,
                          const float* __restrict__ lse, const float* __restrict__ delta,
                          __bf16* __restrict__ dk_chunks, __bf16* __restrict__ dk_anchor,
                          __bf16* __restrict__ dv_chunks, __bf16* __restrict__ dv_anchor, int heads,
                          float c_log2, float scale, PackedPlan plan, SplitKeyUnits ku) {
  using C = BwdCfg<D, T>;
  __shared__ __attribute__((aligned(1024))) char lds[C::kLds];
  __shared__ __attribute__((aligned(16))) float row_lds[kWaves][2 * kBR];   // L, then D, of a block
  const int nq = plan.chunk_tokens, G = plan.frame_tokens;
  const int n_units = plan.n_chunks * ku.upc + ku.n_frames * ku.upf;
  // (contiguous ranges of units of one head per XCD: neighbours stream the same rows)
  const int per = gridDim.x / kXcds, rem = gridDim.x % kXcds, xcd = blockIdx.x % kXcds;
  const int logical = xcd * per + min(xcd, rem) + blockIdx.x / kXcds;
  const int head = logical / n_units, unit = logical - head * n_units;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, l16 = lane & 15, grp = lane >> 4;
  const int64_t row_elems = int64_t(heads) * D;
  const bool is_chunk = unit < plan.n_chunks * ku.upc;
  int owner, k0, n_keys;
  const __bf16 *kbase, *vbase;
  __bf16 *okbase, *ovbase;
  if (is_chunk) {
    owner = unit / ku.upc;
    k0 = (unit % ku.upc) * C::kRows;
    n_keys = nq;
    const int64_t o = int64_t(owner) * nq * row_elems + head * D;
    kbase = static_cast<const __bf16*>(plan.k) + o;
    vbase = static_cast<const __bf16*>(plan.v) + o;
    okbase = dk_chunks + o;
    ovbase = dv_chunks + o;
  } else {
    const int a = unit - plan.n_chunks * ku.upc;
    owner = a / ku.upf;
    k0 = (a % ku.upf) * C::kRows;
    n_keys = G;
    const int64_t o = int64_t(owner) * G * row_elems + head * D;
    kbase = static_cast<const __bf16*>(plan.ak) + o;
    vbase = static_cast<const __bf16*>(plan.av) + o;
    okbase = dk_anchor + o;
    ovbase = dv_anchor + o;
  }
  bf16x8 ks[T][C::KS], vs[T][C::KS];
  load_stationary<D, T>(kbase, row_elems, k0, n_keys, l16, grp, ks);
  load_stationary<D, T>(vbase, row_elems, k0, n_keys, l16, grp, vs);
  f32x4 acc_k[C::DT][T], acc_v[C::DT][T];
#pragma unroll
  for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
    for (int t = 0; t < T; ++t) {
      acc_k[dt][t] = f32x4{};
      acc_v[dt][t] = f32x4{};
    }

  Blocks<D> bl;
  bl.row_bytes = uint32_t(2 * row_elems);
  bl.blk = wave;
  int run = -1;
  int64_t run_tok = 0;     // first token of the current run
  auto next_run = [&]() __attribute__((always_inline)) {
    ++run;
    int c0, c1;
    if (is_chunk) {
      if (run > 0) return false;
      c0 = owner;
      c1 = min(owner + min(plan.window, plan.n_chunks) + 1, plan.n_chunks);
    } else {
      if (run >= kMaxFrameRuns || ku.frame_runs[owner][2 * run + 1] == 0) return false;
      c0 = ku.frame_runs[owner][2 * run];
      c1 = c0 + ku.frame_runs[owner][2 * run + 1];
    }
    run_tok = int64_t(c0) * nq;
    bl.a = reinterpret_cast<const char*>(q + run_tok * row_elems + head * D);
    bl.b = reinterpret_cast<const char*>(dout + run_tok * row_elems + head * D);
    bl.len = (c1 - c0) * nq;
    return true;
  };
  bool more = next_run();
  auto settle = [&]() __attribute__((always_inline)) {
    while (more) {
      const int n = (bl.len + kBR - 1) / kBR;
      if (bl.blk < n) return true;
      bl.blk -= n;
      more = next_run();
    }
    return false;
  };
  char* qt = lds + wave * 2 * C::BLOCK;
  char* gt = qt + C::BLOCK;
  const uint32_t dst = uint32_t(size_t(LDS_PTR(char, qt)));
  float row_val = 0.0f;   // lanes 0 .. 31: L of the fetched block's rows, 32 .. 63: D
  auto fetch = [&]() __attribute__((always_inline)) {
    if (!settle()) return 0;
    const int64_t i = (run_tok + min(bl.blk * kBR + (lane & 31), bl.len - 1)) * heads + head;
    row_val = lane < 32 ? lse[i] : delta[i];
    const int nv = bl.template fetch<T>(dst, lane);
    bl.blk += kWaves;
    return nv;
  };
  for (int nv = fetch(); nv > 0;) {
    row_lds[wave][lane] = row_val;
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    asm volatile("" ::: "memory");
    f32x4 s[2][T], dp[2][T];
    {
      bf16x8 rows[2][C::KS];
      read_rows<D, T>(qt, l16, grp, rows);
      rows_product<D, T>(rows, ks, s);             // S = Q K^T
    }
    {
      bf16x8 rows[2][C::KS];
      read_rows<D, T>(gt, l16, grp, rows);
      rows_product<D, T>(rows, vs, dp);            // dP = dO V^T
    }
    uint32_t pk[T][4], dk[T][4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const f32x4 L = *reinterpret_cast<const f32x4*>(&row_lds[wave][16 * h + 4 * grp]);
      const f32x4 Dq = *reinterpret_cast<const f32x4*>(&row_lds[wave][kBR + 16 * h + 4 * grp]);
#pragma unroll
      for (int t = 0; t < T; ++t) {
        float p[4], ds[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          p[j] = __builtin_amdgcn_exp2f(fmaf(s[h][t][j], c_log2, -L[j]));
          p[j] = 16 * h + 4 * grp + j < nv ? p[j] : 0.0f;
          ds[j] = p[j] * (dp[h][t][j] - Dq[j]);
        }
#pragma unroll
        for (int x = 0; x < 2; ++x) {
          pk[t][2 * h + x] = pack_bf16(p[2 * x], p[2 * x + 1]);
          dk[t][2 * h + x] = pack_bf16(ds[2 * x], ds[2 * x + 1]);
        }
      }
    }
    bf16x8 cols[C::DT];
    read_cols<D>(gt, l16, grp, cols);
    cols_product<D, T>(cols, pk, acc_v);           // dV^T += dO^T P
    read_cols<D>(qt, l16, grp, cols);
    __builtin_amdgcn_s_waitcnt(0xc07f);            // lgkmcnt(0): the block is read
    __builtin_amdgcn_sched_barrier(0);
    nv = fetch();
    __builtin_amdgcn_sched_barrier(0);
    cols_product<D, T>(cols, dk, acc_k);           // dK^T += Q^T dS
  }
  merge_store<D, T>(lds, acc_k, wave, l16, grp, okbase, row_elems, k0, n_keys, scale);
  merge_store<D, T>(lds, acc_v, wave, l16, grp, ovbase, row_elems, k0, n_keys, 1.0f);
}

}  // namespace

hipError_t launch_bwd_split_dq(int tiles, const void* q, const void* dout, const float* lse,
                               const float* delta, void* dq, int heads, int head_dim,
                               float softmax_scale, const PackedPlan& plan, hipStream_t stream) {
  const float c = float(double(softmax_scale) * 1.4426950408889634);
  const int n_qtiles = (plan.chunk_tokens + 16 * tiles - 1) / (16 * tiles);
  const dim3 grid(unsigned(plan.n_chunks * heads * n_qtiles));
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(kThreads), 0, stream, static_cast<const __bf16*>(q),
                       static_cast<const __bf16*>(dout), lse, delta, static_cast<__bf16*>(dq), heads,
                       c, softmax_scale, plan, n_qtiles);
    return hipGetLastError();
  };
  if (head_dim == 64)
    return tiles == 2 ? go(bwd_split_dq_kernel<64, 2>) : go(bwd_split_dq_kernel<64, 1>);
  return tiles == 2 ? go(bwd_split_dq_kernel<128, 2>) : go(bwd_split_dq_kernel<128, 1>);
}

hipError_t launch_bwd_split_dkv(int tiles, const void* q, const void* dout, const float* lse,
                                const float* delta, void* dk, void* dv, void* dak, void* dav,
                                int heads, int head_dim, float softmax_scale, const PackedPlan& plan,
                                const uint8_t (*frame_runs)[16], int n_frames, hipStream_t stream) {
  const float c = float(double(softmax_scale) * 1.4426950408889634);
  if (head_dim != 64) tiles = 1;
  SplitKeyUnits ku;
  std::memset(&ku, 0, sizeof(ku));
  ku.upc = (plan.chunk_tokens + 16 * tiles - 1) / (16 * tiles);
  ku.upf = (plan.frame_tokens + 16 * tiles - 1) / (16 * tiles);
  ku.n_frames = n_frames;
  for (int f = 0; f < n_frames; ++f) std::memcpy(ku.frame_runs[f], frame_runs[f], 16);
  const dim3 grid(unsigned((plan.n_chunks * ku.upc + n_frames * ku.upf) * heads));
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(kThreads), 0, stream, static_cast<const __bf16*>(q),
                       static_cast<const __bf16*>(dout), lse, delta, static_cast<__bf16*>(dk),
                       static_cast<__bf16*>(dak), static_cast<__bf16*>(dv), static_cast<__bf16*>(dav),
                       heads, c, softmax_scale, plan, ku);
    return hipGetLastError();
  };
  if (head_dim == 64)
    return tiles == 2 ? go(bwd_split_dkv_kernel<64, 2>) : go(bwd_split_dkv_kernel<64, 1>);
  return go(bwd_split_dkv_kernel<128, 1>);   // (two tiles do not fit the registers)
}

}  // namespace ff
