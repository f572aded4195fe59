// bf16 renderer attention for launches too small to fill the GPU with the
// 256-query workgroups of attn_bf16.hip: the waves of a workgroup share the
// queries and split the keys.
//
// Work split: a workgroup = 8 waves = QT tiles of 16 queries of one head, the
// key blocks (32 keys) dealt round robin to the waves, each with its own sum and
// O; the eight partial results are merged through LDS.
// A launch has heads * ceil(nq / 16 QT) workgroups, 8 to 16 times those of the
// 256-query kernel, and a wave's serial chain is an eighth of the keys.  In
// exchange every workgroup reads all of its head's K and V (the 256-query
// kernel shares each tile among 256 queries), so the load path bounds the
// kernel once the GPU is full (attention_bf16_split_tiles draws the line).
//
// Operands as in attn_bf16.hip (S^T = K Q^T and O^T += V^T P^T on
// v_mfma_f32_16x16x32_bf16, P^T straight from the softmax registers).  Each
// wave copies its own blocks HBM -> LDS (global_load_lds) and takes a block's K
// and V operands into registers before its products, which frees the LDS for
// the next block's copy: that copy runs under this block's products and
// softmax, and one 16 KB pair per wave is all the LDS a wave needs.  Nothing is
// shared between waves inside the key loop but the first block's max, so it has
// one barrier, in each wave's first step.
//
// Rounding.  Every wave starts from the reference max of the 256-query kernel,
// the column max of the read set's first 32 keys (wave 0's first block), so each
// probability is rounded to bf16 relative to the same reference as there, and
// O is divided by the same sums.  A query's reference moves by its own scores
// only: its result does not depend on which queries share its workgroup, nor on
// QT.  Against a reference of each wave's own this costs 1 us of 8.2 (2 heads x
// 128, 198 queries over 726 keys) and of 18.8 (6 heads x 64, packed clip of 7 x
// 351 tokens).

#include <hip/hip_runtime.h>

#include <float.h>
#include <math.h>

#include "attn_tile.h"
#include "ff_internal.h"

namespace ff {
namespace {

constexpr int kWaves = 8;
constexpr int kThreads = 64 * kWaves;
constexpr int kBK = 32;                  // keys per block
constexpr int kXcds = 8;
constexpr float kRaise = 56.0f;          // log2 units the column max may exceed the reference by:
                                         // sums of 2^56 times the keys stay far inside float32

template <int D, int QT>
struct SplitCfg {
  static constexpr int KS = D / 32;            // 32-wide d slices of S^T
  static constexpr int DT = D / 16;            // 16-row d tiles of O^T
  static constexpr int BLOCK = kBK * 2 * D;    // bytes of one K (or V) block
  static constexpr int COPIES = BLOCK / 1024;  // 1 KB copies of it
  static constexpr int kRows = 16 * QT;
  static constexpr int kPitch = D + 4;         // padded row of the merge buffer (floats)
  static constexpr int kPart = kWaves * kRows * (kPitch + 2) * 4;
  static constexpr int kLds = kWaves * 2 * BLOCK > kPart ? kWaves * 2 * BLOCK : kPart;
};

template <int D, int QT, class Src>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void attn_bf16_split_kernel(const __bf16* __restrict__ q, __bf16* __restrict__ out, int nq,
                            int heads, float scale_log2, Src src, int n_qtiles) {
  constexpr bool kPacked = __is_same(Src, PackedPlan);
  constexpr bool kBatch = __is_same(Src, KvBatch);
  constexpr bool kSets = kPacked || kBatch;
  using C = SplitCfg<D, QT>;
  __shared__ __attribute__((aligned(1024))) char lds[C::kLds];
  __shared__ float ref_max[C::kRows];

  // as in attn_f32.hip: contiguous ranges of workgroups per XCD, or whole
  // (set, head) pairs round robin when the sets' lengths differ
  const int b = blockIdx.x;
  int logical = b;
  if constexpr (kSets) {
    const int n_pairs = gridDim.x / n_qtiles;
    const int n_even = n_pairs - n_pairs % kXcds;
    if (b < n_even * n_qtiles)
      logical = (b % kXcds + kXcds * (b / kXcds / n_qtiles)) * n_qtiles + b / kXcds % n_qtiles;
  } else {
    const int per = gridDim.x / kXcds, rem = gridDim.x % kXcds, xcd = b % kXcds;
    logical = xcd * per + min(xcd, rem) + b / kXcds;
  }
  int chunk = 0;
  if constexpr (kSets) chunk = logical / (heads * n_qtiles);
  const int rest = logical - chunk * heads * n_qtiles;
  const int head = rest / n_qtiles;
  const int q0 = (rest % n_qtiles) * C::kRows;
  if constexpr (kBatch) {
    q = static_cast<const __bf16*>(src.q[chunk]);
    out = static_cast<__bf16*>(src.out[chunk]);
  } else {
    q += int64_t(chunk) * nq * heads * D;
    out += int64_t(chunk) * nq * heads * D;
  }

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, l16 = lane & 15, grp = lane >> 4;

  bf16x8 qreg[QT][C::KS];
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    const __bf16* qp = q + (int64_t(min(q0 + 16 * t + l16, nq - 1)) * heads + head) * D + 8 * grp;
#pragma unroll
    for (int s = 0; s < C::KS; ++s) qreg[t][s] = *reinterpret_cast<const bf16x8*>(qp + 32 * s);
  }
  f32x4 o[C::DT][QT];
  float m_run[QT], l_run[QT];
  f32x4 lsum[QT];            // row sums (every row of the tile holds the sum)
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    m_run[t] = -FLT_MAX;     // (finite: keys that score -inf get weight 0)
    l_run[t] = 0.0f;
    lsum[t] = f32x4{};
#pragma unroll
    for (int dt = 0; dt < C::DT; ++dt) o[dt][t] = f32x4{};
  }

  int n_segs;
  if constexpr (kPacked) n_segs = packed_num_segments(src, chunk);
  else if constexpr (kBatch) n_segs = src.set[chunk].n;
  else n_segs = src.n;
  auto segment = [&](int i) __attribute__((always_inline)) {
    if constexpr (kPacked) return packed_segment(src, chunk, i, heads, D, 2);
    else if constexpr (kBatch) return src.set[chunk].seg[i];
    else return src.seg[i];
  };
  // cursor of the next block to fetch: block blk of segment sg (wave w takes
  // blocks w, w + 8, .. of the read set)
  int sg = 0, blk = wave;
  KvSegment seg = segment(0);
  auto settle = [&]() __attribute__((always_inline)) {
    while (sg < n_segs) {
      const int n = (seg.len + kBK - 1) / kBK;
      if (blk < n) break;
      blk -= n;
      if (++sg < n_segs) seg = segment(sg);
    }
    return sg < n_segs;
  };

  // The wave's K and V block in LDS.  1 KB copies, 16 bytes per lane, lane l at
  // 16 l; the lanes of a quad (K) or octet (V) take consecutive bytes of one row,
  // and their order inside it is permuted so that reads are free of bank
  // conflicts:
  //   K copy (kh, ks): rows 16 kh + l / 4, 64-byte slice ks; position l % 4 holds
  //     chunk (l % 4) ^ (row / 4).  Operand read: row 16 kh + l16, chunk grp.
  //   V copy (G, H): rows 8 G + l / 8, 128-byte slice H; position l % 8 holds chunk
  //     (l % 8) ^ 2 (row / 2).  Transposing read of d tile 4 H + p: lane group grp
  //     reads key rows 4 grp .. +3 (and 16 + those), lane l16 8 bytes of row l16 / 4.
  char* kbuf = lds + wave * 2 * C::BLOCK;
  char* vbuf = kbuf + C::BLOCK;
  const int k_lane = 64 * l16 + 16 * (grp ^ (l16 >> 2));
  int v_lane[4];
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const int r = 4 * grp + (l16 >> 2);
    v_lane[p] = (r >> 3) * (16 * D) + 128 * (r & 7) + 32 * (p ^ ((r & 7) >> 1)) + 8 * (l16 & 3);
  }

  // Copy the cursor's block.  Rows past the segment's end re-read its last row
  // (their scores are masked).  Returns the block's valid keys and moves the
  // cursor on.
  auto fetch = [&]() __attribute__((always_inline)) {
    constexpr uint32_t kSpan = 3072;   // largest immediate offset of four copies
    const uint32_t row_bytes = 2u * uint32_t(seg.tok_stride);
    const int k0 = blk * kBK, last = seg.len - 1 - k0;
    const int64_t off = 2 * int64_t(head) * seg.head_stride + int64_t(k0) * row_bytes - kSpan;
    const char* vb = static_cast<const char*>(seg.v) + off;
    const char* kb = static_cast<const char*>(seg.k) + off;
    const uint32_t kdst = uint32_t(size_t(LDS_PTR(char, kbuf)));
    int ln = lane;   // (keeps the per-lane offsets out of loop-invariant registers)
    asm volatile("" : "+v"(ln));
#pragma unroll
    for (int c = 0; c < C::COPIES; c += 4) {
      uint32_t koff[4], voff[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int kr = 16 * ((c + i) / C::KS) + (ln >> 2);
        const int kch = 4 * ((c + i) % C::KS) + ((ln & 3) ^ (ln >> 4));
        const int vr = 8 * ((c + i) / (D / 64)) + (ln >> 3);
        const int vch = 8 * ((c + i) % (D / 64)) + ((ln & 7) ^ (2 * (ln >> 4)));
        koff[i] = uint32_t(min(kr, last)) * row_bytes + (16u * kch + kSpan - 1024u * i);
        voff[i] = uint32_t(min(vr, last)) * row_bytes + (16u * vch + kSpan - 1024u * i);
      }
      lds_copy_blocks<4>(kdst + 1024 * c, kb, koff);
      lds_copy_blocks<4>(kdst + C::BLOCK + 1024 * c, vb, voff);
    }
    blk += kWaves;
    return last + 1;
  };

  // S^T of a block from its K operands (rows 16 kh + l16, d slice ks), keys past
  // n_valid masked, and the column max of each query
  auto scores = [&](const bf16x8 (&kc)[2][C::KS], int n_valid, f32x4 (&s)[2][QT], float (&mx)[QT])
      __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < C::KS; ++ks)
#pragma unroll
      for (int kh = 0; kh < 2; ++kh)
#pragma unroll
        for (int t = 0; t < QT; ++t)
          s[kh][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kc[kh][ks], qreg[t][ks],
                                                             ks == 0 ? f32x4{} : s[kh][t], 0, 0, 0);
    if (n_valid < kBK)
#pragma unroll
      for (int kh = 0; kh < 2; ++kh)
#pragma unroll
        for (int t = 0; t < QT; ++t)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            s[kh][t][j] = 4 * grp >= n_valid - 16 * kh - j ? -INFINITY : s[kh][t][j];
#pragma unroll
    for (int t = 0; t < QT; ++t) {
      mx[t] = fmaxf(fmaxf(s[0][t][0], s[0][t][1]), fmaxf(s[0][t][2], s[0][t][3]));
      mx[t] = fmaxf(mx[t], fmaxf(fmaxf(s[1][t][0], s[1][t][1]), fmaxf(s[1][t][2], s[1][t][3])));
      mx[t] = max_across_groups(mx[t]) * scale_log2;
    }
  };

  // The barrier behind wave 0's reference max, which every wave passes once: in
  // its first step or, without a block, before the merge.  (Written out: copies
  // in flight need no wait.)
  auto publish_barrier = []() __attribute__((always_inline)) {
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0): the max is written
    asm volatile("s_barrier" ::: "memory");
  };

  // One block: take its K and V into registers, start the copy of the next one
  // into their place (when there is one), then S^T, softmax and O^T.  Returns
  // the next block's valid keys, 0 without one.  The wave's first step also takes
  // the reference max from wave 0, whose first block is the read set's.
  auto step = [&](int n_valid, bool first) __attribute__((always_inline)) {
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    asm volatile("" ::: "memory");
    bf16x8 kc[2][C::KS], va[C::DT];
#pragma unroll
    for (int kh = 0; kh < 2; ++kh)
#pragma unroll
      for (int ks = 0; ks < C::KS; ++ks)
        kc[kh][ks] = *reinterpret_cast<const bf16x8*>(kbuf + k_lane + 1024 * (kh * C::KS + ks));
#pragma unroll
    for (int dt = 0; dt < C::DT; ++dt) {
      const char* vt = vbuf + v_lane[dt % 4] + 1024 * (dt / 4);
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, vt));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, vt + 32 * D));
      const u32x2 lo2 = __builtin_bit_cast(u32x2, lo), hi2 = __builtin_bit_cast(u32x2, hi);
      const u32x4 au = {lo2[0], lo2[1], hi2[0], hi2[1]};
      va[dt] = __builtin_bit_cast(bf16x8, au);
    }
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0): the reads are done
    __builtin_amdgcn_sched_barrier(0);
    const int nv_next = settle() ? fetch() : 0;
    __builtin_amdgcn_sched_barrier(0);
    f32x4 s[2][QT];
    float mx[QT];
    scores(kc, n_valid, s, mx);
    if (first) {
      if (wave == 0 && grp == 0) {
#pragma unroll
        for (int t = 0; t < QT; ++t) ref_max[16 * t + l16] = mx[t];
      }
      publish_barrier();
#pragma unroll
      for (int t = 0; t < QT; ++t) m_run[t] = fmaxf(ref_max[16 * t + l16], -FLT_MAX);
    }
    // a query's reference follows its column max once that is kRaise above it
    bool over = false;
#pragma unroll
    for (int t = 0; t < QT; ++t) over |= mx[t] > m_run[t] + kRaise;
    if (__builtin_amdgcn_ballot_w64(over) != 0) {
#pragma unroll
      for (int t = 0; t < QT; ++t) {
        const float m_new = mx[t] > m_run[t] + kRaise ? mx[t] : m_run[t];
        const float alpha = __builtin_amdgcn_exp2f(m_run[t] - m_new);
        l_run[t] *= alpha;
        lsum[t] *= alpha;
        m_run[t] = m_new;
#pragma unroll
        for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
          for (int j = 0; j < 4; ++j) o[dt][t][j] *= alpha;
      }
    }
    uint32_t pk[QT][4];
#pragma unroll
    for (int t = 0; t < QT; ++t) {
      float lb = 0.0f;
#pragma unroll
      for (int kh = 0; kh < 2; ++kh)
#pragma unroll
        for (int j = 0; j < 4; j += 2) {
          const float p0 = __builtin_amdgcn_exp2f(fmaf(s[kh][t][j], scale_log2, -m_run[t]));
          const float p1 = __builtin_amdgcn_exp2f(fmaf(s[kh][t][j + 1], scale_log2, -m_run[t]));
          pk[t][2 * kh + (j >> 1)] = pack_bf16(p0, p1);
          if constexpr (kPacked) lb += p0 + p1;
        }
      l_run[t] += lb;
    }
    // (all ones: every row of the result is the column sum of P^T)
    const bf16x8 ones = {__bf16(1.0f), __bf16(1.0f), __bf16(1.0f), __bf16(1.0f),
                         __bf16(1.0f), __bf16(1.0f), __bf16(1.0f), __bf16(1.0f)};
#pragma unroll
    for (int t = 0; t < QT; ++t) {
      const u32x4 pu = {pk[t][0], pk[t][1], pk[t][2], pk[t][3]};
      const bf16x8 pb = __builtin_bit_cast(bf16x8, pu);
#pragma unroll
      for (int dt = 0; dt < C::DT; ++dt)
        o[dt][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va[dt], pb, o[dt][t], 0, 0, 0);
      lsum[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pb, lsum[t], 0, 0, 0);
    }
    return nv_next;
  };

  int nv = settle() ? fetch() : 0;
  if (nv == 0) publish_barrier();
  for (bool first = true; nv > 0; first = false) nv = step(nv, first);

  // merge the waves' partial results (over the K and V blocks, once all are read)
  __syncthreads();
  float* part = reinterpret_cast<float*>(lds);
  float* part_m = part + kWaves * C::kRows * C::kPitch;
  float* part_l = part_m + kWaves * C::kRows;
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    // the sum of the rounded probabilities, as O adds them up; of the unrounded
    // ones where the log-sum-exp is written (as in the 256-query kernel)
    float l = lsum[t][0];
    if constexpr (kPacked)
      if (src.lse != nullptr) l = sum_across_groups(l_run[t]);
    const int row = wave * C::kRows + 16 * t + l16;
    if (grp == 0) {
      part_m[row] = m_run[t];
      part_l[row] = l;
    }
#pragma unroll
    for (int dt = 0; dt < C::DT; ++dt)
      *reinterpret_cast<f32x4*>(part + row * C::kPitch + 16 * dt + 4 * grp) = o[dt][t];
  }
  __syncthreads();
  for (int i = threadIdx.x; i < C::kRows * (D / 8); i += kThreads) {
    const int r = i / (D / 8), c = i % (D / 8);
    if (q0 + r >= nq) continue;
    float m = part_m[r];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) m = fmaxf(m, part_m[w * C::kRows + r]);
    float l = 0.0f;
    f32x4 acc[2] = {};
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const int row = w * C::kRows + r;
      const float a = __builtin_amdgcn_exp2f(part_m[row] - m);
      l += a * part_l[row];
#pragma unroll
      for (int x = 0; x < 2; ++x)
        acc[x] += a * *reinterpret_cast<const f32x4*>(part + row * C::kPitch + 8 * c + 4 * x);
    }
    const float inv = 1.0f / l;
    u32x4 w4;
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      w4[2 * x] = pack_bf16(acc[x][0] * inv, acc[x][1] * inv);
      w4[2 * x + 1] = pack_bf16(acc[x][2] * inv, acc[x][3] * inv);
    }
    *reinterpret_cast<u32x4*>(out + (int64_t(q0 + r) * heads + head) * D + 8 * c) = w4;
    if constexpr (kPacked)
      if (src.lse != nullptr && c == 0)
        src.lse[(int64_t(chunk) * nq + q0 + r) * heads + head] = m + log2f(l);
  }
}

template <class Src>
hipError_t launch(int qt, const void* q, void* out, int nq, int heads, int head_dim,
                  float softmax_scale, const Src& src, int sets, hipStream_t stream) {
  const float c = float(double(softmax_scale) * 1.4426950408889634);
  const int n_qtiles = (nq + 16 * qt - 1) / (16 * qt);
  const dim3 grid(unsigned(n_qtiles * heads * sets));
  last_launch.query_tiles = qt;
  last_launch.key_parts = 1;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(kThreads), 0, stream, static_cast<const __bf16*>(q),
                       static_cast<__bf16*>(out), nq, heads, c, src, n_qtiles);
    return hipGetLastError();
  };
  if (head_dim == 64)
    return qt == 2 ? go(attn_bf16_split_kernel<64, 2, Src>) : go(attn_bf16_split_kernel<64, 1, Src>);
  return qt == 2 ? go(attn_bf16_split_kernel<128, 2, Src>) : go(attn_bf16_split_kernel<128, 1, Src>);
}

}  // namespace

// The line between this kernel and the 256-query one is drawn by their
// estimated times, a fixed part (launch, prologue, merge) plus the rounds of
// the GPU times the 64-key tiles one workgroup walks.  The constants are fits
// to 1 to 24 heads x 63 to 1170 queries x 189 to 7020 keys, each kernel forced
// (us): 2 heads x 198 queries x 1188 keys 24.5 against 9.4 (QT 1) and 12.5 (QT
// 2) at d = 128; 12 x 351 x 2106 29.4 / 24.4 / 17.0; 12 x 1170 x 7020 65 / 129 /
// 83, where every CU has work and the copies (each workgroup its own K and V)
// bound this kernel.  (Taken before the waves shared a reference max, which adds
// about 1 us to each form of it: less than the fits' scatter.)
int attention_bf16_split_tiles(int nq, int heads, int head_dim, int sets, double tiles_mean,
                               double tiles_max, double whole_tiles, bool merged) {
  struct Cost { double fixed, tile; };   // us, us per tile
  const bool wide = head_dim == 128;
  const Cost whole = wide ? Cost{7.0, 1.63} : Cost{6.0, 1.01};
  const Cost one = wide ? Cost{4.5, 0.29} : Cost{4.0, 0.17};
  const Cost two = wide ? Cost{6.5, 0.36} : Cost{5.0, 0.23};
  constexpr double kMerge = 9.0;
  constexpr double kMargin = 0.95;   // near a tie the 256-query kernel, which reads less
  const int cus = device_cus();
  const auto split_us = [&](int qt, const Cost& c) {
    const int64_t groups = int64_t((nq + 16 * qt - 1) / (16 * qt)) * heads * sets;
    return c.fixed + c.tile * fmax(tiles_max, tiles_mean * double((groups + cus - 1) / cus));
  };
  const double t0 = kMargin * (whole.fixed + whole_tiles * whole.tile + (merged ? kMerge : 0.0));
  const double t1 = split_us(1, one), t2 = split_us(2, two);
  if (t0 <= t1 && t0 <= t2) return 0;
  return t1 <= t2 ? 1 : 2;
}

hipError_t launch_attention_bf16_split(int qt, const void* q, void* out, int nq, int heads,
                                       int head_dim, float softmax_scale, const KvSegments& segs,
                                       hipStream_t stream) {
  return launch(qt, q, out, nq, heads, head_dim, softmax_scale, segs, 1, stream);
}

hipError_t launch_attention_bf16_split_batch(int qt, int nq, int heads, int head_dim,
                                             float softmax_scale, const KvBatch& b,
                                             hipStream_t stream) {
  return launch(qt, nullptr, nullptr, nq, heads, head_dim, softmax_scale, b, b.n, stream);
}

hipError_t launch_attention_bf16_split_packed(int qt, const void* q, void* out, int heads,
                                              int head_dim, float softmax_scale,
                                              const PackedPlan& plan, hipStream_t stream) {
  return launch(qt, q, out, plan.chunk_tokens, heads, head_dim, softmax_scale, plan, plan.n_chunks,
                stream);
}

}  // namespace ff
