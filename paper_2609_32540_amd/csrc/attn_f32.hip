// Float32 renderer attention (the float32 workloads) on the float32 matrix
// instructions, v_mfma_f32_16x16x4_f32.
//
// Work split: a workgroup = 8 waves = QT tiles of 16 queries of one head.  The
// waves share the queries and split the keys, 16-key blocks dealt round robin,
// each with its own running max, sum and O; the eight partial results are
// merged through LDS at the end.  The matrix rate bounds the kernel (32 cycles
// per 16 x 16 x 4 product, 2 * D * QT / 4 products per 16-key block), so K and
// V go straight from global memory to the registers the products read: one
// 16-byte load per lane feeds four products of each query tile, far below what
// the load path delivers, and no wave ever waits for another one inside the
// key loop.  Splitting keys (not queries) over the waves also fills the GPU
// when there are few queries: a launch has heads * ceil(nq / 16 QT) workgroups.
//
// Operands.  The four lane groups g of a product supply its four summands, and
// their order is free as long as A and B agree, so each lane's summands are
// chosen to be consecutive in memory:
//   S^T = K Q^T     product (t, e) sums d = 16 t + 4 g + e: lane (l16, g) loads
//                   K (and Q) row l16 at d = 16 t + 4 g as one 16-byte vector.
//                   Result: lane (l16, g) register j = key 4 g + j, query l16.
//   O^T += V^T P^T  product j sums keys 4 g + j, so P^T is the softmax register
//                   j itself; row i of d tile (h, e) is d = 64 h + 4 i + e: lane
//                   (l16, g) loads V row 4 g + j at d = 64 h + 4 l16.  Result:
//                   register j of tile (h, e) = d 64 h + 16 g + 4 j + e.
// K of the next block is loaded once the S products have consumed this block's
// K, V of the next block after the P V products: each load has the other half
// of the block (and the SIMD's second wave) to land.
//
// Against the kernel before it (one thread per query, fma from LDS, one
// workgroup per 128 queries): 12 heads x 128, 1170 queries over 7020 keys 14.4
// ms -> 0.54 ms (93 of the 153 TFLOP/s a large float32 product reaches here;
// 444 workgroups are 1.73 rounds of 256 CUs); 2 heads x 64, 192 queries over
// 704 keys 545 us -> 12 us.  Error against float64 5.5e-7 (1.9e-6 before:
// shorter sums).  The max is subtracted from a score before the factor log2 e
// is applied (one fma for both is 3% faster): the largest key's exponent is
// then exactly 0, where the fma would leave the rounding error of max * log2 e,
// which from scores of about 3e9 passes the float32 exponent range.

#include <hip/hip_runtime.h>

#include <float.h>
#include <math.h>

#include "attn_tile.h"
#include "ff_internal.h"

namespace ff {
namespace {

constexpr int kWaves = 8;                 // key groups of a workgroup
constexpr int kThreads = 64 * kWaves;
constexpr int kBK = 16;                   // keys per block
constexpr int kXcds = 8;
constexpr float kLog2e = 1.44269504f;

template <int D, int QT, class Src>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void attn_f32_kernel(const float* __restrict__ q, float* __restrict__ out, int nq, int heads,
                     float scale, Src src, int n_qtiles) {
  constexpr bool kPacked = __is_same(Src, PackedPlan);
  constexpr bool kBatch = __is_same(Src, KvBatch);
  constexpr bool kSets = kPacked || kBatch;
  constexpr int KT = D / 16;              // 16-byte vectors of a K (or Q) row per lane
  constexpr int VH = D / 64;              // 16-byte vectors of a V row per lane
  constexpr int kRows = 16 * QT;          // queries of the workgroup
  constexpr int kPitch = D + 4;           // padded row of the merge buffer (floats)
  __shared__ __attribute__((aligned(16))) float part[kWaves * kRows * kPitch];
  __shared__ float part_m[kWaves * kRows], part_l[kWaves * kRows];

  // Workgroups of one head run on one XCD where possible (they share its L2
  // for the head's K and V): contiguous ranges per XCD, or whole (set, head)
  // pairs round robin when the sets' lengths differ.
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
  const int q0 = (rest % n_qtiles) * kRows;
  if constexpr (kBatch) {
    q = static_cast<const float*>(src.q[chunk]);
    out = static_cast<float*>(src.out[chunk]);
  } else {
    q += int64_t(chunk) * nq * heads * D;
    out += int64_t(chunk) * nq * heads * D;
  }

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, l16 = lane & 15, grp = lane >> 4;

  f32x4 qreg[QT][KT];
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    const float* qp = q + (int64_t(min(q0 + 16 * t + l16, nq - 1)) * heads + head) * D + 4 * grp;
#pragma unroll
    for (int i = 0; i < KT; ++i) qreg[t][i] = *reinterpret_cast<const f32x4*>(qp + 16 * i) * scale;
  }
  f32x4 o[QT][VH][4];
  float m_run[QT], l_run[QT];
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    m_run[t] = -FLT_MAX;   // (finite: a key whose score is -inf then gets weight 0)
    l_run[t] = 0.0f;
#pragma unroll
    for (int h = 0; h < VH; ++h)
#pragma unroll
      for (int e = 0; e < 4; ++e) o[t][h][e] = f32x4{};
  }

  int n_segs;
  if constexpr (kPacked) n_segs = packed_num_segments(src, chunk);
  else if constexpr (kBatch) n_segs = src.set[chunk].n;
  else n_segs = src.n;
  auto segment = [&](int i) __attribute__((always_inline)) {
    if constexpr (kPacked) return packed_segment(src, chunk, i, heads, D, 4);
    else if constexpr (kBatch) return src.set[chunk].seg[i];
    else return src.seg[i];
  };

  // cursor of this wave: block blk of segment sg (blocks are numbered through
  // the segments; wave w takes blocks w, w + 8, ..)
  int sg = 0, blk = wave;
  KvSegment seg = segment(0);
  auto settle = [&]() __attribute__((always_inline)) {   // into the segment that holds blk
    while (sg < n_segs) {
      const int n = (seg.len + kBK - 1) / kBK;
      if (blk < n) break;
      blk -= n;
      if (++sg < n_segs) seg = segment(sg);
    }
  };
  f32x4 kreg[KT], vreg[4][VH];
  // rows past the segment's end re-read its last row (their scores are masked,
  // their V is zeroed)
  auto load_k = [&]() __attribute__((always_inline)) {
    const int row = min(blk * kBK + l16, seg.len - 1);
    const float* p = static_cast<const float*>(seg.k) + head * seg.head_stride +
                     int64_t(row) * seg.tok_stride + 4 * grp;
#pragma unroll
    for (int i = 0; i < KT; ++i) kreg[i] = *reinterpret_cast<const f32x4*>(p + 16 * i);
  };
  auto load_v = [&](const float* base, int tok_stride, int k0, int len) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int row = min(k0 + 4 * grp + j, len - 1);
      const float* p = base + int64_t(row) * tok_stride + 4 * l16;
#pragma unroll
      for (int h = 0; h < VH; ++h) vreg[j][h] = *reinterpret_cast<const f32x4*>(p + 64 * h);
    }
  };
  auto v_base = [&]() __attribute__((always_inline)) {
    return static_cast<const float*>(seg.v) + head * seg.head_stride;
  };

  settle();
  bool have = sg < n_segs;
  if (have) {
    load_k();
    load_v(v_base(), seg.tok_stride, blk * kBK, seg.len);
  }
  while (have) {
    f32x4 s[QT];
#pragma unroll
    for (int t = 0; t < QT; ++t) s[t] = f32x4{};
#pragma unroll
    for (int i = 0; i < KT; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int t = 0; t < QT; ++t)
          s[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(kreg[i][e], qreg[t][i][e], s[t], 0, 0, 0);
    const int n_valid = seg.len - blk * kBK;
    // the next block: its K now, its V once this block's V is consumed
    blk += kWaves;
    settle();
    have = sg < n_segs;
    if (have) load_k();

    bool raised = false;
    float alpha[QT];
#pragma unroll
    for (int t = 0; t < QT; ++t) {
      if (n_valid < kBK)
#pragma unroll
        for (int j = 0; j < 4; ++j) s[t][j] = 4 * grp + j < n_valid ? s[t][j] : -INFINITY;
      float mx = fmaxf(fmaxf(s[t][0], s[t][1]), fmaxf(s[t][2], s[t][3]));
      mx = fmaxf(m_run[t], max_across_groups(mx));
      alpha[t] = __builtin_amdgcn_exp2f((m_run[t] - mx) * kLog2e);
      raised |= mx != m_run[t];
      m_run[t] = mx;
    }
    if (__builtin_amdgcn_ballot_w64(raised) != 0) {
#pragma unroll
      for (int t = 0; t < QT; ++t) {
        l_run[t] *= alpha[t];
#pragma unroll
        for (int h = 0; h < VH; ++h)
#pragma unroll
          for (int e = 0; e < 4; ++e) o[t][h][e] *= alpha[t];
      }
    }
#pragma unroll
    for (int t = 0; t < QT; ++t) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        s[t][j] = __builtin_amdgcn_exp2f((s[t][j] - m_run[t]) * kLog2e);
      l_run[t] += (s[t][0] + s[t][1]) + (s[t][2] + s[t][3]);
    }
    if (n_valid < kBK)   // (probability 0 times an infinite last row would be NaN)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (4 * grp + j >= n_valid)
#pragma unroll
          for (int h = 0; h < VH; ++h) vreg[j][h] = f32x4{};
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int h = 0; h < VH; ++h)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int t = 0; t < QT; ++t)
            o[t][h][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(vreg[j][h][e], s[t][j], o[t][h][e], 0, 0, 0);
    if (have) load_v(v_base(), seg.tok_stride, blk * kBK, seg.len);
  }

  // merge the waves' partial results
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    const float l = sum_across_groups(l_run[t]);
    const int row = wave * kRows + 16 * t + l16;
    if (grp == 0) {
      part_m[row] = m_run[t];
      part_l[row] = l;
    }
#pragma unroll
    for (int h = 0; h < VH; ++h)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const f32x4 w = {o[t][h][0][j], o[t][h][1][j], o[t][h][2][j], o[t][h][3][j]};
        *reinterpret_cast<f32x4*>(part + row * kPitch + 64 * h + 16 * grp + 4 * j) = w;
      }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kRows * (D / 4); i += kThreads) {
    const int r = i / (D / 4), c = i % (D / 4);
    if (q0 + r >= nq) continue;
    float m = part_m[r];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) m = fmaxf(m, part_m[w * kRows + r]);
    float l = 0.0f;
    f32x4 acc = {};
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const float a = __builtin_amdgcn_exp2f((part_m[w * kRows + r] - m) * kLog2e);
      l += a * part_l[w * kRows + r];
      acc += a * *reinterpret_cast<const f32x4*>(part + (w * kRows + r) * kPitch + 4 * c);
    }
    *reinterpret_cast<f32x4*>(out + (int64_t(q0 + r) * heads + head) * D + 4 * c) = acc * (1.0f / l);
  }
}

// Query tiles per workgroup.  Two tiles halve the K and V loads per product;
// one tile gives twice the workgroups.  A launch takes ceil(workgroups / CUs)
// rounds of the GPU (one workgroup per CU), each as long as its tiles, so the
// form with the shorter sum of rounds is used and two tiles on a tie.
int query_tiles(int nq, int heads, int sets) {
  const int cus = device_cus();
  const auto rounds = [&](int qt) {
    return (int64_t((nq + 16 * qt - 1) / (16 * qt)) * heads * sets + cus - 1) / cus;
  };
  return 2 * rounds(2) <= rounds(1) ? 2 : 1;
}

template <class Src>
hipError_t launch(const float* q, float* out, int nq, int heads, int head_dim, float softmax_scale,
                  const Src& src, int sets, hipStream_t stream) {
  if (nq <= 0 || sets <= 0) return hipSuccess;
  const int qt = query_tiles(nq, heads, sets);
  const int n_qtiles = (nq + 16 * qt - 1) / (16 * qt);
  const dim3 grid(unsigned(n_qtiles * heads * sets));
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(kThreads), 0, stream, q, out, nq, heads, softmax_scale, src, n_qtiles);
    return hipGetLastError();
  };
  if (head_dim == 64)
    return qt == 2 ? go(attn_f32_kernel<64, 2, Src>) : go(attn_f32_kernel<64, 1, Src>);
  return qt == 2 ? go(attn_f32_kernel<128, 2, Src>) : go(attn_f32_kernel<128, 1, Src>);
}

}  // namespace

hipError_t launch_attention_f32(const void* q, void* out, int nq, int heads, int head_dim,
                                float softmax_scale, const KvSegments& segs, hipStream_t stream) {
  return launch(static_cast<const float*>(q), static_cast<float*>(out), nq, heads, head_dim,
                softmax_scale, segs, 1, stream);
}

hipError_t launch_attention_f32_batch(int nq, int heads, int head_dim, float softmax_scale,
                                      const KvBatch& b, hipStream_t stream) {
  return launch<KvBatch>(nullptr, nullptr, nq, heads, head_dim, softmax_scale, b, b.n, stream);
}

hipError_t launch_attention_f32_packed(const void* q, void* out, int heads, int head_dim,
                                       float softmax_scale, const PackedPlan& plan,
                                       hipStream_t stream) {
  return launch(static_cast<const float*>(q), static_cast<float*>(out), plan.chunk_tokens, heads,
                head_dim, softmax_scale, plan, plan.n_chunks, stream);
}

}  // namespace ff
