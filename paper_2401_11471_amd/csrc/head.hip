// Classifier head, loss and parameter update of a full training step
// (Algorithm 1: fully connected FP, Loss, fully connected BP, and the update
// of every kernel and of the fully connected weights). The trunk's output y
// ([B][H][W][C] NHWC, flattened per image to K = H*W*C features) feeds one
// fully connected layer (fc_w [n_classes][K], fc_b [n_classes], float32);
// the loss is softmax cross-entropy averaged over the batch; the update is
// plain SGD. Every reduction runs in a fixed order, so results are
// reproducible run to run.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <string>
#include <type_traits>

#include "lrcnn.h"
#include "plan.hpp"

namespace lrcnn {
namespace {

constexpr int kMaxClasses = 64;
// Features per block of the logits pass. The pass reads every class's
// weights once per image (from L2 after the first) and is bound by how many
// blocks share that: VGG-16's 25088 features and 8 images make 104 blocks
// of 2048 (32 blocks of kWsChunk left the chip idle: 143 us, and the float32
// training step on VGG-16's last block 1.43 ms; now 1.22 ms with the fused
// passes below). The partial sums of
// the finer chunks go into dy, which the last pass of the call overwrites:
// K / 2048 x 64 classes x 4 bytes per image always fit its K x 2 bytes. With
// K <= 2048 there is one chunk, and it goes to the workspace, which holds
// the sums of chunks of kWsChunk features; so do the sums of a call whose dy
// shares memory with an input (dy written over y).
constexpr int kChunk = 2048, kWsChunk = 8192;

typedef uint16_t bf16;
__device__ __forceinline__ float ld(const float *p) { return *p; }
__device__ __forceinline__ float ld(const bf16 *p) {
  return __uint_as_float((uint32_t)(*p) << 16);
}
// float32 -> bfloat16, round to nearest, ties to even (NaN kept quiet)
__device__ __forceinline__ void st(float *p, float v) { *p = v; }
__device__ __forceinline__ void st(bf16 *p, float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7f800000u) == 0x7f800000u && (u & 0x007fffffu)) {
    *p = (bf16)((u >> 16) | 0x40u);
    return;
  }
  u += 0x7fffu + ((u >> 16) & 1u);
  *p = (bf16)(u >> 16);
}

// N consecutive values (4: one access)
template <int N>
__device__ __forceinline__ void ldn(const float *p, float (&v)[N]) {
  if constexpr (N == 4) {
    const float4 q = *(const float4 *)p;
    v[0] = q.x, v[1] = q.y, v[2] = q.z, v[3] = q.w;
  } else {
    v[0] = *p;
  }
}
template <int N>
__device__ __forceinline__ void ldn(const bf16 *p, float (&v)[N]) {
  if constexpr (N == 4) {
    const uint2 q = *(const uint2 *)p;
    v[0] = __uint_as_float(q.x << 16), v[1] = __uint_as_float(q.x & 0xffff0000u);
    v[2] = __uint_as_float(q.y << 16), v[3] = __uint_as_float(q.y & 0xffff0000u);
  } else {
    v[0] = ld(p);
  }
}
template <int N>
__device__ __forceinline__ void stn(float *p, const float (&v)[N]) {
  if constexpr (N == 4) *(float4 *)p = make_float4(v[0], v[1], v[2], v[3]);
  else *p = v[0];
}
template <int N>
__device__ __forceinline__ void stn(bf16 *p, const float (&v)[N]) {
  bf16 t[N];
#pragma unroll
  for (int i = 0; i < N; ++i) st(t + i, v[i]);
  if constexpr (N == 4)
    *(uint2 *)p = make_uint2((uint32_t)t[0] | ((uint32_t)t[1] << 16),
                             (uint32_t)t[2] | ((uint32_t)t[3] << 16));
  else *p = t[0];
}

// part[b][chunk][c] = sum over the chunk's features k of y[b, k] * fc_w[c, k]:
// each thread sums its strided vectors of V features, a wave its lanes' sums
// as a fixed tree, and the four waves' sums are added in order. (Thread
// after thread in LDS, the 256 sums of a class took 7 us by themselves.)
template <typename T, int V>
__global__ __launch_bounds__(256) void head_partial_kernel(const T *y, const float *fw,
                                                           long long K, int C, int chunks,
                                                           int chunk, float *part) {
  __shared__ float red[kMaxClasses][4];
  const int ch = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
  const long long k0 = (long long)ch * chunk;
  const long long k1 = k0 + chunk < K ? k0 + chunk : K;
  float acc[kMaxClasses];
#pragma unroll
  for (int c = 0; c < kMaxClasses; ++c) acc[c] = 0.f;
  const T *yb = y + (long long)b * K;
  for (long long k = k0 + tid * V; k < k1; k += 256 * V) {
    float v[V];
    ldn<V>(yb + k, v);
#pragma unroll
    for (int c = 0; c < kMaxClasses; ++c)
      if (c < C) {
        float w[V];
        ldn<V>(fw + (long long)c * K + k, w);
#pragma unroll
        for (int e = 0; e < V; ++e) acc[c] += v[e] * w[e];
      }
  }
#pragma unroll
  for (int c = 0; c < kMaxClasses; ++c)
    if (c < C) {
      float s = acc[c];
#pragma unroll
      for (int d = 32; d > 0; d >>= 1) s += __shfl_down(s, d);
      if ((tid & 63) == 0) red[c][tid >> 6] = s;
    }
  __syncthreads();
  if (tid < C)
    part[((long long)b * chunks + ch) * C + tid] =
        ((red[tid][0] + red[tid][1]) + red[tid][2]) + red[tid][3];
}

// One block: logits (a thread per image and class), softmax, per-sample loss
// and dL/dlogits = (p - onehot)/B for every sample, then the mean loss and
// dL/dfc_b (sums over samples in sample order). A label outside [0, C)
// makes its loss term NaN; nothing is read out of bounds.
__global__ __launch_bounds__(256) void head_softmax_kernel(const float *part, int chunks,
                                                           const float *fb,
                                                           const int32_t *labels, int B,
                                                           int C, float *logits, float *dlog,
                                                           float *lossv, float *loss,
                                                           float *dfb) {
  const int tid = threadIdx.x;
  for (long long i = tid; i < (long long)B * C; i += 256) {
    const long long b = i / C;
    const int c = (int)(i - b * C);
    float s = fb[c];
#pragma unroll 8
    for (int ch = 0; ch < chunks; ++ch) s += part[(b * chunks + ch) * C + c];
    logits[i] = s;
  }
  __syncthreads();
  for (int b = tid; b < B; b += 256) {
    const float *z = logits + (long long)b * C;
    float m = -INFINITY;
#pragma unroll 8
    for (int c = 0; c < C; ++c) m = fmaxf(m, z[c]);
    float se = 0.f;
#pragma unroll 8
    for (int c = 0; c < C; ++c) se += expf(z[c] - m);
    const int lab = labels[b];
    const float lse = m + logf(se);
    lossv[b] = lse - (lab >= 0 && lab < C ? z[lab] : NAN);
#pragma unroll 8
    for (int c = 0; c < C; ++c)
      dlog[(long long)b * C + c] = (expf(z[c] - lse) - (c == lab ? 1.f : 0.f)) / (float)B;
  }
  __syncthreads();
  if (tid == 0) {
    float s = 0.f;
    for (int b = 0; b < B; ++b) s += lossv[b];
    *loss = s / (float)B;
  }
  if (tid < C) {
    float s = 0.f;
    for (int b = 0; b < B; ++b) s += dlog[(long long)b * C + tid];
    dfb[tid] = s;
  }
}

// dy[b, k] = sum_c dlog[b, c] * fc_w[c, k] (storage dtype) and
// dfc_w[c, k] = sum_b dlog[b, c] * y[b, k], V features per thread, in one
// launch (they do not depend on each other). Vectors [from, to) of the two, so
// that a call with a gradient written over an input runs dy before dfc_w.
template <typename T, int V>
__global__ void head_grad_kernel(const float *dlog, const float *fw, const T *y, long long K,
                                 int B, int C, T *dy, float *dfw, long long from, long long to) {
  const long long KV = K / V, ny = (long long)B * KV;
  for (long long i = from + (long long)blockIdx.x * blockDim.x + threadIdx.x; i < to;
       i += (long long)gridDim.x * blockDim.x) {
    const bool isy = i < ny;
    const long long j = isy ? i : i - ny;
    const long long r = j / KV, k = (j - r * KV) * V;
    float s[V], v[V];
#pragma unroll
    for (int e = 0; e < V; ++e) s[e] = 0.f;
    if (isy) {
#pragma unroll 8
      for (int c = 0; c < C; ++c) {
        ldn<V>(fw + (long long)c * K + k, v);
#pragma unroll
        for (int e = 0; e < V; ++e) s[e] += dlog[r * C + c] * v[e];
      }
      stn<V>(dy + r * K + k, s);
    } else {
#pragma unroll 8
      for (int b = 0; b < B; ++b) {
        ldn<V>(y + (long long)b * K + k, v);
#pragma unroll
        for (int e = 0; e < V; ++e) s[e] += dlog[(long long)b * C + r] * v[e];
      }
      stn<V>(dfw + r * K + k, s);
    }
  }
}

// theta <- theta - lr * g for up to kSgdSegs parameter tensors in one launch
// (a launch per tensor costs more than the tensor for all but the largest),
// computed in float32 and stored in theta's dtype. Block runs of 1024
// elements; a segment whose pointers are not 16-byte aligned goes element by
// element.
constexpr int kSgdSegs = 24;
struct SgdSeg {
  void *w;
  const float *g;
  long long n;
  int bf, vec;
};
struct SgdBatch {
  int n;
  SgdSeg seg[kSgdSegs];
  long long start[kSgdSegs + 1];  // first block run of each segment
};
template <typename T>
__device__ __forceinline__ void sgd_run(const SgdSeg &g, long long i0, float lr) {
  T *w = (T *)g.w;
  const long long i = i0 + 4 * threadIdx.x;
  if (g.vec && i + 4 <= g.n) {
    float a[4], d[4];
    ldn<4>(w + i, a);
    ldn<4>(g.g + i, d);
#pragma unroll
    for (int e = 0; e < 4; ++e) a[e] = a[e] - lr * d[e];
    stn<4>(w + i, a);
    return;
  }
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (i + e < g.n) st(w + i + e, ld(w + i + e) - lr * g.g[i + e]);
}
__global__ __launch_bounds__(256) void sgd_kernel(SgdBatch sb, float lr) {
  for (long long r = blockIdx.x; r < sb.start[sb.n]; r += gridDim.x) {
    int s = 0;
    while (s + 1 < sb.n && r >= sb.start[s + 1]) ++s;
    const SgdSeg &g = sb.seg[s];
    const long long i0 = (r - sb.start[s]) * 1024;
    if (g.bf) sgd_run<bf16>(g, i0, lr);
    else sgd_run<float>(g, i0, lr);
  }
}

// Collects the tensors of one update; a tensor that overlaps one already
// collected (shared weights) starts a new launch, so updates stay in order.
struct SgdQueue {
  SgdBatch b{};
  float lr;
  hipStream_t s;
  void flush() {
    if (b.n && b.start[b.n] > 0)
      sgd_kernel<<<(unsigned)(b.start[b.n] < 65536 ? b.start[b.n] : 65536), 256, 0, s>>>(b, lr);
    b.n = 0;
  }
  void add(void *w, const float *g, long long n, bool bf) {
    if (n <= 0) return;
    const uintptr_t lo = (uintptr_t)w, hi = lo + (uintptr_t)n * (bf ? 2 : 4);
    bool over = b.n == kSgdSegs;
    for (int i = 0; i < b.n && !over; ++i) {
      const SgdSeg &q = b.seg[i];
      const uintptr_t ql = (uintptr_t)q.w, qh = ql + (uintptr_t)q.n * (q.bf ? 2 : 4);
      over = lo < qh && ql < hi;
    }
    if (over) flush();
    if (b.n == 0) b.start[0] = 0;
    const bool vec = ((uintptr_t)w & (bf ? 7 : 15)) == 0 && ((uintptr_t)g & 15) == 0;
    b.seg[b.n] = SgdSeg{w, g, n, bf ? 1 : 0, vec ? 1 : 0};
    b.start[b.n + 1] = b.start[b.n] + (n + 1023) / 1024;
    ++b.n;
  }
};

unsigned blocks_for(long long n) {
  long long g = (n + 255) / 256;
  if (g > 65536) g = 65536;
  return (unsigned)(g < 1 ? 1 : g);
}

struct HeadLayout {
  long long K;
  int B, chunks, ws_chunks;
  size_t part, dlog, lossv, total;
};
HeadLayout head_layout(const Plan &P, int C) {
  HeadLayout h;
  const Shape &s = P.shp[P.n - 1];
  h.K = (long long)s.h * s.w * s.c;
  h.B = P.cfg.batch;
  h.chunks = (int)((h.K + kChunk - 1) / kChunk);
  h.ws_chunks = (int)((h.K + kWsChunk - 1) / kWsChunk);
  auto a256 = [](size_t x) { return (x + 255) & ~(size_t)255; };
  h.part = 0;
  h.dlog = a256((size_t)h.B * h.ws_chunks * C * 4);
  h.lossv = a256(h.dlog + (size_t)h.B * C * 4);
  h.total = a256(h.lossv + (size_t)h.B * 4);
  return h;
}

bool misaligned(const void *p) { return ((uintptr_t)p & 15u) != 0; }
bool overlap(const void *a, size_t na, const void *b, size_t nb) {
  return (uintptr_t)a < (uintptr_t)b + nb && (uintptr_t)b < (uintptr_t)a + na;
}

}  // namespace
}  // namespace lrcnn

using lrcnn::Plan;

extern "C" int lrcnn_head_workspace_bytes(const lrcnn_plan_t *plan, int32_t n_classes,
                                          size_t *bytes) {
  if (!plan || !bytes) return lrcnn_fail(LRCNN_EINVAL, "null plan or output");
  if (n_classes < 1 || n_classes > lrcnn::kMaxClasses)
    return lrcnn_fail(LRCNN_EINVAL, "n_classes must be in [1, 64]");
  *bytes = lrcnn::head_layout(*reinterpret_cast<const Plan *>(plan), n_classes).total;
  return LRCNN_OK;
}

extern "C" int lrcnn_head_loss(const lrcnn_plan_t *plan, const void *y, const float *fc_w,
                               const float *fc_b, const int32_t *labels, int32_t n_classes,
                               float *logits, float *loss, void *dy, float *d_fc_w,
                               float *d_fc_b, void *head_ws, size_t head_ws_bytes,
                               void *stream) {
  using namespace lrcnn;
  if (!plan) return lrcnn_fail(LRCNN_EINVAL, "null plan");
  if (n_classes < 1 || n_classes > kMaxClasses)
    return lrcnn_fail(LRCNN_EINVAL, "n_classes must be in [1, 64]");
  const void *ptrs[] = {y, fc_w, fc_b, labels, logits, loss, dy, d_fc_w, d_fc_b, head_ws};
  for (const void *p : ptrs)
    if (!p || misaligned(p)) return lrcnn_fail(LRCNN_EINVAL, "null or misaligned head argument");
  const Plan &P = *reinterpret_cast<const Plan *>(plan);
  const HeadLayout h = head_layout(P, n_classes);
  if (head_ws_bytes < h.total)
    return lrcnn_fail(LRCNN_EWORKSPACE, "head workspace needs " + std::to_string(h.total) +
                                            " bytes, got " + std::to_string(head_ws_bytes));
  hipStream_t s = (hipStream_t)stream;
  char *ws = (char *)head_ws;
  float *dlog = (float *)(ws + h.dlog), *lossv = (float *)(ws + h.lossv);
  const int C = n_classes;
  const bool bf = P.cfg.dtype == LRCNN_BF16;
  // gradients may be written over inputs: dy over y (d_fc_w then comes from
  // what is left there), d_fc_w over fc_w
  const size_t ny = (size_t)h.B * h.K * (bf ? 2 : 4), nw = (size_t)C * h.K * 4;
  const bool dy_in = overlap(dy, ny, y, ny) || overlap(dy, ny, fc_w, nw) ||
                     overlap(dy, ny, fc_b, (size_t)C * 4) || overlap(dy, ny, labels, (size_t)h.B * 4);
  const bool in_place = dy_in || overlap(d_fc_w, nw, fc_w, nw) || overlap(d_fc_w, nw, y, ny);
  const bool in_dy = h.chunks > 1 && !dy_in;
  float *part = in_dy ? (float *)dy : (float *)(ws + h.part);
  const int chunk = in_dy ? kChunk : kWsChunk, chunks = in_dy ? h.chunks : h.ws_chunks;
  dim3 g1(chunks, h.B);
  // (4-wide accesses when every image's and class's row keeps them aligned)
  const bool v4 = h.K % 4 == 0;
  auto partial = [&](auto *yp) {
    using T = std::remove_const_t<std::remove_pointer_t<decltype(yp)>>;
    if (v4) head_partial_kernel<T, 4><<<g1, 256, 0, s>>>(yp, fc_w, h.K, C, chunks, chunk, part);
    else head_partial_kernel<T, 1><<<g1, 256, 0, s>>>(yp, fc_w, h.K, C, chunks, chunk, part);
  };
  auto grads = [&](auto *yp) {
    using T = std::remove_const_t<std::remove_pointer_t<decltype(yp)>>;
    const long long kv = h.K / (v4 ? 4 : 1), mid = h.B * kv, end = mid + C * kv;
    auto run = [&](long long from, long long to) {
      const unsigned g = blocks_for(to - from);
      if (v4)
        head_grad_kernel<T, 4><<<g, 256, 0, s>>>(dlog, fc_w, yp, h.K, h.B, C, (T *)dy, d_fc_w,
                                                 from, to);
      else
        head_grad_kernel<T, 1><<<g, 256, 0, s>>>(dlog, fc_w, yp, h.K, h.B, C, (T *)dy, d_fc_w,
                                                 from, to);
    };
    if (in_place) {
      run(0, mid);
      run(mid, end);
    } else {
      run(0, end);
    }
  };
  if (bf) partial((const bf16 *)y);
  else partial((const float *)y);
  head_softmax_kernel<<<1, 256, 0, s>>>(part, chunks, fc_b, labels, h.B, C, logits, dlog,
                                        lossv, loss, d_fc_b);
  if (bf) grads((const bf16 *)y);
  else grads((const float *)y);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess)
    return lrcnn_fail(LRCNN_EHIP, std::string("head: ") + hipGetErrorString(e));
  return LRCNN_OK;
}

extern "C" int lrcnn_sgd_update(const lrcnn_plan_t *plan, float lr, void *const *w,
                                float *const *dw, float *fc_w, const float *d_fc_w,
                                float *fc_b, const float *d_fc_b, int32_t n_classes,
                                void *stream) {
  using namespace lrcnn;
  if (!plan || !w || !dw) return lrcnn_fail(LRCNN_EINVAL, "null plan or parameter array");
  const Plan &P = *reinterpret_cast<const Plan *>(plan);
  hipStream_t s = (hipStream_t)stream;
  const bool bf = P.cfg.dtype == LRCNN_BF16;
  SgdQueue q;
  q.lr = lr;
  q.s = s;
  for (int v = 1; v < P.n; ++v) {
    const lrcnn_node &d = P.nodes[v];
    if (d.op != LRCNN_OP_CONV) continue;
    if (!w[v] || !dw[v] || misaligned(w[v]) || misaligned(dw[v]))
      return lrcnn_fail(LRCNN_EINVAL, "weights or dw of node " + std::to_string(v) +
                                          " null or misaligned");
    q.add(w[v], dw[v], (long long)d.c_out * d.kh * d.kw * P.shp[d.in0].c, bf);
  }
  if (fc_w || fc_b) {
    if (!fc_w || !d_fc_w || !fc_b || !d_fc_b || n_classes < 1)
      return lrcnn_fail(LRCNN_EINVAL, "head parameters and gradients must all be given");
    const Shape &o = P.shp[P.n - 1];
    const long long nw = (long long)n_classes * o.h * o.w * o.c;
    q.add(fc_w, d_fc_w, nw, false);
    q.add(fc_b, d_fc_b, n_classes, false);
  }
  q.flush();
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess)
    return lrcnn_fail(LRCNN_EHIP, std::string("sgd: ") + hipGetErrorString(e));
  return LRCNN_OK;
}
