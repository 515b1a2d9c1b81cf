// Decoder-block pieces around the fake-ternary linears: RMSNorm, SwiGLU and the
// routing / permutation of the routed-expert MLP (gfx950).  All are streaming
// kernels bound by HBM bandwidth; rows are processed with 16-byte accesses.
#include <cmath>
#include <type_traits>

#include "kernels.h"

namespace catq {

// ------------------------------------------------------------- block sums

template <int NT>
__device__ __forceinline__ float block_sum(float v, float* red) {
  v = wave_sum(v);
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  if (l == 0) red[w] = v;
  __syncthreads();
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < NT / 64; ++i) s += red[i];
  __syncthreads();
  return s;
}

template <int NT>
__device__ __forceinline__ float block_max(float v, float* red) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v = fmaxf(v, __shfl_xor(v, m, 64));
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  if (l == 0) red[w] = v;
  __syncthreads();
  float r = 0.f;
#pragma unroll
  for (int i = 0; i < NT / 64; ++i) r = fmaxf(r, red[i]);
  __syncthreads();
  return r;
}

// -------------------------------------------------- activation quantization
// Symmetric 8-bit absmax fake quantization (the W1.58A8 setting) of each
// group of `group` consecutive values of a row: s = max|x| / 127,
// q = round-half-even(x / s) clamped to [-127, 127] (0 when s = 0),
// y = bf16(q * s); every step in IEEE fp32.  One workgroup per (row, group):
// a pass for the maximum, a second (from L2) for the codes.  y may alias x.
template <typename XT>
__global__ __launch_bounds__(256) void act_quant_kernel(const XT* x, int64_t n, int64_t group,
                                                        bf16* y) {
  __shared__ float red[4];
  const int64_t off = (int64_t)blockIdx.x * n + (int64_t)blockIdx.y * group;
  const XT* xr = x + off;
  bf16* yr = y + off;
  const int64_t nc = group / 8;
  float m = 0.f;
  for (int64_t c = threadIdx.x; c < nc; c += 256) {
    float v[8];
    load8<XT>(xr + c * 8, v);
#pragma unroll
    for (int j = 0; j < 8; ++j) m = fmaxf(m, fabsf(v[j]));
  }
  m = block_max<256>(m, red);
  const float s = m / 127.0f;
  for (int64_t c = threadIdx.x; c < nc; c += 256) {
    float v[8];
    load8<XT>(xr + c * 8, v);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float q = s > 0.f ? fminf(fmaxf(rintf(v[j] / s), -127.f), 127.f) : 0.f;
      v[j] = q * s;
    }
    store8<bf16>(yr + c * 8, v);
  }
}

// ---------------------------------------------------------------- RMSNorm

template <typename XT>
__global__ __launch_bounds__(256) void rmsnorm_fwd_kernel(const XT* x, int64_t n, float eps,
                                                          bf16* y, float* rstd) {
  __shared__ float red[4];
  const int64_t row = blockIdx.x;
  const XT* xr = x + row * n;
  const int64_t nc = n / 8;
  float ss = 0.f;
  for (int64_t c = threadIdx.x; c < nc; c += 256) {
    float v[8];
    load8<XT>(xr + c * 8, v);
#pragma unroll
    for (int j = 0; j < 8; ++j) ss = fmaf(v[j], v[j], ss);
  }
  ss = block_sum<256>(ss, red);
  const float r = 1.0f / sqrtf(ss / (float)n + eps);
  if (threadIdx.x == 0 && rstd) rstd[row] = r;
  for (int64_t c = threadIdx.x; c < nc; c += 256) {
    float v[8];
    load8<XT>(xr + c * 8, v);
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] *= r;
    store8<bf16>(y + row * n + c * 8, v);
  }
}

template <typename XT>
__global__ __launch_bounds__(256) void rmsnorm_bwd_kernel(const XT* x, const float* rstd,
                                                          const bf16* dy, const bf16* dres,
                                                          int64_t n, bf16* dx) {
  __shared__ float red[4];
  const int64_t row = blockIdx.x;
  const int64_t nc = n / 8;
  float sd = 0.f;
  for (int64_t c = threadIdx.x; c < nc; c += 256) {
    float a[8], b[8];
    load8<XT>(x + row * n + c * 8, a);
    load8<bf16>(dy + row * n + c * 8, b);
#pragma unroll
    for (int j = 0; j < 8; ++j) sd = fmaf(a[j], b[j], sd);
  }
  sd = block_sum<256>(sd, red);
  const float r = rstd[row];
  const float coef = r * r * r * sd / (float)n;
  for (int64_t c = threadIdx.x; c < nc; c += 256) {
    float a[8], b[8], d[8];
    load8<XT>(x + row * n + c * 8, a);
    load8<bf16>(dy + row * n + c * 8, b);
    if (dres)
      load8<bf16>(dres + row * n + c * 8, d);
    else
#pragma unroll
      for (int j = 0; j < 8; ++j) d[j] = 0.f;
#pragma unroll
    for (int j = 0; j < 8; ++j) a[j] = fmaf(r, b[j], fmaf(-a[j], coef, d[j]));
    store8<bf16>(dx + row * n + c * 8, a);
  }
}

// ---------------------------------------------------------------- SwiGLU


__global__ __launch_bounds__(256) void swiglu_fwd_kernel(const bf16* gu, int64_t rows, int64_t F,
                                                         bf16* a) {
  const int64_t nc = F / 8;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= rows * nc) return;
  const int64_t r = i / nc, c = i % nc;
  float g[8], u[8];
  load8<bf16>(gu + r * 2 * F + c * 8, g);
  load8<bf16>(gu + r * 2 * F + F + c * 8, u);
#pragma unroll
  for (int j = 0; j < 8; ++j) g[j] = swiglu1(g[j], u[j]);
  store8<bf16>(a + r * F + c * 8, g);
}

__global__ __launch_bounds__(256) void swiglu_bwd_kernel(const bf16* gu, const bf16* da,
                                                         int64_t rows, int64_t F, bf16* dgu) {
  const int64_t nc = F / 8;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= rows * nc) return;
  const int64_t r = i / nc, c = i % nc;
  float g[8], u[8], d[8], dg[8], du[8];
  load8<bf16>(gu + r * 2 * F + c * 8, g);
  load8<bf16>(gu + r * 2 * F + F + c * 8, u);
  load8<bf16>(da + r * F + c * 8, d);
#pragma unroll
  for (int j = 0; j < 8; ++j) swiglu1_bwd(g[j], u[j], d[j], dg[j], du[j]);
  store8<bf16>(dgu + r * 2 * F + c * 8, dg);
  store8<bf16>(dgu + r * 2 * F + F + c * 8, du);
}

// ---------------------------------------------------------------- routing

// Logits in order as integers: a larger logit has a larger key, -0 and +0 the
// same, a NaN the lowest of all (0).
__device__ __forceinline__ unsigned int logit_key(float x) {
  if (x != x) return 0u;
  const unsigned int u = x == 0.0f ? 0u : __float_as_uint(x);
  return (u >> 31) ? ~u : u | 0x80000000u;
}
__device__ __forceinline__ float key_logit(unsigned int key) {
  if (key == 0u) return __builtin_nanf("");
  return __uint_as_float((key >> 31) ? key & 0x7fffffffu : ~key);
}

// One wavefront per token: top-k of the E >= k logits (largest first; equal
// values go to the lower expert id, NaN after every other) and the softmax over
// the k selected logits.  An expert is selected once whatever the logits hold:
// the ids index rows and experts, so they are valid and distinct also where
// logits are NaN or -inf (then it is the weights that turn NaN or 0).  PER logits
// per lane (E <= 64 PER).
template <int PER>
__global__ __launch_bounds__(256) void moe_topk_kernel(const float* logits, int64_t T, int E,
                                                       int k, int32_t* ids, float* w) {
  const int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (t >= T) return;
  unsigned int key[PER];
  unsigned int open = 0;   // bit i: expert lane + 64 i not selected yet
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int e = lane + 64 * i;
    key[i] = e < E ? logit_key(logits[t * E + e]) : 0u;
    open |= e < E ? 1u << i : 0u;
  }
  float sel = -INFINITY;   // lane j: the j-th selected logit and its expert
  int sid = 0;
  for (int j = 0; j < k; ++j) {
    // lane-local best (lowest id among equals), then across lanes
    unsigned int bk = 0u;
    int be = 0x7fffffff;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int e = lane + 64 * i;
      if (((open >> i) & 1u) && (key[i] > bk || (key[i] == bk && e < be))) {
        bk = key[i];
        be = e;
      }
    }
    for (int mk = 32; mk >= 1; mk >>= 1) {
      const unsigned int ok = __shfl_xor(bk, mk, 64);
      const int oe = __shfl_xor(be, mk, 64);
      if (ok > bk || (ok == bk && oe < be)) {
        bk = ok;
        be = oe;
      }
    }
    if (lane == j) {
      sel = key_logit(bk);
      sid = be;
    }
    if ((be & 63) == lane) open &= ~(1u << (be >> 6));
  }
  const float ex = expf(sel - __shfl(sel, 0, 64));
  float sum = 0.f;
  for (int j = 0; j < k; ++j) sum += __shfl(ex, j, 64);
  if (lane < k) {
    ids[t * k + lane] = sid;
    w[t * k + lane] = ex * (1.0f / sum);
  }
}

// Rows by expert: workgroup e counts the ids below e (the expert's first row)
// and its own, then gives every (token, slot) of the expert its row, in token
// order.  Each wave takes a contiguous segment of the ids, 256 at a time with
// one ballot per 64; only the waves' totals are shared, so the two passes cost a
// few loads in latency (a scan of 256 ids at a time through LDS, after a count
// and an offset kernel, took 132 us for 24000 ids of 64 experts, this 10 us).
constexpr int kRankWaves = 16;
__global__ __launch_bounds__(kRankWaves * 64) void moe_rank_kernel(const int32_t* ids, int64_t n,
                                                                   int E, int64_t* off,
                                                                   int32_t* perm_row) {
  __shared__ int64_t below[kRankWaves], mine[kRankWaves];
  const int e = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t seg = ((n + kRankWaves - 1) / kRankWaves + 255) / 256 * 256;
  const int64_t i0 = min(wave * seg, n), i1 = min(i0 + seg, n);
  auto load = [&](int64_t c, int (&id)[4]) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t i = c + 64 * u + lane;
      id[u] = i < i1 ? ids[i] : 0x7fffffff;
    }
  };
  int64_t lt = 0, eq = 0;
  for (int64_t c = i0; c < i1; c += 256) {
    int id[4];
    load(c, id);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      lt += __popcll(__ballot(id[u] < e));
      eq += __popcll(__ballot(id[u] == e));
    }
  }
  if (lane == 0) {
    below[wave] = lt;
    mine[wave] = eq;
  }
  __syncthreads();
  int64_t first = 0, before = 0, total = 0;
#pragma unroll
  for (int w = 0; w < kRankWaves; ++w) {
    first += below[w];
    before += w < wave ? mine[w] : 0;
    total += mine[w];
  }
  if (threadIdx.x == 0) {
    off[e] = first;
    if (e == E - 1) off[E] = first + total;
  }
  int64_t row = first + before;
  for (int64_t c = i0; c < i1; c += 256) {
    int id[4];
    load(c, id);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const unsigned long long m = __ballot(id[u] == e);
      if (id[u] == e)
        perm_row[c + 64 * u + lane] = (int32_t)(row + __popcll(m & ((1ull << lane) - 1)));
      row += __popcll(m);
    }
  }
}

// Rows between token order and expert order.  One block per token (and 2048
// columns): its row is read once and written to its k slots, or its k slots'
// rows are read four at a time (all in flight) and summed in slot order.  One
// block per slot moved one 16-byte load per thread and latency bounded it: 3000
// tokens x 8 slots of 2048 columns, gather 29.6 -> 18.4 us (6 TB/s), combine's
// backward 29.7 -> 18.8 us.  The slots' rows and weights are loaded four at a
// time too: one after the other they are a chain of k latencies, all that a few
// tokens take (64 tokens x 8: gather 3.8 -> 3.3 us, combine's backward 4.4 -> 3.5).
// With one slot there is nothing to batch.
template <typename F>
__device__ __forceinline__ void slot_batches(int k, F&& f) {
  if (k == 1) {
    f(0, std::integral_constant<int, 1>{});
    return;
  }
  for (int s0 = 0; s0 < k; s0 += 4) f(s0, std::integral_constant<int, 4>{});
}

__global__ __launch_bounds__(256) void moe_gather_kernel(const bf16* x, const int32_t* perm,
                                                         int k, int64_t h, bf16* xg) {
  const int64_t t = blockIdx.x;
  const int32_t* dst = perm + t * k;
  for (int64_t c = (int64_t)blockIdx.y * 256 + threadIdx.x; c < h / 8; c += (int64_t)gridDim.y * 256) {
    const u32x4 v = *reinterpret_cast<const u32x4*>(x + t * h + c * 8);
    slot_batches(k, [&](int s0, auto u_c) {
      constexpr int U = decltype(u_c)::value;
      int32_t d[U];
#pragma unroll
      for (int u = 0; u < U; ++u) d[u] = dst[min(s0 + u, k - 1)];
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (s0 + u < k) *reinterpret_cast<u32x4*>(xg + (int64_t)d[u] * h + c * 8) = v;
    });
  }
}

// acc += w[s] * row perm[s] (or the row itself without w) for s = 0 .. k - 1
__device__ __forceinline__ void sum_slots(const bf16* rows, const int32_t* perm, const float* w,
                                          int k, int64_t h, int64_t c, float (&acc)[8]) {
  slot_batches(k, [&](int s0, auto u_c) {
    constexpr int U = decltype(u_c)::value;
    float v[U][8];
#pragma unroll
    for (int u = 0; u < U; ++u)
      load8<bf16>(rows + (int64_t)perm[min(s0 + u, k - 1)] * h + c * 8, v[u]);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (s0 + u >= k) break;
      const float ww = w ? w[s0 + u] : 1.0f;
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[j] = fmaf(ww, v[u][j], acc[j]);
    }
  });
}

template <typename YT>
__global__ __launch_bounds__(256) void moe_combine_kernel(const bf16* yg, const int32_t* perm,
                                                          const float* w, const YT* res, int k,
                                                          int64_t h, YT* y) {
  const int64_t t = blockIdx.x;
  for (int64_t c = (int64_t)blockIdx.y * 256 + threadIdx.x; c < h / 8; c += (int64_t)gridDim.y * 256) {
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (res) load8<YT>(res + t * h + c * 8, acc);
    sum_slots(yg, perm + t * k, w + t * k, k, h, c, acc);
    store8<YT>(y + t * h + c * 8, acc);
  }
}

__global__ __launch_bounds__(256) void moe_combine_bwd_kernel(const bf16* dy, const int32_t* perm,
                                                              const float* w, int k, int64_t h,
                                                              bf16* dyg) {
  const int64_t t = blockIdx.x;
  for (int64_t c = (int64_t)blockIdx.y * 256 + threadIdx.x; c < h / 8; c += (int64_t)gridDim.y * 256) {
    float v[8];
    load8<bf16>(dy + t * h + c * 8, v);
    slot_batches(k, [&](int s0, auto u_c) {
      constexpr int U = decltype(u_c)::value;
      int32_t d[U];
      float ww[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int s = min(s0 + u, k - 1);
        d[u] = perm[t * k + s];
        ww[u] = w[t * k + s];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (s0 + u >= k) break;
        float o[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) o[j] = v[j] * ww[u];
        store8<bf16>(dyg + (int64_t)d[u] * h + c * 8, o);
      }
    });
  }
}

__global__ __launch_bounds__(256) void moe_scatter_add_kernel(const bf16* dxg, const int32_t* perm,
                                                              int k, int64_t h, bf16* dx) {
  const int64_t t = blockIdx.x;
  for (int64_t c = (int64_t)blockIdx.y * 256 + threadIdx.x; c < h / 8; c += (int64_t)gridDim.y * 256) {
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    sum_slots(dxg, perm + t * k, nullptr, k, h, c, acc);
    store8<bf16>(dx + t * h + c * 8, acc);
  }
}

static unsigned chunks_y(int64_t h) {
  const int64_t c = (h / 8 + 255) / 256;
  return (unsigned)(c < 1 ? 1 : c);
}

}  // namespace catq

using namespace catq;

extern "C" catq_status catq_aux_rmsnorm_fwd(const void* x, catq_dtype x_dtype, int64_t rows,
                                            int64_t n, float eps, void* y, float* rstd,
                                            hipStream_t stream) {
  clear_error();
  CATQ_REQUIRE(dtype_ok(x_dtype), CATQ_ERR_DTYPE, "bad dtype");
  CATQ_REQUIRE(x && y, CATQ_ERR_NULL, "x and y must not be NULL");
  CATQ_REQUIRE(count_ok(rows, n) && n % 8 == 0, CATQ_ERR_SHAPE,
               "need rows > 0, n a multiple of 8 and rows*n <= 2^38");
  CATQ_REQUIRE(eps >= 0, CATQ_ERR_VALUE, "eps must be >= 0");
  CATQ_REQUIRE(aligned16(x) && aligned16(y), CATQ_ERR_ALIGN, "misaligned");
  const double xs = x_dtype == CATQ_BF16 ? 2.0 : 4.0;
  const double by = (double)rows * n * (xs + 2.0) + (rstd ? 4.0 * rows : 0.0);
  if (x_dtype == CATQ_BF16)
    CATQ_TRACED(stream, "rmsnorm_fwd_kernel<__bf16>", 0.0, by, rows, n, 0,
                hipLaunchKernelGGL(rmsnorm_fwd_kernel<bf16>, dim3((unsigned)rows), dim3(256), 0,
                                   stream, (const bf16*)x, n, eps, (bf16*)y, rstd));
  else
    CATQ_TRACED(stream, "rmsnorm_fwd_kernel<float>", 0.0, by, rows, n, 0,
                hipLaunchKernelGGL(rmsnorm_fwd_kernel<float>, dim3((unsigned)rows), dim3(256), 0,
                                   stream, (const float*)x, n, eps, (bf16*)y, rstd));
  CATQ_CHECK_LAUNCH("rmsnorm fwd");
  return CATQ_OK;
}

extern "C" catq_status catq_aux_rmsnorm_bwd(const void* x, catq_dtype x_dtype, const float* rstd,
                                            const void* dy, const void* dres, int64_t rows,
                                            int64_t n, void* dx, hipStream_t stream) {
  clear_error();
  CATQ_REQUIRE(dtype_ok(x_dtype), CATQ_ERR_DTYPE, "bad dtype");
  CATQ_REQUIRE(x && rstd && dy && dx, CATQ_ERR_NULL, "NULL argument");
  CATQ_REQUIRE(count_ok(rows, n) && n % 8 == 0, CATQ_ERR_SHAPE,
               "need rows > 0, n a multiple of 8 and rows*n <= 2^38");
  CATQ_REQUIRE(aligned16(x) && aligned16(dy) && aligned16(dres) && aligned16(dx), CATQ_ERR_ALIGN,
               "misaligned");
  const double xs = x_dtype == CATQ_BF16 ? 2.0 : 4.0;
  const double by = (double)rows * n * (xs + 2.0 + (dres ? 2.0 : 0.0) + 2.0) + 4.0 * rows;
  if (x_dtype == CATQ_BF16)
    CATQ_TRACED(stream, "rmsnorm_bwd_kernel<__bf16>", 0.0, by, rows, n, 0,
                hipLaunchKernelGGL(rmsnorm_bwd_kernel<bf16>, dim3((unsigned)rows), dim3(256), 0,
                                   stream, (const bf16*)x, rstd, (const bf16*)dy,
                                   (const bf16*)dres, n, (bf16*)dx));
  else
    CATQ_TRACED(stream, "rmsnorm_bwd_kernel<float>", 0.0, by, rows, n, 0,
                hipLaunchKernelGGL(rmsnorm_bwd_kernel<float>, dim3((unsigned)rows), dim3(256), 0,
                                   stream, (const float*)x, rstd, (const bf16*)dy,
                                   (const bf16*)dres, n, (bf16*)dx));
  CATQ_CHECK_LAUNCH("rmsnorm bwd");
  return CATQ_OK;
}

extern "C" catq_status catq_aux_act_quant(const void* x, catq_dtype x_dtype, int64_t rows,
                                          int64_t n, int64_t group, void* y,
                                          hipStream_t stream) {
  clear_error();
  CATQ_REQUIRE(rows >= 0, CATQ_ERR_SHAPE, "rows must be >= 0");
  if (rows == 0) return CATQ_OK;
  CATQ_REQUIRE(x && y, CATQ_ERR_NULL, "NULL argument");
  CATQ_REQUIRE(dtype_ok(x_dtype), CATQ_ERR_DTYPE, "x must be bf16 or fp32");
  CATQ_REQUIRE(n > 0 && group > 0 && n % group == 0 && group % 8 == 0, CATQ_ERR_SHAPE,
               "group must be a multiple of 8 dividing n");
  CATQ_REQUIRE(rows <= INT32_MAX && n / group <= 65535 && count_ok(rows, n), CATQ_ERR_SHAPE,
               "too many rows or groups");
  CATQ_REQUIRE(aligned16(x) && aligned16(y), CATQ_ERR_ALIGN, "misaligned");
  CATQ_REQUIRE(x_dtype == CATQ_BF16 || x != y, CATQ_ERR_VALUE,
               "an fp32 input cannot be quantized in place (y is bf16)");
  const dim3 grid((unsigned)rows, (unsigned)(n / group));
  const double bytes = (double)rows * (double)n * (2.0 * dtype_size(x_dtype) + 2.0);
  if (x_dtype == CATQ_BF16)
    CATQ_TRACED(stream, "act_quant_kernel<bf16>", 0.0, bytes, rows, n, group,
                hipLaunchKernelGGL(act_quant_kernel<bf16>, grid, dim3(256), 0, stream,
                                   (const bf16*)x, n, group, (bf16*)y));
  else
    CATQ_TRACED(stream, "act_quant_kernel<float>", 0.0, bytes, rows, n, group,
                hipLaunchKernelGGL(act_quant_kernel<float>, grid, dim3(256), 0, stream,
                                   (const float*)x, n, group, (bf16*)y));
  CATQ_CHECK_LAUNCH("act quant");
  return CATQ_OK;
}

extern "C" catq_status catq_aux_swiglu_fwd(const void* gu, int64_t rows, int64_t F, void* a,
                                           hipStream_t stream) {
  clear_error();
  CATQ_REQUIRE(gu && a, CATQ_ERR_NULL, "NULL argument");
  CATQ_REQUIRE(count_ok(rows, 2 * F) && F % 8 == 0, CATQ_ERR_SHAPE,
               "need rows > 0, F a multiple of 8 and rows*2F <= 2^38");
  CATQ_REQUIRE(aligned16(gu) && aligned16(a), CATQ_ERR_ALIGN, "misaligned");
  const int64_t n = rows * (F / 8);
  CATQ_TRACED(stream, "swiglu_fwd_kernel", 0.0, 6.0 * (double)rows * F, rows, F, 0,
              hipLaunchKernelGGL(swiglu_fwd_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256),
                                 0, stream, (const bf16*)gu, rows, F, (bf16*)a));
  CATQ_CHECK_LAUNCH("swiglu fwd");
  return CATQ_OK;
}

extern "C" catq_status catq_aux_swiglu_bwd(const void* gu, const void* da, int64_t rows, int64_t F,
                                           void* dgu, hipStream_t stream) {
  clear_error();
  CATQ_REQUIRE(gu && da && dgu, CATQ_ERR_NULL, "NULL argument");
  CATQ_REQUIRE(count_ok(rows, 2 * F) && F % 8 == 0, CATQ_ERR_SHAPE,
               "need rows > 0, F a multiple of 8 and rows*2F <= 2^38");
  CATQ_REQUIRE(aligned16(gu) && aligned16(da) && aligned16(dgu), CATQ_ERR_ALIGN, "misaligned");
  const int64_t n = rows * (F / 8);
  CATQ_TRACED(stream, "swiglu_bwd_kernel", 0.0, 10.0 * (double)rows * F, rows, F, 0,
              hipLaunchKernelGGL(swiglu_bwd_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256),
                                 0, stream, (const bf16*)gu, (const bf16*)da, rows, F, (bf16*)dgu));
  CATQ_CHECK_LAUNCH("swiglu bwd");
  return CATQ_OK;
}

extern "C" size_t catq_aux_moe_route_workspace_bytes(int64_t T, int32_t E, int32_t k) {
  (void)T;
  (void)k;
  return round_up((size_t)(E > 0 ? E : 1) * sizeof(int64_t), 256);
}

extern "C" catq_status catq_aux_moe_route(const float* logits, int64_t T, int32_t E, int32_t k,
                                          int32_t* expert_ids, float* weights, int32_t* perm_row,
                                          int64_t* row_offsets, void* workspace,
                                          size_t workspace_bytes, hipStream_t stream) {
  clear_error();
  CATQ_REQUIRE(logits && expert_ids && weights && perm_row && row_offsets && workspace,
               CATQ_ERR_NULL, "NULL argument");
  CATQ_REQUIRE(T > 0 && E > 0 && E <= 1024 && k >= 1 && k <= 16 && k <= E, CATQ_ERR_SHAPE,
               "need T > 0, 1 <= k <= min(16, E), E <= 1024");
  CATQ_REQUIRE(count_ok(T, k) && T * k < (int64_t)1 << 31 && count_ok(T, E), CATQ_ERR_SHAPE,
               "too many routed rows");
  CATQ_REQUIRE(workspace_bytes >= catq_aux_moe_route_workspace_bytes(T, E, k), CATQ_ERR_WORKSPACE,
               "workspace too small");
  auto topk = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3((unsigned)((T + 3) / 4)), dim3(256), 0, stream, logits, T, E, k,
                       expert_ids, weights);
  };
  if (E <= 64)
    topk(moe_topk_kernel<1>);
  else if (E <= 128)
    topk(moe_topk_kernel<2>);
  else if (E <= 256)
    topk(moe_topk_kernel<4>);
  else
    topk(moe_topk_kernel<16>);
  CATQ_CHECK_LAUNCH("moe top-k");
  hipLaunchKernelGGL(moe_rank_kernel, dim3((unsigned)E), dim3(kRankWaves * 64), 0, stream,
                     expert_ids, T * k, E, row_offsets, perm_row);
  CATQ_CHECK_LAUNCH("moe rank");
  return CATQ_OK;
}

extern "C" catq_status catq_aux_moe_gather(const void* x, const int32_t* perm_row, int64_t T,
                                           int32_t k, int64_t h, void* xg, hipStream_t stream) {
  clear_error();
  CATQ_REQUIRE(x && perm_row && xg, CATQ_ERR_NULL, "NULL argument");
  CATQ_REQUIRE(count_ok(T, k, h) && h % 8 == 0, CATQ_ERR_SHAPE,
               "need T, k, h > 0, h a multiple of 8 and T*k*h <= 2^38");
  CATQ_REQUIRE(aligned16(x) && aligned16(xg), CATQ_ERR_ALIGN, "misaligned");
  hipLaunchKernelGGL(moe_gather_kernel, dim3((unsigned)T, chunks_y(h)), dim3(256), 0, stream,
                     (const bf16*)x, perm_row, k, h, (bf16*)xg);
  CATQ_CHECK_LAUNCH("moe gather");
  return CATQ_OK;
}

extern "C" catq_status catq_aux_moe_combine(const void* yg, const int32_t* perm_row,
                                            const float* weights, const void* res, int64_t T,
                                            int32_t k, int64_t h, void* y, catq_dtype y_dtype,
                                            hipStream_t stream) {
  clear_error();
  CATQ_REQUIRE(dtype_ok(y_dtype), CATQ_ERR_DTYPE, "bad dtype");
  CATQ_REQUIRE(yg && perm_row && weights && y, CATQ_ERR_NULL, "NULL argument");
  CATQ_REQUIRE(count_ok(T, k, h) && h % 8 == 0, CATQ_ERR_SHAPE,
               "need T, k, h > 0, h a multiple of 8 and T*k*h <= 2^38");
  CATQ_REQUIRE(aligned16(yg) && aligned16(res) && aligned16(y), CATQ_ERR_ALIGN, "misaligned");
  if (y_dtype == CATQ_BF16)
    hipLaunchKernelGGL(moe_combine_kernel<bf16>, dim3((unsigned)T, chunks_y(h)), dim3(256), 0,
                       stream, (const bf16*)yg, perm_row, weights, (const bf16*)res, k, h,
                       (bf16*)y);
  else
    hipLaunchKernelGGL(moe_combine_kernel<float>, dim3((unsigned)T, chunks_y(h)), dim3(256), 0,
                       stream, (const bf16*)yg, perm_row, weights, (const float*)res, k, h,
                       (float*)y);
  CATQ_CHECK_LAUNCH("moe combine");
  return CATQ_OK;
}

extern "C" catq_status catq_aux_moe_combine_bwd(const void* dy, const int32_t* perm_row,
                                                const float* weights, int64_t T, int32_t k,
                                                int64_t h, void* dyg, hipStream_t stream) {
  clear_error();
  CATQ_REQUIRE(dy && perm_row && weights && dyg, CATQ_ERR_NULL, "NULL argument");
  CATQ_REQUIRE(count_ok(T, k, h) && h % 8 == 0, CATQ_ERR_SHAPE,
               "need T, k, h > 0, h a multiple of 8 and T*k*h <= 2^38");
  CATQ_REQUIRE(aligned16(dy) && aligned16(dyg), CATQ_ERR_ALIGN, "misaligned");
  hipLaunchKernelGGL(moe_combine_bwd_kernel, dim3((unsigned)T, chunks_y(h)), dim3(256), 0,
                     stream, (const bf16*)dy, perm_row, weights, k, h, (bf16*)dyg);
  CATQ_CHECK_LAUNCH("moe combine bwd");
  return CATQ_OK;
}

extern "C" catq_status catq_aux_moe_scatter_add(const void* dxg, const int32_t* perm_row, int64_t T,
                                                int32_t k, int64_t h, void* dx,
                                                hipStream_t stream) {
  clear_error();
  CATQ_REQUIRE(dxg && perm_row && dx, CATQ_ERR_NULL, "NULL argument");
  CATQ_REQUIRE(count_ok(T, k, h) && h % 8 == 0, CATQ_ERR_SHAPE,
               "need T, k, h > 0, h a multiple of 8 and T*k*h <= 2^38");
  CATQ_REQUIRE(aligned16(dxg) && aligned16(dx), CATQ_ERR_ALIGN, "misaligned");
  hipLaunchKernelGGL(moe_scatter_add_kernel, dim3((unsigned)T, chunks_y(h)), dim3(256), 0, stream,
                     (const bf16*)dxg, perm_row, k, h, (bf16*)dx);
  CATQ_CHECK_LAUNCH("moe scatter add");
  return CATQ_OK;
}
