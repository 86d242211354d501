// Embedding gather, RMSNorm, and RoPE with the tree K/V write into the cache.
//
// RMSNorm: y = x / sqrt(mean(x^2) + eps) * gain, fp32 math, rounded once to the
// activation type.  The residual stream x stays fp32 between layers.
// RoPE (rotate-half): the pair (i, i + hd/2) of every query and key head is rotated by
// pos * base^(-2i/hd); the angle and its sine/cosine are evaluated in double so that
// large positions (16k-token prefixes) keep full fp32 accuracy, once per step into a
// (cos, sin) table of fp32 pairs per tree row.  The rotation itself normally runs in the
// QKV projection's epilogue; the kernel here serves the fp32 model and products sliced
// along K.  The projection is rounded once: q to the activation type, k and v to the
// cache dtype.  Tree row r of session b sits at position prefix_len + depth(r) and its
// key/value go to slot prefix_len + r.
#include "common.h"

namespace {

// Four consecutive elements as float4 (the row bases are 16-byte aligned: d % 64 == 0).
AS_DEVICE float4 load4(const float *p, int c) { return *(const float4 *)(p + 4 * c); }
AS_DEVICE float4 load4(const bf16 *p, int c) {
  typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
  const bf16x4 v = *(const bf16x4 *)(p + 4 * c);
  return make_float4((float)v[0], (float)v[1], (float)v[2], (float)v[3]);
}
AS_DEVICE void store4(float *p, int c, float4 v) { *(float4 *)(p + 4 * c) = v; }
// Four consecutive activations of row `row`: fp32 row-major, fp16 in the activation layout.
AS_DEVICE void store_act4(float *p, int row, int c, int, int d, float4 v) {
  store4(p + (size_t)row * d, c, v);
}
AS_DEVICE void store_act4(f16 *p, int row, int c, int rows, int d, float4 v) {
  typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
  *(f16x4 *)(p + act_off(row, 4 * c, rows, d)) =
      f16x4{(f16)v.x, (f16)v.y, (f16)v.z, (f16)v.w};
}

// One row per block, four elements a thread per step (d % 64 == 0).
template <typename T>
__global__ void embed_kernel(const T *__restrict__ embed, const int32_t *__restrict__ tok,
                             float *__restrict__ x, int d) {
  const int row = blockIdx.x;
  const T *src = embed + (size_t)tok[row] * d;
  float *dst = x + (size_t)row * d;
  for (int c = threadIdx.x; c < (d >> 2); c += blockDim.x) store4(dst, c, load4(src, c));
}

// One 256-thread block per row (neighbouring rows on one XCD: their pieces share lines of
// the activation layout); d is a multiple of 64.  A row of up to 8192 values is read
// once (float4 per thread and step, kept in registers), longer rows are read twice.
template <typename Tin, typename TG, typename Tout>
__global__ __launch_bounds__(256) void rmsnorm_kernel(const Tin *__restrict__ x,
                                                      const TG *__restrict__ gain,
                                                      Tout *__restrict__ out, int d, float eps) {
  constexpr int MAXJ = 8;
  const int rows = gridDim.x, row = xcd_tile(blockIdx.x, rows), tid = threadIdx.x;
  const int d4 = d >> 2;
  const Tin *xr = x + (size_t)row * d;
  float4 v[MAXJ];
  float ss = 0.f;
#pragma unroll
  for (int j = 0; j < MAXJ; ++j) {
    const int c = tid + 256 * j;
    if (c < d4) {
      v[j] = load4(xr, c);
      ss += v[j].x * v[j].x + v[j].y * v[j].y + v[j].z * v[j].z + v[j].w * v[j].w;
    }
  }
  for (int c = tid + 256 * MAXJ; c < d4; c += 256) {
    const float4 t = load4(xr, c);
    ss += t.x * t.x + t.y * t.y + t.z * t.z + t.w * t.w;
  }
  __shared__ float red[4];
  ss = wave_sum(ss);
  if ((tid & 63) == 0) red[tid >> 6] = ss;
  __syncthreads();
  const float tot = (red[0] + red[1]) + (red[2] + red[3]);
  const float scale = 1.0f / sqrtf(tot / (float)d + eps);
#pragma unroll
  for (int j = 0; j < MAXJ; ++j) {
    const int c = tid + 256 * j;
    if (c < d4) {
      const float4 g = load4(gain, c);
      store_act4(out, row, c, rows, d,
                 make_float4(v[j].x * scale * g.x, v[j].y * scale * g.y, v[j].z * scale * g.z,
                             v[j].w * scale * g.w));
    }
  }
  for (int c = tid + 256 * MAXJ; c < d4; c += 256) {
    const float4 t = load4(xr, c), g = load4(gain, c);
    store_act4(out, row, c, rows, d,
               make_float4(t.x * scale * g.x, t.y * scale * g.y, t.z * scale * g.z,
                           t.w * scale * g.w));
  }
}

__global__ void rope_table_kernel(const int32_t *__restrict__ pos,
                                  const double *__restrict__ inv_freq, float2 *__restrict__ rot,
                                  int rows, int half) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= rows * half) return;
  const int row = idx / half, i = idx - row * half;
  double sd, cd;
  sincos((double)pos[row] * inv_freq[i], &sd, &cd);
  rot[idx] = make_float2((float)cd, (float)sd);
}

// grid: (H + 2 Hkv heads, sessions, chunks of ROPE_ROWS tree rows); block: 256 threads.  One
// block takes ROPE_ROWS tree rows of one head of the projection: a rotated query or key
// head, four frequencies a thread, or a value head, whose columns go through LDS so that
// they land as runs of consecutive slots in the head-dim-major value cache.  One block a
// head rather than one a kv head with its group of query heads: a latency-bound kernel of
// few rows then has 48 blocks a session instead of 8 (8B shape).  head_dim is 64 or 128.
constexpr int ROPE_ROWS = 16, ROPE_THREADS = 256;
AS_DEVICE float4 sum_slices(const float *p, int nsl, size_t stride) {
  float4 a = *(const float4 *)p;
  for (int s = 1; s < nsl; ++s) {
    const float4 v = *(const float4 *)(p + s * stride);
    a.x += v.x; a.y += v.y; a.z += v.z; a.w += v.w;
  }
  return a;
}
template <typename TW, typename TA, int HD>
__global__ __launch_bounds__(ROPE_THREADS) void rope_kv_kernel(const float *__restrict__ qkv,
                                                      int nsl, TA *__restrict__ q_out,
                                                      TreeMeta meta, TW *__restrict__ ck,
                                                      TW *__restrict__ cv, int n1, int H, int Hkv,
                                                      int capacity,
                                                      const float2 *__restrict__ rot) {
  constexpr int HALF = HD / 2;
  __shared__ float vs[ROPE_ROWS][HD + 1];
  const int gh = blockIdx.x, b = blockIdx.y, r0 = blockIdx.z * ROPE_ROWS, tid = threadIdx.x;
  const int nr = min(ROPE_ROWS, n1 - r0);  // rows of this block
  const int rows = gridDim.y * n1;
  const size_t W = (size_t)(H + 2 * Hkv) * HD, slice = W * rows;  // qkv row, slice
  const size_t row0 = (size_t)b * n1 + r0;
  const float *base = qkv + row0 * W + (size_t)gh * HD;
  const int S = meta.sess_S[b];
  if (gh < H + Hkv) {
    typedef TA a4 __attribute__((ext_vector_type(4)));
    typedef TW w4 __attribute__((ext_vector_type(4)));
    for (int e = tid; e < nr * (HALF / 4); e += ROPE_THREADS) {
      const int r = e / (HALF / 4), i = e % (HALF / 4) * 4;
      const float4 a1 = sum_slices(base + r * W + i, nsl, slice);
      const float4 a2 = sum_slices(base + r * W + i + HALF, nsl, slice);
      const float4 c01 = *(const float4 *)(rot + (row0 + r) * HALF + i);
      const float4 c23 = *(const float4 *)(rot + (row0 + r) * HALF + i + 2);
      const float x1[4] = {a1.x, a1.y, a1.z, a1.w}, x2[4] = {a2.x, a2.y, a2.z, a2.w};
      const float cc[4] = {c01.x, c01.z, c23.x, c23.z}, sn[4] = {c01.y, c01.w, c23.y, c23.w};
      float y1[4], y2[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        y1[j] = x1[j] * cc[j] - x2[j] * sn[j];
        y2[j] = x2[j] * cc[j] + x1[j] * sn[j];
      }
      if (gh < H) {
        TA *qo = q_out + (row0 + r) * H * HD + (size_t)gh * HD;
        *(a4 *)(qo + i) = a4{from_f32<TA>(y1[0]), from_f32<TA>(y1[1]), from_f32<TA>(y1[2]),
                             from_f32<TA>(y1[3])};
        *(a4 *)(qo + i + HALF) = a4{from_f32<TA>(y2[0]), from_f32<TA>(y2[1]),
                                    from_f32<TA>(y2[2]), from_f32<TA>(y2[3])};
      } else {
        TW *kd = ck + (((size_t)b * Hkv + gh - H) * capacity + S + r0 + r) * HD;
        *(w4 *)(kd + i) = w4{from_f32<TW>(y1[0]), from_f32<TW>(y1[1]), from_f32<TW>(y1[2]),
                             from_f32<TW>(y1[3])};
        *(w4 *)(kd + i + HALF) = w4{from_f32<TW>(y2[0]), from_f32<TW>(y2[1]),
                                    from_f32<TW>(y2[2]), from_f32<TW>(y2[3])};
      }
    }
    return;
  }
  for (int e = tid; e < nr * (HD / 4); e += ROPE_THREADS) {  // this head's values, row-major
    const int r = e / (HD / 4), d = e % (HD / 4) * 4;
    const float4 v = sum_slices(base + r * W + d, nsl, slice);
    vs[r][d] = v.x; vs[r][d + 1] = v.y; vs[r][d + 2] = v.z; vs[r][d + 3] = v.w;
  }
  __syncthreads();
  TW *vb = cv + ((size_t)b * Hkv + gh - H - Hkv) * HD * capacity + S + r0;
  for (int e = tid; e < HD * ROPE_ROWS; e += ROPE_THREADS) {
    const int dd = e / ROPE_ROWS, r = e % ROPE_ROWS;
    if (r < nr) vb[(size_t)dd * capacity + r] = from_f32<TW>(vs[r][dd]);
  }
}

// One thread per eight-column piece of a row, 16 rows x 4 pieces a wave: 64-byte reads of
// each row, contiguous 1 KB writes.
__global__ __launch_bounds__(256) void cast_bf16_f16_kernel(const bf16 *__restrict__ in,
                                                            f16 *__restrict__ out, int rows,
                                                            int d) {
  const long long u = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const int k32 = d >> 5, l = (int)(u & 63);
  const long long blk = u >> 6;
  const int rb = (int)(blk / k32), kb = (int)(blk - (long long)rb * k32);
  const int row = rb * 16 + (l & 15), col = kb * 32 + (l >> 4) * 8;
  if (row >= rows) return;
  *(f16x8 *)(out + act_off(row, col, rows, d)) =
      bf16x8_to_f16x8(*(const bf16x8 *)(in + (size_t)row * d + col));
}

}  // namespace

namespace acespec {

hipError_t launch_rope_table(const int32_t *pos, const double *inv_freq, float2 *rot, int rows,
                             int half, hipStream_t s) {
  const int n = rows * half;
  hipLaunchKernelGGL(rope_table_kernel, dim3((n + 255) / 256), dim3(256), 0, s, pos, inv_freq,
                     rot, rows, half);
  return hipGetLastError();
}

hipError_t launch_cast_bf16_f16(const bf16 *in, f16 *out, int rows, int d, hipStream_t s) {
  const long long n = (long long)((rows + 15) / 16) * (d / 32) * 64;  // d is a multiple of 64
  hipLaunchKernelGGL(cast_bf16_f16_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                     in, out, rows, d);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_embed(const T *embed, const int32_t *tok, float *x, int rows, int d,
                        hipStream_t s) {
  hipLaunchKernelGGL(embed_kernel<T>, dim3(rows), dim3(256), 0, s, embed, tok, x, d);
  return hipGetLastError();
}

template <typename TW, typename TIN>
hipError_t launch_rmsnorm(const TIN *x, const TW *gain, typename ActOf<TW>::type *out, int rows,
                          int d, float eps, hipStream_t s) {
  hipLaunchKernelGGL((rmsnorm_kernel<TIN, TW, typename ActOf<TW>::type>), dim3(rows), dim3(256),
                     0, s, x, gain, out, d, eps);
  return hipGetLastError();
}

template <typename TW>
hipError_t launch_rope_kv(const float *qkv, int nsl, typename ActOf<TW>::type *q_out,
                          const TreeMeta &meta, TW *cache_k, TW *cache_v, int B, int n1, int H,
                          int Hkv, int hd, int capacity, const float2 *rot, hipStream_t s) {
  if ((hd != 64 && hd != 128) || H % Hkv) return hipErrorInvalidValue;
  const dim3 grid(H + 2 * Hkv, B, (n1 + ROPE_ROWS - 1) / ROPE_ROWS);
  auto kernel = hd == 64 ? rope_kv_kernel<TW, typename ActOf<TW>::type, 64>
                         : rope_kv_kernel<TW, typename ActOf<TW>::type, 128>;
  hipLaunchKernelGGL(kernel, grid, dim3(ROPE_THREADS), 0, s, qkv, nsl, q_out, meta, cache_k,
                     cache_v, n1, H, Hkv, capacity, rot);
  return hipGetLastError();
}

template hipError_t launch_embed<float>(const float *, const int32_t *, float *, int, int,
                                        hipStream_t);
template hipError_t launch_embed<bf16>(const bf16 *, const int32_t *, float *, int, int,
                                       hipStream_t);
template hipError_t launch_rmsnorm<float, float>(const float *, const float *, float *, int, int,
                                                 float, hipStream_t);
template hipError_t launch_rmsnorm<bf16, float>(const float *, const bf16 *, f16 *, int, int,
                                                float, hipStream_t);
template hipError_t launch_rmsnorm<bf16, bf16>(const bf16 *, const bf16 *, f16 *, int, int,
                                               float, hipStream_t);
template hipError_t launch_rope_kv<float>(const float *, int, float *, const TreeMeta &, float *,
                                          float *, int, int, int, int, int, int, const float2 *,
                                          hipStream_t);
template hipError_t launch_rope_kv<bf16>(const float *, int, f16 *, const TreeMeta &, bf16 *,
                                         bf16 *, int, int, int, int, int, int, const float2 *,
                                         hipStream_t);

}  // namespace acespec
