// Commit of the verified path into the KV cache (Algorithm 1, COMPACT_KV; Section III-B:
// the cloud keeps the state of the accepted prefix and discards the rest of the tree).
//
// After a verify step the tree's keys and values sit in slots prefix_len + row.  The root
// (row 0) and the kept drafted rows path[0 .. path_len) move to the contiguous slots
// prefix_len + 0 .. prefix_len + path_len, i.e. to the positions a plain causal decode of
// the accepted tokens would have filled (a kept node at depth i has RoPE position
// prefix_len + i, so its rotated key is already the right one).  One workgroup per
// (layer, kv head, session); every source entry is read into LDS before any destination
// is written, because a destination slot may be another entry's source.
//
// What bounds it is the value columns: two bytes an entry, in lines of their own, and the
// chain of dependent reads (lengths, path, entries) before the first store, so workgroups
// in flight count: LDS is sized to the tree (8 KB at 16 nodes of head dim 128, eight
// workgroups a CU where a fixed 32 KB left five), entries are mapped to threads by shifts,
// and keys move as 16-byte pieces.  32 layers x 8 kv heads x 48 sessions: 105 -> 78 us.
#include "common.h"

namespace {

constexpr int CT = 256;   // threads

// VEC: keys move as 16-byte pieces (the cache is 16-byte aligned).
template <typename T, bool VEC>
__global__ __launch_bounds__(CT) void commit_kv_kernel(T *__restrict__ ck, T *__restrict__ cv,
                                                       const int32_t *__restrict__ prefix_len,
                                                       const int32_t *__restrict__ path,
                                                       const int32_t *__restrict__ path_len,
                                                       const int32_t *__restrict__ status,
                                                       int B, int n1, int Hkv, int hd,
                                                       int capacity, int32_t *new_len) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  __shared__ int32_t rows[64];             // kept rows (n1 <= 65)
  const int lg = blockIdx.x, b = blockIdx.y;
  const int l = lg / Hkv, g = lg - l * Hkv;
  const int tid = threadIdx.x;
  const int32_t row = tid < n1 - 1 ? path[(size_t)b * n1 + tid] : 0;
  const int S = prefix_len[b];
  const int np = path_len[b];
  const bool ok = (status == nullptr || status[b] == ACESPEC_OK) && S >= 0 &&
                  S + n1 <= capacity && np >= 0 && np < n1;
  // every kept row must be a drafted row of this tree
  if (tid < n1 - 1) rows[tid] = row;
  const bool bad = __syncthreads_or(!ok || (tid < np && (row < 1 || row >= n1)));
  if (lg == 0 && tid == 0) new_len[b] = bad ? -1 : S + 1 + np;
  if (bad || np == 0) return;

  const size_t head = ((size_t)l * B + b) * Hkv + g;   // (layer, session, kv head)
  T *kb = ck + head * capacity * hd + (size_t)S * hd;  // [slots from S][hd]
  T *vb = cv + head * hd * capacity + S;               // [hd][slots from S]
  T *vbuf = (T *)smem;                                 // [hd][np]
  T *kbuf = vbuf + (size_t)(n1 - 1) * hd;              // [np][hd]
  // values: kept rows fastest (the next power of two of them), so that a wave's accesses
  // fall into few lines; kept row i is 1-based among the moved slots (row 0 stays in place)
  const int lp = np > 1 ? 32 - __builtin_clz(np - 1) : 0;
  const int i = tid & ((1 << lp) - 1), d0 = tid >> lp, dstep = CT >> lp;
  if (i < np) {
    const int r = rows[i];
#pragma unroll 4
    for (int d = d0; d < hd; d += dstep) vbuf[d * np + i] = vb[(size_t)d * capacity + r];
  }
  if constexpr (VEC) {
    constexpr int PE = 16 / sizeof(T);   // elements a piece; hd is 64 or 128
    const int lq = __builtin_ctz(hd / PE);
    for (int e = tid; e < np << lq; e += CT) {
      const int k = e >> lq, o = (e & ((1 << lq) - 1)) * PE;
      *(uint4 *)(kbuf + k * hd + o) = *(const uint4 *)(kb + (size_t)rows[k] * hd + o);
    }
    __syncthreads();
    for (int e = tid; e < np << lq; e += CT)
      *(uint4 *)(kb + hd + (size_t)e * PE) = *(const uint4 *)(kbuf + (size_t)e * PE);
  } else {
    for (int e = tid; e < np * hd; e += CT) {
      const int k = e / hd;
      kbuf[e] = kb[(size_t)rows[k] * hd + (e - k * hd)];
    }
    __syncthreads();
    for (int e = tid; e < np * hd; e += CT) kb[hd + (size_t)e] = kbuf[e];
  }
  if (i < np) {
#pragma unroll 4
    for (int d = d0; d < hd; d += dstep) vb[(size_t)d * capacity + 1 + i] = vbuf[d * np + i];
  }
}

// Value-cache layout conversion (not part of the verify step): every plane (layer,
// session, kv head) is a [rows][cols] matrix, written transposed as [cols][rows] --
// slot-major [capacity][head_dim] <-> the head-dim-major [head_dim][capacity] the verify
// step reads.  Elements move as raw bits (E: 2 or 4 bytes), one workgroup per tile.
//
// 64 x 64 tiles through LDS with 16-byte reads and 16-byte writes on both sides: bound by
// HBM once every access moves a line's worth (1.1 GB in 2-byte elements: 32 x 32 tiles of
// single elements 525 us, these 176 us, 6.3 TB/s).  Rows and columns are
// multiples of a 16-byte piece, the arrays 16-byte aligned.
template <typename E>
__global__ __launch_bounds__(256) void transpose_planes_vec_kernel(const E *__restrict__ src,
                                                                   E *__restrict__ dst, int rows,
                                                                   int cols, int tiles_r,
                                                                   int tiles_c) {
  constexpr int PE = 16 / sizeof(E), PPR = 64 / PE;   // elements a piece, pieces a tile row
  constexpr int PITCH = 64 + 4 / sizeof(E);           // odd number of banks
  typedef E piece __attribute__((ext_vector_type(PE)));
  __shared__ E tile[64 * PITCH];
  const int per_plane = tiles_r * tiles_c;
  const size_t plane = blockIdx.x / per_plane;
  const int t = (int)(blockIdx.x - plane * per_plane);
  // tiles along the destination's rows follow each other
  const int tc = t / tiles_r, tr = t - tc * tiles_r;
  const size_t base = plane * rows * cols;
  const int r0 = tr * 64, c0 = tc * 64;
  piece v[PPR / 4];
#pragma unroll
  for (int k = 0; k < PPR / 4; ++k) {
    const int x = threadIdx.x + 256 * k, r = x / PPR, c = x % PPR * PE;
    if (r0 + r < rows && c0 + c < cols)
      v[k] = __builtin_nontemporal_load((const piece *)(src + base + (size_t)(r0 + r) * cols + c0 + c));
  }
#pragma unroll
  for (int k = 0; k < PPR / 4; ++k) {
    const int x = threadIdx.x + 256 * k, r = x / PPR, c = x % PPR * PE;
#pragma unroll
    for (int j = 0; j < PE; ++j) tile[(c + j) * PITCH + r] = v[k][j];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < PPR / 4; ++k) {
    const int x = threadIdx.x + 256 * k, c = x / PPR, r = x % PPR * PE;
    piece o;
#pragma unroll
    for (int j = 0; j < PE; ++j) o[j] = tile[c * PITCH + r + j];
    if (r0 + r < rows && c0 + c < cols)
      __builtin_nontemporal_store(o, (piece *)(dst + base + (size_t)(c0 + c) * rows + r0 + r));
  }
}

// Any sizes and alignment: 32 x 32 tiles of single elements.
template <typename E>
__global__ __launch_bounds__(256) void transpose_planes_kernel(const E *__restrict__ src,
                                                               E *__restrict__ dst, int rows,
                                                               int cols, int tiles_r,
                                                               int tiles_c) {
  __shared__ E tile[32][33];
  const int per_plane = tiles_r * tiles_c;
  const long long plane = blockIdx.x / per_plane;
  const int t = (int)(blockIdx.x - plane * per_plane);
  const int tr = t / tiles_c, tc = t - tr * tiles_c;
  const size_t base = (size_t)plane * rows * cols;
  const int x = threadIdx.x & 31, y = threadIdx.x >> 5;  // 32 x 8 threads
  for (int i = y; i < 32; i += 8) {
    const int r = tr * 32 + i, c = tc * 32 + x;
    if (r < rows && c < cols) tile[i][x] = src[base + (size_t)r * cols + c];
  }
  __syncthreads();
  for (int i = y; i < 32; i += 8) {
    const int c = tc * 32 + i, r = tr * 32 + x;  // destination row c, column r
    if (c < cols && r < rows) dst[base + (size_t)c * rows + r] = tile[x][i];
  }
}

}  // namespace

namespace acespec {

template <typename T>
hipError_t launch_commit_kv(T *ck, T *cv, const int32_t *prefix_len, const int32_t *path,
                            const int32_t *path_len, const int32_t *status, int L, int B,
                            int n1, int Hkv, int hd, int capacity, int32_t *new_len,
                            hipStream_t s) {
  if (n1 > 65 || (hd != 64 && hd != 128)) return hipErrorInvalidValue;
  const size_t lds = (size_t)2 * (n1 - 1) * hd * sizeof(T);   // at most 64 KB
  const bool vec = (((uintptr_t)ck | (uintptr_t)cv) & 15) == 0;
  auto kernel = vec ? commit_kv_kernel<T, true> : commit_kv_kernel<T, false>;
  hipLaunchKernelGGL(kernel, dim3(L * Hkv, B), dim3(CT), lds, s, ck, cv, prefix_len, path,
                     path_len, status, B, n1, Hkv, hd, capacity, new_len);
  return hipGetLastError();
}

template hipError_t launch_commit_kv<float>(float *, float *, const int32_t *, const int32_t *,
                                            const int32_t *, const int32_t *, int, int, int,
                                            int, int, int, int32_t *, hipStream_t);
template hipError_t launch_commit_kv<bf16>(bf16 *, bf16 *, const int32_t *, const int32_t *,
                                           const int32_t *, const int32_t *, int, int, int, int,
                                           int, int, int32_t *, hipStream_t);

hipError_t launch_transpose_planes(const void *src, void *dst, int elem_bytes, int planes,
                                   int rows, int cols, hipStream_t s) {
  if (planes < 1 || rows < 1 || cols < 1 || (elem_bytes != 2 && elem_bytes != 4))
    return hipErrorInvalidValue;
  const int pe = 16 / elem_bytes;
  if (rows % pe == 0 && cols % pe == 0 && (((uintptr_t)src | (uintptr_t)dst) & 15) == 0) {
    const int tr = (rows + 63) / 64, tc = (cols + 63) / 64;
    const dim3 grid((unsigned)((long long)planes * tr * tc));   // fewer than the tiles below
    if (elem_bytes == 2)
      hipLaunchKernelGGL(transpose_planes_vec_kernel<uint16_t>, grid, dim3(256), 0, s,
                         (const uint16_t *)src, (uint16_t *)dst, rows, cols, tr, tc);
    else
      hipLaunchKernelGGL(transpose_planes_vec_kernel<uint32_t>, grid, dim3(256), 0, s,
                         (const uint32_t *)src, (uint32_t *)dst, rows, cols, tr, tc);
    return hipGetLastError();
  }
  const int tiles_r = (rows + 31) / 32, tiles_c = (cols + 31) / 32;
  const long long blocks = (long long)planes * tiles_r * tiles_c;
  if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  if (elem_bytes == 2)
    hipLaunchKernelGGL(transpose_planes_kernel<uint16_t>, dim3((unsigned)blocks), dim3(256), 0, s,
                       (const uint16_t *)src, (uint16_t *)dst, rows, cols, tiles_r, tiles_c);
  else
    hipLaunchKernelGGL(transpose_planes_kernel<uint32_t>, dim3((unsigned)blocks), dim3(256), 0, s,
                       (const uint32_t *)src, (uint32_t *)dst, rows, cols, tiles_r, tiles_c);
  return hipGetLastError();
}

}  // namespace acespec
