// Fused vocabulary-wide verification: one workgroup per tree row, nothing of size
// [rows, vocab] is written back.
//
// For row r with logits z (fp32) the target distribution is p~ = softmax(z / T) cut to
// the top-p nucleus (the smallest most-probable set whose mass reaches top_p, ties in
// probability broken by lower token id, crossing token kept) and renormalised: p_r.
// The row produces
//   - the top-k payload: the k most probable ids and p_r on them renormalised (the sparse
//     partial distribution the cloud returns downlink, Section III-B),
//   - a bonus sample from p_r (inverse CDF in token-id order),
// and decides each drafted child n of r (token x, draft distribution Q = q[r]) by the
// speculative acceptance test of Chen et al. (cited in Section II):
//   accept[n] = u0 * Q(x) < p_r(x)         (u0 < min(1, p/q)),
//   resample[n] = inverse CDF of max(0, p_r - Q) at u1 (of p_r if that has no mass).
//
// Arithmetic: e = exp2((z - max) * log2(e) / T) in fp32 (the factor log2(e) / T and the
// nucleus normaliser each carried as a pair of floats); probability mass is summed in
// 2^-40 fixed point (64-bit integers), so every reduction is exact, order independent
// and run-to-run deterministic.  The nucleus and top-k thresholds are found by a radix
// select on the order-preserving 32-bit key of z (12 + 11 + 9 bits, histograms in LDS
// weighted by mass for top-p and by count for top-k), which finds the exact threshold
// logit and the number of tied ids to keep (ids ascending).  The inverse CDFs run over
// 256-id segments: segment masses are prefix-summed in LDS, and the chosen segment is
// re-read and scanned across a wavefront.
// Occupancy: 512 threads, 51 KB of LDS (the histograms of each pass and the segment
// tables share storage; the refinement levels are sized to fit under pass 1's) and at most
// 80 VGPRs per row (ten values spill: thread constants, reloaded between the passes and
// three times a step of the last one), so three rows are in flight per CU and their scans and selections
// overlap each other's passes over memory (two rows a CU give about 1.45x the throughput
// of one, three about 10 % more than two); the row passes keep the next step's loads in
// flight while processing the current one.
#include "common.h"

namespace {

constexpr int VT = 512;             // threads per row (three rows in flight per CU)
constexpr int NWV = VT / 64;        // waves
constexpr int SEG = 256;            // ids per segment (one float4 per lane)
constexpr int SEGMAX = 1024;        // vocab <= 262144
constexpr int KMAX = 256;

typedef unsigned long long u64;

// Block-wide scans and selections.
struct VScan {
  u64 wsum[NWV];
  float wmax[NWV];
  u64 above_p;             // selection results
  uint32_t above_k;
  int sel_p, sel_k;
};
// The top-k ids found by a segment pass.
struct VTop {
  uint32_t cand_key[KMAX];
  int32_t cand_id[KMAX];
  uint32_t cand_in[KMAX];
  uint32_t ncand;
};
struct VSmem : VScan, VTop {
  // The threshold histograms (passes 1-3) and the per-segment tables (tie pass, pass 4)
  // are never live together; sharing their storage keeps three rows in flight per CU.
  union {
    struct {  // pass 1: bits 31..20 of the key
      uint32_t cnt[4096];
      u64 mass[4096];
    } h;
    struct {  // passes 2 and 3: bits 19..9, then 8..0, inside the selected bins
      uint32_t cnt[2048];
      u64 mass[2048];
      uint32_t cntk[2048];
    } r;
    struct {
      u64 seg_p[SEGMAX];       // per-segment mass of p_r, then its exclusive prefix
      u64 seg_r[SEGMAX];       // same for the residual max(0, p_r - Q)
      uint32_t tie_p[SEGMAX];  // per-segment count of ids tied at the top-p threshold (prefix)
      uint32_t tie_k[SEGMAX];
    } g;
  };
  uint32_t nbin;           // elements of the selected top-p / top-k bins (pass 2)
  int flag;                // data-error code of the row (0 = none)
};

AS_DEVICE u64 fixw(float v) { return __float2ull_rn(v * AS_FX_SCALE); }
// fixw(v) as a float, exactly: for v <= 1 the product is at most 2^40, and either it is
// already an integer (>= 2^23) or its rounding is below 2^24, so the value is representable.
AS_DEVICE float fixw_f(float v) { return rintf(v * AS_FX_SCALE); }

// Four weights' fixed-point masses: below 2^32 each, as nearly always, a conversion each.
AS_DEVICE void fix4(const float (&e)[4], u64 (&w)[4]) {
  float f[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) f[j] = fixw_f(e[j]);
  if (fmaxf(fmaxf(f[0], f[1]), fmaxf(f[2], f[3])) < 4294967296.f) {
#pragma unroll
    for (int j = 0; j < 4; ++j) w[j] = (uint32_t)f[j];
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) w[j] = (u64)f[j];
  }
}

AS_DEVICE float key_to_f32(uint32_t key) {  // inverse of f32_key
  return __uint_as_float((key & 0x80000000u) ? (key & 0x7FFFFFFFu) : ~key);
}

// Block-wide exclusive scan (u64).  All threads must call it.
AS_DEVICE u64 block_scan_excl(u64 v, VScan &sm, u64 &total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  u64 x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const u64 y = __shfl_up(x, o);
    if (lane >= o) x += y;
  }
  if (lane == 63) sm.wsum[wave] = x;
  __syncthreads();
  u64 off = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < NWV; ++w) {
    const u64 s = sm.wsum[w];
    off += w < wave ? s : 0;
    tot += s;
  }
  __syncthreads();
  total = tot;
  return off + x - v;
}

AS_DEVICE u64 block_sum(u64 v, VScan &sm) {
  u64 t;
  block_scan_excl(v, sm, t);
  return t;
}

AS_DEVICE float block_max(float v, VScan &sm) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  v = wave_max(v);
  if (lane == 0) sm.wmax[wave] = v;
  __syncthreads();
  float m = sm.wmax[0];
#pragma unroll
  for (int w = 1; w < NWV; ++w) m = fmaxf(m, sm.wmax[w]);
  __syncthreads();
  return m;
}

// Descending radix step: bins b = nb-1 .. 0 hold (count, mass).  Finds the bin where the
// running mass from the top first reaches `target` (mass mode) or where the running
// count first reaches `target` (count mode); returns the bin and the amount strictly
// above it.  nb is 4096, 2048, 1024 or 512.
template <bool MASS>
AS_DEVICE void select_bin(VScan &sm, const uint32_t *cnt, const u64 *mass, int nb, u64 target,
                          u64 base, int &sel, u64 &above) {
  const int t = threadIdx.x;
  if (t == 0) {  // defined result even if no bin qualifies (cannot happen for valid sums)
    if (MASS) { sm.sel_p = 0; sm.above_p = base; }
    else { sm.sel_k = 0; sm.above_k = (uint32_t)base; }
  }
  const int per = nb / VT > 0 ? nb / VT : 1;   // bins per thread
  const bool owner = t * per < nb;
  u64 local = 0;
  if (owner) {
    for (int j = 0; j < per; ++j) {
      const int bin = nb - 1 - (t * per + j);
      local += MASS ? mass[bin] : (u64)cnt[bin];
    }
  }
  u64 tot;
  u64 run = base + block_scan_excl(local, sm, tot);
  if (owner) {
    for (int j = 0; j < per; ++j) {
      const int bin = nb - 1 - (t * per + j);
      const u64 v = MASS ? mass[bin] : (u64)cnt[bin];
      if (run < target && run + v >= target) {
        if (MASS) { sm.sel_p = bin; sm.above_p = run; }
        else { sm.sel_k = bin; sm.above_k = (uint32_t)run; }
      }
      run += v;
    }
  }
  __syncthreads();
  sel = MASS ? sm.sel_p : sm.sel_k;
  above = MASS ? sm.above_p : (u64)sm.above_k;
  __syncthreads();
}

struct Sel {
  uint32_t tau_p, tau_k;   // exact threshold keys
  u64 above_p;             // mass strictly above tau_p
  uint32_t above_k;        // count strictly above tau_k
  uint32_t j_p, j_k;       // tied ids (ascending) kept at the thresholds
  uint32_t c_p, c_k;       // tie counts at the thresholds
  float M;                 // row max
  float c_hi, c_lo;        // log2(e) / T as a float pair
  float inv_hi, inv_lo;    // 1 / nucleus mass (fixed point units) as a float pair
};

// The raw v_exp_f32: for exponents >= -126 it is exactly exp2f (whose extra steps only
// rescale subnormal results), and anything below 2^-41 rounds to 0 in fixed point anyway.
// The exponent (z - M) log2(e) / T takes the factor as a float pair, so its error is the
// rounding of z - M and of the final sum only (random from element to element, not a
// tilt of the whole distribution).
AS_DEVICE float elem_e(float z, const Sel &s) {
  const float d = z - s.M;
  return __builtin_amdgcn_exp2f(fmaf(d, s.c_hi, d * s.c_lo));
}

// p_r of one element given its nucleus membership: the weight's fixed-point value times
// 1 / (nucleus mass), the latter again as a float pair.
AS_DEVICE float elem_p(float z, bool in, const Sel &s) {
  const float f = fixw_f(elem_e(z, s));
  return in ? fmaf(f, s.inv_hi, f * s.inv_lo) : 0.f;
}

// Nucleus / top-k membership given the element's rank among ids tied at the threshold.
AS_DEVICE bool in_nucleus(uint32_t key, uint32_t tie_rank, const Sel &s) {
  return key > s.tau_p || (key == s.tau_p && tie_rank < s.j_p);
}
AS_DEVICE bool in_topk(uint32_t key, uint32_t tie_rank, const Sel &s) {
  return key > s.tau_k || (key == s.tau_k && tie_rank < s.j_k);
}

// Wave-level exclusive prefix of per-lane counts.
AS_DEVICE uint32_t wave_excl_u32(uint32_t v) {
  const int lane = threadIdx.x & 63;
  uint32_t x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o);
    if (lane >= o) x += y;
  }
  return x - v;
}
AS_DEVICE u64 wave_incl_u64(u64 v) {
  const int lane = threadIdx.x & 63;
  u64 x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const u64 y = __shfl_up(x, o);
    if (lane >= o) x += y;
  }
  return x;
}

// Per-lane tie ranks of the 4 elements a lane holds in segment s (ids s*256+lane*4+i).
AS_DEVICE void tie_ranks(const uint32_t key[4], bool valid, uint32_t tau, uint32_t base,
                         uint32_t rank[4]) {
  uint32_t n = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) n += (valid && key[i] == tau) ? 1u : 0u;
  uint32_t r = base + wave_excl_u32(n);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    rank[i] = r;
    r += (valid && key[i] == tau) ? 1u : 0u;
  }
}

// Inverse CDF inside segment s: the smallest id whose running mass exceeds `target`,
// where `excl` is the mass before the segment.  mode 0: p_r, mode 1: max(0, p_r - Q).
// Executed by one whole wave; returns the id (in every lane).
AS_DEVICE int seg_inverse_cdf(const float *z, const float *q, int V, int s, u64 excl, u64 target,
                              int mode, const Sel &sel, const VSmem &sm) {
  const int lane = threadIdx.x & 63;
  const int id0 = s * SEG + lane * 4;
  const bool valid = id0 < V;
  float4 z4 = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
  float4 q4 = make_float4(0.f, 0.f, 0.f, 0.f);
  if (valid) {
    z4 = *(const float4 *)(z + id0);
    if (mode == 1) q4 = *(const float4 *)(q + id0);
  }
  const float zz[4] = {z4.x, z4.y, z4.z, z4.w};
  const float qq[4] = {q4.x, q4.y, q4.z, q4.w};
  uint32_t key[4], rank[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) key[i] = f32_key(zz[i]);
  if (sel.c_p > 1) tie_ranks(key, valid, sel.tau_p, sm.g.tie_p[s], rank);
  else {
#pragma unroll
    for (int i = 0; i < 4; ++i) rank[i] = 0;
  }
  u64 w[4];
  u64 lt = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float p = valid ? elem_p(zz[i], in_nucleus(key[i], rank[i], sel), sel) : 0.f;
    const float v = mode == 1 ? fmaxf(p - qq[i], 0.f) : p;
    w[i] = valid ? fixw(v) : 0;
    lt += w[i];
  }
  const u64 incl = excl + wave_incl_u64(lt);
  u64 run = incl - lt;
  int found = 0x7fffffff;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    run += w[i];
    if (found == 0x7fffffff && run > target && w[i] > 0) found = id0 + i;
  }
  // smallest id over the wave
  int f = found;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) f = min(f, __shfl_xor(f, o));
  return f < V ? f : V - 1;
}

// Finds the segment whose [excl, excl + mass) contains target (mass > 0); arrays hold
// exclusive prefixes.  Any lane may call it.
AS_DEVICE int find_segment(const u64 *excl, int nseg, u64 target) {
  int lo = 0, hi = nseg - 1;  // last segment with excl <= target
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (excl[mid] <= target) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// Loads the VR float4 this thread handles in one step of a pass over the row, all issued
// before any is used: one load in flight per thread leaves the passes bound by memory
// latency rather than bandwidth.  Past the end of the row the row's last float4 is
// loaded again (V is a multiple of 4): every load is unconditional, so the compiler can
// wait for the older loads only, and the callers skip those entries.
constexpr int VR = 2;  // float4 a thread per step of the row passes (the segment pass: VU)
constexpr int VU = 2;
AS_DEVICE void load_step(const float *z, int V, int i0, float4 (&v)[VR]) {
#pragma unroll
  for (int u = 0; u < VR; ++u) {
    const int i = i0 + u * VT * 4;
    v[u] = *(const float4 *)(z + (i < V ? i : V - 4));
  }
}

// A pass over the row, VR float4 per thread a step: the next step's loads are issued
// before the current step is processed, so a thread always has loads in flight.
struct RowStream {
  const float *z;
  int V, i0;
  float4 cur[VR], nxt[VR];
  AS_DEVICE RowStream(const float *z_, int V_, int start) : z(z_), V(V_), i0(start) {
    load_step(z, V, i0, cur);
  }
  AS_DEVICE bool more() const { return i0 < V; }
  AS_DEVICE void prefetch() { load_step(z, V, i0 + VT * 4 * VR, nxt); }
  AS_DEVICE void advance() {
#pragma unroll
    for (int u = 0; u < VR; ++u) cur[u] = nxt[u];
    i0 += VT * 4 * VR;
  }
};

// Sum over the 16 lanes of a row, in every lane.
AS_DEVICE uint32_t row16_sum(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true);   // lane ^ 1
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true);   // lane ^ 2
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, true);  // half mirror
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, true);  // mirror
  return v;
}
AS_DEVICE u64 row16_sum(u64 v) {
#pragma unroll
  for (int o = 1; o < 16; o <<= 1) v += __shfl_xor(v, o);
  return v;
}
// 2^40 v as an integer, for v given in units of 2^-40 and already whole.
AS_DEVICE u64 whole_u64(float f) { return (u64)f; }
constexpr float SMALL_FX = 268435456.f;   // 2^28

// Segments [sb, se) of a row in which no ids are tied at the thresholds: 16 lanes a
// segment, four segments a wave and step, so that the sums over lanes cost a sixth of those
// over a wave.  The masses are the integers that segment_pass adds up: p 2^40 comes straight
// from the scaled normaliser (scaling by a power of two commutes with the roundings), and
// masses below 2^-12, nearly all, are added as 32-bit integers, the others of a group of
// four ids as 64-bit ones.  What bounds the pass is this arithmetic (about 25 instructions
// an id with the residual, 50 before).
AS_DEVICE bool segment_pass_untied(const float *z, const float *q, int V, int sb, int se,
                                   bool resid, const Sel &sel, VTop &sm, u64 *seg_p, u64 *seg_r) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 4, p16 = lane & 15;
  const float i_hi = sel.inv_hi * AS_FX_SCALE, i_lo = sel.inv_lo * AS_FX_SCALE;
  bool badq = false;
  for (int s0 = sb + wave * 4; s0 < se; s0 += NWV * 4) {
    const int s = s0 + g, id0 = s * SEG + p16 * 4;
    const int lim = s < se ? V : 0;
    float4 z4[4], q4[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int id = id0 + k * 64, ld = id < lim ? id : V - 4;
      // last pass over the row and its draft q: streamed past L2 and the MALL
      z4[k] = ld_stream(z + ld);
      if (resid) q4[k] = ld_stream(q + ld);
    }
    uint32_t sp = 0, sr = 0;
    u64 sp64 = 0, sr64 = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int id = id0 + k * 64;
      const bool valid = id < lim;
      const float zz[4] = {z4[k].x, z4[k].y, z4[k].z, z4[k].w};
      float P[4], R[4];
      bool top = false;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint32_t key = f32_key(zz[j]);
        const float f = fixw_f(elem_e(zz[j], sel));
        P[j] = valid && key >= sel.tau_p ? fmaf(f, i_hi, f * i_lo) : 0.f;
        top |= key >= sel.tau_k;
      }
      if (resid) {
        const float qq[4] = {q4[k].x, q4[k].y, q4[k].z, q4[k].w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          badq |= valid && !(qq[j] >= 0.f && qq[j] <= 3.402823466e38f);
          R[j] = rintf(fmaxf(fmaf(qq[j], -AS_FX_SCALE, P[j]), 0.f));
        }
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) P[j] = rintf(P[j]);
      if (fmaxf(fmaxf(P[0], P[1]), fmaxf(P[2], P[3])) < SMALL_FX) {
        sp += ((uint32_t)P[0] + (uint32_t)P[1]) + ((uint32_t)P[2] + (uint32_t)P[3]);
        if (resid) sr += ((uint32_t)R[0] + (uint32_t)R[1]) + ((uint32_t)R[2] + (uint32_t)R[3]);
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          sp64 += whole_u64(P[j]);
          if (resid) sr64 += whole_u64(R[j]);
        }
      }
      if (top && valid) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const uint32_t key = f32_key(zz[j]);
          if (key >= sel.tau_k) {
            const uint32_t slot = atomicAdd(&sm.ncand, 1u);
            if (slot < KMAX) {
              sm.cand_key[slot] = key;
              sm.cand_id[slot] = id + j;
              sm.cand_in[slot] = key >= sel.tau_p ? 1u : 0u;
            }
          }
        }
      }
    }
    u64 tp, tr = 0;
    if (__ballot((sp64 | sr64) != 0) == 0) {
      // 16 sums below 2^32: their 16-bit halves add up in 32 bits
      tp = ((u64)row16_sum(sp >> 16) << 16) + row16_sum(sp & 0xFFFFu);
      if (resid) tr = ((u64)row16_sum(sr >> 16) << 16) + row16_sum(sr & 0xFFFFu);
    } else {
      tp = row16_sum(sp64 + sp);
      if (resid) tr = row16_sum(sr64 + sr);
    }
    if (p16 == 0 && s < se) {
      seg_p[s] = tp;
      seg_r[s] = tr;
    }
  }
  return badq;
}

// Segments [sb, se) of a row, one wave a segment: the fixed-point masses of p_r (seg_p) and
// of the residual (seg_r, when resid), and the top-k ids, appended to sm.cand_*.  tie_base
// gives the number of ids tied at the two thresholds before a segment (asked for only where
// ids are tied).  Every draft probability read is checked: returns whether this thread saw a
// NaN, infinite or negative one.  The VU segments of a step are loaded before any is used;
// past the end of the row the last float4 is loaded again (unconditional loads), those lanes
// are not valid.
template <typename TieBase>
AS_DEVICE bool segment_pass(const float *z, const float *q, int V, int sb, int se, bool resid,
                            const Sel &sel, VTop &sm, TieBase tie_base, u64 *seg_p, u64 *seg_r) {
  // (rows of fewer segments than the workgroup's 16-lane groups leave some of those idle: 2048
  // rows of 1024 ids take 101 us in all this way and 106 that, of 8192 ids 138 and 134)
  if (sel.c_p <= 1 && sel.c_k <= 1 && V >= NWV * 4 * SEG)
    return segment_pass_untied(z, q, V, sb, se, resid, sel, sm, seg_p, seg_r);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  bool badq = false;
  for (int s0 = sb + wave; s0 < se; s0 += NWV * VU) {
    float4 z4u[VU], q4u[VU];
#pragma unroll
    for (int u = 0; u < VU; ++u) {
      const int id0 = (s0 + u * NWV) * SEG + lane * 4;
      const int ld = id0 < V ? id0 : V - 4;
      // last pass over the row and its draft q: streamed past L2 and the MALL (the
      // earlier passes keep the default policy, so their re-reads may hit the MALL)
      z4u[u] = ld_stream(z + ld);
      q4u[u] = resid ? ld_stream(q + ld) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int u = 0; u < VU; ++u) {
      const int s = s0 + u * NWV;
      if (s >= se) break;
      const int id0 = s * SEG + lane * 4;
      const bool valid = id0 < V;
      const float4 z4 = z4u[u], q4 = q4u[u];
      const float zz[4] = {z4.x, z4.y, z4.z, z4.w};
      const float qq[4] = {q4.x, q4.y, q4.z, q4.w};
      uint32_t key[4], rp[4], rk[4], tp = 0, tk = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) key[j] = f32_key(zz[j]);
      if (sel.c_p > 1 || sel.c_k > 1) tie_base(s, tp, tk);
      if (sel.c_p > 1) tie_ranks(key, valid, sel.tau_p, tp, rp);
      else {
#pragma unroll
        for (int j = 0; j < 4; ++j) rp[j] = 0;
      }
      if (sel.c_k > 1) tie_ranks(key, valid, sel.tau_k, tk, rk);
      else {
#pragma unroll
        for (int j = 0; j < 4; ++j) rk[j] = 0;
      }
      u64 sp_ = 0, sr_ = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (!valid) continue;
        const bool inn = in_nucleus(key[j], rp[j], sel);
        const float p = elem_p(zz[j], inn, sel);
        sp_ += fixw(p);
        if (resid) {
          badq |= !(qq[j] >= 0.f && qq[j] <= 3.402823466e38f);
          sr_ += fixw(fmaxf(p - qq[j], 0.f));
        }
        if (in_topk(key[j], rk[j], sel)) {
          const uint32_t slot = atomicAdd(&sm.ncand, 1u);
          if (slot < KMAX) {
            sm.cand_key[slot] = key[j];
            sm.cand_id[slot] = id0 + j;
            sm.cand_in[slot] = inn ? 1u : 0u;
          }
        }
      }
      sp_ = wave_sum_u64(sp_);
      sr_ = wave_sum_u64(sr_);
      if (lane == 0) {
        seg_p[s] = sp_;
        seg_r[s] = sr_;
      }
    }
  }
  return badq;
}

// The largest mass target of the nucleus: ceil(top_p * S), within [1, S].
AS_DEVICE u64 nucleus_target(float top_p, u64 S) {
  u64 T = (u64)ceil((double)top_p * (double)S);
  if (T < 1) T = 1;
  return T > S ? S : T;
}

// Whether row r has drafted children (the tail: every row has one).  Every lane of the wave
// calls it and looks at a row of its own: one row after the other, each a load of its own,
// took 9 us of a 65-row tree's 45 (65 rows of 4096 ids).
AS_DEVICE bool row_has_child(const acespec::VocabArgs &a, size_t srow0, int r) {
  if (a.tail) return true;
  bool any = false;
  for (int c = r + 1 + (threadIdx.x & 63); c < a.n1; c += 64) any |= a.par[srow0 + c] == r;
  return __any(any);
}

// The row's maximum from the LM head's column tiles (+inf when a logit is not finite).
AS_DEVICE float tile_row_max(const acespec::VocabArgs &a, int row, VScan &sm) {
  const float *tm = a.tile_max + (size_t)row * a.ntile;
  float mx = -INFINITY;
  for (int t = threadIdx.x; t < a.ntile; t += VT) mx = max_or_inf(mx, tm[t]);
  return block_max(mx, sm);
}

// ------------------------------------------------------------------------------------
// Few rows: one workgroup a row leaves most CUs idle and is a chain of latencies over the
// whole row (17 rows of 128256 ids: 150 us).  The passes are split over `chunks` workgroups
// a row, a kernel each, with the same integer sums and the same exact thresholds, so the
// results are those of the whole-row kernel, bit for bit:
//   hist     each chunk's histogram over 1024 bins of the exponent (M - z) log2(e) / T, 0.04
//            wide (finer where it matters than the key's top bits, and evenly filled)
//   bins     one workgroup a row: sums the chunks' histograms, finds the bins in which the
//            top-p mass and the k-th id fall
//   collect  keys and ids of those two bins' elements (a few hundred)
//   select   one workgroup a row: exact thresholds from that list
//   segments each chunk's part of pass 4
//   finish   vocab_verify_kernel<true>, from the prefix sums on
// A row whose list overflows, or with more than TIES ids tied at a threshold, is marked and
// done whole by the last kernel.
// ------------------------------------------------------------------------------------
constexpr int NBIN = 1024;
constexpr float BIN_PER = 25.f;     // bins per unit of the base-2 exponent
constexpr int LCAP = 4096;          // listed elements a row
constexpr int TIES = 16;
struct RowState {
  uint32_t nlist, ntop, whole, badq;   // whole: the last kernel does the row by itself
  int bp, bk;
  u64 T_p, ap, ak;
  Sel sel;
  uint32_t nan;
  int32_t tie_p[TIES], tie_k[TIES];    // ids tied at the thresholds (when more than one)
  uint32_t top_key[KMAX];
  int32_t top_id[KMAX];
  uint32_t top_in[KMAX];
};

// Monotone in z (each step is): larger logits, larger bins.
AS_DEVICE int exp_bin(float z, float M, float c_hi) {
  const float t = (z - M) * c_hi * -BIN_PER;
  return NBIN - 1 - (int)fminf(t, (float)(NBIN - 1));
}

struct SplitView {   // one row's part of the scratch
  RowState *st;
  uint32_t *cnt;     // [chunks][NBIN]
  u64 *mass;         // [chunks][NBIN]
  uint2 *list;       // [LCAP] key, id
  u64 *seg_p, *seg_r;
};
__host__ __device__ constexpr size_t split_row_bytes(int chunks, int nseg) {
  return ((sizeof(RowState) + 255) & ~(size_t)255) + (size_t)chunks * NBIN * 12 +
         (size_t)LCAP * 8 + (((size_t)nseg * 16 + 255) & ~(size_t)255);
}
AS_DEVICE SplitView split_view(const acespec::VocabArgs &a, int row) {
  const int nseg = (a.V + SEG - 1) / SEG;
  char *p = (char *)a.split + (size_t)row * split_row_bytes(a.chunks, nseg);
  SplitView v;
  v.st = (RowState *)p;
  p += (sizeof(RowState) + 255) & ~(size_t)255;
  v.mass = (u64 *)p;
  p += (size_t)a.chunks * NBIN * 8;
  v.cnt = (uint32_t *)p;
  p += (size_t)a.chunks * NBIN * 4;
  v.list = (uint2 *)p;
  p += (size_t)LCAP * 8;
  v.seg_p = (u64 *)p;
  v.seg_r = v.seg_p + nseg;
  return v;
}
// Segments of chunk c.
AS_DEVICE void chunk_range(const acespec::VocabArgs &a, int c, int &sb, int &se) {
  const int nseg = (a.V + SEG - 1) / SEG;
  sb = (int)((long long)nseg * c / a.chunks);
  se = (int)((long long)nseg * (c + 1) / a.chunks);
}

__global__ __launch_bounds__(VT) void vocab_hist_kernel(acespec::VocabArgs a) {
  __shared__ VScan sm;
  __shared__ uint32_t cnt[NBIN];
  __shared__ u64 mass[NBIN];
  const int row = blockIdx.x / a.chunks, c = blockIdx.x - row * a.chunks, tid = threadIdx.x;
  const SplitView v = split_view(a, row);
  Sel sel;
  sel.M = tile_row_max(a, row, sm);
  sel.c_hi = a.c_hi;
  sel.c_lo = a.c_lo;
  if (c == 0 && tid == 0) {
    v.st->nlist = v.st->ntop = v.st->badq = 0;
    v.st->whole = v.st->nan = !(sel.M <= 3.402823466e38f);
    v.st->sel.M = sel.M;
  }
  if (!(sel.M <= 3.402823466e38f)) return;
  for (int i = tid; i < NBIN; i += VT) {
    cnt[i] = 0;
    mass[i] = 0;
  }
  __syncthreads();
  int sb, se;
  chunk_range(a, c, sb, se);
  const int i_end = min(se * SEG, a.V);
  const float *z = a.logits + (size_t)row * a.V;
  for (RowStream rs(z, i_end, sb * SEG + tid * 4); rs.more(); rs.advance()) {
    rs.prefetch();
#pragma unroll
    for (int u = 0; u < VR; ++u) {
      if (rs.i0 + u * VT * 4 >= i_end) break;
      const float zz[4] = {rs.cur[u].x, rs.cur[u].y, rs.cur[u].z, rs.cur[u].w};
      float e[4];
      u64 w[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) e[j] = elem_e(zz[j], sel);
      fix4(e, w);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int b = exp_bin(zz[j], sel.M, sel.c_hi);
        atomicAdd(&cnt[b], 1u);
        atomicAdd(&mass[b], w[j]);
      }
    }
  }
  __syncthreads();
  for (int i = tid; i < NBIN; i += VT) {
    v.cnt[(size_t)c * NBIN + i] = cnt[i];
    v.mass[(size_t)c * NBIN + i] = mass[i];
  }
}

__global__ __launch_bounds__(VT) void vocab_bins_kernel(acespec::VocabArgs a) {
  __shared__ VScan sm;
  __shared__ uint32_t cnt[NBIN];
  __shared__ u64 mass[NBIN];
  const int row = blockIdx.x, tid = threadIdx.x;
  const SplitView v = split_view(a, row);
  if (v.st->nan) return;
  u64 tot = 0;
  for (int i = tid; i < NBIN; i += VT) {
    uint32_t n = 0;
    u64 m = 0;
#pragma unroll 8
    for (int c = 0; c < a.chunks; ++c) {
      n += v.cnt[(size_t)c * NBIN + i];
      m += v.mass[(size_t)c * NBIN + i];
    }
    cnt[i] = n;
    mass[i] = m;
    tot += m;
  }
  const u64 T_p = nucleus_target(a.top_p, block_sum(tot, sm));
  int bp, bk;
  u64 ap, ak;
  select_bin<true>(sm, cnt, mass, NBIN, T_p, 0, bp, ap);
  select_bin<false>(sm, cnt, mass, NBIN, (u64)a.k, 0, bk, ak);
  if (tid == 0) {
    v.st->bp = bp;
    v.st->bk = bk;
    v.st->T_p = T_p;
    v.st->ap = ap;
    v.st->ak = ak;
  }
}

__global__ __launch_bounds__(VT) void vocab_collect_kernel(acespec::VocabArgs a) {
  __shared__ uint2 list[LCAP / 2];
  __shared__ uint32_t n, at;
  const int row = blockIdx.x / a.chunks, c = blockIdx.x - row * a.chunks, tid = threadIdx.x;
  const SplitView v = split_view(a, row);
  if (v.st->nan) return;
  const int bp = v.st->bp, bk = v.st->bk;
  const float M = v.st->sel.M;
  if (tid == 0) n = 0;
  __syncthreads();
  int sb, se;
  chunk_range(a, c, sb, se);
  const int i_end = min(se * SEG, a.V);
  const float *z = a.logits + (size_t)row * a.V;
  for (RowStream rs(z, i_end, sb * SEG + tid * 4); rs.more(); rs.advance()) {
    rs.prefetch();
#pragma unroll
    for (int u = 0; u < VR; ++u) {
      if (rs.i0 + u * VT * 4 >= i_end) break;
      const float zz[4] = {rs.cur[u].x, rs.cur[u].y, rs.cur[u].z, rs.cur[u].w};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int b = exp_bin(zz[j], M, a.c_hi);
        if (b == bp || b == bk) {
          const uint32_t slot = atomicAdd(&n, 1u);
          if (slot < LCAP / 2) list[slot] = make_uint2(f32_key(zz[j]), rs.i0 + u * VT * 4 + j);
        }
      }
    }
  }
  __syncthreads();
  if (n == 0) return;
  // past LCAP (or more than fit here): the row is done whole
  if (tid == 0) at = atomicAdd(&v.st->nlist, n <= LCAP / 2 ? n : LCAP + 1);
  __syncthreads();
  for (uint32_t i = tid; i < min(n, LCAP / 2u) && at + i < LCAP; i += VT) v.list[at + i] = list[i];
}

__global__ __launch_bounds__(VT) void vocab_select_kernel(acespec::VocabArgs a) {
  __shared__ VSmem sm;
  __shared__ uint32_t keys[LCAP];
  __shared__ uint32_t lo_p, hi_p, lo_k, hi_k, np, nk;
  const int row = blockIdx.x, tid = threadIdx.x;
  const SplitView v = split_view(a, row);
  RowState &st = *v.st;
  if (st.nan) return;
  const uint32_t n = st.nlist;
  if (n > LCAP) {
    if (tid == 0) st.whole = 1;
    return;
  }
  Sel sel;
  sel.M = st.sel.M;
  sel.c_hi = a.c_hi;
  sel.c_lo = a.c_lo;
  const int bp = st.bp, bk = st.bk;
  const u64 T_p = st.T_p;
  if (tid == 0) {
    lo_p = lo_k = ~0u;
    hi_p = hi_k = 0;
    np = nk = 0;
  }
  __syncthreads();
  uint32_t mn_p = ~0u, mx_p = 0, mn_k = ~0u, mx_k = 0;
  for (uint32_t i = tid; i < n; i += VT) {
    const uint32_t key = v.list[i].x;
    keys[i] = key;
    const int b = exp_bin(key_to_f32(key), sel.M, sel.c_hi);
    if (b == bp) { mn_p = min(mn_p, key); mx_p = max(mx_p, key); }
    if (b == bk) { mn_k = min(mn_k, key); mx_k = max(mx_k, key); }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    mn_p = min(mn_p, (uint32_t)__shfl_xor((int)mn_p, o));
    mx_p = max(mx_p, (uint32_t)__shfl_xor((int)mx_p, o));
    mn_k = min(mn_k, (uint32_t)__shfl_xor((int)mn_k, o));
    mx_k = max(mx_k, (uint32_t)__shfl_xor((int)mx_k, o));
  }
  if ((tid & 63) == 0) {
    atomicMin(&lo_p, mn_p);
    atomicMax(&hi_p, mx_p);
    atomicMin(&lo_k, mn_k);
    atomicMax(&hi_k, mx_k);
  }
  __syncthreads();
  // radix steps over key - lo, 11 bits at a time from the top of the bins' key ranges; a
  // step's last sub-range ends at its bin's highest key, for the list holds the other bin's
  // elements too, and those above this bin are counted in above_* already
  const uint32_t end_p = hi_p, end_k = hi_k;
  uint32_t bp_lo = lo_p, bk_lo = lo_k, w_p = end_p - lo_p, w_k = end_k - lo_k;  // width - 1
  u64 above_p = st.ap, above_k = st.ak;
  while (true) {
    const uint32_t w = max(w_p, w_k);
    const int bits = 32 - (w ? __clz((int)w) : 32), sh = bits > 11 ? bits - 11 : 0;
    __syncthreads();
    for (int i = tid; i < 2048; i += VT) {
      sm.r.cnt[i] = 0;
      sm.r.mass[i] = 0;
      sm.r.cntk[i] = 0;
    }
    __syncthreads();
    for (uint32_t i = tid; i < n; i += VT) {
      const uint32_t key = keys[i], dp = key - bp_lo, dk = key - bk_lo;
      if (key >= bp_lo && dp <= w_p) {
        atomicAdd(&sm.r.cnt[dp >> sh], 1u);
        atomicAdd(&sm.r.mass[dp >> sh], fixw(elem_e(key_to_f32(key), sel)));
      }
      if (key >= bk_lo && dk <= w_k) atomicAdd(&sm.r.cntk[dk >> sh], 1u);
    }
    __syncthreads();
    int sp, sk;
    u64 ap2, ak2;
    select_bin<true>(sm, sm.r.cnt, sm.r.mass, 2048, T_p, above_p, sp, ap2);
    select_bin<false>(sm, sm.r.cntk, sm.r.mass, 2048, (u64)a.k, above_k, sk, ak2);
    above_p = ap2;
    above_k = ak2;
    bp_lo += (uint32_t)sp << sh;
    bk_lo += (uint32_t)sk << sh;
    if (sh == 0) {
      sel.tau_p = bp_lo;
      sel.tau_k = bk_lo;
      sel.c_p = sm.r.cnt[sp];
      sel.c_k = sm.r.cntk[sk];
      const u64 w_tau = sm.r.mass[sp] / (sel.c_p ? sel.c_p : 1);
      const u64 need = T_p - above_p;  // > 0
      u64 j = w_tau ? (need + w_tau - 1) / w_tau : 1;
      if (j < 1) j = 1;
      if (j > sel.c_p) j = sel.c_p;
      sel.above_p = above_p;
      sel.above_k = (uint32_t)above_k;
      sel.j_p = (uint32_t)j;
      sel.j_k = (uint32_t)((u64)a.k - above_k);
      const double inv = 1.0 / (double)(above_p + j * w_tau);
      sel.inv_hi = (float)inv;
      sel.inv_lo = (float)(inv - (double)sel.inv_hi);
      break;
    }
    w_p = min((1u << sh) - 1, end_p - bp_lo);
    w_k = min((1u << sh) - 1, end_k - bk_lo);
  }
  const bool many = sel.c_p > TIES || sel.c_k > TIES;
  if (tid == 0) {
    st.sel = sel;
    if (many) st.whole = 1;
  }
  if (many) return;
  for (uint32_t i = tid; i < n; i += VT) {
    const uint2 e = v.list[i];
    if (sel.c_p > 1 && e.x == sel.tau_p) st.tie_p[atomicAdd(&np, 1u)] = (int32_t)e.y;
    if (sel.c_k > 1 && e.x == sel.tau_k) st.tie_k[atomicAdd(&nk, 1u)] = (int32_t)e.y;
  }
}

// Ids of a tie list before segment s.
AS_DEVICE uint32_t ties_before(const int32_t *ids, uint32_t n, int s) {
  uint32_t r = 0;
  for (uint32_t i = 0; i < n; ++i) r += ids[i] < s * SEG;
  return r;
}

__global__ __launch_bounds__(VT, 8) void vocab_segments_kernel(acespec::VocabArgs a) {
  __shared__ VTop sm;
  __shared__ uint32_t at;
  const int row = blockIdx.x / a.chunks, c = blockIdx.x - row * a.chunks, tid = threadIdx.x;
  const SplitView v = split_view(a, row);
  RowState &st = *v.st;
  if (st.whole) return;
  const Sel sel = st.sel;
  if (tid == 0) sm.ncand = 0;
  __syncthreads();
  const int b = row / a.n1;
  const bool resid = !a.q_scalar && row_has_child(a, (size_t)b * a.n1, row - b * a.n1);
  int sb, se;
  chunk_range(a, c, sb, se);
  const bool badq = segment_pass(
      a.logits + (size_t)row * a.V, resid ? a.q + (size_t)row * a.V : nullptr, a.V, sb, se, resid,
      sel, sm,
      [&](int s, uint32_t &tp, uint32_t &tk) {
        tp = sel.c_p > 1 ? ties_before(st.tie_p, sel.c_p, s) : 0;
        tk = sel.c_k > 1 ? ties_before(st.tie_k, sel.c_k, s) : 0;
      },
      v.seg_p, v.seg_r);
  if (badq) st.badq = 1;
  __syncthreads();
  const uint32_t n = min(sm.ncand, (uint32_t)KMAX);
  if (n == 0) return;
  if (tid == 0) at = atomicAdd(&st.ntop, n);
  __syncthreads();
  if (tid < (int)n && at + tid < (uint32_t)KMAX) {
    st.top_key[at + tid] = sm.cand_key[tid];
    st.top_id[at + tid] = sm.cand_id[tid];
    st.top_in[at + tid] = sm.cand_in[tid];
  }
}

// (six waves a SIMD: three 8-wave rows per CU, which caps the kernel at 80 VGPRs)
// SPLIT: the row's thresholds, segment masses and top-k ids come from the kernels above.
template <bool SPLIT>
__global__ __launch_bounds__(VT, 6) void vocab_verify_kernel(acespec::VocabArgs a) {
  __shared__ VSmem sm;
  const int row = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int V = a.V;
  const float *z = a.logits + (size_t)row * V;
  const int nseg = (V + SEG - 1) / SEG;

  if (tid == 0) sm.flag = 0;
  Sel sel;
  sel.M = SPLIT ? split_view(a, row).st->sel.M : tile_row_max(a, row, sm);
  sel.c_hi = a.c_hi;
  sel.c_lo = a.c_lo;
  const bool tail = a.tail != 0;
  const int b = row / a.n1, r = row - b * a.n1;
  const size_t srow0 = (size_t)b * a.n1;
  if (!(sel.M <= 3.402823466e38f)) {
    // A logit of this row is NaN or infinite (an activation overflowed upstream): the row
    // gets no decisions, the session's status reports it.  Outputs stay defined.
    const int k = a.k;
    if (tid < k) {
      a.topk_ids[(size_t)row * k + tid] = -1;
      a.topk_probs[(size_t)row * k + tid] = 0.f;
    }
    if (tid == 0) {
      a.bonus[row] = -1;
      a.rowflag[row] = ACESPEC_ENONFINITE;
      if (!tail && r == 0) {
        a.accept[row] = 1;
        a.resample[row] = -1;
      }
    }
    const int c_lo = tail ? 0 : r + 1, c_hi = tail ? 1 : a.n1;
    for (int ci = c_lo + tid; ci < c_hi; ci += VT) {
      const int child = tail ? row : (int)(srow0 + ci);
      if (!tail && a.par[srow0 + ci] != r) continue;
      a.accept[child] = 0;
      a.resample[child] = -1;
    }
    return;
  }

  const bool has_child = row_has_child(a, srow0, r);

  // (a list that does not hold exactly the top-k ids is not used: its other slots are an
  // earlier call's)
  const RowState *st0 = SPLIT ? split_view(a, row).st : nullptr;
  if (SPLIT && !st0->whole && st0->ntop == (uint32_t)a.k) {
    const SplitView v = split_view(a, row);
    const RowState &st = *st0;
    sel = st.sel;
    for (int s = tid; s < nseg; s += VT) {
      sm.g.seg_p[s] = v.seg_p[s];
      sm.g.seg_r[s] = v.seg_r[s];
      if (sel.c_p > 1) sm.g.tie_p[s] = ties_before(st.tie_p, sel.c_p, s);
    }
    if (tid < a.k) {
      sm.cand_key[tid] = st.top_key[tid];
      sm.cand_id[tid] = st.top_id[tid];
      sm.cand_in[tid] = st.top_in[tid];
    }
    if (tid == 0 && st.badq) sm.flag = ACESPEC_EBADDRAFT;
    __syncthreads();
  } else {
  // ---- pass 1: total mass, 12-bit histograms ---------------------------------------
  for (int i = tid; i < 4096; i += VT) {
    sm.h.cnt[i] = 0;
    sm.h.mass[i] = 0;
  }
  if (tid == 0) sm.ncand = 0;
  __syncthreads();
  for (RowStream rs(z, V, tid * 4); rs.more(); rs.advance()) {
    rs.prefetch();
    const int i0 = rs.i0;
    const float4 (&vv)[VR] = rs.cur;
#pragma unroll
    for (int u = 0; u < VR; ++u) {
      if (i0 + u * VT * 4 >= V) break;
      const float zz[4] = {vv[u].x, vv[u].y, vv[u].z, vv[u].w};
      float e[4];
      u64 w[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) e[j] = elem_e(zz[j], sel);
      fix4(e, w);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint32_t key = f32_key(zz[j]);
        atomicAdd(&sm.h.cnt[key >> 20], 1u);
        atomicAdd(&sm.h.mass[key >> 20], w[j]);
      }
    }
  }
  __syncthreads();
  u64 tot = 0;
  for (int i = tid; i < 4096; i += VT) tot += sm.h.mass[i];
  const u64 S_fx = block_sum(tot, sm);
  const u64 T_p = nucleus_target(a.top_p, S_fx);
  const u64 K = (u64)a.k;

  int bp, bk;
  u64 ap, ak;
  select_bin<true>(sm, sm.h.cnt, sm.h.mass, 4096, T_p, 0, bp, ap);
  select_bin<false>(sm, sm.h.cnt, sm.h.mass, 4096, K, 0, bk, ak);

  // ---- pass 2: refine bits 19..9 inside the selected bins ------------------------------
  // The keys of those bins' elements also go to a per-row scratch list (kept in L2), so
  // that pass 3 can read them instead of the row when they fit.
  __syncthreads();  // pass 1's bins are read; their storage is reused
  for (int i = tid; i < 2048; i += VT) {
    sm.r.cnt[i] = 0;
    sm.r.mass[i] = 0;
    sm.r.cntk[i] = 0;
  }
  if (tid == 0) sm.nbin = 0;
  uint32_t *cl = a.cand ? a.cand + (size_t)row * a.cand_cap : nullptr;
  __syncthreads();
  for (RowStream rs(z, V, tid * 4); rs.more(); rs.advance()) {
    rs.prefetch();
    const int i0 = rs.i0;
    const float4 (&vv)[VR] = rs.cur;
#pragma unroll
    for (int u = 0; u < VR; ++u) {
      if (i0 + u * VT * 4 >= V) break;
      const float zz[4] = {vv[u].x, vv[u].y, vv[u].z, vv[u].w};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint32_t key = f32_key(zz[j]);
        const int hi = key >> 20, mid = (key >> 9) & 0x7FF;
        if (hi == bp) {
          atomicAdd(&sm.r.cnt[mid], 1u);
          atomicAdd(&sm.r.mass[mid], fixw(elem_e(zz[j], sel)));
        }
        if (hi == bk) atomicAdd(&sm.r.cntk[mid], 1u);
        if (cl && (hi == bp || hi == bk)) {
          const uint32_t slot = atomicAdd(&sm.nbin, 1u);
          if (slot < (uint32_t)a.cand_cap) cl[slot] = key;
        }
      }
    }
  }
  __syncthreads();
  int sp, sk;
  u64 ap2, ak2;
  select_bin<true>(sm, sm.r.cnt, sm.r.mass, 2048, T_p, ap, sp, ap2);
  select_bin<false>(sm, sm.r.cntk, sm.r.mass, 2048, K, ak, sk, ak2);
  const uint32_t pre_p = ((uint32_t)bp << 11) | (uint32_t)sp;  // key bits 31..9
  const uint32_t pre_k = ((uint32_t)bk << 11) | (uint32_t)sk;

  // ---- pass 3: refine bits 8..0 ------------------------------------------------------
  for (int i = tid; i < 512; i += VT) {
    sm.r.cnt[i] = 0;
    sm.r.mass[i] = 0;
    sm.r.cntk[i] = 0;
  }
  const uint32_t nbin = sm.nbin;  // final: pass 2 ended with a barrier
  __syncthreads();
  if (cl && nbin <= (uint32_t)a.cand_cap) {
    // the candidates' keys (a key maps back to its logit exactly)
    for (uint32_t i = tid; i < nbin; i += VT) {
      const uint32_t key = cl[i];
      if ((key >> 9) == pre_p) {
        atomicAdd(&sm.r.cnt[key & 0x1FF], 1u);
        atomicAdd(&sm.r.mass[key & 0x1FF], fixw(elem_e(key_to_f32(key), sel)));
      }
      if ((key >> 9) == pre_k) atomicAdd(&sm.r.cntk[key & 0x1FF], 1u);
    }
  } else
  for (RowStream rs(z, V, tid * 4); rs.more(); rs.advance()) {
    rs.prefetch();
    const int i0 = rs.i0;
    const float4 (&vv)[VR] = rs.cur;
#pragma unroll
    for (int u = 0; u < VR; ++u) {
      if (i0 + u * VT * 4 >= V) break;
      const float zz[4] = {vv[u].x, vv[u].y, vv[u].z, vv[u].w};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint32_t key = f32_key(zz[j]);
        if ((key >> 9) == pre_p) {
          atomicAdd(&sm.r.cnt[key & 0x1FF], 1u);
          atomicAdd(&sm.r.mass[key & 0x1FF], fixw(elem_e(zz[j], sel)));
        }
        if ((key >> 9) == pre_k) atomicAdd(&sm.r.cntk[key & 0x1FF], 1u);
      }
    }
  }
  __syncthreads();
  int lp, lk;
  u64 ap3, ak3;
  select_bin<true>(sm, sm.r.cnt, sm.r.mass, 512, T_p, ap2, lp, ap3);
  select_bin<false>(sm, sm.r.cntk, sm.r.mass, 512, K, ak2, lk, ak3);
  sel.tau_p = (pre_p << 9) | (uint32_t)lp;
  sel.tau_k = (pre_k << 9) | (uint32_t)lk;
  sel.c_p = sm.r.cnt[lp];
  sel.c_k = sm.r.cntk[lk];
  sel.above_p = ap3;
  sel.above_k = (uint32_t)ak3;
  {
    const u64 w_tau = sm.r.mass[lp] / (sel.c_p ? sel.c_p : 1);
    const u64 need = T_p - ap3;  // > 0
    u64 j = w_tau ? (need + w_tau - 1) / w_tau : 1;
    if (j < 1) j = 1;
    if (j > sel.c_p) j = sel.c_p;
    sel.j_p = (uint32_t)j;
    sel.j_k = (uint32_t)(K - ak3);
    const u64 SN = ap3 + j * w_tau;
    const double inv = 1.0 / (double)SN;
    sel.inv_hi = (float)inv;
    sel.inv_lo = (float)(inv - (double)sel.inv_hi);
  }
  __syncthreads();

  // ---- optional pass: tie ranks at the thresholds (ids ascending) ------------------------
  const bool ties = sel.c_p > 1 || sel.c_k > 1;
  if (ties) {
    for (int s = wave; s < nseg; s += NWV) {
      const int id0 = s * SEG + lane * 4;
      uint32_t np = 0, nk = 0;
      if (id0 < V) {
        const float4 v = *(const float4 *)(z + id0);
        const float zz[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const uint32_t key = f32_key(zz[j]);
          np += key == sel.tau_p;
          nk += key == sel.tau_k;
        }
      }
      np = (uint32_t)wave_sum_i32((int)np);
      nk = (uint32_t)wave_sum_i32((int)nk);
      if (lane == 0) {
        sm.g.tie_p[s] = np;
        sm.g.tie_k[s] = nk;
      }
    }
    __syncthreads();
    if (tid == 0) {  // exclusive prefixes over segments (sequential: rare path)
      uint32_t rp = 0, rk = 0;
      for (int s = 0; s < nseg; ++s) {
        const uint32_t a0 = sm.g.tie_p[s], b0 = sm.g.tie_k[s];
        sm.g.tie_p[s] = rp;
        sm.g.tie_k[s] = rk;
        rp += a0;
        rk += b0;
      }
    }
    __syncthreads();
  }

  // ---- pass 4: id-ordered segments: masses of p_r and of the residual, top-k ids ----------
  const bool resid = !a.q_scalar && has_child;
  const bool badq = segment_pass(
      z, resid ? a.q + (size_t)row * V : nullptr, V, 0, nseg, resid, sel, sm,
      [&](int sg, uint32_t &tp, uint32_t &tk) { tp = sm.g.tie_p[sg]; tk = sm.g.tie_k[sg]; },
      sm.g.seg_p, sm.g.seg_r);
  if (__syncthreads_or(badq) && tid == 0) sm.flag = ACESPEC_EBADDRAFT;
  }
  // Scalar mode: the uplink carries only q-hat of each drafted token (one float per
  // child row); the cloud then tests acceptance and does no sampling, so the residual
  // mass (the only reader of a dense q row) is not needed.
  const bool dense_q = a.q_scalar == nullptr;
  const float *q = dense_q ? a.q + (size_t)row * V : nullptr;
  // exclusive prefixes over segments
  u64 Ptot, Rtot;
  {
    constexpr int SPT = SEGMAX / VT;  // consecutive segments per thread
    u64 lp[SPT], lr[SPT], vp = 0, vr = 0;
#pragma unroll
    for (int j = 0; j < SPT; ++j) {
      const int sg = tid * SPT + j;
      lp[j] = sg < nseg ? sm.g.seg_p[sg] : 0;
      lr[j] = sg < nseg ? sm.g.seg_r[sg] : 0;
      vp += lp[j];
      vr += lr[j];
    }
    u64 ep = block_scan_excl(vp, sm, Ptot);
    u64 er = block_scan_excl(vr, sm, Rtot);
#pragma unroll
    for (int j = 0; j < SPT; ++j) {
      const int sg = tid * SPT + j;
      if (sg < nseg) {
        sm.g.seg_p[sg] = ep;
        sm.g.seg_r[sg] = er;
      }
      ep += lp[j];
      er += lr[j];
    }
  }
  __syncthreads();

  // ---- top-k payload: exactly k candidates, sorted by (key desc, id asc) -----------------
  const int k = a.k;
  {
    u64 wc = 0;
    int rank = 0, cid = 0;
    if (tid < k) {
      const uint32_t mk = sm.cand_key[tid];
      cid = sm.cand_id[tid];
      for (int j = 0; j < k; ++j) {
        const uint32_t ok = sm.cand_key[j];
        rank += (ok > mk) || (ok == mk && sm.cand_id[j] < cid);
      }
      wc = fixw(elem_p(key_to_f32(mk), sm.cand_in[tid] != 0, sel));
    }
    const u64 ksum = block_sum(wc, sm);
    if (tid < k) {
      a.topk_ids[(size_t)row * k + rank] = cid;
      a.topk_probs[(size_t)row * k + rank] = ksum ? (float)((double)wc / (double)ksum) : 0.f;
    }
  }

  // ---- bonus sample from p_r --------------------------------------------------------------
  const float *u = a.u;
  if (wave == 0) {
    int id = -1;
    if (dense_q) {
      const u64 target = (u64)floor((double)u[(size_t)row * 3 + 2] * (double)Ptot);
      const int sg = find_segment(sm.g.seg_p, nseg, target);
      id = seg_inverse_cdf(z, q, V, sg, sm.g.seg_p[sg], target, 0, sel, sm);
    }
    if (lane == 0) a.bonus[row] = id;
  }

  // ---- children: accept test and residual resample ------------------------------------------
  if (!tail && r == 0 && tid == 0) {
    a.accept[row] = 1;
    a.resample[row] = -1;
  }
  // Waves 1.. take the children in turn (wave 0 drew the bonus).
  if (has_child && wave >= 1) {
    int seen = 0;
    const int c_lo = tail ? 0 : r + 1, c_hi = tail ? 1 : a.n1;
    for (int ci = c_lo; ci < c_hi; ++ci) {
      int child;
      if (tail) {
        child = row;
      } else {
        if (a.par[srow0 + ci] != r) continue;
        child = (int)(srow0 + ci);
      }
      const bool mine = (seen % (NWV - 1)) + 1 == wave;
      ++seen;
      if (!mine) continue;
      int x = a.tok[child];
      x = x < 0 ? 0 : (x >= V ? V - 1 : x);
      // p_r(x): nucleus membership needs x's rank among ids tied at the threshold
      const float zx = z[x];
      const uint32_t kx = f32_key(zx);
      uint32_t rx = 0;
      if (kx == sel.tau_p && sel.c_p > 1) {
        const int sx = x / SEG;
        const int id0 = sx * SEG + lane * 4;
        const bool valid = id0 < V;
        const float4 z4 = valid ? *(const float4 *)(z + id0) : make_float4(0.f, 0.f, 0.f, 0.f);
        const uint32_t keys[4] = {f32_key(z4.x), f32_key(z4.y), f32_key(z4.z), f32_key(z4.w)};
        uint32_t rk4[4];
        tie_ranks(keys, valid, sel.tau_p, sm.g.tie_p[sx], rk4);
        const int src = (x - sx * SEG) >> 2;
        const uint32_t mine_rank = rk4[0] * ((x & 3) == 0) + rk4[1] * ((x & 3) == 1) +
                                   rk4[2] * ((x & 3) == 2) + rk4[3] * ((x & 3) == 3);
        rx = __shfl(mine_rank, src);
      }
      const float px = elem_p(zx, in_nucleus(kx, rx, sel), sel);
      const float qx = dense_q ? q[x] : a.q_scalar[child];
      if (!dense_q && !(qx >= 0.f && qx <= 1.f) && lane == 0) sm.flag = ACESPEC_EBADDRAFT;
      const float u0 = u[(size_t)child * 3 + 0], u1 = u[(size_t)child * 3 + 1];
      const bool acc = u0 * qx < px;
      int res = -1;
      if (!dense_q) {
        // no cloud-side resampling in the scalar protocol
      } else if (Rtot > 0) {
        const u64 target = (u64)floor((double)u1 * (double)Rtot);
        const int sg = find_segment(sm.g.seg_r, nseg, target);
        res = seg_inverse_cdf(z, q, V, sg, sm.g.seg_r[sg], target, 1, sel, sm);
      } else {
        const u64 target = (u64)floor((double)u1 * (double)Ptot);
        const int sg = find_segment(sm.g.seg_p, nseg, target);
        res = seg_inverse_cdf(z, q, V, sg, sm.g.seg_p[sg], target, 0, sel, sm);
      }
      if (lane == 0) {
        a.accept[child] = acc ? 1 : 0;
        a.resample[child] = res;
      }
    }
  }
  __syncthreads();
  if (tid == 0) a.rowflag[row] = sm.flag;
}

}  // namespace

namespace acespec {

// Chunks of a row, 1: whole rows.  Six launches take about 43 us however small they are, a
// whole row of 20000 ids 42, of 32000 ids 54, of 128256 ids 140, as long as each row has a
// CU to itself; the rows' bytes take over from there, the sooner the shorter the row.  Split
// against whole, us: 16384 ids, 1 row 41 / 37; 20000 ids, 17 rows 43 / 44, 48 rows 47 / 45;
// 24000 ids, 17 rows 45 / 48, 128 rows 52 / 50; 32000 ids, 128 rows 54 / 58; 128256 ids, 17
// rows 54 / 143.  From 48000 ids on, 512 rows with top_p below 1 (50272 ids 123 / 138, 128256
// ids 249 / 312), 384 with top_p 1, whose threshold lies among few ids, so that whole rows
// need one pass less (384 rows 97 / 92 and 172 / 173, 448 rows 111 / 93 and 204 / 178).
// Beyond 512 rows there are not two chunks a row for the workgroups that the CUs hold.
int vocab_chunks(int rows, int V, float top_p) {
  const int most = V < 20000 ? 0 : V < 24000 ? 32 : V < 48000 ? 128
                                     : top_p < 1.f ? kVocabSplitRows : 384;
  if (rows < 1 || rows > most) return 1;
  const int nseg = (V + SEG - 1) / SEG;
  int c = 1024 / rows;   // every CU holds four of the chunks' workgroups
  if (c > 32) c = 32;
  if (c > nseg / 8) c = nseg / 8;
  return c < 1 ? 1 : c;
}
size_t vocab_split_bytes(int rows, int V) {
  const int c = vocab_chunks(rows, V, 0.f);   // (the most that any top_p takes)
  return c > 1 ? (size_t)rows * split_row_bytes(c, (V + SEG - 1) / SEG) : 0;
}

hipError_t launch_vocab(const VocabArgs &args, hipStream_t s) {
  if (args.V > SEGMAX * SEG || args.k > KMAX || args.k < 1 || !args.tile_max)
    return hipErrorInvalidValue;
  VocabArgs a = args;
  a.chunks = vocab_chunks(a.rows, a.V, a.top_p);
  const dim3 rows(a.rows), parts(a.rows * a.chunks), block(VT);
  if (a.chunks == 1 || !a.split || vocab_split_bytes(a.rows, a.V) > a.split_bytes) {
    hipLaunchKernelGGL(vocab_verify_kernel<false>, rows, block, 0, s, a);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(vocab_hist_kernel, parts, block, 0, s, a);
  hipLaunchKernelGGL(vocab_bins_kernel, rows, block, 0, s, a);
  hipLaunchKernelGGL(vocab_collect_kernel, parts, block, 0, s, a);
  hipLaunchKernelGGL(vocab_select_kernel, rows, block, 0, s, a);
  hipLaunchKernelGGL(vocab_segments_kernel, parts, block, 0, s, a);
  hipLaunchKernelGGL(vocab_verify_kernel<true>, rows, block, 0, s, a);
  return hipGetLastError();
}

}  // namespace acespec
