// Embedding gather, per-position correction rules and commit bookkeeping.
//
// Correction (paper Sec. 3.3, "Verification as Auto Correction"): every
// drafted position k is decided independently and in parallel, one
// workgroup per position:
//   (A) greedy  : argmax of the scoring logits (ties -> lowest code)
//   (B) sample  : inverse-CDF sample of p = softmax(top_k(logits / T))
//   (C) accept/reject: keep the token t with probability min(p(t)/q(t), 1),
//       else sample the residual [p - q]_+; a rejected position stores this
//       round's logits as its next reference q (an accepted one keeps q).
// q is the stored reference warped like p, or a point mass at t.
// Probabilities, sums and the inverse CDF are float64; the top-k set is
// found by a radix select (11, 11 and 10 bits) over order-preserving float
// keys, ties at the boundary resolved towards lower codes.  Uniforms: 24-bit SplitMix64
// outputs at a counter built from (sequence, position, round, stream)
// (Steele, Lea & Flood, OOPSLA 2014).
#include "ssd_internal.h"

namespace ssd {

__device__ __forceinline__ uint16_t f2bf_m(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// ---------------- embedding ----------------
__device__ __forceinline__ int token_of(const TokIn& tok, int t, int V) {
  const int b = t / tok.K, k = t - b * tok.K;
  const int id = tok.ids[(size_t)(b % tok.rows) * tok.stride + k];
  return id < 0 ? 0 : (id >= V ? V - 1 : id);
}

// hi/lo bf16 planes of eight consecutive values, 16 bytes a plane
__device__ __forceinline__ void store_split8(uint16_t* p, size_t i, size_t plane, const float (&v)[8]) {
  uint32_t hi[4], lo[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint16_t a = f2bf_m(v[2 * j]), b = f2bf_m(v[2 * j + 1]);
    hi[j] = (uint32_t)a | ((uint32_t)b << 16);
    lo[j] = (uint32_t)f2bf_m(v[2 * j] - __uint_as_float((uint32_t)a << 16)) |
            ((uint32_t)f2bf_m(v[2 * j + 1] - __uint_as_float((uint32_t)b << 16)) << 16);
  }
  *(uint4*)(p + i) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
  *(uint4*)(p + plane + i) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
}

// sum over the workgroup's 256 threads in a fixed order, valid in thread 0
__device__ __forceinline__ float block_sum_256(float s, float* red) {
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  return red[0];
}

// bf16 models (d a multiple of 256, at most 8192): eight columns a thread,
// 16-byte loads and stores.  The row passes through LDS so that x^2 is summed
// thread by thread over columns t, t + 256, ... and then by halves, the order
// of the one-column kernel (the same 1/rms bits).  1024 rows of 4096: 14.6 us
// against 21.4 us with one column a thread.
__global__ __launch_bounds__(256) void embed_kernel(const uint16_t* emb, TokIn tok, int* zero, int n_zero, int d,
                                                    int V, const float* g, float* x, uint16_t* xn, size_t xn_plane,
                                                    int tiled, float* ssq) {
  __shared__ __attribute__((aligned(16))) float row[8192];
  __shared__ float red[256];
  const int t = blockIdx.x;
  const int id = token_of(tok, t, V);
  if (t == 0)
    for (int i = threadIdx.x; i < n_zero; i += 256) zero[i] = 0;
  for (int c = threadIdx.x * 8; c < d; c += 2048) {
    const uint4 w = *(const uint4*)(emb + (size_t)id * d + c);
    const float4 ga = *(const float4*)(g + c), gb = *(const float4*)(g + c + 4);
    const uint32_t u[4] = {w.x, w.y, w.z, w.w};
    const float gg[8] = {ga.x, ga.y, ga.z, ga.w, gb.x, gb.y, gb.z, gb.w};
    float v[8], gv[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      v[j] = __uint_as_float(j & 1 ? u[j / 2] & 0xFFFF0000u : u[j / 2] << 16);
      gv[j] = gg[j] * v[j];
    }
    const float4 lo = make_float4(v[0], v[1], v[2], v[3]), hi = make_float4(v[4], v[5], v[6], v[7]);
    *(float4*)(row + c) = lo;
    *(float4*)(row + c + 4) = hi;
    *(float4*)(x + (size_t)t * d + c) = lo;
    *(float4*)(x + (size_t)t * d + c + 4) = hi;
    store_split8(xn, act_index(tiled, t, c, d), xn_plane, gv);
  }
  __syncthreads();
  float s = 0.f;
  for (int i = threadIdx.x; i < d; i += 256) s += row[i] * row[i];
  s = block_sum_256(s, red);
  if (threadIdx.x == 0) ssq[t] = s;
}

__global__ __launch_bounds__(256) void embed_f32_kernel(const float* emb, TokIn tok, int* zero, int n_zero, int d,
                                                        int V, const float* g, float* x, float* xn, float* ssq) {
  __shared__ float red[256];
  const int t = blockIdx.x;
  const int id = token_of(tok, t, V);
  if (t == 0)
    for (int i = threadIdx.x; i < n_zero; i += 256) zero[i] = 0;
  float s = 0.f;
  for (int i = threadIdx.x; i < d; i += 256) {
    const float v = emb[(size_t)id * d + i];
    x[(size_t)t * d + i] = v;
    xn[(size_t)t * d + i] = g[i] * v;
    s += v * v;
  }
  s = block_sum_256(s, red);
  if (threadIdx.x == 0) ssq[t] = s;
}

void embed(const Dims& dm, const void* emb, const TokIn& tok, int* zero, int n_zero, int M, const float* g, float* x,
           void* xn, size_t xn_plane, int tiled, float* ssq, hipStream_t st) {
  if (dm.bf16)
    hipLaunchKernelGGL(embed_kernel, dim3(M), dim3(256), 0, st, (const uint16_t*)emb, tok, zero, n_zero, dm.d, dm.V, g, x,
                       (uint16_t*)xn, xn_plane, tiled, ssq);
  else
    hipLaunchKernelGGL(embed_f32_kernel, dim3(M), dim3(256), 0, st, (const float*)emb, tok, zero, n_zero, dm.d, dm.V, g,
                       x, (float*)xn, ssq);
}

// one 16-byte piece a thread: at most a few rows, a launch's latency
__global__ __launch_bounds__(256) void last_rows_kernel(const float* x, int K, int d, float* out) {
  const int c = (blockIdx.x * 256 + threadIdx.x) * 4, b = blockIdx.y;
  if (c < d) *(float4*)(out + (size_t)b * d + c) = *(const float4*)(x + ((size_t)b * K + K - 1) * d + c);
}

void last_rows(const float* x, int B, int K, int d, float* out, hipStream_t st) {
  hipLaunchKernelGGL(last_rows_kernel, dim3((d + 1023) / 1024, B), dim3(256), 0, st, x, K, d, out);
}

__global__ __launch_bounds__(256) void ssq_kernel(const float* x, int d, float* ssq) {
  __shared__ float red[256];
  const int t = blockIdx.x;
  float s = 0.f;
  for (int i = threadIdx.x; i < d; i += 256) {
    float v = x[(size_t)t * d + i];
    s += v * v;
  }
  s = block_sum_256(s, red);
  if (threadIdx.x == 0) ssq[t] = s;
}

void norm_rows_f32(const float* x, int M, int d, float* ssq, hipStream_t st) {
  hipLaunchKernelGGL(ssq_kernel, dim3(M), dim3(256), 0, st, x, d, ssq);
}

// ---------------- block helpers (256 threads) ----------------
constexpr int NT_SEL = 256;

__device__ __forceinline__ uint32_t fkey(float f) {
  uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ uint64_t sm_mix(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// output number c+1 of the SplitMix64 stream seeded with `seed`, top 24 bits in [0,1)
__device__ __forceinline__ double uniform24(unsigned long long seed, int b, int pos, unsigned round, int stream) {
  const uint64_t c = ((uint64_t)b << 44) | ((uint64_t)pos << 20) | ((uint64_t)(round & 0xFFFFu) << 4) | (uint64_t)stream;
  const uint64_t z = sm_mix(seed + (c + 1ull) * 0x9E3779B97F4A7C15ull);
  return (double)(z >> 40) * (1.0 / 16777216.0);
}

struct SelShared {
  float fred[NT_SEL / 64];
  int ired[NT_SEL / 64];
};

// argmax with ties to the lowest index over row[0..V)
// Lowest index among the maxima.  Thread t scans elements 4t + 1024 j .. +3
// in ascending order (16-byte loads: each wave load is one contiguous 1 KiB
// span); the reductions below keep the lower index among equal values, so
// the result does not depend on how the elements are dealt to threads.
__device__ int block_argmax(const float* row, int V, SelShared& sh) {
  float bv = -INFINITY;
  int bi = 0x7fffffff;
  if ((V & 3) == 0 && (((uintptr_t)row) & 15) == 0) {
    auto take = [&](const float4 x, int v) {
      if (x.x > bv || bi == 0x7fffffff) {
        bv = x.x;
        bi = v;
      }
      if (x.y > bv) {
        bv = x.y;
        bi = v + 1;
      }
      if (x.z > bv) {
        bv = x.z;
        bi = v + 2;
      }
      if (x.w > bv) {
        bv = x.w;
        bi = v + 3;
      }
    };
    // eight loads in flight, then taken in order (a load used right away is
    // waited for alone)
    constexpr int UB = 8, STR = NT_SEL * 4;
    int v = threadIdx.x * 4;
    for (; v + (UB - 1) * STR < V; v += UB * STR) {
      float4 x[UB];
#pragma unroll
      for (int u = 0; u < UB; ++u) x[u] = *(const float4*)(row + v + u * STR);
#pragma unroll
      for (int u = 0; u < UB; ++u) take(x[u], v + u * STR);
    }
    for (; v < V; v += STR) take(*(const float4*)(row + v), v);
  } else {
    for (int v = threadIdx.x; v < V; v += NT_SEL) {
      const float x = row[v];
      if (x > bv || bi == 0x7fffffff) {
        bv = x;
        bi = v;
      }
    }
  }
  for (int o = 32; o > 0; o >>= 1) {
    float ov = __shfl_xor(bv, o);
    int oi = __shfl_xor(bi, o);
    if (ov > bv || (ov == bv && oi < bi)) {
      bv = ov;
      bi = oi;
    }
  }
  __syncthreads();
  if ((threadIdx.x & 63) == 0) {
    sh.fred[threadIdx.x >> 6] = bv;
    sh.ired[threadIdx.x >> 6] = bi;
  }
  __syncthreads();
  float rv = sh.fred[0];
  int ri = sh.ired[0];
  for (int w = 1; w < NT_SEL / 64; ++w) {
    if (sh.fred[w] > rv || (sh.fred[w] == rv && sh.ired[w] < ri)) {
      rv = sh.fred[w];
      ri = sh.ired[w];
    }
  }
  __syncthreads();
  return ri;
}

// ---------------- rules (B) and (C): warped distributions ----------------
// One workgroup of 16 waves per position.  A row is read in 16-byte loads,
// wave w walking the w-th contiguous segment, so every pass over it is
// coalesced and index order is wave order, then lane order.  A kept set is
// held as a threshold key and the index of its last boundary tie, a test any
// thread can make for any code; where it has at most SMP_LIST codes it is
// also compacted into LDS in index order, and the float64 exponentials (about
// 50 instructions each) run over those codes instead of the whole row.
// Four 32-token rows, 16384 codes, top 2000, rule C: 360 -> 50 us a launch (59
// with every pass reading the row again); two 24-token rows, rule B: 151 -> 25.
constexpr int SMP_T = 1024, SMP_W = SMP_T / 64;
constexpr int SMP_LIST = 4096;
constexpr int SMP_HELD = 256 * SMP_W;  // codes a workgroup holds per group of a wave
constexpr int SMP_BINS = 2048;

struct SmpShared {
  int hist[SMP_BINS];
  int idx[SMP_LIST];   // kept codes in index order, and their logits
  float val[SMP_LIST];
  double dred[SMP_W];
  int ired[2][SMP_W];
  float fred[SMP_W];
  unsigned bc[4];
};

// row elements v .. v + 3 (V a multiple of four and the row 16-byte aligned: one load); n of them exist
struct Quad {
  float x[4];
  int n;
};
__device__ __forceinline__ Quad load_quad(const float* row, int v, int V, bool vec) {
  Quad q;
  q.n = max(0, min(4, V - v));
  if (vec) {
    if (q.n > 0) {
      const float4 f = *(const float4*)(row + v);
      q.x[0] = f.x, q.x[1] = f.y, q.x[2] = f.z, q.x[3] = f.w;
    }
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (e < q.n) q.x[e] = row[v + e];
  }
  return q;
}

// The segment of this wave, in groups of 256 codes (four per lane).  NG > 0:
// read once and held (rows of up to 4096 NG codes: the kept set takes five
// passes over them), in registers and, with 128 of them a lane, 48 (NG = 4) or
// 180 (NG = 8) bytes of scratch; NG = 0: read again by every pass.
template <int NG>
struct Seg {
  const float* row;
  int beg, groups, V;
  bool vec;
  Quad held[NG > 0 ? NG : 1];
  __device__ __forceinline__ Seg(const float* r, int v) : row(r), V(v) {
    const int all = (V + 255) / 256, per = (all + SMP_W - 1) / SMP_W, w = threadIdx.x >> 6;
    beg = w * per * 256;
    groups = max(0, min(per, all - w * per));
    vec = (V & 3) == 0 && (((uintptr_t)row) & 15) == 0;
    if constexpr (NG > 0) {
#pragma unroll
      for (int i = 0; i < NG; ++i) {
        held[i] = Quad{};
        if (i < groups) held[i] = load_quad(row, code(i), V, vec);
      }
    }
  }
  // first of this lane's four codes in group i
  __device__ __forceinline__ int code(int i) const { return beg + i * 256 + (threadIdx.x & 63) * 4; }
  // fn(first code, quad) over the groups in order (every lane of the wave together)
  template <int U = 4, typename F>
  __device__ __forceinline__ void each(F fn) const {
    if constexpr (NG > 0) {
#pragma unroll
      for (int i = 0; i < NG; ++i)
        if (i < groups) fn(code(i), held[i]);
    } else {
#pragma unroll U
      for (int i = 0; i < groups; ++i) fn(code(i), load_quad(row, code(i), V, vec));
    }
  }
};

__device__ double smp_sum(double v, SmpShared& sh) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh.dred[threadIdx.x >> 6] = v;
  __syncthreads();
  double r = 0.0;
#pragma unroll
  for (int w = 0; w < SMP_W; ++w) r += sh.dred[w];
  return r;
}

// A warped distribution p_v = [v kept] exp(z_v - mz) / Z, z = row / T.
struct Dist {
  const float* row;
  double T, mz, Z;
  uint32_t thr;  // kept: keys above thr, and keys equal to it up to index cut
  int cut;
  bool all;
  int n;         // kept codes listed in LDS (-1: not listed)
  __device__ __forceinline__ bool keep(uint32_t key, int v) const {
    return all || key > thr || (key == thr && v <= cut);
  }
  __device__ __forceinline__ double prob(float x) const { return exp((double)x / T - mz) / Z; }
  // probability of any code
  __device__ __forceinline__ double at(int v) const {
    const float x = row[v];
    return keep(fkey(x), v) ? prob(x) : 0.0;
  }
};

// Kept set and normaliser of top_k(row / T).  Every thread returns the same
// Dist; the LDS list belongs to the last call.
template <int NG>
__device__ Dist make_dist(const float* row, int V, int top_k, double T, SmpShared& sh) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const Seg<NG> sg(row, V);
  Dist d;
  d.row = row;
  d.T = T;
  d.all = top_k <= 0 || top_k >= V;
  d.thr = 0;
  d.cut = V;
  d.n = -1;
  d.Z = 1.0;
  float mx = -INFINITY;
  int need = 0;
  if (d.all) {
    sg.each([&](int, const Quad& q) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (e < q.n) mx = fmaxf(mx, q.x[e]);
    });
  } else {
    uint32_t prefix = 0, mask = 0;
    int remaining = top_k;
#pragma unroll 1
    for (int pass = 0; pass < 3; ++pass) {
      const int shift = pass == 0 ? 21 : pass == 1 ? 10 : 0;
      const uint32_t dm = pass == 2 ? 1023u : 2047u;
      __syncthreads();  // the previous user of the shared arrays is done
      sh.hist[tid] = 0;
      sh.hist[tid + SMP_T] = 0;
      __syncthreads();
      sg.each([&](int, const Quad& q) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (e < q.n) {
            const uint32_t key = fkey(q.x[e]);
            if (pass == 0) mx = fmaxf(mx, q.x[e]);
            if ((key & mask) == prefix) atomicAdd(&sh.hist[(key >> shift) & dm], 1);
          }
      });
      __syncthreads();
      // digits in descending order, two per thread: the one whose running
      // count first reaches `remaining`
      const int b0 = SMP_BINS - 1 - 2 * tid;
      const int h0 = sh.hist[b0], h1 = sh.hist[b0 - 1];
      int inc = h0 + h1;
      for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(inc, o);
        if (lane >= o) inc += t;
      }
      if (lane == 63) sh.ired[0][wave] = inc;
      __syncthreads();
      int before = 0;
#pragma unroll
      for (int w = 0; w < SMP_W; ++w) before += w < wave ? sh.ired[0][w] : 0;
      inc += before;
      const int exc = inc - h0 - h1;
      if (exc < remaining && inc >= remaining) {  // one thread
        const bool second = exc + h0 < remaining;
        sh.bc[0] = second ? b0 - 1 : b0;
        sh.bc[1] = remaining - (second ? exc + h0 : exc);
        sh.bc[2] = second ? h1 : h0;
      }
      __syncthreads();
      prefix |= sh.bc[0] << shift;
      mask |= dm << shift;
      remaining = (int)sh.bc[1];
    }
    d.thr = prefix;
    need = remaining;                        // keys equal to thr that are kept
    const int ties = (int)sh.bc[2];          // of this many
    const bool list = top_k <= SMP_LIST;
    if (list || ties != need) {
      // keys above and equal to thr per wave; then the kept codes' places in index order
      int gt = 0, eq = 0;
      sg.each([&](int, const Quad& q) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (e < q.n) {
            const uint32_t key = fkey(q.x[e]);
            gt += key > d.thr;
            eq += key == d.thr;
          }
      });
      for (int o = 32; o > 0; o >>= 1) {
        gt += __shfl_xor(gt, o);
        eq += __shfl_xor(eq, o);
      }
      if (lane == 0) {
        sh.ired[0][wave] = gt;
        sh.ired[1][wave] = eq;
      }
      __syncthreads();
      int gtb = 0, eqb = 0;
#pragma unroll
      for (int w = 0; w < SMP_W; ++w) {
        gtb += w < wave ? sh.ired[0][w] : 0;
        eqb += w < wave ? sh.ired[1][w] : 0;
      }
      int at = gtb + min(eqb, need);  // place of this wave's next kept code
      const uint64_t below = (1ull << lane) - 1;
      sg.each([&](int v, const Quad& q) {
        bool kg[4], ke[4];
        int eq_below = eqb, eq_all = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t key = e < q.n ? fkey(q.x[e]) : 0u;
          kg[e] = e < q.n && key > d.thr;
          ke[e] = e < q.n && key == d.thr;
          const uint64_t m = __ballot(ke[e]);
          eq_below += __popcll(m & below);
          eq_all += __popcll(m);
        }
        int k_below = at, k_all = 0;
        bool kept[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          kept[e] = kg[e] || (ke[e] && eq_below < need);
          if (ke[e] && eq_below == need - 1) sh.bc[3] = (unsigned)(v + e);  // the last kept tie: one lane
          eq_below += ke[e];
          const uint64_t m = __ballot(kept[e]);
          k_below += __popcll(m & below);
          k_all += __popcll(m);
        }
        if (list) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (kept[e]) {
              sh.idx[k_below] = v + e;
              sh.val[k_below] = q.x[e];
              ++k_below;
            }
        }
        at += k_all;
        eqb += eq_all;
      });
      __syncthreads();
      d.cut = (int)sh.bc[3];
      if (list) d.n = top_k;
    }
  }
  // largest logit, then the normaliser over the kept codes
  for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
  if (lane == 0) sh.fred[wave] = mx;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < SMP_W; ++w) mx = fmaxf(mx, sh.fred[w]);
  d.mz = (double)mx / T;
  double z = 0.0;
  if (d.n >= 0) {
    for (int i = tid; i < d.n; i += SMP_T) z += exp((double)sh.val[i] / T - d.mz);
  } else {
    Seg<0>(row, V).template each<1>([&](int v, const Quad& q) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (e < q.n && d.keep(fkey(q.x[e]), v + e)) z += exp((double)q.x[e] / T - d.mz);
    });
  }
  d.Z = smp_sum(z, sh);
  return d;
}

// Inverse CDF over the kept codes of p (whose list, if any, is in LDS) with
// weights wf(v, p_v): the smallest code whose running sum exceeds u * total,
// else the last code of positive weight.  *total: the sum of the weights.
template <typename WF>
__device__ int smp_invcdf(const Dist& p, int V, double u, WF wf, double* total, SmpShared& sh) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const bool list = p.n >= 0;
  // this thread's weights in index order: four consecutive list entries, or
  // (a wave's codes) the sum of its segment
  constexpr int EPT = SMP_LIST / SMP_T;
  double w[EPT], s = 0.0;
  int last = -1;
  if (list) {
    const int per = (p.n + SMP_T - 1) / SMP_T;
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      const int i = tid * per + e;
      w[e] = 0.0;
      if (e < per && i < p.n) {
        w[e] = wf(sh.idx[i], p.prob(sh.val[i]));
        s += w[e];
        if (w[e] > 0.0) last = sh.idx[i];
      }
    }
  } else {
    Seg<0>(p.row, V).each<1>([&](int v, const Quad& q) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (e < q.n && p.keep(fkey(q.x[e]), v + e)) {
          const double x = wf(v + e, p.prob(q.x[e]));
          s += x;
          if (x > 0.0) last = v + e;
        }
    });
  }
  // running sums: over the lanes of a wave (list order), then over the waves
  double inc = s;
  for (int o = 1; o < 64; o <<= 1) {
    const double t = __shfl_up(inc, o);
    if (lane >= o) inc += t;
  }
  __syncthreads();
  if (lane == 63) sh.dred[wave] = inc;
  __syncthreads();
  double base = 0.0, tot = 0.0;
#pragma unroll
  for (int x = 0; x < SMP_W; ++x) {
    if (x == wave) base = tot;
    tot += sh.dred[x];
  }
  *total = tot;
  const double target = u * tot;
  int cand = 0x7fffffff;
  if (list) {
    const int per = (p.n + SMP_T - 1) / SMP_T;
    double c = base + (inc - s);
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      const int i = tid * per + e;
      c += w[e];
      if (e < per && i < p.n && c > target && cand == 0x7fffffff) cand = sh.idx[i];
    }
  } else if (base + sh.dred[wave] > target) {
    // the wave walks its segment in index order until the sum passes the target
    double run = base;
    bool found = false;
    Seg<0>(p.row, V).each<1>([&](int v, const Quad& q) {
      if (found) return;
      double x[4], t = 0.0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        x[e] = e < q.n && p.keep(fkey(q.x[e]), v + e) ? wf(v + e, p.prob(q.x[e])) : 0.0;
        t += x[e];
      }
      double ti = t;
      for (int o = 1; o < 64; o <<= 1) {
        const double y = __shfl_up(ti, o);
        if (lane >= o) ti += y;
      }
      double c = run + (ti - t);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        c += x[e];
        if (e < q.n && c > target && cand == 0x7fffffff) cand = v + e;
      }
      run += __shfl(ti, 63);
      found = __ballot(cand != 0x7fffffff) != 0;
    });
  }
  for (int o = 32; o > 0; o >>= 1) {
    cand = min(cand, __shfl_xor(cand, o));
    last = max(last, __shfl_xor(last, o));
  }
  if (lane == 0) {
    sh.ired[0][wave] = cand;
    sh.ired[1][wave] = last;
  }
  __syncthreads();
#pragma unroll
  for (int x = 0; x < SMP_W; ++x) {
    cand = min(cand, sh.ired[0][x]);
    last = max(last, sh.ired[1][x]);
  }
  return cand != 0x7fffffff ? cand : last;
}

// position k of sequence b is already chosen (a fixed first position or an end-of-line token)
__device__ __forceinline__ bool sel_fixed(const SelectArgs& a, int b, int k) {
  return k < a.n_fixed || (a.eol_period > 0 && (a.f[b] + k - a.eol_base) % a.eol_period == a.eol_period - 1);
}

// scoring logits of position k of sequence b: the output at k - 1, the carry for k = 0
__device__ __forceinline__ const float* sel_logits(const SelectArgs& a, int b, int k) {
  return k == 0 ? a.carry + (size_t)b * a.Vimg : a.logits + ((size_t)b * a.K + k - 1) * a.Vimg;
}

// rule (A), and the strict mode's argmax
__global__ __launch_bounds__(NT_SEL) void select_greedy_kernel(SelectArgs a) {
  __shared__ SelShared sh;
  const int k = blockIdx.x, b = blockIdx.y;
  const int V = a.Vimg;
  const size_t idx = (size_t)b * a.K + k;
  if (sel_fixed(a, b, k)) {
    if (threadIdx.x == 0) a.accept[idx] = 0;
    return;
  }
  int* tok = a.tokens + (size_t)b * a.tok_stride + k;
  int t = *tok - a.img_lo;
  t = t < 0 ? 0 : (t >= V ? V - 1 : t);
  const int newt = block_argmax(sel_logits(a, b, k), V, sh);
  if (threadIdx.x == 0) {
    if (a.truncate) a.amax[idx] = newt;
    *tok = newt + a.img_lo;
    a.accept[idx] = newt == t ? 1 : 0;
    if (newt == t) atomicAdd(&a.count[b], 1);
  }
}

// rules (B) and (C)
template <int NG>
__global__ __launch_bounds__(SMP_T) void select_sample_kernel(SelectArgs a) {
  __shared__ SmpShared sh;
  const int k = blockIdx.x, b = blockIdx.y;
  const int V = a.Vimg;
  const size_t idx = (size_t)b * a.K + k;
  if (sel_fixed(a, b, k)) {
    if (threadIdx.x == 0) a.accept[idx] = 0;
    return;
  }
  const float* L = sel_logits(a, b, k);
  int* tok = a.tokens + (size_t)b * a.tok_stride + k;
  int t = *tok - a.img_lo;
  t = t < 0 ? 0 : (t >= V ? V - 1 : t);
  const int pos = a.f[b] + k;
  const double u1 = uniform24(a.seed, b, pos, a.round, 1);
  int newt = t;
  bool acc = false;
  double tot;
  if (a.rule == SSD_SAMPLE) {
    const Dist p = make_dist<NG>(L, V, a.top_k, a.temperature, sh);
    newt = smp_invcdf(p, V, u1, [](int, double pv) { return pv; }, &tot, sh);
    acc = newt == t;
  } else {
    const int slot = pos % a.ring;
    const bool has_ref = a.ref_flag[(size_t)b * a.ring + slot] != 0;
    float* refrow = a.ref + ((size_t)b * a.ring + slot) * V;
    Dist q{};
    double qt = 1.0;  // a point mass at t without a reference
    if (has_ref) {
      q = make_dist<NG>(refrow, V, a.top_k, a.temperature, sh);
      qt = q.at(t);
    }
    const Dist p = make_dist<NG>(L, V, a.top_k, a.temperature, sh);
    const double pt = p.at(t);
    const double alpha = qt > 0.0 ? fmin(pt / qt, 1.0) : (pt > 0.0 ? 1.0 : 0.0);
    const double u0 = uniform24(a.seed, b, pos, a.round, 0);
    if (u0 < alpha) {
      acc = true;
    } else {
      // residual [p - q]_+, positive only where p keeps a code
      const int r = smp_invcdf(
          p, V, u1,
          [&](int v, double pv) {
            const double x = pv - (has_ref ? q.at(v) : (v == t ? 1.0 : 0.0));
            return x > 0.0 ? x : 0.0;
          },
          &tot, sh);
      if (!(tot > 0.0)) {
        acc = true;  // zero residual mass (rounding only): keep the token
      } else {
        newt = r;
        // the rejected position's reference becomes this round's backbone logits (every read of it is done)
        if ((V & 3) == 0)
          for (int v = threadIdx.x * 4; v < V; v += SMP_T * 4) *(float4*)(refrow + v) = *(const float4*)(L + v);
        else
          for (int v = threadIdx.x; v < V; v += SMP_T) refrow[v] = L[v];
        if (threadIdx.x == 0) a.ref_flag[(size_t)b * a.ring + slot] = 1;
      }
    }
  }
  if (threadIdx.x == 0) {
    *tok = newt + a.img_lo;
    a.accept[idx] = acc ? 1 : 0;
    if (acc) atomicAdd(&a.count[b], 1);
  }
}

void select_tokens(const SelectArgs& a, hipStream_t st) {
  if (a.rule == SSD_GREEDY || a.truncate)
    hipLaunchKernelGGL(select_greedy_kernel, dim3(a.K, a.B), dim3(NT_SEL), 0, st, a);
  else if (a.Vimg <= 4 * SMP_HELD)
    hipLaunchKernelGGL(select_sample_kernel<4>, dim3(a.K, a.B), dim3(SMP_T), 0, st, a);
  else if (a.Vimg <= 8 * SMP_HELD)
    hipLaunchKernelGGL(select_sample_kernel<8>, dim3(a.K, a.B), dim3(SMP_T), 0, st, a);
  else
    hipLaunchKernelGGL(select_sample_kernel<0>, dim3(a.K, a.B), dim3(SMP_T), 0, st, a);
}

// truncate mode: accepted run, new frontier and carry
__global__ __launch_bounds__(256) void truncate_kernel(SelectArgs a, int* f, float* carry) {
  __shared__ int kk_s;
  const int b = blockIdx.x;
  if (threadIdx.x == 0) {
    int kk = a.n_fixed;
    while (kk < a.K && a.accept[(size_t)b * a.K + kk]) ++kk;
    kk_s = kk;
    a.count[b] = kk - a.n_fixed;
  }
  __syncthreads();
  const int kk = kk_s;
  if (kk >= 1) {
    const float* src = a.logits + ((size_t)b * a.K + kk - 1) * a.Vimg;
    for (int v = threadIdx.x; v < a.Vimg; v += 256) carry[(size_t)b * a.Vimg + v] = src[v];
  }
  __syncthreads();
  if (threadIdx.x == 0) f[b] += kk;
}

void truncate_finalize(const SelectArgs& a, int* f, hipStream_t st) {
  hipLaunchKernelGGL(truncate_kernel, dim3(a.B), dim3(256), 0, st, a, f, (float*)a.carry);
}

// commit: carry <- logits row (b * rps + last); f += f_inc; drop the references of the committed positions
// Workgroups (x, b): the carry row of sequence b is copied by all gridDim.x
// workgroups of b in 16-byte vectors; workgroup 0 alone clears the reference
// flags of the committed positions and advances the frontier.
__global__ __launch_bounds__(256) void commit_kernel(int Vimg, const float* logits, int rps, int last, float* carry,
                                                     int* f, int f_inc, int* ref_flag, int ring) {
  const int b = blockIdx.y;
  const float* src = logits + ((size_t)b * rps + last) * Vimg;
  float* dst = carry + (size_t)b * Vimg;
  if ((Vimg & 3) == 0) {
    for (int v = (blockIdx.x * 256 + threadIdx.x) * 4; v < Vimg; v += gridDim.x * 1024)
      *(float4*)(dst + v) = *(const float4*)(src + v);
  } else {
    for (int v = blockIdx.x * 256 + threadIdx.x; v < Vimg; v += gridDim.x * 256) dst[v] = src[v];
  }
  if (blockIdx.x != 0) return;
  const int f0 = f[b];
  if (ref_flag)
    for (int k = threadIdx.x; k < f_inc && k < ring; k += 256) ref_flag[(size_t)b * ring + (f0 + k) % ring] = 0;
  __syncthreads();
  if (threadIdx.x == 0) f[b] = f0 + f_inc;
}

// workgroups per sequence: one per 1024 carry values, at most 16
static int commit_groups(int Vimg) { return std::max(1, std::min(16, (Vimg + 1023) / 1024)); }

void commit_update(int B, int K, int Vimg, const float* logits, float* carry, int* f, int* ref_flag, int ring,
                   hipStream_t st) {
  // K > 0: logits rows are [B][K], carry from row K-1, f += K.
  // K < 0: logits rows are [B][1] (last row only), f += -K.
  int rps = K > 0 ? K : 1, last = K > 0 ? K - 1 : 0, inc = K > 0 ? K : -K;
  hipLaunchKernelGGL(commit_kernel, dim3(commit_groups(Vimg), B), dim3(256), 0, st, Vimg, logits, rps, last, carry, f,
                     inc, ref_flag, ring);
}

void commit_prefix(int B, int rps, int Kc, int Vimg, const float* logits, float* carry, int* f, int* ref_flag,
                   int ring, hipStream_t st) {
  hipLaunchKernelGGL(commit_kernel, dim3(commit_groups(Vimg), B), dim3(256), 0, st, Vimg, logits, rps, Kc - 1, carry,
                     f, Kc, ref_flag, ring);
}

// Classifier-free guidance: guided logits l_u + w (l_c - l_u) of each image b
// (conditional stream b, unconditional stream Bi + b).  Workgroup (r, b): rows
// r < K of the pass's logits [2*Bi*K][V] (row = stream * K + r), r = K the
// carry [2*Bi][V].  K = 0 mixes the carry only.
__global__ __launch_bounds__(256) void cfg_mix_kernel(int Bi, int K, int Vimg, float w, const float* logits,
                                                      const float* carry, float* out_logits, float* out_carry) {
  const int r = blockIdx.x, b = blockIdx.y;
  const float *c, *u;
  float* o;
  if (r < K) {
    c = logits + ((size_t)b * K + r) * Vimg;
    u = logits + ((size_t)(Bi + b) * K + r) * Vimg;
    o = out_logits + ((size_t)b * K + r) * Vimg;
  } else {
    c = carry + (size_t)b * Vimg;
    u = carry + (size_t)(Bi + b) * Vimg;
    o = out_carry + (size_t)b * Vimg;
  }
  if ((Vimg & 3) == 0) {
    const float4* c4 = reinterpret_cast<const float4*>(c);
    const float4* u4 = reinterpret_cast<const float4*>(u);
    float4* o4 = reinterpret_cast<float4*>(o);
    for (int v = threadIdx.x; v < Vimg / 4; v += 256) {
      const float4 x = c4[v], y = u4[v];
      o4[v] = make_float4(y.x + w * (x.x - y.x), y.y + w * (x.y - y.y), y.z + w * (x.z - y.z), y.w + w * (x.w - y.w));
    }
  } else {
    for (int v = threadIdx.x; v < Vimg; v += 256) o[v] = u[v] + w * (c[v] - u[v]);
  }
}

void cfg_mix(int Bi, int K, int Vimg, float w, const float* logits, const float* carry, float* out_logits,
             float* out_carry, hipStream_t st) {
  hipLaunchKernelGGL(cfg_mix_kernel, dim3(K + 1, Bi), dim3(256), 0, st, Bi, K, Vimg, w, logits, carry, out_logits,
                     out_carry);
}

// Which XCD (accelerator complex die) each workgroup runs on: the XCC_ID
// hardware register (bits [3:0]).  Used once at start-up to verify the
// round-robin workgroup-to-XCD dispatch the split-K reductions rely on.
__global__ void xcc_probe_kernel(int* out) {
  if (threadIdx.x == 0) out[blockIdx.x] = (int)(__builtin_amdgcn_s_getreg(20 | (0 << 6) | ((4 - 1) << 11)) & 0xF);
}

void xcc_probe(int* out, int n_wg, hipStream_t st) {
  hipLaunchKernelGGL(xcc_probe_kernel, dim3(n_wg), dim3(64), 0, st, out);
}

// Rotary table of a session: angles and their cosine and sine in float64,
// rounded to fp32.  One thread per pair on the device: a session of 4352
// positions and 64 pairs takes 6.7 us, against 8.4 ms for the same loop on
// the host (278528 pow, cos and sin calls) plus the copy and its wait.
__global__ __launch_bounds__(256) void rope_table_kernel(float2* tab, int positions, int half, double theta) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (size_t)positions * half) return;
  const int p = (int)(i / half), j = (int)(i - (size_t)p * half);
  const double ang = (double)p * pow(theta, -(double)j / half);
  tab[i] = make_float2((float)cos(ang), (float)sin(ang));
}

void rope_table(float2* tab, int positions, int half, double theta, hipStream_t st) {
  const size_t n = (size_t)positions * half;
  hipLaunchKernelGGL(rope_table_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, tab, positions, half,
                     theta);
}

__global__ __launch_bounds__(256) void fill_u32_kernel(unsigned* p, size_t n, unsigned v) {
  const size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (i + 4 <= n)
    *(uint4*)(p + i) = make_uint4(v, v, v, v);
  else
    for (size_t j = i; j < n; ++j) p[j] = v;
}

// (p 16-byte aligned: an array of the library)
void fill_u32(unsigned* p, size_t n, unsigned v, hipStream_t st) {
  if (n == 0) return;
  hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)((n + 1023) / 1024)), dim3(256), 0, st, p, n, v);
}

// rows of src [B][K][Vimg] become the references of positions f+k (only_new: keep existing ones); sixteen waves
// a row, 16-byte copies where both sides allow them (rows of 16384 codes: 6.6 us against 18.3 us with four waves
// copying words)
__global__ __launch_bounds__(1024) void set_ref_kernel(int rows_per_b, int Vimg, const float* src, const int* f,
                                                       float* ref, int* ref_flag, int ring, int only_new) {
  const int k = blockIdx.x, b = blockIdx.y;
  const int slot = (f[b] + k) % ring;
  int* fl = ref_flag + (size_t)b * ring + slot;
  if (only_new && *fl) return;
  const float* s = src + ((size_t)b * rows_per_b + k) * Vimg;
  float* d = ref + ((size_t)b * ring + slot) * Vimg;
  if ((Vimg & 3) == 0 && (((uintptr_t)s | (uintptr_t)d) & 15) == 0) {
#pragma unroll 4
    for (int v = threadIdx.x * 4; v < Vimg; v += 4096) *(float4*)(d + v) = *(const float4*)(s + v);
  } else {
    for (int v = threadIdx.x; v < Vimg; v += 1024) d[v] = s[v];
  }
  __syncthreads();
  if (threadIdx.x == 0) *fl = 1;
}

void set_ref_rows(int B, int K, int rows_per_b, int Vimg, const float* src, const int* f, float* ref, int* ref_flag,
                  int ring, int only_new, hipStream_t st) {
  hipLaunchKernelGGL(set_ref_kernel, dim3(K, B), dim3(1024), 0, st, rows_per_b, Vimg, src, f, ref, ref_flag, ring,
                     only_new);
}

// first image token from the carry: argmax (rule A) or a sample of the warped carry (uniform stream 2, round 0)
__global__ __launch_bounds__(NT_SEL) void first_argmax_kernel(int Vimg, int img_lo, const float* carry, int* out_abs,
                                                              int out_stride) {
  __shared__ SelShared sh;
  const int b = blockIdx.x;
  const int v = block_argmax(carry + (size_t)b * Vimg, Vimg, sh);
  if (threadIdx.x == 0) out_abs[(size_t)b * out_stride] = v + img_lo;
}

__global__ __launch_bounds__(SMP_T) void first_sample_kernel(int Vimg, int img_lo, const float* carry, int top_k,
                                                             double T, unsigned long long seed, const int* f,
                                                             int* out_abs, int out_stride) {
  __shared__ SmpShared sh;
  const int b = blockIdx.x;
  const Dist p = make_dist<0>(carry + (size_t)b * Vimg, Vimg, top_k, T, sh);
  double tot;
  const int v = smp_invcdf(p, Vimg, uniform24(seed, b, f[b], 0u, 2), [](int, double pv) { return pv; }, &tot, sh);
  if (threadIdx.x == 0) out_abs[(size_t)b * out_stride] = v + img_lo;
}

// Draft-head input z = [h; e] as split bf16 planes [R][2d]: h fp32 (hi/lo),
// e the bf16 embedding row of the token (exact in the hi plane).  Eight
// columns a thread: 512 rows of d 4096 in 6.9 us against 19.1 us with one.
__global__ __launch_bounds__(256) void draft_input_kernel(const float* h, const uint16_t* emb, const int* tok, int d,
                                                          uint16_t* z, size_t plane, int tiled) {
  const int r = blockIdx.x;
  const uint16_t* er = emb + (size_t)tok[r] * d;
  for (int c = threadIdx.x * 8; c < d; c += 2048) {
    const float4 a = *(const float4*)(h + (size_t)r * d + c), b = *(const float4*)(h + (size_t)r * d + c + 4);
    const uint4 e = *(const uint4*)(er + c);
    const float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    store_split8(z, act_index(tiled, r, c, 2 * d), plane, v);
    const size_t i = act_index(tiled, r, d + c, 2 * d);
    *(uint4*)(z + i) = e;
    *(uint4*)(z + plane + i) = make_uint4(0, 0, 0, 0);
  }
}

void draft_input(const float* h, const void* emb, const int* tok, int R, int d, void* z, size_t plane, int tiled,
                 hipStream_t st) {
  hipLaunchKernelGGL(draft_input_kernel, dim3(R), dim3(256), 0, st, h, (const uint16_t*)emb, tok, d, (uint16_t*)z,
                     plane, tiled);
}

// fp32 models: z = [h; e] as plain fp32 rows [R][2d]
__global__ __launch_bounds__(256) void draft_input_f32_kernel(const float* h, const float* emb, const int* tok, int d,
                                                              float* z) {
  const int r = blockIdx.x;
  const float* hr = h + (size_t)r * d;
  const float* er = emb + (size_t)tok[r] * d;
  float* zr = z + (size_t)r * 2 * d;
  for (int i = threadIdx.x; i < d; i += blockDim.x) {
    zr[i] = hr[i];
    zr[d + i] = er[i];
  }
}

void draft_input_f32(const float* h, const float* emb, const int* tok, int R, int d, float* z, hipStream_t st) {
  hipLaunchKernelGGL(draft_input_f32_kernel, dim3(R), dim3(256), 0, st, h, emb, tok, d, z);
}

void first_token(int B, int Vimg, int img_lo, const float* carry, int rule, int top_k, double temperature,
                 unsigned long long seed, const int* f, int* out_abs, int out_stride, hipStream_t st) {
  if (rule == SSD_GREEDY)
    hipLaunchKernelGGL(first_argmax_kernel, dim3(B), dim3(NT_SEL), 0, st, Vimg, img_lo, carry, out_abs, out_stride);
  else
    hipLaunchKernelGGL(first_sample_kernel, dim3(B), dim3(SMP_T), 0, st, Vimg, img_lo, carry, top_k, temperature, seed,
                       f, out_abs, out_stride);
}

// The greedy argmax a of a logits row (lowest code among equal maxima) placed
// at image index x = f[b] - P + pos_off of sequence b: with `keep` it is a
// planted draft (a where keep[x] is set, else the other code
// repl[x] + (repl[x] >= a)), without it the token itself (the pending token of
// strict verification).  `active` (optional) gates sequences: an inactive one
// is skipped, and a planted replacement (or x outside [0, x_end)) deactivates
// it.  One workgroup per sequence.
__global__ __launch_bounds__(NT_SEL) void place_argmax_kernel(PlaceArgs a) {
  __shared__ SelShared sh;
  const int b = blockIdx.x;
  if (a.active && a.active[b] == 0) return;
  const int x = a.f[b] - a.P + a.pos_off;
  if (x < 0 || x >= a.x_end) {
    if (a.active && threadIdx.x == 0) a.active[b] = 0;
    return;
  }
  const int am = block_argmax(a.logits + (size_t)b * a.row_stride, a.Vimg, sh);
  int t = am;
  bool kept = true;
  if (a.keep) {
    kept = a.keep[(size_t)b * a.x_end + x] != 0;
    if (!kept) {
      const int r = a.repl[(size_t)b * a.x_end + x];
      t = r + (r >= am ? 1 : 0);
    }
  }
  if (threadIdx.x == 0) {
    const int id = t + a.img_lo;
    a.img[(size_t)b * a.img_stride + x] = id;
    if (a.table) a.table[(size_t)b * a.x_end + x] = id;
    if (a.next_tok) a.next_tok[b] = id;
    if (a.active && !kept) a.active[b] = 0;
  }
}

void place_argmax(const PlaceArgs& a, int B, hipStream_t st) {
  hipLaunchKernelGGL(place_argmax_kernel, dim3(B), dim3(NT_SEL), 0, st, a);
}

// tok[b][k] = img[b][f[b] - P + k], k < K (blocks at per-sequence frontiers)
__global__ __launch_bounds__(64) void gather_block_kernel(const int* img, int img_stride, const int* f, int P, int K,
                                                          int* tok) {
  const int b = blockIdx.x;
  const int* src = img + (size_t)b * img_stride + (f[b] - P);
  for (int k = threadIdx.x; k < K; k += 64) tok[(size_t)b * K + k] = src[k];
}

void gather_block(const int* img, int img_stride, const int* f, int P, int K, int B, int* tok, hipStream_t st) {
  hipLaunchKernelGGL(gather_block_kernel, dim3(B), dim3(64), 0, st, img, img_stride, f, P, K, tok);
}

__global__ void add_i32_kernel(int* p, int n, int delta) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] += delta;
}

void add_i32(int* p, int n, int delta, hipStream_t st) {
  if (n <= 0 || delta == 0) return;
  hipLaunchKernelGGL(add_i32_kernel, dim3((n + 255) / 256), dim3(256), 0, st, p, n, delta);
}

}  // namespace ssd
