// Projection GEMMs of the backbone forward pass, y[t][n] = sum_k in[t][k] W[n][k],
// with the epilogues the verify step needs fused into the final write:
//   QKV    : 1/rms scale, rotary embedding at the token's raster position,
//            q to the query buffer, k/v (bf16) into the KV cache slots [f, f+K)
//   RESID  : x += y; xn = g_next * x; per-block sums of x^2 for the next 1/rms
//   SWIGLU : h = silu(gate / rms) * (up / rms)
//   LOGITS : logits = y / rms  (fp32)
//
// bf16 path (gfx950 MFMA v_mfma_f32_16x16x32_bf16): weights are prepacked into
// 16x32 operand tiles (one 16-byte load per lane fetches a whole A operand) and
// activations arrive as hi/lo bf16 planes (fp32 precision), so each A tile
// meets two B operands.  Passes of up to ROWS_MAX rows stream the weights
// (gemm_rows.h); larger ones run on the tiled kernels here.
#include <cstdlib>
#include <cstring>

#include "gemm_rows.h"
#include "tiles.h"

namespace ssd {

// stored state: bf16 for bf16 models (KV cache)
template <bool BF>
__device__ __forceinline__ void st_state(void* base, size_t i, float v) {
  if (BF)
    ((uint16_t*)base)[i] = f2bf(v);
  else
    ((float*)base)[i] = v;
}

// activation: hi/lo bf16 planes for bf16 models, fp32 otherwise
template <bool BF>
__device__ __forceinline__ void st_split(void* base, size_t plane, size_t i, float v) {
  if (BF) {
    uint16_t hi = f2bf(v);
    ((uint16_t*)base)[i] = hi;
    ((uint16_t*)base)[plane + i] = f2bf(v - bf2f(hi));
  } else {
    ((float*)base)[i] = v;
  }
}

__device__ __forceinline__ float rms_scale(const EpiArgs& e, int t) {
  if (!e.ssq) return 1.f;
  float s = 0.f;
  const size_t c = (size_t)e.ssq_off + (size_t)t * e.ssq_step;
  for (int p = 0; p < e.ssq_parts; ++p) s += e.ssq[(size_t)p * e.ssq_ld + c];
  return 1.0f / sqrtf(s * e.inv_d + e.eps);
}

// Epilogue of the output pair (n, n+1), n even, for token t with accumulators
// (v0, v1) and rms scale r.  Returns the squared new residual values (RESID).
template <bool BF>
__device__ __forceinline__ float epi_pair(const EpiArgs& e, int t, int n, float v0, float v1, float r) {
  switch (e.kind) {
    case EPI_QKV: {
      const int b = t / e.Kblk, k = t - b * e.Kblk;
      const int pos = e.f[b] + k;
      const int D = e.D, half = D >> 1;
      const int qN = e.Hq * D, kN = e.Hkv * D;
      v0 *= r;
      v1 *= r;
      if (n < qN + kN) {
        const bool isq = n < qN;
        const int nn = isq ? n : n - qN;
        const int head = nn / D, j = (nn - head * D) >> 1;
        const float2 cs = e.rope[(size_t)pos * half + j];
        const float a = v0 * cs.x - v1 * cs.y;  // dim j
        const float c = v1 * cs.x + v0 * cs.y;  // dim j + D/2
        if (isq) {
          size_t base = (((size_t)b * e.Hq + head) * e.Kblk + k) * D;
          st_split<BF>(e.q, e.q_plane, base + j, a);
          st_split<BF>(e.q, e.q_plane, base + j + half, c);
        } else {
          size_t base = (((size_t)b * e.Hkv + head) * e.Lmax + pos) * D;
          st_state<BF>(e.kc, base + j, a);
          st_state<BF>(e.kc, base + j + half, c);
        }
      } else {
        const int nv = n - qN - kN;
        const int head = nv / D, dd = nv - head * D;
        size_t base = (((size_t)b * e.Hkv + head) * D + dd) * e.Lmax + pos;
        st_state<BF>(e.vc, base, v0);
        st_state<BF>(e.vc, base + e.Lmax, v1);
      }
      return 0.f;
    }
    case EPI_RESID: {
      size_t i = (size_t)t * e.ld + n;
      float2 xo = e.x ? *(const float2*)(e.x + i) : make_float2(0.f, 0.f);
      float x0 = xo.x + v0, x1 = xo.y + v1;
      *(float2*)(e.xo + i) = make_float2(x0, x1);
      st_split<BF>(e.xn, e.xn_plane, i, e.gnext[n] * x0);
      st_split<BF>(e.xn, e.xn_plane, i + 1, e.gnext[n + 1] * x1);
      return x0 * x0 + x1 * x1;
    }
    case EPI_SWIGLU: {
      float g = v0 * r, u = v1 * r;
      float s = g / (1.0f + expf(-g));
      st_split<BF>(e.h, e.h_plane, (size_t)t * e.ld + (n >> 1), s * u);
      return 0.f;
    }
    default: {  // EPI_LOGITS
      size_t i = (size_t)t * e.ld + n;
      *(float2*)(e.logits + i) = make_float2(v0 * r, v1 * r);
      return 0.f;
    }
  }
}

struct GemmKArgs {
  const u32x4* W;
  int N, K, KB;
  int S, kchunks, n_fb;
  const uint16_t* in;
  size_t in_plane;
  int ld_in;
  int M, t0;
  int xcd;
  int ft0;  // eight-wave tiles: first 16-feature tile of the launch (its partials and counters count from its first tile)
  float* part;
  unsigned* counters;
  EpiArgs epi;
};

// Tiled GEMM for more than ROWS_MAX token rows (prefills, batches), and for wide
// projections of fewer (gemm_plan_bf16):
// there the weights are worth reusing from registers and LDS rather than
// streaming once per 64-row tile, and from a few hundred rows on the product
// is bound by the matrix cores, not by the weight stream.  Each
// workgroup owns a 128-row x (32 NT)-feature output tile over the whole K
// range and every operand byte it loads feeds many MFMAs.  Four waves in a
// 2 x 2 arrangement, each 64 rows (four 16-row tiles) x 16 NT features; K
// advances in 64-input stages: the stage's token rows (both planes) sit in
// LDS, double-buffered, and each wave's weight fragments (prepacked, one
// 16-byte load per lane each) go straight to registers, the next stage's
// loads in flight while the current stage is multiplied.  All row tiles of a
// feature tile run on one XCD (xcd_grid with the row tiles as the group), so
// its weights come from HBM once and from that XCD's L2 after.  When the
// tiles cannot fill the CUs (few rows, narrow outputs) the K range is split
// over S workgroups of the same XCD; the last of them sums the partials in
// split order and runs the epilogue.
// LDS rows of one stage are unpadded (64 inputs, eight 16-byte chunks); chunk
// c of row r sits at chunk c ^ ((r >> 1) & 7), so that the 16 rows an MFMA
// operand read touches at one logical chunk hit distinct banks in groups of
// 16 and of 32 lanes, and each row's stores stay one 128-byte span
constexpr int TILE_ROWS = 128, TILE_KT = 64, TILE_LD = TILE_KT;
constexpr int TILE_PL = TILE_ROWS * TILE_LD;  // one plane of one stage (bf16)

template <int NT>
struct TileStage {
  u32x4 x[8];         // token rows: 4 rows x 2 planes per thread
  u32x4 w[NT][2];     // weight fragments: NT feature tiles x 2 k-blocks
};

// Buffer loads: a scalar base, 32-bit lane offsets and a scalar offset for
// the stage's K position, the plane and the feature tile.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_rsrc(const void* b) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(b), 0, 0x7FFFFFFF, 0x00020000);
}

template <int NT>
__device__ __forceinline__ void tile_load(TileStage<NT>& st, __amdgpu_buffer_rsrc_t xh, __amdgpu_buffer_rsrc_t xl,
                                          const int (&xoff)[4], __amdgpu_buffer_rsrc_t wr, int lane_b, int wtile_b,
                                          int KB, int k0) {
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    st.x[2 * p] = __builtin_amdgcn_raw_buffer_load_b128(xh, xoff[p], k0 * 2, 0);
    st.x[2 * p + 1] = __builtin_amdgcn_raw_buffer_load_b128(xl, xoff[p], k0 * 2, 0);
  }
  const int kb0 = k0 / 32;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
      st.w[nt][kb] = __builtin_amdgcn_raw_buffer_load_b128(wr, lane_b, wtile_b + (nt * KB + kb0 + kb) * 1024, 0);
}

template <int NT>
__device__ __forceinline__ void tile_load_x(TileStage<NT>& st, __amdgpu_buffer_rsrc_t xh, __amdgpu_buffer_rsrc_t xl,
                                            const int (&xoff)[4], int k0) {
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    st.x[2 * p] = __builtin_amdgcn_raw_buffer_load_b128(xh, xoff[p], k0 * 2, 0);
    st.x[2 * p + 1] = __builtin_amdgcn_raw_buffer_load_b128(xl, xoff[p], k0 * 2, 0);
  }
}

template <int NT>
__device__ __forceinline__ void tile_load_w(TileStage<NT>& st, __amdgpu_buffer_rsrc_t wr, int lane_b, int wtile_b,
                                            int KB, int k0) {
  const int kb0 = k0 / 32;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
      st.w[nt][kb] = __builtin_amdgcn_raw_buffer_load_b128(wr, lane_b, wtile_b + (nt * KB + kb0 + kb) * 1024, 0);
}

template <int NT>
__device__ __forceinline__ void tile_store_x(const TileStage<NT>& st, uint16_t* xs, int tid) {
  const int cg = tid & 7, rr = tid >> 3;
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const int r = rr + 32 * p;
    const int pc = cg ^ ((r >> 1) & 7);
    *(u32x4*)(xs + r * TILE_LD + pc * 8) = st.x[2 * p];
    *(u32x4*)(xs + TILE_PL + r * TILE_LD + pc * 8) = st.x[2 * p + 1];
  }
}

template <int NT>
__device__ __forceinline__ void tile_mma(floatx4 (&acc)[NT][4], const TileStage<NT>& st, const uint16_t* xs, int wm,
                                         int lane) {
  const int row = wm * 64 + (lane & 15);
#pragma unroll
  for (int kb = 0; kb < 2; ++kb) {
    bf16x8 bhi[4], blo[4];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      // rows row + 16 mt share (row >> 1) & 7 = ((lane & 15) >> 1)
      const uint16_t* p = xs + (row + mt * 16) * TILE_LD + (((kb * 4 + (lane >> 4)) ^ ((lane & 15) >> 1)) * 8);
      bhi[mt] = __builtin_bit_cast(bf16x8, *(const u32x4*)p);
      blo[mt] = __builtin_bit_cast(bf16x8, *(const u32x4*)(p + TILE_PL));
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const bf16x8 w = __builtin_bit_cast(bf16x8, st.w[nt][kb]);
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) {
        acc[nt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, bhi[mt], acc[nt][mt], 0, 0, 0);
        acc[nt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, blo[mt], acc[nt][mt], 0, 0, 0);
      }
    }
  }
}

// DEPTH 2: two register stages, loads one stage ahead; DEPTH 4: four
// register stages, loads three stages ahead (64-feature tiles only, which
// still fit two workgroups per CU with them)
template <int NT, int DEPTH>
__global__ __launch_bounds__(256, 2) void gemm_tile_kernel(GemmKArgs a) {
  __shared__ __attribute__((aligned(16))) uint16_t xs[2][2 * TILE_PL];
  __shared__ float rscale[TILE_ROWS];
  __shared__ float sq_red[2][TILE_ROWS];

  __shared__ int is_last;
  const int m_tiles = (a.M + TILE_ROWS - 1) / TILE_ROWS;
  int fb, member;
  xcd_unmap(blockIdx.x, m_tiles * a.S, a.xcd, fb, member);
  if (fb >= a.n_fb) return;
  const int mtile = member / a.S, split = member - mtile * a.S;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: scalar addressing
  const int wm = w & 1, wn = w >> 1;
  const int r0 = mtile * TILE_ROWS;                 // first row of the tile
  const int nb0 = fb * 2 * NT + wn * NT;            // first 16-feature tile of this wave
  const int t0w = a.t0 + r0 + wm * 64;              // first row of this wave (absolute)
  const int Mw = a.M - r0 - wm * 64 < 64 ? a.M - r0 - wm * 64 : 64;  // rows of this wave (<= 0: none)
  const int Mt = a.M - r0 < TILE_ROWS ? a.M - r0 : TILE_ROWS;
  const EpiArgs& e = a.epi;
  const int nst = a.K / TILE_KT / a.S, st0 = split * nst;  // this split's stages (a multiple of DEPTH)

  floatx4 acc[NT][4];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) acc[nt][mt] = floatx4{0.f, 0.f, 0.f, 0.f};

  // lane offsets of the token rows this thread copies (rows past M repeat
  // row M - 1; their results are never stored) and of its weight fragments
  const __amdgpu_buffer_rsrc_t xh = tile_rsrc(a.in), xl = tile_rsrc(a.in + a.in_plane), wr = tile_rsrc(a.W);
  int xoff[4];
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const int r = r0 + (tid >> 3) + 32 * p;
    xoff[p] = ((r < a.M ? r : a.M - 1) * a.ld_in + (tid & 7) * 8) * 2;
  }
  const int lane_b = lane * 16, wtile_b = nb0 * a.KB * 1024;
  auto load = [&](TileStage<NT>& st, int stage) {
    tile_load<NT>(st, xh, xl, xoff, wr, lane_b, wtile_b, a.KB, (st0 + stage) * TILE_KT);
  };
  auto load_x = [&](TileStage<NT>& st, int stage) { tile_load_x<NT>(st, xh, xl, xoff, (st0 + stage) * TILE_KT); };
  auto load_w = [&](TileStage<NT>& st, int stage) {
    tile_load_w<NT>(st, wr, lane_b, wtile_b, a.KB, (st0 + stage) * TILE_KT);
  };
  // 1/rms of the tile's rows (the LDS of stage buffer 1 serves as the
  // reduction scratch; it is written only after the next barrier)
  auto rms = [&]() {
    if (e.ssq)
      rms_prologue<TILE_ROWS>(e, Mt, a.t0 + r0, (float(*)[TILE_ROWS])(void*)xs[1], rscale);
    else if (tid < TILE_ROWS)
      rscale[tid] = 1.f;
  };
  // DEPTH stages per trip, so that the register stages have fixed names and
  // the loop body has no branch (a branch makes the compiler move the
  // accumulators between register files every trip); stage c sits in LDS
  // buffer c % 2
  if constexpr (DEPTH == 3) {
    // weights two stages ahead in three register slots (w0..w2), token rows
    // one stage ahead (xr); a trip runs three stages, so the LDS buffer of
    // its first stage alternates between trips
    TileStage<NT> w0, w1, w2, xr;
    load(w0, 0);
    load_w(w1, 1);
    rms();
    tile_store_x<NT>(w0, xs[0], tid);
    lds_barrier();
    int c = 0;
    uint16_t* xa = xs[0];  // buffer of stage c
    uint16_t* xb = xs[1];
    for (; c + 4 < nst; c += 3) {
      load_x(xr, c + 1);
      load_w(w2, c + 2);
      tile_mma<NT>(acc, w0, xa, wm, lane);
      tile_store_x<NT>(xr, xb, tid);
      lds_barrier();
      load_x(xr, c + 2);
      load_w(w0, c + 3);
      tile_mma<NT>(acc, w1, xb, wm, lane);
      tile_store_x<NT>(xr, xa, tid);
      lds_barrier();
      load_x(xr, c + 3);
      load_w(w1, c + 4);
      tile_mma<NT>(acc, w2, xa, wm, lane);
      tile_store_x<NT>(xr, xb, tid);
      lds_barrier();
      uint16_t* t = xa;
      xa = xb;
      xb = t;
    }
    // 2, 3 or 4 stages left: w0 holds stage c (its rows in xa), w1 stage c + 1
    const int left = nst - c;
    load_x(xr, c + 1);
    if (left >= 3) load_w(w2, c + 2);
    tile_mma<NT>(acc, w0, xa, wm, lane);
    tile_store_x<NT>(xr, xb, tid);
    lds_barrier();
    if (left >= 3) {
      load_x(xr, c + 2);
      if (left == 4) load_w(w0, c + 3);
    }
    tile_mma<NT>(acc, w1, xb, wm, lane);
    if (left >= 3) {
      tile_store_x<NT>(xr, xa, tid);
      lds_barrier();
      if (left == 4) load_x(xr, c + 3);
      tile_mma<NT>(acc, w2, xa, wm, lane);
      if (left == 4) {
        tile_store_x<NT>(xr, xb, tid);
        lds_barrier();
        tile_mma<NT>(acc, w0, xb, wm, lane);
      }
    }
  } else if constexpr (DEPTH == 2) {
    TileStage<NT> s0, s1;
    load(s0, 0);
    rms();
    tile_store_x<NT>(s0, xs[0], tid);
    lds_barrier();
    int c = 0;
    for (; c + 2 < nst; c += 2) {
      load(s1, c + 1);
      tile_mma<NT>(acc, s0, xs[0], wm, lane);
      tile_store_x<NT>(s1, xs[1], tid);
      lds_barrier();
      load(s0, c + 2);
      tile_mma<NT>(acc, s1, xs[1], wm, lane);
      tile_store_x<NT>(s0, xs[0], tid);
      lds_barrier();
    }
    load(s1, c + 1);
    tile_mma<NT>(acc, s0, xs[0], wm, lane);
    tile_store_x<NT>(s1, xs[1], tid);
    lds_barrier();
    tile_mma<NT>(acc, s1, xs[1], wm, lane);
  } else {
    TileStage<NT> s0, s1, s2, s3;
    load(s0, 0);
    load(s1, 1);
    load(s2, 2);
    rms();
    tile_store_x<NT>(s0, xs[0], tid);
    lds_barrier();
    int c = 0;
    for (; c + 4 < nst; c += 4) {
      load(s3, c + 3);
      tile_mma<NT>(acc, s0, xs[0], wm, lane);
      tile_store_x<NT>(s1, xs[1], tid);
      lds_barrier();
      load(s0, c + 4);
      tile_mma<NT>(acc, s1, xs[1], wm, lane);
      tile_store_x<NT>(s2, xs[0], tid);
      lds_barrier();
      load(s1, c + 5);
      tile_mma<NT>(acc, s2, xs[0], wm, lane);
      tile_store_x<NT>(s3, xs[1], tid);
      lds_barrier();
      load(s2, c + 6);
      tile_mma<NT>(acc, s3, xs[1], wm, lane);
      tile_store_x<NT>(s0, xs[0], tid);
      lds_barrier();
    }
    load(s3, c + 3);
    tile_mma<NT>(acc, s0, xs[0], wm, lane);
    tile_store_x<NT>(s1, xs[1], tid);
    lds_barrier();
    tile_mma<NT>(acc, s1, xs[1], wm, lane);
    tile_store_x<NT>(s2, xs[0], tid);
    lds_barrier();
    tile_mma<NT>(acc, s2, xs[0], wm, lane);
    tile_store_x<NT>(s3, xs[1], tid);
    lds_barrier();
    tile_mma<NT>(acc, s3, xs[1], wm, lane);
  }

  if (a.S > 1) {
    // split-K: publish this split's fragments; the last arrival of the tile
    // sums all splits in split order (deterministic)
    const int grp = fb * m_tiles + mtile;
    constexpr int FRAG = NT * 4 * 64 * 4;  // floats per wave
    float* P = a.part + ((size_t)grp * a.S * 4 + w) * FRAG + lane * 4;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) *(floatx4*)(P + (size_t)split * 4 * FRAG + (nt * 4 + mt) * 256) = acc[nt][mt];
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (tid == 0) {
      if (!a.xcd) __threadfence();  // splits on different XCDs: write back through L2
      const unsigned prev = atomicAdd(&a.counters[grp], 1u);
      is_last = prev == (unsigned)(a.S - 1);
      if (is_last && !a.xcd) __threadfence();
    }
    __syncthreads();
    if (!is_last) return;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) acc[nt][mt] = floatx4{0.f, 0.f, 0.f, 0.f};
    for (int sp = 0; sp < a.S; ++sp) {
      floatx4 v[NT][4];
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) v[nt][mt] = *(const floatx4*)(P + (size_t)sp * 4 * FRAG + (nt * 4 + mt) * 256);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) acc[nt][mt] += v[nt][mt];
    }
    if (tid == 0) a.counters[grp] = 0u;
  }

  float sq[4] = {0.f, 0.f, 0.f, 0.f};
  if (NT == 2 && e.kind == EPI_RESID) {
    // the new residual x stored in place (16 bytes a lane); both planes of
    // g * x (8 bytes a lane and plane) go through the wave's NT x 4 KiB of the
    // stage buffers and come back as 16 bytes of one row a lane: NT x 32
    // contiguous bytes per row and plane (64-feature tiles only: with 128
    // features the registers this takes spill inside the K loop)
    __syncthreads();  // every wave is done with the stage buffers
    if (Mw > 0) {
      EpiOps<NT, 4> op;
      epi_load<NT, 4>(e, nb0, a.N, Mw, t0w, lane, op);
      constexpr int RL = NT * 16;  // features of a wave row
      uint16_t* stg = &xs[0][0] + w * (2 * 64 * RL);  // [plane][64 rows][RL]
      const int nq = 4 * (lane >> 4);
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) {
        const int row = mt * 16 + (lane & 15);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          const floatx4 v = acc[nt][mt];
          const float4 xo = op.a[nt][mt], g = op.g[nt];
          const float4 xv = make_float4(xo.x + v[0], xo.y + v[1], xo.z + v[2], xo.w + v[3]);
          if (row < Mw) *(float4*)(e.xo + (size_t)(t0w + row) * e.ld + (nb0 + nt) * 16 + nq) = xv;
          uint32_t h0, l0, h1, l1;
          split2(g.x * xv.x, g.y * xv.y, h0, l0);
          split2(g.z * xv.z, g.w * xv.w, h1, l1);
          *(uint2*)(stg + row * RL + nt * 16 + nq) = make_uint2(h0, h1);
          *(uint2*)(stg + 64 * RL + row * RL + nt * 16 + nq) = make_uint2(l0, l1);
          sq[mt] += (xv.x * xv.x + xv.y * xv.y) + (xv.z * xv.z + xv.w * xv.w);
        }
      }
      asm volatile("" ::: "memory");  // a wave's LDS accesses run in order: its reads see all its lanes' writes
      uint16_t* xn = (uint16_t*)e.xn;
      constexpr int CH = RL / 8, RPI = 64 / CH;  // 16-byte chunks per row, rows per instruction
      const int c = lane % CH;
#pragma unroll
      for (int pl = 0; pl < 2; ++pl)
#pragma unroll
        for (int k = 0; k < 64 / RPI; ++k) {
          const int row = k * RPI + lane / CH;
          const uint4 v = *(const uint4*)(stg + pl * 64 * RL + row * RL + c * 8);
          if (row < Mw) *(uint4*)(xn + (pl ? e.xn_plane : 0) + (size_t)(t0w + row) * e.ld + nb0 * 16 + c * 8) = v;
        }
    }
  } else if (Mw > 0) {
    EpiOps<NT, 4> op;
    epi_block_starts<NT, 4>(e, Mw, t0w, lane, op);
    epi_load<NT, 4>(e, nb0, a.N, Mw, t0w, lane, op);
    epi_store<NT, 4>(e, acc, op, nb0, a.N, Mw, t0w, lane, rscale + wm * 64, sq);
  }
  if (e.kind == EPI_RESID) {
    // per-row sums of x^2 over this tile's features: lanes of one row, then
    // the two waves of one row half, in a fixed order
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      float v = sq[mt];
      v += __shfl_xor(v, 16);
      v += __shfl_xor(v, 32);
      if (lane < 16) sq_red[wn][wm * 64 + mt * 16 + lane] = v;
    }
    __syncthreads();
    if (tid < Mt) e.ssq_out[(size_t)fb * e.ssq_out_ld + a.t0 + r0 + tid] = sq_red[0][tid] + sq_red[1][tid];
  }
}

// ---------------- wide tiles with both operands through an LDS DMA ring ----------------
// Eight waves (two per SIMD, one workgroup per CU) own a 128-row x 256-feature
// output tile: 2 (rows) x 4 (features) waves of 64 x 64, the wave tile of
// gemm_tile_kernel<4, 3>.  A 64-input stage -- the token rows of both planes
// (32 KiB) and the 32 packed 1 KiB weight tiles of the 256 features (32 KiB)
// -- comes by LDS DMA into a ring of two stages, the next stage's copies in
// flight while the current one is multiplied; every operand byte crosses the
// L2 once per workgroup (with the 128 x 128 tiles the token rows crossed it
// once per 128 features and each weight fragment once per wave that uses
// it).  A token DMA instruction fills eight rows x 128 bytes (whole cache
// lines), its lanes choosing the global chunk so that LDS holds the rows in
// the swizzled layout the operand reads expect (chunk c of row r at c ^ ((r
// >> 1) & 7)); a weight tile lands in its stored lane order, so both operand
// reads are one conflict-free ds_read_b128 per fragment.  The reads are
// issued as separate instructions with their own waits, so that the
// compiler does not make them wait for every LDS DMA copy in flight.
// A narrower variant (NT = 3: waves of 64 x 48, tiles of 128 x 192, 24 weight
// tiles a stage in the same ring) fills grids that the 256-feature tiles
// leave part empty.
constexpr int T8_STAGES = 2, T8_THREADS = 512;
constexpr int T8_STAGE_BYTES = 2 * TILE_PL * 2 + 32 * 1024;  // one stage: both token planes, then up to 32 weight tiles

// the eight token operand fragments of one k-block at addr: [mt * 2 + plane],
// row tiles 16 rows (2 KiB) apart, the planes TILE_PL elements apart
__device__ __forceinline__ void ds_read_tiles2(u32x4 (&x)[8], uint32_t addr) {
  constexpr int PL = TILE_PL * 2, RT = 16 * TILE_LD * 2;
  x[0] = ds_read16_at<0>(addr);
  x[1] = ds_read16_at<PL>(addr);
  x[2] = ds_read16_at<RT>(addr);
  x[3] = ds_read16_at<PL + RT>(addr);
  x[4] = ds_read16_at<2 * RT>(addr);
  x[5] = ds_read16_at<PL + 2 * RT>(addr);
  x[6] = ds_read16_at<3 * RT>(addr);
  x[7] = ds_read16_at<PL + 3 * RT>(addr);
}

// K loop of one tile segment: stages st0 .. st0 + nst - 1 of the 128 token
// rows from r0 against the 64 NT features from 16-feature tile ft, summed
// into acc.  pro() runs once the first stage's copies are in flight (the
// tile's 1/rms, whose LDS scratch is the ring's second buffer); on return
// every wave is past the last stage's barrier, so the buffer of stage nst is
// free.
template <int NT, class Pro>
__device__ __forceinline__ void t8_kloop(const GemmKArgs& a, int ft, int r0, int st0, int nst, uint16_t* xs,
                                         floatx4 (&acc)[NT][4], Pro&& pro) {
  static_assert(NT == 3 || NT == 4, "waves of 48 or 64 features");
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform
  const int wm = w & 1, wn = w >> 1;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) acc[nt][mt] = floatx4{0.f, 0.f, 0.f, 0.f};

  const __amdgpu_buffer_rsrc_t xh = tile_rsrc(a.in), xl = tile_rsrc(a.in + a.in_plane), wr = tile_rsrc(a.W);
  // token DMA: 32 instructions a stage (2 planes x 16 blocks of 8 rows), four
  // per wave; lane l of block rb takes row rb * 8 + l / 8 and stored chunk
  // l % 8, i.e. the logical chunk (l % 8) ^ ((row >> 1) & 7) (rows past M
  // repeat row M - 1; their results are never stored)
  int xoff[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int i = w * 4 + j, rb = i & 15;
    const int row = rb * 8 + (lane >> 3);
    const int r = r0 + row;
    const int c = (lane & 7) ^ ((row >> 1) & 7);
    xoff[j] = ((r < a.M ? r : a.M - 1) * a.ld_in + c * 8) * 2;
  }
  auto issue_x = [&](int stage) {
    uint16_t* dst = xs + (size_t)(stage % T8_STAGES) * (T8_STAGE_BYTES / 2);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int i = w * 4 + j, pl = i >> 4, rb = i & 15;
      dma16(pl ? xl : xh, dst + pl * TILE_PL + rb * 512, xoff[j], (st0 + stage) * TILE_KT * 2);
    }
    // the stage's 8 NT weight tiles (4 NT feature tiles x 2 k-blocks), NT per wave
    const int kb0 = (st0 + stage) * TILE_KT / 32;
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const int i = w * NT + j, f = i >> 1, kb = i & 1;
      dma16(wr, dst + 2 * TILE_PL + i * 512, lane * 16, ((ft + f) * a.KB + kb0 + kb) * 1024);
    }
  };
  // operand reads: row wm * 64 + lane % 16 (+ 16 mt), logical chunk kb * 4 +
  // lane / 16 stored at that ^ ((row >> 1) & 7), which no mt changes
  const uint32_t xs0 = lds_addr(xs);
  uint32_t xrd[2];
#pragma unroll
  for (int kb = 0; kb < 2; ++kb)
    xrd[kb] = xs0 + (uint32_t)(((wm * 64 + (lane & 15)) * TILE_LD +
                                (((kb * 4 + (lane >> 4)) ^ ((lane & 15) >> 1)) * 8)) * 2);
  // weight tile (f, kb) of the stage sits at (2 f + kb) KiB after its token
  // planes; this wave's feature tiles are f = NT wn .. NT wn + NT - 1
  const uint32_t wrd = xs0 + (uint32_t)(2 * TILE_PL * 2 + wn * NT * 2048 + lane * 16);
  auto mma = [&](int stage) {
    const uint32_t so = (uint32_t)((stage % T8_STAGES) * T8_STAGE_BYTES);
    u32x4 x0[8], x1[8], b0[NT], b1[NT];  // token [mt * 2 + plane] and weight [nt] fragments of k-blocks 0 and 1
    ds_read_tiles2(x0, xrd[0] + so);
    b0[0] = ds_read16_at<0>(wrd + so);
    b0[1] = ds_read16_at<2048>(wrd + so);
    b0[2] = ds_read16_at<4096>(wrd + so);
    if constexpr (NT == 4) b0[NT - 1] = ds_read16_at<6144>(wrd + so);
    ds_read_tiles2(x1, xrd[1] + so);
    b1[0] = ds_read16_at<1024>(wrd + so);
    b1[1] = ds_read16_at<3072>(wrd + so);
    b1[2] = ds_read16_at<5120>(wrd + so);
    if constexpr (NT == 4) b1[NT - 1] = ds_read16_at<7168>(wrd + so);
    lgkm_wait<8 + NT>(x0);  // k-block 0's reads done, k-block 1's (8 + NT) may be outstanding
    lgkm_wait<8 + NT>(b0);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) {
        const bf16x8 wf = __builtin_bit_cast(bf16x8, b0[nt]);
        acc[nt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, __builtin_bit_cast(bf16x8, x0[mt * 2]), acc[nt][mt], 0, 0, 0);
        acc[nt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, __builtin_bit_cast(bf16x8, x0[mt * 2 + 1]), acc[nt][mt], 0, 0, 0);
      }
    __builtin_amdgcn_sched_barrier(0);  // the first k-block's MFMAs stay above the second wait
    lgkm_wait<0>(x1);
    lgkm_wait<0>(b1);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) {
        const bf16x8 wf = __builtin_bit_cast(bf16x8, b1[nt]);
        acc[nt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, __builtin_bit_cast(bf16x8, x1[mt * 2]), acc[nt][mt], 0, 0, 0);
        acc[nt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, __builtin_bit_cast(bf16x8, x1[mt * 2 + 1]), acc[nt][mt], 0, 0, 0);
      }
  };

  issue_x(0);
  pro();
  // stage c: this wave's copies of stage c are done (none are issued after
  // them yet), the barrier publishes everyone's copies and tells that every
  // wave is done with stage c - 1, whose ring buffer then takes stage c + 1
  for (int c = 0; c < nst; ++c) {
    wait_vmcnt<0>();
    dma_barrier();
    if (c + 1 < nst) issue_x(c + 1);
    mma(c);
  }
}

// x * sigmoid(x) from the hardware exp2 and reciprocal (each within about
// one ulp; the limits 0 and x hold for large |x|)
__device__ __forceinline__ float silu_hw(float x) {
  return x * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(x * -1.44269504088896341f));
}

// Epilogue of the tile (fb, rows r0 ..) from its sums; stg: a free ring
// buffer (64 KiB).  Every thread of the workgroup calls it (one barrier for
// the residual's row sums).
template <int NT>
__device__ __forceinline__ void t8_epilogue(const GemmKArgs& a, int fb, int ft, int r0, const floatx4 (&acc)[NT][4],
                                            const float* rscale, float (*sq_red)[TILE_ROWS], uint16_t* stg_all) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = w & 1, wn = w >> 1;
  const int nb0 = ft + wn * NT;  // first 16-feature tile of this wave
  const int t0w = a.t0 + r0 + wm * 64;
  const int Mw = a.M - r0 - wm * 64 < 64 ? a.M - r0 - wm * 64 : 64;
  const int Mt = a.M - r0 < TILE_ROWS ? a.M - r0 : TILE_ROWS;
  const EpiArgs& e = a.epi;
  float sq[4] = {0.f, 0.f, 0.f, 0.f};
  if (e.kind == EPI_SWIGLU) {
    // a lane's four features of one fragment are two gate/up pairs, i.e. two
    // adjacent outputs (4 bytes a plane): the wave's 64 x 32 outputs go
    // through its own 8 KiB of the free ring buffer and come back as 16
    // bytes of one row a lane, stored as 64 contiguous bytes per row and plane
    if (Mw > 0) {
      uint16_t* stg = stg_all + w * 4096;  // [plane][64 rows][32]
      const int q = lane >> 4;
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) {
        const int row = mt * 16 + (lane & 15);
        const float r = rscale[wm * 64 + row];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          const floatx4 v = acc[nt][mt];
          const float g0 = v[0] * r, u0 = v[1] * r, g1 = v[2] * r, u1 = v[3] * r;
          uint32_t hi, lo;
          split2(silu_hw(g0) * u0, silu_hw(g1) * u1, hi, lo);
          *(uint32_t*)(stg + row * 32 + nt * 8 + 2 * q) = hi;
          *(uint32_t*)(stg + 2048 + row * 32 + nt * 8 + 2 * q) = lo;
        }
      }
      asm volatile("" ::: "memory");  // a wave's LDS accesses run in order: its reads see all its lanes' writes
      uint16_t* h = (uint16_t*)e.h;
      const int c = lane & 3;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int row = k * 16 + (lane >> 2);
        const uint4 hi = *(const uint4*)(stg + row * 32 + c * 8);
        const uint4 lo = *(const uint4*)(stg + 2048 + row * 32 + c * 8);
        if (row < Mw && c < NT) {  // a wave's 8 NT outputs of a row are NT chunks
          const size_t i = act_index(e.tiled, t0w + row, nb0 * 8 + c * 8, e.ld);
          *(uint4*)(h + i) = hi;
          *(uint4*)(h + e.h_plane + i) = lo;
        }
      }
    }
  } else if (e.kind == EPI_RESID) {
    // the new residual x stored in place (16 bytes a lane); the planes of
    // g * x (8 bytes a lane and plane) go through the wave's 8 KiB of the
    // free ring buffer one plane at a time and come back as 16 bytes of one
    // row a lane: 128 contiguous bytes per row and plane
    if (Mw > 0) {
      EpiOps<NT, 4> op;
      epi_load<NT, 4>(e, nb0, a.N, Mw, t0w, lane, op);
      uint16_t* stg = stg_all + w * 4096;  // [64 rows][64 features], one plane
      const int nq = 4 * (lane >> 4);
      uint2 lo[NT][4];
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) {
        const int row = mt * 16 + (lane & 15);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          const floatx4 v = acc[nt][mt];
          const float4 xo = op.a[nt][mt], g = op.g[nt];
          const float4 xv = make_float4(xo.x + v[0], xo.y + v[1], xo.z + v[2], xo.w + v[3]);
          if (row < Mw) *(float4*)(e.xo + (size_t)(t0w + row) * e.ld + (nb0 + nt) * 16 + nq) = xv;
          uint32_t h0, l0, h1, l1;
          split2(g.x * xv.x, g.y * xv.y, h0, l0);
          split2(g.z * xv.z, g.w * xv.w, h1, l1);
          *(uint2*)(stg + row * 64 + nt * 16 + nq) = make_uint2(h0, h1);
          lo[nt][mt] = make_uint2(l0, l1);
          sq[mt] += (xv.x * xv.x + xv.y * xv.y) + (xv.z * xv.z + xv.w * xv.w);
        }
      }
      uint16_t* xn = (uint16_t*)e.xn;
      const int c = lane & 7;
#pragma unroll
      for (int pl = 0; pl < 2; ++pl) {
        if (pl) {
#pragma unroll
          for (int mt = 0; mt < 4; ++mt)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) *(uint2*)(stg + (mt * 16 + (lane & 15)) * 64 + nt * 16 + nq) = lo[nt][mt];
        }
        asm volatile("" ::: "memory");  // a wave's LDS accesses run in order: its reads see all its lanes' writes
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const int row = k * 8 + (lane >> 3);
          const uint4 v = *(const uint4*)(stg + row * 64 + c * 8);
          if (row < Mw && c < 2 * NT)
            *(uint4*)(xn + (pl ? e.xn_plane : 0) + act_index(e.tiled, t0w + row, nb0 * 16 + c * 8, e.ld)) = v;
        }
        asm volatile("" ::: "memory");  // the lo plane's writes stay behind the hi plane's reads
      }
    }
  } else if (NT == 4 && e.kind == EPI_QKV && nb0 * 16 < e.Hq * e.D && (e.D & 63) == 0) {
    // query features (a wave's 64 features lie in one head: rotary pairs j0 ..
    // j0 + 31 and their partners j0 + D/2 ..): the rotated values, 4 bytes a
    // lane and plane before, go through the wave's 8 KiB of the free ring
    // buffer one plane at a time, [64 tokens][dims j0 .. j0 + 31, then
    // j0 + D/2 ..], and come back as the 8 dims of one tiled-q lane chunk
    // (16 bytes) a lane
    if (Mw > 0) {
      EpiOps<NT, 4> op;
      epi_block_starts<NT, 4>(e, Mw, t0w, lane, op);
      epi_load<NT, 4>(e, nb0, a.N, Mw, t0w, lane, op);
      const int D = e.D, half = D >> 1;
      const int n0 = nb0 * 16, head = n0 / D, j0 = (n0 - head * D) >> 1;
      const int g = e.Hq / e.Hkv, hkv = head / g, hg = head - hkv * g;
      uint16_t* stg = stg_all + w * 4096;
      const int nq = 4 * (lane >> 4);
      uint2 lo[NT][4];  // lo planes of (j, j + 1) and (j + D/2, j + 1 + D/2), for the second pass
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) {
        const int row = mt * 16 + (lane & 15);
        const float r = rscale[wm * 64 + row];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          const floatx4 v = acc[nt][mt];
          const float4 cs = op.a[nt][mt];
          const float x0 = v[0] * r, y0 = v[1] * r, x1 = v[2] * r, y1 = v[3] * r;
          const float a0 = x0 * cs.x - y0 * cs.y, c0 = y0 * cs.x + x0 * cs.y;
          const float a1 = x1 * cs.z - y1 * cs.w, c1 = y1 * cs.z + x1 * cs.w;
          uint32_t h0, l0, h1, l1;
          split2(a0, a1, h0, l0);
          split2(c0, c1, h1, l1);
          const int jj = nt * 8 + nq / 2;  // pair offset from j0 (even)
          *(uint32_t*)(stg + row * 64 + jj) = h0;
          *(uint32_t*)(stg + row * 64 + 32 + jj) = h1;
          lo[nt][mt] = make_uint2(l0, l1);
        }
      }
      uint16_t* qb = (uint16_t*)e.q;
      const int c = lane & 7;
      const int col = c < 4 ? j0 + c * 8 : j0 + half + (c - 4) * 8;
#pragma unroll
      for (int pl = 0; pl < 2; ++pl) {
        if (pl) {
#pragma unroll
          for (int mt = 0; mt < 4; ++mt)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
              const int row = mt * 16 + (lane & 15), jj = nt * 8 + nq / 2;
              *(uint32_t*)(stg + row * 64 + jj) = lo[nt][mt].x;
              *(uint32_t*)(stg + row * 64 + 32 + jj) = lo[nt][mt].y;
            }
        }
        asm volatile("" ::: "memory");  // a wave's LDS accesses run in order: its reads see all its lanes' writes
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const int row = k * 8 + (lane >> 3);
          const uint4 v = *(const uint4*)(stg + row * 64 + c * 8);
          if (row < Mw) {
            const int t = t0w + row, b = t / e.Kblk, kk = t - b * e.Kblk;
            const size_t base = ((size_t)b * e.Hkv + hkv) * (size_t)e.qrows_pad * D;
            *(uint4*)(qb + (pl ? e.q_plane : 0) + base + tile16x32_index(hg * e.Kblk + kk, col, D)) = v;
          }
        }
        asm volatile("" ::: "memory");  // the lo plane's writes stay behind the hi plane's reads
      }
    }
  } else if (Mw > 0) {
    EpiOps<NT, 4> op;
    epi_block_starts<NT, 4>(e, Mw, t0w, lane, op);
    epi_load<NT, 4>(e, nb0, a.N, Mw, t0w, lane, op);
    epi_store<NT, 4>(e, acc, op, nb0, a.N, Mw, t0w, lane, rscale + wm * 64, sq);
  }
  if (e.kind == EPI_RESID) {
    // per-row sums of x^2 over this tile's features: lanes of one row, then
    // the four waves of one row half, in a fixed order
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      float v = sq[mt];
      v += __shfl_xor(v, 16);
      v += __shfl_xor(v, 32);
      if (lane < 16) sq_red[wn][wm * 64 + mt * 16 + lane] = v;
    }
    __syncthreads();
    if (tid < Mt)
      e.ssq_out[(size_t)fb * e.ssq_out_ld + a.t0 + r0 + tid] =
          ((sq_red[0][tid] + sq_red[1][tid]) + sq_red[2][tid]) + sq_red[3][tid];
  }
}

// the tile's 1/rms of its rows (1 without a norm), scratch: 8 KiB of LDS
__device__ __forceinline__ void t8_rms(const GemmKArgs& a, int r0, float* scratch, float* rscale) {
  const int Mt = a.M - r0 < TILE_ROWS ? a.M - r0 : TILE_ROWS;
  if (a.epi.ssq)
    rms_prologue<TILE_ROWS, T8_THREADS>(a.epi, Mt, a.t0 + r0, (float(*)[TILE_ROWS])(void*)scratch, rscale);
  else if (threadIdx.x < TILE_ROWS)
    rscale[threadIdx.x] = 1.f;
}

// One workgroup per output tile and K split (grid of xcd_grid(n_fb,
// m_tiles * S)): the splits' sums meet in the last arrival.  Feature block fb
// of the launch covers the 4 NT 16-feature tiles from a.ft0 + 4 NT fb; its
// per-row x^2 part (residual epilogue) is number ft / (4 NT), which counts
// the blocks of the whole projection when every launch of it has one width.
template <int NT>
__global__ __launch_bounds__(T8_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2)))
void gemm_tile8_kernel(GemmKArgs a) {
  __shared__ __attribute__((aligned(16))) uint16_t xs[T8_STAGES * T8_STAGE_BYTES / 2];
  __shared__ float rscale[TILE_ROWS];
  __shared__ float sq_red[4][TILE_ROWS];
  __shared__ int is_last;
  const int m_tiles = (a.M + TILE_ROWS - 1) / TILE_ROWS;
  int fb, member;
  xcd_unmap(blockIdx.x, m_tiles * a.S, a.xcd, fb, member);
  if (fb >= a.n_fb) return;
  const int mtile = member / a.S, split = member - mtile * a.S;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform
  const int r0 = mtile * TILE_ROWS;
  const int nst = a.K / TILE_KT / a.S;

  const int ft = a.ft0 + fb * 4 * NT;  // the tile's first 16-feature tile
  floatx4 acc[NT][4];
  t8_kloop<NT>(a, ft, r0, split * nst, nst, xs, acc,
               [&] { t8_rms(a, r0, (float*)(void*)(xs + T8_STAGE_BYTES / 2), rscale); });

  if (a.S > 1) {
    // split-K: publish this split's fragments; the last arrival of the tile
    // sums all splits in split order (deterministic)
    const int grp = fb * m_tiles + mtile;
    constexpr int FRAG = NT * 4 * 64 * 4;  // floats per wave
    float* P = a.part + ((size_t)grp * a.S * 8 + w) * FRAG + lane * 4;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) *(floatx4*)(P + (size_t)split * 8 * FRAG + (nt * 4 + mt) * 256) = acc[nt][mt];
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (tid == 0) {
      if (!a.xcd) __threadfence();  // splits on different XCDs: write back through L2
      const unsigned prev = atomicAdd(&a.counters[grp], 1u);
      is_last = prev == (unsigned)(a.S - 1);
      if (is_last && !a.xcd) __threadfence();
    }
    __syncthreads();
    if (!is_last) return;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) acc[nt][mt] = floatx4{0.f, 0.f, 0.f, 0.f};
    for (int sp = 0; sp < a.S; ++sp) {
      floatx4 v[NT][4];
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) v[nt][mt] = *(const floatx4*)(P + (size_t)sp * 8 * FRAG + (nt * 4 + mt) * 256);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) acc[nt][mt] += v[nt][mt];
    }
    if (tid == 0) a.counters[grp] = 0u;
  }
  t8_epilogue<NT>(a, ft / (4 * NT), ft, r0, acc, rscale, sq_red, xs + (size_t)(nst % T8_STAGES) * (T8_STAGE_BYTES / 2));
}

// the 128 x 256 LDS-DMA tiles where they apply (SSD_GEMM_T8=0 keeps every
// plan on the 128 x 128 tiles, for comparisons)
static bool tile8_enabled() {
  static const bool on = [] {
    const char* v = std::getenv("SSD_GEMM_T8");
    return !(v && std::strcmp(v, "0") == 0);
  }();
  return on;
}
// the 128 x 192 tiles where they fill a grid better (SSD_GEMM_T8N=0: never)
static bool tile8_narrow_enabled() {
  static const bool on = [] {
    const char* v = std::getenv("SSD_GEMM_T8N");
    return !(v && std::strcmp(v, "0") == 0);
  }();
  return on;
}

static GemmPlan gemm_plan_tiles(int M, int N, int K, int xcd);

GemmPlan gemm_plan_guided(int M, int N, int K, int xcd) {
  return M <= 64 ? gemm_rows_plan(M, N, K, xcd) : gemm_plan_tiles(M, N, K, xcd);
}

GemmPlan gemm_plan_bf16(int M, int N, int K, int xcd) {
  if (M <= 64) return gemm_rows_plan(M, N, K, xcd);
  if (M <= ROWS_MAX) {
    // one 128-row tile: the few-row kernel with two row groups, or the 128 x 256
    // tiles where their modelled time is less (8 us, 1.4 us a 64-input stage, whose
    // weights come from HBM here, and 0.43 us a MB of partial sums out and back).
    // At 128 rows of the 8B widths: gate/up 77 us on the tiles, 99 on the few-row
    // kernel; output layer 86 and 101; but QKV 37 (64-feature tiles) and 30.  1B
    // widths at 96 and 128 rows, on the 64-feature tiles and here: QKV 24.5 ->
    // 18.8 and 25.7 -> 21.4 us, O 15.4 -> 11.3 and 15.8 -> 12.7, gate/up 31.1 ->
    // 21.5 and 33.0 -> 25.3, down 26.8 -> 18.1 and 28.5 -> 20.6.
    double ns;
    const GemmPlan r = gemm_rows_plan(M, N, K, xcd, &ns);
    const GemmPlan t = gemm_plan_tiles(M, N, K, xcd);
    const double parts = t.S > 1 ? 8.0 * t.S * TILE_ROWS * N : 0.0;
    if (t.tile == 3 && !t.tail_fb && 8e3 + 1400.0 * t.kchunks + 0.43e-3 * parts < ns) return t;
    return r;
  }
  return gemm_plan_tiles(M, N, K, xcd);
}

static GemmPlan gemm_plan_tiles(int M, int N, int K, int xcd) {
  GemmPlan p{};
  p.xcd = xcd;
  p.tile = 0;
  p.tail_fb = 0;
  p.tail_S = 1;
  p.tail_nt = 0;
  if (K % (2 * TILE_KT) == 0 && N % 256 == 0 && (size_t)N * K * 2 < (1ull << 31) && tile8_enabled()) {
    // 128 x 256 tiles, eight waves, both operands by LDS DMA, one workgroup
    // per CU: K split by the largest divisor of the stage count that keeps
    // the grid within 256 workgroups, wherever each workgroup still runs at
    // least 32 stages.  Measured on the 8B shapes at 512 rows against the
    // 128 x 128 tiles: gate/up 269 -> 231 us, down 167 -> 122, output layer
    // 274 -> 234, QKV 82 -> 77; O (16 stages per workgroup) 55 -> 62, so it
    // stays on them.
    const int mt = (M + TILE_ROWS - 1) / TILE_ROWS;
    const int nfb = N / 256, nst = K / TILE_KT;
    int S = 1;
    for (int s = 2; s <= 16; ++s)
      if (nst % s == 0 && (long)nfb * mt * s <= 256) S = s;
    if (nst / S >= 32) {
      p.tile = 3;
      p.NT = 4;
      p.MT = TILE_ROWS / 16;
      p.WV = T8_THREADS / 64;
      p.bn = 256;
      p.n_fb = nfb;
      p.m_tiles = mt;
      p.S = S;
      p.KCB = TILE_KT / 32;
      p.kchunks = nst / S;
      p.depth = T8_STAGES;  // ring stages
      // 128 x 192 tiles (waves of 64 x 48) where the 256-feature grid leaves
      // CUs idle and the narrower one fills more of them with no more stages
      // per workgroup (8B QKV: 96 tiles in two splits on 192 CUs at 512 rows,
      // 128 in two splits on all 256 instead).  Only where N > K, which keeps
      // them off the residual projections (N = d, K >= d), whose per-row x^2
      // parts count 256-feature blocks.
      const bool narrow = tile8_narrow_enabled() && N > K;
      if (narrow && N % 192 == 0) {
        const int nfb3 = N / 192;
        int S3 = 0;
        for (int s = 1; s <= 16; ++s)
          if (nst % s == 0 && (long)nfb3 * mt * s <= 256 && nst / s >= 32) S3 = s;
        if (S3 && nst / S3 <= nst / S && (long)nfb3 * mt * S3 > (long)nfb * mt * S) {
          p.NT = 3;
          p.bn = 192;
          p.n_fb = nfb3;
          p.S = S3;
          p.kchunks = nst / S3;
          return p;
        }
      }
      // whole tiles in as many full rounds of 256 as there are, the feature
      // blocks left over K-split so that they fill the last round, where
      // that saves the busiest CU a quarter of a round and more (8B gate/up
      // at 1024 rows: 768 tiles, then 128 in two splits of 32 stages); where
      // no split fits, as 128 x 192 tiles if those fill more of the round
      // (8B gate/up at 512 rows: 256 tiles, then 192 of 256 features as 256
      // of 192)
      const long tiles = (long)nfb * mt, full = tiles / 256;
      if (S == 1 && full >= 1 && tiles % 256 && (256 * full) % mt == 0) {
        const int fb_a = (int)(256 * full / mt), r = (nfb - fb_a) * mt;
        int st = 1;
        for (int s = 2; s <= 16; ++s)
          if (nst % s == 0 && (long)r * s <= 256 && nst / s >= 16) st = s;
        const int fr = (nfb - fb_a) * 256;
        if (st > 1 && nst / st + nst / 8 <= nst * 3 / 4) {
          p.tail_fb = fb_a;
          p.tail_S = st;
        } else if (narrow && fr % 192 == 0 && (long)(fr / 192) * mt <= 256 && (long)(fr / 192) * mt > r) {
          p.tail_fb = fb_a;
          p.tail_nt = 3;
        }
      }
      return p;
    }
  }
  if (K % (2 * TILE_KT) == 0 && N % 64 == 0 && (size_t)N * K * 2 < (1ull << 31)) {
    // 128-feature tiles wherever they give at least 160 workgroups (measured
    // on the 8B and 1B shapes: up to 35 % faster than 64-feature tiles
    // there, slower on grids that leave CUs idle); then K splits until the
    // grid has 256 workgroups
    const int mt = (M + TILE_ROWS - 1) / TILE_ROWS;
    const long w4 = (long)(N / 128) * mt;
    const bool four = N % 128 == 0 && w4 >= 160;
    p.tile = 1;
    p.NT = four ? 4 : 2;
    p.MT = TILE_ROWS / 16;
    p.WV = 4;
    p.bn = 32 * p.NT;
    p.n_fb = N / p.bn;
    p.m_tiles = mt;
    // the split: the smallest divisor of the stage count (at most 16, an
    // even count of stages per split) that brings the grid to 256
    // workgroups, else the largest such divisor (1B down projection at 128
    // rows: 88 stages in 11 splits, 352 workgroups)
    p.S = 1;
    const int nst = K / TILE_KT;
    for (int s = 2; s <= 16 && (long)p.n_fb * mt * p.S < 256; ++s)
      if (nst % s == 0 && (nst / s) % 2 == 0) p.S = s;
    p.KCB = TILE_KT / 32;
    p.kchunks = nst / p.S;
    // four-stage pipeline for 64-feature tiles (measured on the 8B shapes at
    // 512 rows: O 75 -> 59 us, down 241 -> 177); 128-feature tiles would need
    // one workgroup per CU for it, which measured slower
    p.depth = p.NT == 4 ? 3 : (p.kchunks % 4 == 0 ? 4 : 2);
    return p;
  }
  return gemm_rows_plan(M, N, K, xcd);
}

size_t gemm_partials_floats(const GemmPlan& p, int M) {
  if (p.tile && p.tail_fb) return p.tail_nt ? 0 : (size_t)p.tail_S * (p.n_fb - p.tail_fb) * p.m_tiles * TILE_ROWS * p.bn;
  if (p.S <= 1) return 0;
  if (p.tile) return (size_t)p.S * p.m_tiles * TILE_ROWS * p.n_fb * p.bn;
  (void)M;
  return (size_t)p.S * p.n_fb * p.NT * p.MT * 256;
}

void gemm_bf16(const GemmPlan& p, const void* Wpacked, int N, int K, const ActIn& in, int M, const EpiArgs& epi,
               float* partials, unsigned* counters, hipStream_t st) {
  if (p.tile) {
    // row-major inputs: every rstep-th row from row0
    const int ld_in = in.ld * in.rstep;
    const uint16_t* first = in.p + (size_t)in.row0 * in.ld;
    // buffer addressing reaches 2 GiB from each plane's base: rows beyond
    // that go to further launches (chunks of whole row tiles)
    const size_t row_b = (size_t)ld_in * 2;
    int rows = (int)std::min<size_t>((size_t)M, ((1ull << 31) - (size_t)K * 2) / row_b);
    rows = std::max(TILE_ROWS, rows / TILE_ROWS * TILE_ROWS);
    for (int t0 = 0; t0 < M; t0 += rows) {
      GemmKArgs a{};
      a.W = (const u32x4*)Wpacked;
      a.N = N;
      a.K = K;
      a.KB = K / 32;
      a.S = p.S;
      a.kchunks = p.kchunks;
      a.n_fb = p.n_fb;
      a.in = first + (size_t)t0 * ld_in;
      a.in_plane = in.plane;
      a.ld_in = ld_in;
      a.M = std::min(rows, M - t0);
      a.t0 = t0;
      a.xcd = p.xcd;
      a.part = partials;
      a.counters = counters;
      a.epi = epi;
      const dim3 grid(xcd_grid(p.n_fb, (a.M + TILE_ROWS - 1) / TILE_ROWS * p.S, p.xcd));
      if (p.tile == 3 && p.tail_fb && a.M == M) {
        // whole tiles of the first feature blocks, then the rest K-split
        const int mt = (a.M + TILE_ROWS - 1) / TILE_ROWS;
        a.n_fb = p.tail_fb;
        launch_timed(gemm_tile8_kernel<4>, dim3(xcd_grid(a.n_fb, mt, p.xcd)), dim3(T8_THREADS), st, a);
        a.ft0 = p.tail_fb * 16;
        if (p.tail_nt == 3) {
          a.n_fb = (N - p.tail_fb * 256) / 192;
          launch_timed(gemm_tile8_kernel<3>, dim3(xcd_grid(a.n_fb, mt, p.xcd)), dim3(T8_THREADS), st, a);
        } else {
          a.n_fb = p.n_fb - p.tail_fb;
          a.S = p.tail_S;
          a.kchunks = K / TILE_KT / p.tail_S;
          launch_timed(gemm_tile8_kernel<4>, dim3(xcd_grid(a.n_fb, mt * a.S, p.xcd)), dim3(T8_THREADS), st, a);
        }
      } else if (p.tile == 3 && p.NT == 3)
        launch_timed(gemm_tile8_kernel<3>, grid, dim3(T8_THREADS), st, a);
      else if (p.tile == 3)
        launch_timed(gemm_tile8_kernel<4>, grid, dim3(T8_THREADS), st, a);
      else if (p.NT == 4)
        launch_timed(gemm_tile_kernel<4, 3>, grid, dim3(256), st, a);
      else if (p.depth == 4)
        launch_timed(gemm_tile_kernel<2, 4>, grid, dim3(256), st, a);
      else
        launch_timed(gemm_tile_kernel<2, 2>, grid, dim3(256), st, a);
    }
    return;
  }
  // few-row kernel: up to ROWS_MAX rows a launch (more only for shapes the tiled kernels do not take)
  for (int t0 = 0; t0 < M; t0 += ROWS_MAX) {
    RowsKArgs a{};
    a.W = Wpacked;
    a.N = N;
    a.KB = K / 32;
    a.n_fb = p.n_fb;
    a.S = p.S;
    a.xcd = p.S > 1 ? p.xcd : 0;
    a.in = in;
    a.M = std::min(M - t0, ROWS_MAX);
    a.t0 = t0;
    a.part = partials;
    a.counters = counters;
    a.epi = epi;
    gemm_rows(p.MT, p.NT, a, st);
  }
}

// ---------------- fp32 path (small fp32 models) ----------------
// Output tiles of 16 features x 16 MT tokens on v_mfma_f32_16x16x4_f32 (fp32
// products and sums).  At the few rows of a verify pass the launch is bound by
// one memory round trip, so a workgroup's four waves split the K range (wave w
// takes the 16-input chunks w, w + 4, ...), load both operands straight into
// registers with 16-byte loads, four chunks in flight while four are
// multiplied, and meet in LDS.  A lane's vector holds inputs 4 (lane / 16) ..
// + 3 of its row, so MFMA e of a chunk multiplies inputs e, 4 + e, 8 + e,
// 12 + e of both operands.  The order of every sum depends on K alone, never
// on the row count or MT: a block of several tokens gives the bits of its
// tokens one by one.  At d 256, up to 16 rows: 6.4 us a launch against 52.9 us for
// one thread per output pair walking its weight rows 4 bytes at a time.
constexpr int F32_CH = 16, F32_UB = 4;  // inputs per chunk, chunks in flight per wave

template <int MT>
__global__ __launch_bounds__(256) void gemm_f32_mfma_kernel(const float* __restrict__ W, int N, int K,
                                                            const float* __restrict__ in, int ld_in, int M, EpiArgs e) {
  constexpr int MP = MT * 16;
  __shared__ float part[4][MT][16][17];  // [wave][token tile][token][feature]
  __shared__ float red[16][MP];
  __shared__ float rscale[MP];
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int fb = blockIdx.x, t0 = blockIdx.y * MP;
  const int row = lane & 15, kq = (lane >> 4) * 4;
  const float* wp = W + (size_t)min(fb * 16 + row, N - 1) * K;  // rows past N, M: clamped, never stored
  const float* xp[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) xp[mt] = in + (size_t)min(t0 + mt * 16 + row, M - 1) * ld_in;

  // 1/rms: thread group g sums parts g, g + 16, ... of a token, the groups meet in order
  if (e.ssq) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const int tl = mt * 16 + (tid & 15), g = tid >> 4;
      const size_t c = (size_t)e.ssq_off + (size_t)min(t0 + tl, M - 1) * e.ssq_step;
      float v = 0.f;
      for (int p = g; p < e.ssq_parts; p += 16) v += e.ssq[(size_t)p * e.ssq_ld + c];
      red[g][tl] = v;
    }
  }

  const int nch = (K + F32_CH - 1) / F32_CH;
  const int mine = (nch - w + 3) / 4;  // chunks of this wave
  floatx4 acc[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) acc[mt] = floatx4{0.f, 0.f, 0.f, 0.f};
  floatx4 wa[2][F32_UB], xa[2][MT][F32_UB];
  auto load = [&](int buf, int i0) {
#pragma unroll
    for (int u = 0; u < F32_UB; ++u) {
      const int k = (w + 4 * (i0 + u)) * F32_CH + kq;  // inputs past K: loaded from the row's start, taken as zero
      const int kc = k < K ? k : 0;
      const float keep = k < K ? 1.f : 0.f;
      wa[buf][u] = *(const floatx4*)(wp + kc);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) xa[buf][mt][u] = *(const floatx4*)(xp[mt] + kc);
      if (keep == 0.f) {
        wa[buf][u] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) xa[buf][mt][u] = floatx4{0.f, 0.f, 0.f, 0.f};
      }
    }
  };
  auto mma = [&](int buf) {
#pragma unroll
    for (int u = 0; u < F32_UB; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          acc[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(wa[buf][u][i], xa[buf][mt][u][i], acc[mt], 0, 0, 0);
  };
  load(0, 0);
  for (int i0 = 0; i0 < mine; i0 += 2 * F32_UB) {
    load(1, i0 + F32_UB);  // past the wave's last chunk: zeros
    mma(0);
    load(0, i0 + 2 * F32_UB);
    mma(1);
  }
  // lane: features 4 (lane / 16) .. + 3 of token lane % 16
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int i = 0; i < 4; ++i) part[w][mt][row][kq + i] = acc[mt][i];
  __syncthreads();
  if (tid < MP) {
    float a = 0.f;
    if (e.ssq) {
#pragma unroll
      for (int g = 0; g < 16; ++g) a += red[g][tid];
    }
    rscale[tid] = e.ssq ? 1.0f / sqrtf(a * e.inv_d + e.eps) : 1.f;
  }
  __syncthreads();
  // eight lanes per token, an output pair each
  for (int i = tid; i < MP * 8; i += 256) {
    const int tl = i >> 3, n = (i & 7) * 2;
    const int t = t0 + tl, nn = fb * 16 + n;
    float sq = 0.f;
    if (t < M && nn < N) {
      float v[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int mt = tl >> 4, tr = tl & 15;
        v[j] = ((part[0][mt][tr][n + j] + part[1][mt][tr][n + j]) + part[2][mt][tr][n + j]) + part[3][mt][tr][n + j];
      }
      sq = epi_pair<false>(e, t, nn, v[0], v[1], rscale[tl]);
    }
    if (e.kind == EPI_RESID) {
      sq += __shfl_xor(sq, 1);
      sq += __shfl_xor(sq, 2);
      sq += __shfl_xor(sq, 4);
      if (n == 0 && t < M) e.ssq_out[(size_t)fb * e.ssq_out_ld + t] = sq;
    }
  }
}

// One thread per (token, output pair); plain fp32 FMAs in k order (rows that
// 16-byte loads cannot take: K or the row stride not a multiple of four).
__global__ void gemm_f32_kernel(const float* W, int N, int K, const float* in, int ld_in, int M, EpiArgs e) {
  const int pair = blockIdx.x * blockDim.x + threadIdx.x;
  const int t = blockIdx.y;
  const int n = pair * 2;
  if (n >= N || t >= M) return;
  const float* x = in + (size_t)t * ld_in;
  const float* w0 = W + (size_t)n * K;
  const float* w1 = w0 + K;
  float a0 = 0.f, a1 = 0.f;
  for (int k = 0; k < K; ++k) {
    float xv = x[k];
    a0 = fmaf(xv, w0[k], a0);
    a1 = fmaf(xv, w1[k], a1);
  }
  float r = rms_scale(e, t);
  epi_pair<false>(e, t, n, a0, a1, r);
}

int gemm_f32(const float* W, int N, int K, const float* in, int ld_in, int M, const EpiArgs& epi, hipStream_t st) {
  // 16-byte operand rows: K, the row stride and both bases (a rule on the
  // model's shape, so that every pass of a model sums in one order)
  if (K % 4 == 0 && ld_in % 4 == 0 && (((uintptr_t)W | (uintptr_t)in) & 15) == 0) {
    const int fb = f32_feature_blocks(N);
    // 64-token tiles reuse a weight row four times; below that the launch is
    // latency and the smaller tile has more workgroups
    if (M > 64)
      hipLaunchKernelGGL(gemm_f32_mfma_kernel<4>, dim3(fb, (M + 63) / 64), dim3(256), 0, st, W, N, K, in, ld_in, M, epi);
    else
      hipLaunchKernelGGL(gemm_f32_mfma_kernel<1>, dim3(fb, (M + 15) / 16), dim3(256), 0, st, W, N, K, in, ld_in, M, epi);
    return epi.kind == EPI_RESID ? fb : 0;
  }
  int pairs = N / 2;
  dim3 grid((pairs + 127) / 128, M);
  hipLaunchKernelGGL(gemm_f32_kernel, grid, dim3(128), 0, st, W, N, K, in, ld_in, M, epi);
  if (epi.kind != EPI_RESID) return 0;
  norm_rows_f32(epi.xo, M, N, epi.ssq_out, st);
  return 1;
}

// ---------------- weight packing ----------------
__global__ void pack_tiles_kernel(const uint16_t* src, const int* rowmap, int N, int K, u32x4* dst) {
  const int KB = K / 32;
  const size_t tiles = (size_t)(N / 16) * KB;
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t tile = gid >> 6;
  const int lane = gid & 63;
  if (tile >= tiles) return;
  const int nb = (int)(tile / KB), kb = (int)(tile % KB);
  const int row = rowmap[nb * 16 + (lane & 15)];
  const uint16_t* p = src + (size_t)row * K + kb * 32 + (lane >> 4) * 8;
  u32x4 v;
  v.x = (uint32_t)p[0] | ((uint32_t)p[1] << 16);
  v.y = (uint32_t)p[2] | ((uint32_t)p[3] << 16);
  v.z = (uint32_t)p[4] | ((uint32_t)p[5] << 16);
  v.w = (uint32_t)p[6] | ((uint32_t)p[7] << 16);
  dst[tile * 64 + lane] = v;
}

void pack_bf16_tiles(const uint16_t* src, const int* rowmap, int N, int K, void* dst, hipStream_t st) {
  size_t threads = (size_t)(N / 16) * (K / 32) * 64;
  hipLaunchKernelGGL(pack_tiles_kernel, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, st, src, rowmap, N, K,
                     (u32x4*)dst);
}

__global__ void gather_rows_kernel(const float* src, const int* rowmap, int N, int K, float* dst) {
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (size_t)N * K) return;
  const int n = (int)(gid / K), k = (int)(gid % K);
  dst[gid] = src[(size_t)rowmap[n] * K + k];
}

void gather_rows_f32(const float* src, const int* rowmap, int N, int K, float* dst, hipStream_t st) {
  size_t total = (size_t)N * K;
  hipLaunchKernelGGL(gather_rows_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, src, rowmap, N, K,
                     dst);
}

}  // namespace ssd
