// Projection GEMMs of passes of at most ROWS_MAX token rows (one row of a few
// images, autoregressive steps, small prefills), with the epilogues of
// kernels_gemm.hip.
//
// At these row counts a launch streams its weights once and is bound by HBM,
// by the token rows every workgroup reads again from L2, and by the chain of
// dependent memory round trips around the stream.  A workgroup of eight waves
// owns 16 NT output features and up to 64 rows (128 in two row groups, below);
// its waves split its K range, each loads its weight tiles and token fragments straight into registers (a
// ring of R k-blocks in flight), and they meet in LDS, summed in wave order
// (deterministic).  Every operand byte is loaded once per workgroup and, with
// the whole K range in it, no partial sum leaves it: no publish, count and
// reload round trips.  Narrow outputs of many rows split K over S workgroups
// as well (the last arrival sums them in split order), since a wide feature
// block then saves more token traffic than the hand-off costs.
//
// The inputs of these passes are stored as 16x32 operand tiles (act_index): a
// token fragment is 1 KiB contiguous.  From row-major planes the same loads
// touch 16 rows a power of two apart, 64 bytes each: a layer of the 1B widths
// at 48 rows took 109 us against 74 us.  A layer (with its attention) against
// the earlier split-K streaming kernels: 1B widths at 1, 24 and 64 rows 48.3 ->
// 43, 59.2 -> 53.4 and 89.3 -> 73.4 us; 7B widths at 33 and 64 rows 215.9 -> 118
// and 233.5 -> 142; 8B widths at 48 rows 238 -> 155.
//
// 65 to 128 rows: four waves for each half of the rows (48 or 64), every K share
// read by one wave of each.  A launch costs the bytes its workgroups draw
// through the L2s (its times over feature widths and splits fit 66 GB/s a CU
// with all CUs drawing: a fit, not a counter), hence plain weight loads, which
// the second row group may find in L1, and feature blocks no wider than the row
// groups' accumulators.
// Against the 128 x 64 tiles with LDS stages that ran these rows, 96 and 128
// rows: a 1B layer without attention 97.8 -> 69.7 and 103 -> 80 us, a 7B layer
// 222 -> 155 and 232 -> 182, 8B QKV 35 -> 26.9 and 37.2 -> 30.3.
#pragma once

#include "tiles.h"

namespace ssd {

constexpr int RW_NW = 8;  // waves

// MT: row tiles of a wave; RH: groups of MT row tiles (a workgroup's rows), NW / RH waves each
// OCC: waves per SIMD, 2 (one workgroup per CU) or 4 (two, 128 registers each)
template <int MT, int NT, int R, int OCC, int RH>
__global__ __launch_bounds__(RW_NW * 64) __attribute__((amdgpu_waves_per_eu(OCC, OCC)))
void gemm_rows_kernel(RowsKArgs a) {
  constexpr int NW = RW_NW, KW = NW / RH, NTH = NW * 64, MP = RH * MT * 16;
  constexpr int RP = MT == 3 ? RH * 64 : MP;         // rows of the 1/rms thread groups
  constexpr int G = NTH / RP;                        // groups, each summing QP parts of every row
  constexpr int QP = RH > 1 ? 16 : (MT <= 2 ? 256 : 128) / G;
  constexpr int FW = NT * MT;                        // accumulator fragments of a wave
  constexpr int FR = RH * FW;                        // and of the workgroup
  constexpr int FPW = (FR + NW - 1) / NW;            // fragments a wave finishes
  constexpr bool FOLD = FW > 18;                     // the upper waves add to the lower ones first (LDS)
  constexpr int PW = FOLD ? KW / 2 : KW;
  __shared__ __attribute__((aligned(16))) float part[PW][FR][64 * 4];
  __shared__ float rms_red[G][RP];
  __shared__ float rscale[RP];
  __shared__ float sq_red[NT][MP];
  __shared__ int is_last;

  int fb, split;
  xcd_unmap(blockIdx.x, a.S, a.xcd, fb, split);
  if (fb >= a.n_fb) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kw = w / RH, rh = w % RH;                // the wave's K share and row group
  const EpiArgs& e = a.epi;
  const int tiles = a.N / 16, ft = fb * NT;
  const int t0 = a.t0, M = a.M;  // at most MP rows

  // workgroup fragment q: row group q / FW, in it feature tile q % FW / MT and row tile q % MT
  auto row_tile = [](int q) { return q / FW * MT + q % FW % MT; };
  auto feat_tile = [](int q) { return q % FW / MT; };
  // block starts of the fragments this wave finishes, then the x^2 parts
  EpiOps<1, 1> op[FPW];
#pragma unroll
  for (int j = 0; j < FPW; ++j) {
    const int q = w + j * NW, mt = row_tile(q < FR ? q : 0);
    epi_block_starts<1, 1>(e, max(M - mt * 16, 1), t0 + min(mt * 16, M - 1), lane, op[j]);
  }
  float rv[QP];
  {
    const int t = tid % RP, g = tid / RP;
    const bool has = e.ssq != nullptr;
    const float* base = has ? e.ssq : (const float*)a.in.p;
    const size_t c = has ? (size_t)e.ssq_off + (size_t)(t0 + min(t, M - 1)) * e.ssq_step : 0;
    const size_t ld = has ? (size_t)e.ssq_ld : 0;
#pragma unroll
    for (int i = 0; i < QP; ++i) {
      const int p = g * QP + i;
      rv[i] = base[(size_t)(p < e.ssq_parts ? p : 0) * ld + c];
    }
  }
  __builtin_amdgcn_sched_barrier(0);

  // this wave's k-blocks [k0, k0 + n) of the split's: counts differ by one at
  // most, so only the last group of R can be short
  const int kbs = a.KB / a.S, least = kbs / KW, more = kbs - least * KW;
  const int k0 = split * kbs + kw * least + min(kw, more), n = least + (kw < more ? 1 : 0);
  const int groups = max(1, (least + (more ? 1 : 0) + R - 1) / R);
  const u32x4* wp[NT];                               // tiles past the last reload it; their results are not stored
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) wp[nt] = (const u32x4*)a.W + (size_t)min(ft + nt, tiles - 1) * a.KB * 64;
  const uint16_t* xp[MT];                            // rows past M repeat row M - 1
  const int kstep = a.in.tiled ? 512 : 32;           // elements between k-blocks of a row
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int r = a.in.row0 + (t0 + min((rh * MT + mt) * 16 + (lane & 15), M - 1)) * a.in.rstep;
    xp[mt] = a.in.p + (a.in.tiled ? (size_t)(r >> 4) * a.KB * 512 + ((lane >> 4) * 16 + (r & 15)) * 8
                                  : (size_t)r * a.in.ld + (lane >> 4) * 8);
  }
  const size_t plane = a.in.plane;

  u32x4 rw[R][NT], rx[R][MT], rl[R][MT];
  auto load = [&](int u, int i) {
    const int kb = min(k0 + i, a.KB - 1);            // past the wave's last block: never used
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      // read once by the workgroup, or once per row group: the later reads may find it in L1
      if constexpr (RH == 1)
        rw[u][nt] = __builtin_nontemporal_load(wp[nt] + (size_t)kb * 64 + lane);
      else
        rw[u][nt] = *(wp[nt] + (size_t)kb * 64 + lane);
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      rx[u][mt] = *(const u32x4*)(xp[mt] + (size_t)kb * kstep);
      rl[u][mt] = *(const u32x4*)(xp[mt] + plane + (size_t)kb * kstep);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  floatx4 acc[NT][MT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[nt][mt] = floatx4{0.f, 0.f, 0.f, 0.f};
  auto mma = [&](int u) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const bf16x8 wf = __builtin_bit_cast(bf16x8, rw[u][nt]);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        acc[nt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, __builtin_bit_cast(bf16x8, rx[u][mt]), acc[nt][mt], 0, 0, 0);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        acc[nt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, __builtin_bit_cast(bf16x8, rl[u][mt]), acc[nt][mt], 0, 0, 0);
    }
  };
#pragma unroll
  for (int u = 0; u < R; ++u) load(u, u);
  // the x^2 parts were loaded first, so their sums wait for nothing else
  {
    const int t = tid % RP, g = tid / RP;
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < QP; ++i) s += g * QP + i < e.ssq_parts ? rv[i] : 0.f;
    if (e.ssq && e.ssq_parts > G * QP) {             // more parts than one batch (narrow blocks of a wide model)
      const float* col = e.ssq + (size_t)e.ssq_off + (size_t)(t0 + min(t, M - 1)) * e.ssq_step;
      for (int p = G * QP + g; p < e.ssq_parts; p += G) s += col[(size_t)p * e.ssq_ld];
    }
    rms_red[g][t] = s;
  }
  for (int g = 0; g + 1 < groups; ++g) {
#pragma unroll
    for (int u = 0; u < R; ++u) {
      mma(u);
      load(u, (g + 1) * R + u);
    }
  }
#pragma unroll
  for (int u = 0; u < R; ++u)
    if ((groups - 1) * R + u < n) mma(u);

  // the waves meet: every wave leaves its fragments (FOLD: the upper waves
  // leave theirs, the lower ones add them to their own first)
  auto leave = [&](int slot) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) *(floatx4*)&part[slot][rh * FW + nt * MT + mt][lane * 4] = acc[nt][mt];
  };
  if constexpr (FOLD) {
    if (kw >= PW) leave(kw - PW);
    lds_barrier();
    if (kw < PW) {
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[nt][mt] += *(const floatx4*)&part[kw][rh * FW + nt * MT + mt][lane * 4];
      leave(kw);
    }
  } else {
    leave(kw);
  }
  // epilogue operands while the waves meet
  auto operands = [&]() {
#pragma unroll
    for (int j = 0; j < FPW; ++j) {
      const int q = w + j * NW, qc = q < FR ? q : 0, mt = row_tile(qc);
      epi_load<1, 1>(e, min(ft + feat_tile(qc), tiles - 1), a.N, max(M - mt * 16, 1), t0 + min(mt * 16, M - 1), lane, op[j]);
    }
  };
  if (a.S == 1) operands();
  lds_barrier();
  if (tid < RP) {
    float s = 0.f;
#pragma unroll
    for (int g = 0; g < G; ++g) s += rms_red[g][tid];
    rscale[tid] = e.ssq ? 1.0f / sqrtf(s * e.inv_d + e.eps) : 1.f;
  }
  floatx4 v[FPW];
#pragma unroll
  for (int j = 0; j < FPW; ++j) {
    const int q = w + j * NW, qc = q < FR ? q : 0;
    v[j] = *(const floatx4*)&part[0][qc][lane * 4];
#pragma unroll
    for (int x = 1; x < PW; ++x) v[j] += *(const floatx4*)&part[x][qc][lane * 4];
  }
  if (a.S > 1) {
    // publish this split's sums; the last arrival of the block sums the splits in order
    float* P = a.part + (size_t)fb * a.S * FR * 256 + lane * 4;
#pragma unroll
    for (int j = 0; j < FPW; ++j)
      if (w + j * NW < FR) *(floatx4*)(P + ((size_t)split * FR + w + j * NW) * 256) = v[j];
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (tid == 0) {
      if (!a.xcd) __threadfence();  // splits on different XCDs: write back through L2
      const unsigned prev = atomicAdd(&a.counters[fb], 1u);
      is_last = prev == (unsigned)(a.S - 1);
      if (is_last) a.counters[fb] = 0u;  // every split has arrived: re-arm
      if (is_last && !a.xcd) __threadfence();
    }
    __syncthreads();
    if (!is_last) return;
    operands();
#pragma unroll
    for (int j = 0; j < FPW; ++j) v[j] = floatx4{0.f, 0.f, 0.f, 0.f};
    constexpr int U = RH > 1 ? 2 : 4;
    for (int s0 = 0; s0 < a.S; s0 += U) {  // U splits' loads in flight (indexes clamped, the surplus masked)
      floatx4 pv[U][FPW];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int j = 0; j < FPW; ++j) {
          const int q = w + j * NW;
          pv[u][j] = *(const floatx4*)(P + ((size_t)min(s0 + u, a.S - 1) * FR + (q < FR ? q : 0)) * 256);
        }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int j = 0; j < FPW; ++j) v[j] += pv[u][j] * (s0 + u < a.S ? 1.f : 0.f);
    }
  } else {
    lds_barrier();  // rscale
  }
#pragma unroll
  for (int j = 0; j < FPW; ++j) {
    const int q = w + j * NW;
    if (q >= FR) break;
    const int nt = feat_tile(q), mt = row_tile(q);
    float sq[1] = {0.f};
    if (mt * 16 < M) {
      const floatx4 o[1][1] = {{v[j]}};
      epi_store<1, 1>(e, o, op[j], ft + nt, a.N, M - mt * 16, t0 + mt * 16, lane, rscale + mt * 16, sq);
    }
    if (e.kind == EPI_RESID) {
      float s = sq[0];
      s += __shfl_xor(s, 16);
      s += __shfl_xor(s, 32);
      if (lane < 16) sq_red[nt][mt * 16 + lane] = s;
    }
  }
  if (e.kind == EPI_RESID) {
    lds_barrier();
    if (tid < M) {
      float s = 0.f;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) s += ft + nt < tiles ? sq_red[nt][tid] : 0.f;
      e.ssq_out[(size_t)fb * e.ssq_out_ld + t0 + tid] = s;
    }
  }
}

template <int MT, int NT, int OCC, int RH>
static void launch_rows(const RowsKArgs& a, hipStream_t st) {
  // ring depth: as many k-blocks as the registers beside the accumulators hold
  constexpr int PER = (NT + 2 * MT) * 4, LEFT = (OCC == 4 ? 128 - 30 : 256 - 44) - NT * MT * 4;
  constexpr int R = LEFT / PER >= 8 ? 8 : LEFT / PER >= 4 ? 4 : LEFT / PER >= 3 ? 3 : 2;
  launch_timed(gemm_rows_kernel<MT, NT, R, OCC, RH>, dim3(xcd_grid(a.n_fb, a.S, a.xcd)), dim3(RW_NW * 64), st, a);
}

template <int MT, int OCC, int RH>
static void launch_rows_nt(int NT, const RowsKArgs& a, hipStream_t st) {
  switch (NT) {
    case 1: launch_rows<MT, 1, OCC, RH>(a, st); break;
    case 2: launch_rows<MT, 2, OCC, RH>(a, st); break;
    case 3: launch_rows<MT, 3, OCC, RH>(a, st); break;
    case 4: launch_rows<MT, 4, OCC, RH>(a, st); break;
    default: launch_rows<MT, 6, OCC, RH>(a, st); break;
  }
}

// MT: row tiles of the plan (1 to 4; 6 and 8 as two row groups of 3 and 4)
void gemm_rows(int MT, int NT, const RowsKArgs& a, hipStream_t st) {
  // up to 16 rows more workgroups than CUs run two to a CU, one's stream over
  // the other's epilogue (1B output layer, one row: 13.6 us with 512
  // workgroups of 32 features, 17.4 us with 256 of 64 alone on their CUs);
  // with a CU each, the registers go into a deeper ring
  switch (MT) {
    case 1:
      if (a.n_fb * a.S > 256)
        launch_rows_nt<1, 4, 1>(NT, a, st);
      else
        launch_rows_nt<1, 2, 1>(NT, a, st);
      break;
    case 2: launch_rows_nt<2, 2, 1>(NT, a, st); break;
    case 3: launch_rows_nt<3, 2, 1>(NT, a, st); break;
    case 4: launch_rows_nt<4, 2, 1>(NT, a, st); break;
    case 6: launch_rows_nt<3, 2, 2>(NT, a, st); break;
    default: launch_rows_nt<4, 2, 2>(NT, a, st); break;
  }
}

// Feature tiles per workgroup and K splits of an M-row projection: the least
// of a launch's modelled time over NT and S.  Its terms are a fit to the
// launches of the 1B, 7B and 8B widths at 24 to 64 rows over all NT and S (the
// choice is 1 % off the best one on the average, 10 % at most): weights from
// HBM at 5.3 TB/s together and 30 GB/s a CU; every workgroup's weights and
// token rows, and the splits' partial sums out and back, through the L2s at
// 17 TB/s together and 44 GB/s a CU (66 from 33 rows on, whose deeper token
// tiles keep more loads in flight); 4 us and 0.4 us a split for the hand-off;
// 1 us for each further round of workgroups and for 1024 of them.  From 65 rows
// on (two row groups, fitted at 96 and 128 rows: the choice is 1 % off the best
// on the average, 8 % at most) both row groups' weight reads count, the hand-off
// is 1 us, 0.2 us a feature tile and 0.75 us a MB of partial sums, and 128 rows by 96 features, whose
// registers spill, take 20 % more.  Rows count
// in classes, so that the plans of the class bounds cover every row count
// (workspace sizes).
GemmPlan gemm_rows_plan(int M, int N, int K, int xcd, double* ns) {
  int MT = (std::min(M, ROWS_MAX) + 15) / 16;
  if (MT > 4) MT = MT > 6 ? 8 : 6;
  const int rows = MT * 16;
  const int KB = K / 32, tiles = N / 16;
  double best = 1e30;
  int NT = 1, S = 1;
  for (int nt : {1, 2, 3, 4, 6})
    for (int s = 1; s <= 16; ++s) {
      if (KB % s || (s > 1 && KB / s < RW_NW)) continue;
      const long wgs = (long)((tiles + nt - 1) / nt) * s, rounds = (wgs + 255) / 256;
      const double each = (nt * 32.0 * (MT > 4 ? 2 : 1) + rows * 4.0) * (K / s);  // bytes a workgroup reads
      const double parts = s > 1 ? 8.0 * s * rows * N : 0.0;                      // partial sums out and back
      double stream = std::max({(double)N * K * 2 / 5300, (wgs * each + parts) / 17000, rounds * each / (MT < 3 ? 44 : 66),
                                rounds * nt * 32.0 * (K / s) / 30});
      if (MT == 8 && nt == 6) stream *= 1.2;
      const double split = s == 1 ? 0 : MT > 4 ? 1000 + 200 * nt + parts * 0.75e-3 : 4000 + 400 * s;
      const double t = stream + split + (rounds - 1) * 1000.0 + wgs;
      if (t < best) {
        best = t;
        NT = nt;
        S = s;
      }
    }
  GemmPlan p{};
  p.xcd = xcd;
  p.MT = MT;
  p.NT = NT;
  p.WV = RW_NW;
  p.S = S;
  p.KCB = KB / S;
  p.kchunks = 1;
  p.bn = NT * 16;
  p.n_fb = (tiles + NT - 1) / NT;
  p.tail_S = 1;
  if (ns) *ns = best;
  return p;
}

}  // namespace ssd
