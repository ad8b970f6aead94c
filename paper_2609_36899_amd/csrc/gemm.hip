// Weight-streaming projections: out[s][m][n] = sum_{k in split s} A[m][k] W[n][k].
//
// Each decode step reads the weights once for the whole active batch (paper:
// Introduction; Design Principles, "Specialization in Heterogeneous Pools"),
// so at decode batch sizes the weight stream from HBM is the bound.  bf16
// weights are stored packed so that this stream is long contiguous runs:
// columns form groups of 128 (8 strips of 16), a 16-column x 32-k block is
// 1 KiB in the lane order of the v_mfma_f32_16x16x32_bf16 B operand (one
// 16-byte load per lane at lane * 8 is exactly one fragment), and the eight
// blocks of one k-block of a group are adjacent, so a group's weight tile for
// a k-step of 64 is one contiguous 16 KiB run (layout at pack_weight_kernel).
// Row-wise [N][K] weights give 128-byte runs in many rows at once and stream
// 10-25% slower.
//
// Kernels by batch rows: the streaming kernel (up to 32 rows, weights straight
// into registers), the 64- to 256-row LDS tiles, and the
// 256 x 256 tile above that.  When the column tiles alone cannot fill 256 CUs
// the K axis is split and the fp32 partial sums are reduced in a fixed order
// by the next kernel.
#include "hip_common.h"
#include "kernels.h"

namespace pdec {

namespace {

constexpr int kGroupCols = 128;  // columns per packed group (8 strips of 16)

// Group g of a bf16 weight given as up to three packed segments.
struct GroupRef {
  const uint16_t* base;  // the group's K/32 x 8 blocks of 512 elements
  int col0;              // its first output column
  int col_end;           // end of its segment's output columns
};
__device__ __forceinline__ GroupRef group_ref(const WSegs& w, int g, int K) {
  int s = 0;
  while (s < w.n_seg - 1 && g >= w.grp_end[s]) ++s;
  const int g0 = s ? w.grp_end[s - 1] : 0, c0 = s ? w.row_end[s - 1] : 0;
  return {(const uint16_t*)w.ptr[s] + (int64_t)(g - g0) * kGroupCols * K,
          c0 + (g - g0) * kGroupCols, w.row_end[s]};
}

// Packed bf16 layout (group-major): element (n, k) of an [N][K] matrix is at
//   (((G * K/32 + b) * 8 + s) * 64 + q * 16 + c) * 8 + e,
//   n = 128 G + 16 s + c,  k = 32 b + 8 q + e,
// columns past N zero.  A 16 x 32 block (s, b) is 1 KiB in the lane order of
// the MFMA B operand, and the eight blocks of one k-block of a group are
// adjacent: per k-step of 64 a group's weight tile is one contiguous 16 KiB
// run, so the streams a projection reads from HBM are few and long.
__global__ __launch_bounds__(256) void pack_weight_kernel(const uint16_t* __restrict__ W, int N,
                                                          int K, uint16_t* __restrict__ P) {
  const int KB = K / 32;
  const int64_t chunk = (int64_t)blockIdx.x * 256 + threadIdx.x;  // one 8-element chunk
  if (chunk >= (int64_t)((N + kGroupCols - 1) / kGroupCols) * KB * 8 * 64) return;
  const int l = (int)(chunk & 63);
  const int64_t r = chunk >> 6;
  const int s = (int)(r & 7);
  const int64_t gb = r >> 3;
  const int b = (int)(gb % KB), G = (int)(gb / KB);
  const int n = G * kGroupCols + 16 * s + (l & 15), k = 32 * b + 8 * (l >> 4);
  u32x4 v = {0u, 0u, 0u, 0u};
  if (n < N) v = *(const u32x4*)(W + (int64_t)n * K + k);
  *(u32x4*)(P + chunk * 8) = v;
}

// SwiGLU-fused form (GLU = true, gate and up given as the two segments of
// w, N = the FFN width F, no K split): work group v takes half h = v % 2 of
// group G = v / 2 of both matrices, and each wave the same 16 columns of the
// gate and of the up matrix.  The two results of a column then sit in one
// lane, and the epilogue writes silu(gate) * up as bf16 to u [M][F]: the
// fp32 gate/up products never reach memory.
__device__ __forceinline__ float silu_mul(float g, float u) { return g / (1.f + expf(-g)) * u; }

// Small batches (M <= 32): a work group owns one 128-column group, each of
// its four waves two strips of it and every row of the batch (MT tiles of 16
// rows), so no two waves share weight bytes and no LDS or barrier is needed.
// The weight fragments and the matching activation fragments (L2-resident)
// of the next NS k-steps are in flight in a register ring.  The steady-state
// loop is branch-free (the prefetch index is clamped to the last step) and
// pinned to consume-then-refill order per slot, so the compiler keeps all NS
// slots in flight instead of draining the ring.
template <int MT, int NS, bool GLU>
__global__ __launch_bounds__(256) void gemm_bf16_stream(int M, int N, int K, int k_split,
                                                        const uint16_t* __restrict__ A,
                                                        int64_t lda, WSegs w,
                                                        float* __restrict__ out,
                                                        uint16_t* __restrict__ glu_out) {
  constexpr int WS = 2;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int c16 = lane & 15, q4 = lane >> 4;
  const int kbeg = blockIdx.z * k_split;
  const int n_iter = (min(K, kbeg + k_split) - kbeg) / 64;
  if (n_iter <= 0) return;  // no barriers in this kernel

  // Strip s of this wave, k-block kb: wp[s] + kb * 4096 (a k-block of a
  // group is 8 strips of 512 elements).  Plain: strips 2 wave and 2 wave + 1
  // of group blockIdx.x.  GLU: strip 4 h + wave of the gate and of the up
  // matrix's group G.
  const uint16_t* wp[WS];
  int col_s[WS], col_end;
  if constexpr (GLU) {
    const int G = blockIdx.x >> 1, h = blockIdx.x & 1;
    const int64_t off =
        (int64_t)G * kGroupCols * K + ((int64_t)(kbeg / 32) * 8 + 4 * h + wave) * 512 + lane * 8;
    wp[0] = (const uint16_t*)w.ptr[0] + off;
    wp[1] = (const uint16_t*)w.ptr[1] + off;
    col_s[0] = col_s[1] = G * kGroupCols + (4 * h + wave) * 16 + c16;
    col_end = N;
  } else {
    const GroupRef gr = group_ref(w, blockIdx.x, K);
    wp[0] = gr.base + ((int64_t)(kbeg / 32) * 8 + 2 * wave) * 512 + lane * 8;
    wp[1] = wp[0] + 512;
    col_s[0] = gr.col0 + 2 * wave * 16 + c16;
    col_s[1] = col_s[0] + 16;
    col_end = gr.col_end;
  }
  const uint16_t* ap[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t)
    ap[t] = A + (int64_t)min(t * 16 + c16, M - 1) * lda + kbeg + q4 * 8;

  f32x4 acc[MT][WS];
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int s = 0; s < WS; ++s) acc[t][s] = f32x4{0.f, 0.f, 0.f, 0.f};
  bf16x8 rw[NS][WS][2], ra[NS][MT][2];
  auto load = [&](int i, bf16x8(&wr)[WS][2], bf16x8(&ar)[MT][2]) {
#pragma unroll
    for (int s = 0; s < WS; ++s) {
      wr[s][0] = load_stream<bf16x8>(wp[s] + (int64_t)(2 * i) * 4096);
      wr[s][1] = load_stream<bf16x8>(wp[s] + (int64_t)(2 * i + 1) * 4096);
    }
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      ar[t][0] = *(const bf16x8*)(ap[t] + i * 64);
      ar[t][1] = *(const bf16x8*)(ap[t] + i * 64 + 32);
    }
  };
  auto mma = [&](const bf16x8(&wr)[WS][2], const bf16x8(&ar)[MT][2]) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int s = 0; s < WS; ++s)
          acc[t][s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ar[t][h], wr[s][h], acc[t][s], 0, 0, 0);
  };
  const int last = n_iter - 1;
#pragma unroll
  for (int s = 0; s < NS; ++s) load(min(s, last), rw[s], ra[s]);
  int it0 = 0;
  for (; it0 + NS <= n_iter; it0 += NS) {
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      mma(rw[s], ra[s]);
      load(min(it0 + s + NS, last), rw[s], ra[s]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  const int rem = n_iter - it0;
#pragma unroll
  for (int s = 0; s < NS; ++s)
    if (s < rem) mma(rw[s], ra[s]);

  if constexpr (GLU) {
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        const int row = t * 16 + 4 * q4 + rr;
        if (row < M && col_s[0] < col_end)
          glu_out[(int64_t)row * N + col_s[0]] = f32_to_bf16(silu_mul(acc[t][0][rr], acc[t][1][rr]));
      }
  } else {
    float* o = out + (int64_t)blockIdx.z * M * N;
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
      for (int s = 0; s < WS; ++s)
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
          const int row = t * 16 + 4 * q4 + rr;
          if (row < M && col_s[s] < col_end) o[(int64_t)row * N + col_s[s]] = acc[t][s][rr];
        }
  }
}

// Few rows and few columns (at most 16 rows and 256 strips; o and, up to nine
// rows, down of the 8B shape): one work group per 16-column strip, its eight
// waves taking an eighth of K each and adding up through LDS in wave order.  The
// strips alone fill the GPU, so nothing is split over the grid: no partial sums
// in memory, no pass that adds them, one slab for the consumer.  A wave keeps
// eight k-blocks of 32 (1 KiB of weights and as much of activations each) in
// flight, with K = 4096 half of its share; 16 in flight was no faster, nor was
// placing a group's strips on one XCD.  Each work group reads all of A, at 16
// rows as many bytes as its weights, which is what ends the form (see
// strip_form).  o (4096 x 4096), us per weight_projection, streaming kernel and
// split sum against this: 9.9 / 7.8 at 1 row, 10.6 / 9.2 at 16.
constexpr int kStripWaves = 8;
__global__ __launch_bounds__(64 * kStripWaves) void gemm_bf16_strip(
    int M, int N, int K, const uint16_t* __restrict__ A, int64_t lda, WSegs w,
    float* __restrict__ out) {
  constexpr int NS = 8;
  __shared__ __attribute__((aligned(16))) f32x4 red[kStripWaves][64];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int c16 = lane & 15, q4 = lane >> 4;
  const int strip = blockIdx.x & 7;
  const GroupRef gr = group_ref(w, blockIdx.x >> 3, K);
  const int kb_all = K / 32, per = (kb_all + kStripWaves - 1) / kStripWaves;
  const int kb0 = min(wave * per, kb_all), n = min(per, kb_all - kb0);  // this wave's k-blocks
  const uint16_t* wp = gr.base + ((int64_t)kb0 * 8 + strip) * 512 + lane * 8;
  const uint16_t* ap = A + (int64_t)min(c16, M - 1) * lda + kb0 * 32 + q4 * 8;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  if (n > 0) {
    bf16x8 rw[NS], ra[NS];
    // As in the streaming kernel: branch-free refills (clamped to the last
    // block) pinned behind the slot's use keep all NS slots in flight.
    const int last = n - 1;
    auto load = [&](int i, bf16x8& wr, bf16x8& ar) {
      wr = load_stream<bf16x8>(wp + (int64_t)i * 4096);
      ar = *(const bf16x8*)(ap + i * 32);
    };
#pragma unroll
    for (int s = 0; s < NS; ++s) load(min(s, last), rw[s], ra[s]);
    int it = 0;
    for (; it + NS < n; it += NS) {
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ra[s], rw[s], acc, 0, 0, 0);
        load(min(it + s + NS, last), rw[s], ra[s]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int s = 0; s < NS; ++s)
      if (s < n - it) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ra[s], rw[s], acc, 0, 0, 0);
  }
  red[wave][lane] = acc;
  __syncthreads();
  if (wave > 0) return;
#pragma unroll
  for (int v = 1; v < kStripWaves; ++v) acc += red[v][lane];
  const int col = gr.col0 + strip * 16 + c16;
#pragma unroll
  for (int rr = 0; rr < 4; ++rr)
    if (4 * q4 + rr < M && col < gr.col_end) out[(int64_t)(4 * q4 + rr) * N + col] = acc[rr];
}

// Larger batches (M > 32): ROWS x 128 output tiles, waves in a (ROWS / 16 MT) x 2
// grid of 16 MT x 64 sub-tiles (64 x 64, and 32 x 64 for the 64-row tile).  Per
// k-step of 64 the A tile and the W tile are staged once through LDS and each is
// shared by the waves that need it.  The tiles travel from memory straight into
// LDS (16-byte LDS-DMA loads, no register staging), through a ring of D stages:
// while step it is computed, steps it+1 .. it+D-1 are in flight.  One barrier per
// step: after it, every wave has finished step it-1, whose stage then takes step
// it+D-1.  Up to 64 rows the weight stream is the bound and what is in flight
// sets its rate: the 128-row tile's two stages give gate/up 5.3 TB/s at 64 rows
// (44.4 us), five of this tile (D = 6, 24 KiB stages) 5.7 (40.9).  From 128 rows on a
// fourth stage measured level or slower.
// The W tile (one packed group, 2 k-blocks x 8 strips) is one contiguous
// 16 KiB run in HBM, copied in packed order (fragment reads from LDS are
// linear, hence free of bank conflicts) with the non-temporal hint, so the
// weight stream does not push the re-read A tiles out of L2; the A tile is
// row-major with its 16-byte chunks XOR-swizzled by row (the swizzle is applied
// to the source address, as the DMA writes each wave's 64 chunks contiguously).
// Up to 256 rows one tile covers the batch, so W is read from HBM exactly once
// per step.  Larger batches take several M-blocks, laid out so the M-blocks of one
// column tile are dispatched back to back (ids L and L+8 share an XCD).
// GLU (gate and up as the two segments of w, N = F, no K split): column tile
// v holds half v % 2 of group v / 2 of both matrices, its eight strips
// staged as gate, up, gate, up, ... so that each wave's four strips are two
// (gate, up) pairs of the same columns; the epilogue writes silu(gate) * up
// as bf16 to u [M][F].
template <int ROWS, int MT, int D, bool GLU>
__global__ __launch_bounds__(8 * ROWS / MT) void gemm_bf16_tile(int M, int N, int K, int k_split,
                                                          int n_mb, int n_nb,
                                                          const uint16_t* __restrict__ A,
                                                          int64_t lda, WSegs w,
                                                          float* __restrict__ out,
                                                          uint16_t* __restrict__ glu_out) {
  constexpr int NT = 4;
  constexpr int THREADS = 8 * ROWS / MT;           // (ROWS / 16 MT) x 2 waves
  constexpr int ACH = ROWS * 8 / THREADS;          // A chunks per thread per stage (MT)
  constexpr int WCH = (1024 + THREADS - 1) / THREADS;  // W chunks per thread (16 KiB tile)
  constexpr int LPS = ACH + WCH;                   // loads per thread per stage
  // 384 threads: the last W load of the waves past the tile repeats chunks into
  // padding, so that every wave has the same number of loads in flight.
  constexpr int SA = ROWS * 64, STAGE = SA + WCH * THREADS * 8;
  static_assert(D >= 3 && D <= 6 && STAGE * 2 * D <= 160 * 1024, "stages fit the LDS");
  // One array per stage: the compiler then tells the stages' LDS apart and
  // does not wait for every DMA in flight before reading a landed stage.
  __shared__ __attribute__((aligned(16))) uint16_t lds0[STAGE];
  __shared__ __attribute__((aligned(16))) uint16_t lds1[STAGE];
  __shared__ __attribute__((aligned(16))) uint16_t lds2[STAGE];
  __shared__ __attribute__((aligned(16))) uint16_t lds3[D > 3 ? STAGE : 8];
  __shared__ __attribute__((aligned(16))) uint16_t lds4[D > 4 ? STAGE : 8];
  __shared__ __attribute__((aligned(16))) uint16_t lds5[D > 5 ? STAGE : 8];
  auto stage_ptr = [&](int b) -> uint16_t* {
    return b == 0 ? lds0 : b == 1 ? lds1 : b == 2 ? lds2 : b == 3 ? lds3 : b == 4 ? lds4 : lds5;
  };
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int c16 = lane & 15, q4 = lane >> 4;
  const int L = blockIdx.x;
  const int grp = L / (8 * n_mb), rem = L % (8 * n_mb);
  const int mb = rem / 8, nb = grp * 8 + rem % 8;
  if (nb >= n_nb) return;  // padding of the id layout; uniform over the group
  const int kbeg = blockIdx.z * k_split;
  const int n_iter = (min(K, kbeg + k_split) - kbeg) / 64;
  if (n_iter <= 0) return;
  const int m_blk = mb * ROWS;
  const int wm = wave >> 1, wn = wave & 1;
  GroupRef gr;
  if constexpr (GLU) gr = {nullptr, (nb >> 1) * kGroupCols + (nb & 1) * 64, N};
  else gr = group_ref(w, nb, K);

  // Chunk id = j * THREADS + tid lands at LDS chunk id of the stage (the DMA
  // of wave w, load j, fills chunks j * THREADS + 64 w .. +63).  A: chunk id
  // is row id >> 3, slot id & 7, holding source chunk slot ^ (row & 7).
  const uint16_t* asrc[ACH];
#pragma unroll
  for (int j = 0; j < ACH; ++j) {
    const int id = j * THREADS + tid, r = id >> 3, slot = id & 7;
    asrc[j] = A + (int64_t)min(m_blk + r, M - 1) * lda + kbeg + ((slot ^ (r & 7)) * 8);
  }
  // W: chunk id of step i is chunk id of the step's 16 KiB run (k-block
  // 2i + (id >> 9), strip (id >> 6) & 7, lane id & 63).
  const uint16_t* wsrc[WCH];
#pragma unroll
  for (int j = 0; j < WCH; ++j) {
    const int id = (j * THREADS + tid) & 1023;
    if constexpr (GLU) {  // staged strip sp: strip 4 h + sp / 2 of gate (sp even) or up
      const int kb = id >> 9, sp = (id >> 6) & 7, ln = id & 63;
      wsrc[j] = (const uint16_t*)w.ptr[sp & 1] + (int64_t)(nb >> 1) * kGroupCols * K +
                ((int64_t)(kbeg / 32 + kb) * 8 + 4 * (nb & 1) + (sp >> 1)) * 512 + ln * 8;
    } else {
      wsrc[j] = gr.base + (int64_t)(kbeg / 32) * 4096 + id * 8;
    }
  }
  int aoff[MT][2];
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int ra = wm * 16 * MT + t * 16 + c16, cc = h * 4 + q4;
      aoff[t][h] = ra * 64 + ((cc ^ (ra & 7)) * 8);
    }

  f32x4 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  auto issue1 = [&](int i, int b, int j) {  // load j of step i into stage b, W first
    uint16_t* base = stage_ptr(b) + wave * 64 * 8;
    if (j < WCH)
      dma16_stream(wsrc[j] + (int64_t)i * 8192, base + SA + j * THREADS * 8);
    else
      dma16(asrc[j - WCH] + i * 64, base + (j - WCH) * THREADS * 8);
  };
  auto issue = [&](int i, int b) {
#pragma unroll
    for (int j = 0; j < LPS; ++j) issue1(i, b, j);
  };
  // The step in stage b, with the loads of step i_next: one behind each row of MFMAs
  // where they fit (all at once, eight waves stall on the 64 bytes a cycle of the
  // texture path; us, spread / at once: gate/up of the 8B shape at 160 rows 55 / 60,
  // of the 14B shape at 200 rows 104 / 107, down of the 8B shape at 1463 rows 170 /
  // 185), or all ahead of them (the 64-row tile, which lives on loads in flight).
  constexpr bool kSpread = 2 * MT >= LPS;
  auto compute = [&](int b, int i_next, int b_next) {
    if constexpr (!kSpread) {
      issue(i_next, b_next);
      __builtin_amdgcn_sched_barrier(0);
    }
    const uint16_t* la = stage_ptr(b);
    const uint16_t* lw = la + SA;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      bf16x8 af[MT], bf[NT];
#pragma unroll
      for (int t = 0; t < MT; ++t) af[t] = *(const bf16x8*)(la + aoff[t][h]);
#pragma unroll
      for (int t = 0; t < NT; ++t)
        bf[t] = *(const bf16x8*)(lw + ((h * 8 + wn * 4 + t) * 64 + lane) * 8);
#pragma unroll
      for (int i = 0; i < MT; ++i) {
#pragma unroll
        for (int j = 0; j < NT; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], bf[j], acc[i][j], 0, 0, 0);
        if constexpr (kSpread) {
          if (h * MT + i < LPS) issue1(i_next, b_next, h * MT + i);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  };
  // Every step issues one stage (the prefetch index clamped to the last
  // step, so the tail re-reads it into a stage nobody reads), which keeps
  // the count of loads in flight fixed: waiting until D - 2 stages are
  // outstanding means this wave's part of step it has landed; the barrier
  // then covers the other waves' parts.
  const int last = n_iter - 1;
#pragma unroll
  for (int s = 0; s < D - 1; ++s) issue(min(s, last), s);
  int it = 0;
  for (; it + D <= n_iter; it += D) {
#pragma unroll
    for (int s = 0; s < D; ++s) {
      wait_vmem<(D - 2) * LPS>();
      wg_barrier();
      compute(s, min(it + s + D - 1, last), (s + D - 1) % D);
    }
  }
  const int tail = n_iter - it;  // uniform over the work group
#pragma unroll
  for (int s = 0; s < D; ++s)
    if (s < tail) {
      wait_vmem<(D - 2) * LPS>();
      wg_barrier();
      compute(s, min(it + s + D - 1, last), (s + D - 1) % D);
    }
  wait_vmem<0>();  // no LDS write may still be in flight when the group ends

  if constexpr (GLU) {
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int p = 0; p < NT / 2; ++p) {
        const int col = gr.col0 + (2 * wn + p) * 16 + c16;
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
          const int row = m_blk + wm * 16 * MT + i * 16 + 4 * q4 + rr;
          if (row < M && col < gr.col_end)
            glu_out[(int64_t)row * N + col] =
                f32_to_bf16(silu_mul(acc[i][2 * p][rr], acc[i][2 * p + 1][rr]));
        }
      }
  } else {
    float* o = out + (int64_t)blockIdx.z * M * N;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        const int col = gr.col0 + wn * 64 + j * 16 + c16;
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
          const int row = m_blk + wm * 16 * MT + i * 16 + 4 * q4 + rr;
          if (row < M && col < gr.col_end) o[(int64_t)row * N + col] = acc[i][j][rr];
        }
      }
  }
}

// Batches above 256 rows (prefill chunks, B = 512 decode): 256 x 256 output
// tiles, four waves in a 2 x 2 grid of 128 x 128 sub-tiles (a wave's columns are
// one packed group, NT = 8 strips).  A large grid of these runs at the card's
// power limit (1.6-1.8 GHz here), so what a multiply moves counts as well as what
// it waits for.  A wave of 128 x 128 reads 16 KiB of fragments from LDS for 64
// MFMAs, a third less than two of 64 x 128; an A stage holds k-blocks in pairs, so
// that its loads take whole 128-byte lines (64-byte rows made half as many requests
// to L2 again); v_mfma_f32_32x32x16 took fewer cycles but 8% more time, at a lower
// clock.  One wave per SIMD has no other wave to cover its LDS reads, so it reads
// the fragments of the next k-block while this one's multiply (256 accumulator
// registers and two sets of 64 fragment registers; buffer addressing leaves room
// for them), a read per three MFMAs and, in the second half of a stage, a load per
// three: all 16 loads in half the time stall at the 64 bytes a cycle that the
// texture path takes (5% slower).
// 4096 rows, us, against eight waves of 64 x 128 and k-blocks staged singly: o of
// the 8B shape 102 / 117, down 335 / 372 (1.43 PFLOP/s), gate/up 721 / 770.
// Stages hold two k-blocks of 32: A 256 rows x 128 B and W 2 groups x 2 blocks x 8
// strips (two contiguous 16 KiB runs), in a ring of two.  Column tile v covers
// groups 2v and 2v + 1 (the second clamped to a valid group and its outputs
// dropped when the group count is odd); GLU: column tile v is group v of both
// matrices, wave column wn taking half wn of it with its strips staged as gate,
// up, gate, up, ... (four (gate, up) pairs per wave), and the epilogue writes
// silu(gate) * up as bf16.
// Work group ids L and L + 8 share an XCD, whose 32 CUs run bands of up to
// kBandRows M-blocks by four columns of tiles: the 12 tile edges of such a square
// come through its L2 instead of the 18 of 16 M-blocks by two columns (what down
// at 4096 rows reads past L2: 0.75 GB against 1.0).  K >= 128, a multiple of 64.
constexpr int kBandRows = 8;
template <bool GLU>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void gemm_bf16_wide(
    int M, int N, int K, int n_mb, int n_nb, int row_x, int n_groups, const uint16_t* __restrict__ A,
    int64_t lda, WSegs w, float* __restrict__ out, uint16_t* __restrict__ glu_out) {
  constexpr int MT = 8, NT = 8, THREADS = 256, ROWS = 256;
  constexpr int ACH = ROWS * 8 / THREADS;  // A chunks per thread per stage (8)
  constexpr int WCH = 2048 / THREADS;      // W chunks per thread per stage (8)
  constexpr int LPS = ACH + WCH;
  constexpr int SA = ROWS * 64, STAGE = SA + 2 * 2 * 8 * 512;  // elements
  __shared__ __attribute__((aligned(16))) uint16_t lds0[STAGE];
  __shared__ __attribute__((aligned(16))) uint16_t lds1[STAGE];
  auto stage_ptr = [&](int b) -> uint16_t* { return b == 0 ? lds0 : lds1; };
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // scalar, as all it leads to
  const int c16 = lane & 15, q4 = lane >> 4;
  // XCD x takes columns c, c + cols_x, .. and one of row_x equal parts of the
  // M-blocks; seq numbers its tiles: bands of M-blocks, a band's columns in turn.
  const int x = blockIdx.x % 8, seq = blockIdx.x / 8, cols_x = 8 / row_x;
  const int part = n_mb / row_x, nb_x = (n_nb + cols_x - 1) / cols_x;
  const int band = seq / (kBandRows * nb_x), in_band = seq % (kBandRows * nb_x);
  const int band_h = min(kBandRows, part - band * kBandRows);
  const int mb = x / cols_x * part + band * kBandRows + in_band % band_h;
  const int nb = in_band / band_h * cols_x + x % cols_x;
  if (nb >= n_nb) return;  // padding of the id layout; uniform over the group
  const int n_stages = K / 64;
  const int m_blk = mb * ROWS;
  const int wm = wave >> 1, wn = wave & 1;

  // This wave's output columns: strip t covers col0 + 16 t .. + 15 (plain) or
  // the pair p = t / 2 covers col0 + 16 p .. + 15 (GLU).
  int col0, col_end;
  if constexpr (GLU) {
    col0 = nb * kGroupCols + wn * 64;
    col_end = N;
  } else {
    const int gw = 2 * nb + wn;
    const GroupRef gr = group_ref(w, min(gw, n_groups - 1), K);
    col0 = gr.col0;
    col_end = gw < n_groups ? gr.col_end : 0;  // a clamped second group writes nothing
  }

  // A: chunk id = row * 8 + slot, holding source chunk slot ^ (row & 7).
  // Load j takes rows 32 j .. 32 j + 31; rows past M lie outside the buffer.  The
  // row is part of the lane's offset, which the bounds check counts; the uniform
  // offset, which the check may leave out, only moves along a row.
  const Buffer abuf = make_buffer(A + (int64_t)m_blk * lda,
                                  (uint32_t)min(ROWS, M - m_blk) * (uint32_t)(lda * 2));
  int aofs[ACH];
#pragma unroll
  for (int j = 0; j < ACH; ++j)
    aofs[j] = (32 * j + (tid >> 3)) * (int)(lda * 2) + (((tid & 7) ^ ((tid >> 3) & 7)) * 16);
  // W: chunk id = ((g2 * 2 + kb) * 8 + sp) * 64 + lane of staged group g2 (the
  // wave column that reads it), k-block kb, staged strip sp.  Load j brings strip
  // sp = 4 (j % 2) + wave of k-block (j / 2) % 2 and group j / 4; GLU: strip
  // 4 g2 + sp / 2 of gate (sp even) or up, for a wave always the same matrix.
  Buffer wbuf[2];
  int wofs;  // of the lane in the strips of load 0
  if constexpr (GLU) {
    wbuf[0] = wbuf[1] = make_buffer(
        (const uint16_t*)w.ptr[wave & 1] + (int64_t)nb * kGroupCols * K, (uint32_t)K * 256u);
    wofs = (wave >> 1) * 1024 + lane * 16;
  } else {
#pragma unroll
    for (int g2 = 0; g2 < 2; ++g2)
      wbuf[g2] = make_buffer(group_ref(w, min(2 * nb + g2, n_groups - 1), K).base,
                             (uint32_t)K * 256u);
    wofs = wave * 1024 + lane * 16;
  }
  // Fragments of k-block h of a stage.  Rows are 128 bytes: the eight consecutive
  // lanes of a read are eight rows and one logical chunk, swizzled to eight
  // distinct 16-byte bank groups.
  int aoff[2];  // row tile t: + t * 1024 elements (16 rows; the swizzle repeats every 8)
#pragma unroll
  for (int h = 0; h < 2; ++h)
    aoff[h] = (wm * 128 + c16) * 64 + (((4 * h + q4) ^ (c16 & 7)) * 8);
  const int woff = SA + wn * 16 * 512 + lane * 8;

  f32x4 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  auto issue1 = [&](int i, int b, int j) {  // load j of stage i into slot b
    uint16_t* base = stage_ptr(b) + wave * 64 * 8;
    if (j < ACH) {
      dma16_buf<false>(abuf, aofs[j], i * 128, base + j * THREADS * 8);
    } else {
      const int jw = j - ACH, kb = (jw >> 1) & 1, hi = jw & 1, g2 = jw >> 2;
      const int strip = GLU ? kb * 8 + 4 * g2 + 2 * hi : kb * 8 + 4 * hi;
      dma16_buf<true>(wbuf[g2], wofs, i * 16384 + strip * 1024, base + SA + jw * THREADS * 8);
    }
  };
  // Fragment r of the 16 of a k-block in order of use: the first A row tile, the W
  // strips, the other row tiles.
  bf16x8 fa[2][MT], fb[2][NT];
  auto read1 = [&](int b, int h, int r) {
    const uint16_t* p = stage_ptr(b);
    if (r == 0)
      fa[h][0] = *(const bf16x8*)(p + aoff[h]);
    else if (r <= NT)
      fb[h][r - 1] = *(const bf16x8*)(p + woff + h * 4096 + (r - 1) * 512);
    else
      fa[h][r - NT] = *(const bf16x8*)(p + aoff[h] + (r - NT) * 1024);
  };
  auto mma1 = [&](int h, int x) {
    const int i = x / NT, j = x % NT;
    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[h][i], fb[h][j], acc[i][j], 0, 0, 0);
  };
  // Stage st, in slot b, its first k-block's fragments already in registers.  First
  // half: multiply them and read the second k-block's.  Then this wave is done with
  // the slot and, with its loads in flight at zero, its part of stage st + 1 has
  // landed; behind the barrier that holds for all waves.  Second half: multiply,
  // read the first fragments of stage st + 1 and refill the slot with stage st + 2
  // (both clamped to the last stage: what the clamped ones bring is not used).
  const int last = n_stages - 1;
  auto stage = [&](int st, int b) {
#pragma unroll
    for (int x = 0; x < MT * NT; ++x) {
      mma1(0, x);
      if (x % 3 == 0 && x / 3 < MT + NT) read1(b, 1, x / 3);
      __builtin_amdgcn_sched_barrier(0);
    }
    wait_vmem<0>();
    wg_barrier();
    __builtin_amdgcn_sched_barrier(0);
    const int pre = min(st + 2, last);
#pragma unroll
    for (int x = 0; x < MT * NT; ++x) {
      mma1(1, x);
      if (x % 3 == 0 && x / 3 < LPS) issue1(pre, b, x / 3);
      if (x % 3 == 1 && x / 3 < MT + NT) read1(b ^ 1, 0, x / 3);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto fill = [&](int b) {  // stage 0 into slot b, stage 1 into the other; the first fragments
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int j = 0; j < LPS; ++j) issue1(s, b ^ s, j);
    wait_vmem<LPS>();
    wg_barrier();
#pragma unroll
    for (int r = 0; r < MT + NT; ++r) read1(b, 0, r);
  };
  // An odd number of stages runs the first ahead of the loop in slot 1, which leaves
  // the loop whole turns of the ring and one exit (with a tail behind it the
  // compiler moves accumulators between registers on every turn).
  int st = n_stages & 1;
  if (st) {
    fill(1);
    stage(0, 1);
  } else {
    fill(0);
  }
  do {
    stage(st, 0);
    stage(st + 1, 1);
    st += 2;
  } while (st < n_stages);
  wait_vmem<0>();  // no LDS write may still be in flight when the group ends

  if constexpr (GLU) {
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int p = 0; p < NT / 2; ++p) {
        const int col = col0 + p * 16 + c16;
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
          const int row = m_blk + wm * 128 + i * 16 + 4 * q4 + rr;
          if (row < M && col < col_end)
            glu_out[(int64_t)row * N + col] =
                f32_to_bf16(silu_mul(acc[i][2 * p][rr], acc[i][2 * p + 1][rr]));
        }
      }
  } else {
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        const int col = col0 + j * 16 + c16;
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
          const int row = m_blk + wm * 128 + i * 16 + 4 * q4 + rr;
          if (row < M && col < col_end) out[(int64_t)row * N + col] = acc[i][j][rr];
        }
      }
  }
}

// fp32 weights are row-major [N][K] (the packed layout is for bf16 only).
__device__ __forceinline__ const void* seg_row(const WSegs& w, int n, int64_t row_elems,
                                               int elem_bytes) {
  int start = 0;
  for (int s = 0; s < w.n_seg; ++s) {
    if (n < w.row_end[s])
      return (const char*)w.ptr[s] + (int64_t)(n - start) * row_elems * elem_bytes;
    start = w.row_end[s];
  }
  return w.ptr[0];
}

// fp32: 32 x 64 tiles through LDS, 2 x 4 outputs per thread.
__global__ __launch_bounds__(256) void gemm_f32_tiled(int M, int N, int K, int k_split,
                                                      const float* __restrict__ A, int64_t lda,
                                                      WSegs w, float* __restrict__ out) {
  __shared__ float As[16][33];
  __shared__ float Ws[16][65];
  const int tid = threadIdx.x;
  const int m0 = blockIdx.y * 32, n0 = blockIdx.x * 64;
  const int kbeg = blockIdx.z * k_split;
  const int kend = min(K, kbeg + k_split);
  const int tm = tid >> 4, tn = tid & 15;
  float acc[2][4] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
  for (int k0 = kbeg; k0 < kend; k0 += 16) {
    for (int e = tid; e < 32 * 16; e += 256) {
      const int mm = e >> 4, kk = e & 15, row = m0 + mm, k = k0 + kk;
      As[kk][mm] = (row < M && k < kend) ? A[(int64_t)row * lda + k] : 0.f;
    }
    for (int e = tid; e < 64 * 16; e += 256) {
      const int nn = e >> 4, kk = e & 15, n = n0 + nn, k = k0 + kk;
      Ws[kk][nn] = (n < N && k < kend) ? ((const float*)seg_row(w, n, K, 4))[k] : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
      const float a0 = As[kk][tm * 2], a1 = As[kk][tm * 2 + 1];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float b = Ws[kk][tn * 4 + j];
        acc[0][j] += a0 * b;
        acc[1][j] += a1 * b;
      }
    }
    __syncthreads();
  }
  float* o = out + (int64_t)blockIdx.z * M * N;
  for (int i = 0; i < 2; ++i)
    for (int j = 0; j < 4; ++j) {
      const int row = m0 + tm * 2 + i, col = n0 + tn * 4 + j;
      if (row < M && col < N) o[(int64_t)row * N + col] = acc[i][j];
    }
}

// The exchange steps of gemm_f32_rows from N values a lane on: lanes with the bit
// keep the upper half.  A recursion over the sizes and not a loop: a loop is
// unrolled after the array has become an indexed one, where every select of two
// elements is a chain over all of them (32 values: 13 us at 16 rows of the small
// decoder's gate/up, 4.1 now; its step, 4 rows, 99 / 80).
template <int N, int V>
__device__ __forceinline__ void halve_values(float (&v)[V], int lane) {
  if constexpr (N > 1) {
    constexpr int half = N / 2, bit = 32 * N / V;
    const bool up = lane & bit;
#pragma unroll
    for (int i = 0; i < half; ++i) {
      const float lo = v[i], hi = v[i + half];
      v[i] = (up ? hi : lo) + __shfl_xor(up ? lo : hi, bit, 64);
    }
    halve_values<half>(v, lane);
  }
}

// fp32, up to 16 rows: a wave owns NC columns and every row (MP >= M), its lanes
// take K in steps of 256 (four elements of each weight row and activation row), and
// the NC * MP lane sums are reduced together: each of the first log2(NC * MP)
// exchange steps halves the number of values a lane carries, so 16 values cost
// 17 exchanges instead of 96, and lane i ends with one finished value.  One wave
// per work group and no K split: these products are latency (the tiled kernel's
// loop of loads, barriers and 16-deep products took 11.6 us on average for the
// small decoder's projections, 4 rows, plus the split sums in its consumers;
// this takes 3.1).  GLU: NC columns of the gate matrix and of the up matrix,
// gate in the lower half of the values, so the halves of the wave end with g and
// up of the same outputs and one more exchange gives silu(g) * up.
template <int NC, int MP, bool GLU>
__global__ __launch_bounds__(64) void gemm_f32_rows(int M, int N, int K,
                                                    const float* __restrict__ A, int64_t lda,
                                                    WSegs w, float* __restrict__ out) {
  constexpr int NW = GLU ? 2 * NC : NC, V = NW * MP;
  const int lane = threadIdx.x, n0 = blockIdx.x * NC;
  const float* wr[NW];
#pragma unroll
  for (int c = 0; c < NW; ++c) {
    const int n = min(n0 + c % NC, N - 1);  // columns past N are computed, not written
    wr[c] = GLU ? (const float*)w.ptr[c / NC] + (int64_t)n * K
                : (const float*)seg_row(w, n, K, 4);
  }
  float v[V];
#pragma unroll
  for (int i = 0; i < V; ++i) v[i] = 0.f;
#pragma unroll 2
  for (int k = lane * 4; k < K; k += 256) {  // K % 4 == 0
    f32x4_any a[MP], b[NW];
#pragma unroll
    for (int c = 0; c < NW; ++c) b[c] = *(const f32x4_any*)(wr[c] + k);
#pragma unroll
    for (int m = 0; m < MP; ++m)
      a[m] = *(const f32x4_any*)(A + (int64_t)min(m, M - 1) * lda + k);
#pragma unroll
    for (int c = 0; c < NW; ++c)
#pragma unroll
      for (int m = 0; m < MP; ++m) {
        float s = v[c * MP + m];
        s = fmaf(a[m].x, b[c].x, s);
        s = fmaf(a[m].y, b[c].y, s);
        s = fmaf(a[m].z, b[c].z, s);
        v[c * MP + m] = fmaf(a[m].w, b[c].w, s);
      }
  }
  halve_values<V>(v, lane);
  float r = v[0];
#pragma unroll
  for (int b = 32 / V; b > 0; b /= 2) r += __shfl_xor(r, b, 64);
  const int idx = lane / (64 / V);  // this lane's value: column idx / MP, row idx % MP
  if constexpr (GLU) {
    const float u = __shfl_xor(r, 32, 64);
    r = r / (1.f + expf(-r)) * u;  // in the lower half of the wave
  }
  const int c = idx / MP, m = idx % MP, n = n0 + c;
  if (lane % (64 / V) == 0 && c < NC && n < N && m < M) out[(int64_t)m * N + n] = r;
}

}  // namespace

// Kernel choice for bf16, from measurements on the 8B projection shapes:
//  * M <= 32: the streaming kernel (two strips per wave, ring depth 2), or the
//    strip kernel (strip_form);
//    6.0-6.6 TB/s of weights up to M = 16;
//  * larger M: the 64- to 256-row tiles (plan_tile), and above 256 rows the
//    256 x 256 tile where its grid fills the GPU.
constexpr int kStreamMaxRows = 32;

// Row tiles of the 128-column kernel: 64, 128, 192 or 256 rows, so that up to 256
// rows W is read once per step by the smallest tile that holds the batch.
// Measured (us, against the 128-row tile up to 128 rows and the 256-row tile above):
// gate/up 40.9 / 44.4 at 64 rows, 58.9 / 63.8 at 192, down 37.0 / 39.9 at 160.  Up
// to 64 rows a long K split over the grid (down: 28 k-steps of 64 per work group) is
// 2-3% faster on the 128-row tile.
//
// Above 256 rows (kRowStep steps) the tile and the K splits are chosen together.
// The grid rarely fills whole rounds of the 256 CUs, and what a round costs is
// close to linear in the tile's rows; over 300-2048 rows of qkv, o and down of the
// 8B shape, and all three tiles, the times follow within about 5%
//   (24 + 0.165 rows) K / 4096 us per full round, a last round filled by p
//   counting 0.58 + 0.4 p, divided by the splits,
// plus the splits' partial sums written and read at about 5 TB/s.  Against
// 256-row tiles with the splits planned alone: qkv 97.7 / 108.3 at 1400 rows (two
// rounds of 192 instead of one and an eighth of 256), 44.6 / 52.1 at 600 (128-row
// tiles), down 174 / 191 at 1400 and 60.7 / 68.3 at 300.  Not everywhere: o at 2048
// rows, one full round of 256-row tiles either way, takes 65-69 us where 65.1 was
// measured before the loads were spread.
//
// The 256 x 256 tile enters the same comparison, unsplit and at 102 us a round (o of
// the 8B shape at 4096 rows, one round: 102 us; 115 on eight waves of 64 x 128), from
// two k-steps of 64 on, which its ring of stages needs.  Taken where that is
// estimated less: gate/up and the LM head at most row counts, qkv of the 8B shape
// at 2048 rows (192 tiles, 98 us against 125 on 128-column tiles) and 4096 (194 /
// 215), down of the 14B shape at 2048 (350 / 443).  Left where it would leave most
// CUs idle (o, down, qkv below about 1200 rows) and at gate/up of the 14B shape
// with 300 rows, 272 wide tiles: 183 us on 128-column tiles, 273 on wide ones.
struct TilePlan {
  int rows, splits;  // rows of the 128-column tile
  bool wide;         // the 256 x 256 tile instead (splits = 1)
};
constexpr int kRowStep = 64;  // above 256 rows the plan is the same within a step
// Rounds of 256 work groups that n cost.
double grid_rounds(int64_t n) {
  return (double)(n / 256) + (n % 256 ? 0.58 + 0.4 * (double)(n % 256) / 256 : 0.0);
}
TilePlan plan_tile(int M, int K, int64_t groups, bool glu, bool may_widen) {
  if (M <= 256) {
    // One round of work groups: a partial second one costs 15-30%.
    const int splits = (int)std::min<int64_t>(8, std::max<int64_t>(1, 256 / groups));
    const int rows = M <= 64 && (glu || splits == 1 || K < 8192) ? 64
                     : M <= 128                                  ? 128
                     : M <= 192                                  ? 192
                                                                 : 256;
    return {rows, splits, false};
  }
  const int m = (M + kRowStep - 1) / kRowStep * kRowStep;
  TilePlan best{256, 1, false};
  double least = 1e30;
  const int64_t wide = (groups + 1) / 2 * ((m + 255) / 256);
  if (may_widen && K >= 128) {
    least = grid_rounds(wide) * 102 * K / 4096;
    best.wide = true;
  }
  for (int rows = 256; rows >= 128; rows -= 64) {
    const int64_t tiles = groups * ((m + rows - 1) / rows);
    for (int s = 1; s <= 8 && (s == 1 || tiles * s <= 1024); ++s) {
      const double us = grid_rounds(tiles * s) * (24 + 0.165 * rows) * K / 4096 / s +
                        (s - 1) * (double)m * (double)groups * kGroupCols * 8 / 5e6;
      if (us < least * (best.wide ? 0.95 : 0.99)) least = us, best = {rows, s, false};
    }
  }
  return best;
}

// Where the strip kernel takes a projection: its strips fit the 256 CUs once
// (320 strips, 5120 columns, left a quarter of the CUs two: 13.5 us against 12.1
// at one row) and the activations every work group reads, M * K * 2 bytes, stay
// under 256 KiB (down of the 8B shape, K 14336, us against the streaming kernel
// and its split sum: 20.2 / 22.2 at 1 row, 21.7 / 22.8 at 8, 24.4 / 23.1 at 12).
static bool strip_form(int M, int K, int64_t groups) {
  return M <= 16 && groups <= 32 && (int64_t)M * K <= 131072;
}

// The fp32 kernel for few rows reads four elements of weight and activation rows
// at a time, whatever their alignment (the split count is planned from the shape
// alone); above 16 rows its per-wave weight reads would be repeated by more waves
// than the tiled kernel's.
constexpr int kF32RowsMax = 16;
static bool f32_rows_shape(int M, int K) { return M <= kF32RowsMax && K % 4 == 0; }

int gemm_plan_splits(int dtype, int M, int N, int K, int* k_split, bool glu) {
  const int kq = (dtype == 1) ? 64 : 16;
  const int ksteps = (K + kq - 1) / kq;
  int s = 1;
  if (dtype == 1) {
    // Work groups per split: one per 128-column group (times the M-blocks).
    int64_t groups = (N + kGroupCols - 1) / kGroupCols;
    if (!glu && strip_form(M, K, groups)) {  // K is split inside its work groups
      *k_split = K;
      return 1;
    }
    if (M > kStreamMaxRows)
      s = plan_tile(M, K, groups, glu, true).splits;
    else  // one round of work groups, as above
      s = (int)std::min<int64_t>(8, std::max<int64_t>(1, 256 / groups));
  } else {
    const int64_t groups = (int64_t)((N + 63) / 64) * ((M + 31) / 32);
    if (f32_rows_shape(M, K))
      s = 1;  // gemm_f32_rows
    else if (groups < 512) s = (int)std::min<int64_t>((512 + groups - 1) / groups, 8);
  }
  s = std::max(1, std::min(s, ksteps));
  const int steps_per = (ksteps + s - 1) / s;
  *k_split = steps_per * kq;
  return (K + *k_split - 1) / *k_split;
}

hipError_t launch_pack_weight(int dtype, int N, int K, const void* w, void* packed,
                              hipStream_t stream) {
  if (N <= 0 || K <= 0) return hipSuccess;
  if (dtype != 1)
    return hipMemcpyAsync(packed, w, (size_t)N * K * 4, hipMemcpyDeviceToDevice, stream);
  const int64_t chunks = (int64_t)((N + kGroupCols - 1) / kGroupCols) * (K / 32) * 8 * 64;
  pack_weight_kernel<<<(unsigned)((chunks + 255) / 256), 256, 0, stream>>>(
      (const uint16_t*)w, N, K, (uint16_t*)packed);
  return hipGetLastError();
}

namespace {

// The bf16 kernels over n_groups column groups (GLU: half-groups).
template <bool GLU>
hipError_t launch_gemm_bf16(int M, int N, int K, const uint16_t* a, int64_t lda, const WSegs& w,
                            int n_groups, float* out, uint16_t* glu_out, int splits, int k_split,
                            hipStream_t stream, hipEvent_t ev_start, hipEvent_t ev_stop) {
  if constexpr (!GLU) {
    if (splits == 1 && strip_form(M, K, n_groups))
      return launch_timed(gemm_bf16_strip, dim3(n_groups * 8), dim3(64 * kStripWaves), stream,
                          ev_start, ev_stop, M, N, K, a, lda, w, out);
  }
  if (M <= kStreamMaxRows) {
    const dim3 grid(n_groups, 1, splits);
    if (M <= 16)
      return launch_timed(gemm_bf16_stream<1, 2, GLU>, grid, dim3(256), stream, ev_start,
                          ev_stop, M, N, K, k_split, a, lda, w, out, glu_out);
    return launch_timed(gemm_bf16_stream<2, 2, GLU>, grid, dim3(256), stream, ev_start, ev_stop,
                        M, N, K, k_split, a, lda, w, out, glu_out);
  }
  const TilePlan plan = plan_tile(M, K, n_groups, GLU, splits == 1);
  if (plan.wide) {
    // GLU: n_groups counts half-groups; a wide column tile is one whole group.
    const int n_mb = (M + 255) / 256, n_nb = GLU ? n_groups / 2 : (n_groups + 1) / 2;
    // Columns by XCD alone would give each fewer than four: two halves of the
    // M-blocks keep its share of the grid near square.
    const int row_x = n_mb >= 2 * kBandRows && n_mb % 2 == 0 && n_nb < 32 ? 2 : 1;
    const int cols_x = 8 / row_x;
    const dim3 grid(8 * ((n_nb + cols_x - 1) / cols_x) * (n_mb / row_x));
    return launch_timed(gemm_bf16_wide<GLU>, grid, dim3(256), stream, ev_start, ev_stop, M, N, K,
                        n_mb, n_nb, row_x, n_groups, a, lda, w, out, glu_out);
  }
  const int rows = plan.rows;
  const int n_mb = (M + rows - 1) / rows, n_nb = n_groups;
  const dim3 grid(((n_nb + 7) / 8) * 8 * n_mb, 1, splits);
#define PDEC_TILE(ROWS_, MT_, D_)                                                              \
  return launch_timed(gemm_bf16_tile<ROWS_, MT_, D_, GLU>, grid, dim3(8 * ROWS_ / MT_), stream, \
                      ev_start, ev_stop, M, N, K, k_split, n_mb, n_nb, a, lda, w, out, glu_out)
  if (rows == 64) PDEC_TILE(64, 2, 6);
  if (rows == 128) PDEC_TILE(128, 4, 3);
  if (rows == 192) PDEC_TILE(192, 4, 3);
  PDEC_TILE(256, 4, 3);
#undef PDEC_TILE
}

}  // namespace

namespace {

// The fused gate/up grid has one work group per half column-group of both
// matrices (up to 256 rows: one M-block).  When that count is whole rounds
// of the 256 CUs plus a last round at most half full (F = 17408: 272
// half-groups), the last round runs nearly as long as a full one while most
// CUs idle: at K = 5120 and 128 rows, 272 half-groups took 112 us against
// 70 us for 256.  Those tail columns then take the plain kernels with their
// K axis split (up to 16 ways, so that the tail fills one round of short
// work groups) and a SwiGLU pass over the summed partials.
struct GluPlan {
  int fused_halves;  // half-groups of the fused launch (a multiple of 256 when split)
  int tail_halves;   // half-groups left to the split launch (0: none)
  int splits, k_split;
};

GluPlan plan_glu(int M, int F, int K) {
  const int halves = 2 * ((F + kGroupCols - 1) / kGroupCols);
  GluPlan p{halves, 0, 1, K};
  const int tail = halves % 256;
  if (M > 256 || halves < 256 || tail == 0 || tail > 128) return p;
  const int ksteps = K / 64, want = std::min(16, 256 / tail);
  const int per = (ksteps + want - 1) / want;  // k-steps of 64 per split
  const int splits = (ksteps + per - 1) / per;
  if (splits < 2) return p;
  return {halves - tail, tail, splits, per * 64};
}

}  // namespace

int64_t swiglu_tail_part_elems(int M, int F, int K) {
  const GluPlan g = plan_glu(M, F, K);
  if (g.tail_halves == 0) return 0;
  const int64_t ft = F - (int64_t)(g.fused_halves / 2) * kGroupCols;  // tail columns per matrix
  return (int64_t)g.splits * M * 2 * ft;
}

hipError_t launch_gemm_swiglu(int M, int F, int K, const void* A, int64_t lda, const void* w_gate,
                              const void* w_up, void* u, float* tail_part, hipStream_t stream,
                              hipEvent_t ev_start, hipEvent_t ev_stop) {
  if (M <= 0 || F <= 0) return hipSuccess;
  WSegs w{};
  w.ptr[0] = w_gate;
  w.ptr[1] = w_up;
  w.row_end[0] = F;
  w.row_end[1] = 2 * F;
  w.n_seg = 2;
  const GluPlan g = plan_glu(M, F, K);
  if (g.tail_halves == 0 || !tail_part)
    return launch_gemm_bf16<true>(M, F, K, (const uint16_t*)A, lda, w, 2 * ((F + 127) / 128),
                                  nullptr, (uint16_t*)u, 1, K, stream, ev_start, ev_stop);
  // Whole groups [0, g0) of both matrices fused; groups [g0, ...) split.
  hipError_t e = launch_gemm_bf16<true>(M, F, K, (const uint16_t*)A, lda, w, g.fused_halves,
                                        nullptr, (uint16_t*)u, 1, K, stream, ev_start, nullptr);
  if (e != hipSuccess) return e;
  const int g0 = g.fused_halves / 2, ft = F - g0 * kGroupCols, tg = (ft + kGroupCols - 1) / kGroupCols;
  WSegs t{};
  t.ptr[0] = (const uint16_t*)w_gate + (int64_t)g0 * kGroupCols * K;
  t.ptr[1] = (const uint16_t*)w_up + (int64_t)g0 * kGroupCols * K;
  t.row_end[0] = ft;
  t.row_end[1] = 2 * ft;
  t.grp_end[0] = tg;
  t.grp_end[1] = 2 * tg;
  t.n_seg = 2;
  e = launch_gemm_bf16<false>(M, 2 * ft, K, (const uint16_t*)A, lda, t, 2 * tg, tail_part, nullptr,
                              g.splits, g.k_split, stream, nullptr, nullptr);
  if (e != hipSuccess) return e;
  e = launch_swiglu(1, M, ft, tail_part, g.splits, (uint16_t*)u + (int64_t)g0 * kGroupCols, stream,
                    F);
  if (e == hipSuccess && ev_stop) e = hipEventRecord(ev_stop, stream);
  return e;
}

namespace {

// 16 lane values per wave (8 columns of one row, 4 of up to four rows, ...).
template <bool GLU>
hipError_t launch_f32_rows(int M, int N, int K, const float* A, int64_t lda, const WSegs& w,
                           float* out, hipStream_t stream, hipEvent_t ev_start,
                           hipEvent_t ev_stop) {
#define PDEC_F32_ROWS(NC_, MP_)                                                                \
  return launch_timed(gemm_f32_rows<NC_, MP_, GLU>, dim3((N + NC_ - 1) / NC_), dim3(64), stream, \
                      ev_start, ev_stop, M, N, K, A, lda, w, out)
  if (M == 1) PDEC_F32_ROWS(4, 1);
  if (M == 2) PDEC_F32_ROWS(4, 2);
  if (M <= 4) PDEC_F32_ROWS((GLU ? 2 : 4), 4);
  if (M <= 8) PDEC_F32_ROWS(2, 8);
  PDEC_F32_ROWS(1, 16);
#undef PDEC_F32_ROWS
}

}  // namespace

bool launch_gemm_f32_swiglu(int M, int F, int K, const float* A, const float* w_gate,
                            const float* w_up, float* u, hipStream_t stream, hipError_t* err,
                            hipEvent_t ev_start, hipEvent_t ev_stop) {
  *err = hipSuccess;
  if (!f32_rows_shape(M, K)) return false;
  WSegs w{};
  w.ptr[0] = w_gate;
  w.ptr[1] = w_up;
  w.row_end[0] = F;
  w.row_end[1] = 2 * F;
  w.n_seg = 2;
  *err = launch_f32_rows<true>(M, F, K, A, K, w, u, stream, ev_start, ev_stop);
  return true;
}

hipError_t launch_gemm(int dtype, int M, int N, int K, const void* A, int64_t lda,
                       const WSegs& w_in, float* out, int splits, int k_split, hipStream_t stream,
                       hipEvent_t ev_start, hipEvent_t ev_stop) {
  if (M <= 0 || N <= 0) return hipSuccess;
  const dim3 block(256);
  if (dtype == 1) {
    // Each segment is padded to whole groups; count them.
    WSegs w = w_in;
    int start = 0, n_groups = 0;
    for (int s = 0; s < w.n_seg; ++s) {
      n_groups += (w.row_end[s] - start + kGroupCols - 1) / kGroupCols;
      w.grp_end[s] = n_groups;
      start = w.row_end[s];
    }
    return launch_gemm_bf16<false>(M, N, K, (const uint16_t*)A, lda, w, n_groups, out, nullptr,
                                   splits, k_split, stream, ev_start, ev_stop);
  } else {
    if (splits == 1 && f32_rows_shape(M, K))
      return launch_f32_rows<false>(M, N, K, (const float*)A, lda, w_in, out, stream, ev_start,
                                    ev_stop);
    const dim3 grid((N + 63) / 64, (M + 31) / 32, splits);
    return launch_timed(gemm_f32_tiled, grid, block, stream, ev_start, ev_stop, M, N, K, k_split,
                        (const float*)A, lda, w_in, out);
  }
  return hipGetLastError();
}

}  // namespace pdec
