// Red cells and direct (Toeplitz) gray tiles of the relaxed online
// convolution, for gfx950.
//
// Layout: state S[m][t][c] with c = b*D + d (time-major, one B*D slab per
// position and layer), filters Hf[m][k][d] (lag-major).  A thread owns one
// column (m, c): every element it writes has no other writer in the launch,
// so results are deterministic and no atomics are used.  Consecutive threads
// take consecutive c, so every row access of a wavefront is one contiguous
// 256-byte segment.
//
// Red cell (Alg. 1 red line, Alg. 3 inner loop): z_t = fmaf(h_0, y_t, acc_t),
// then the slot of position t is overwritten with y_t (the in-place storage
// of Sec. 3.3: b^l_t lives in a^l_t's slot until it is consumed).
//
// Gray tile (Eq. taus) for i = t+1, side U: for j < dst_len,
//   S[i+j] += sum_{k<U} y[i-U+k] * h[U+j-k]     (lags 1..2U-1).
#include <type_traits>
#include <utility>

#include "lcsm_internal.h"

namespace lcsm {
namespace {

constexpr int kThreads = 256;

// Output split of the fused tile: SPLIT threads share one column, each
// computing U/SPLIT of the U outputs (bounds the per-thread work and
// registers at the larger fused sides).
template <int U>
struct Split {
  static constexpr int value = U >= 64 ? 8 : (U >= 32 ? 4 : (U >= 16 ? 2 : 1));
};

// RED: do the red cell at position t first (the tile's newest input y_t then
// comes from the register, not from memory).  U == 0: no tile.
// 1 <= U <= kFusedMaxU: the tile i = t+1 (U outputs from U inputs and 2U-1
// lags) is computed by SPLIT threads per column, thread part p taking the
// outputs j in [p U/SPLIT, (p+1) U/SPLIT); part 0 also does the red cell.
// Every load (inputs, lags, the red cell's accumulator and the tile's
// destination accumulators) is issued before the first store, so the step
// costs one memory round trip; the slots read and written are distinct rows.
// Grid (channel blocks, B, M * SPLIT): no integer division on the critical
// path, consecutive lanes take consecutive channels.  With a channel-block
// count that is not a multiple of 8 the batch rows of one block run on
// different XCDs, and each XCD's L2 fetches the same lag rows.  Remapping the
// workgroup ids so that they share one XCD removes those reads, but its
// integer divisions ahead of the first load cost about 0.5 us per launch on
// these latency-bound steps (a 32768-position, 18-layer generation: 135 ->
// 151 ms), so the grid keeps the hardware order.
//
// These launches last 2 to 3 us, of which a good part passes before the first
// load: the host hands over what it knows (St = row t of layer 0, the layer
// strides), lanes past D load column D - 1 instead of leaving early (one wait for
// the arguments instead of two), rows and the layer's pointers are uniform, so
// that an address is a scalar base and the lane's 32-bit offset, and FULL (the
// destination not clipped: every row and lag exists) needs no clamping.  Same
// box, before and after: 8192 positions of 6144 columns 20.46 -> 19.91 ms, 65536 of
// 18432 columns 207.9 -> 204.4, 32768 of 55296 columns 126.7 -> 125.2.
template <int U, bool RED, bool FULL>
__global__ __launch_bounds__(kThreads) void k_step_fused(const float* __restrict__ y,
                                                        float* __restrict__ z,
                                                        float* __restrict__ St,
                                                        const float* __restrict__ Hf, size_t ls,
                                                        size_t hls, int BD, int D, int rows,
                                                        int lags) {
  constexpr int SP = U > 0 ? Split<U>::value : 1;
  constexpr int UJ = U > 0 ? U / SP : 1;  // outputs per thread
  const unsigned c0 = blockIdx.x * kThreads, left = (unsigned)D - c0;
  const bool live = threadIdx.x < left;
  const unsigned off = 4 * (live ? threadIdx.x : left - 1);  // bytes, below 4 kThreads
  auto at = [&](const float* base) -> float& {
    return *reinterpret_cast<float*>(reinterpret_cast<char*>(const_cast<float*>(base)) + off);
  };
  const int m = SP > 1 ? (int)blockIdx.z / SP : (int)blockIdx.z;
  const int part = SP > 1 ? (int)blockIdx.z - m * SP : 0;
  const int j0 = part * UJ;
  const unsigned bc = blockIdx.y * (unsigned)D + c0;  // below B D
  const size_t slab = (size_t)m * BD + bc;
  float* row0 = St + (size_t)m * ls + bc;  // row t
  const float* hc = Hf + (size_t)m * hls + c0;
  auto row = [&](int k) -> float& { return at(row0 + (long long)k * BD); };

  constexpr int NY = U > 0 ? U : 1;
  constexpr int NH = U > 0 ? UJ + U : 1;  // lags j0+1 .. j0+UJ+U-1 at hh[1..]
  float yb[NY];
  float hh[NH];
  float zo[UJ];
  const bool red = RED && part == 0;
  // Every load is unconditional, with its row or lag clamped into range
  // (values past the end are never used): loads under a condition are issued
  // only after the earlier ones have returned, a second round trip per step.
  // rows, lags: how many rows after t and lags there are (the tile's outputs
  // are the first min(U, rows)); the arguments fill one line of 64 bytes.
  float yt, acc = 0.f, h0 = 0.f;
  if constexpr (RED) {
    yt = at(y + slab);
    acc = row(0);
    h0 = at(hc);
  } else {
    yt = row(0);
  }
  if constexpr (U > 0) {
    // rows t+1-U .. t-1 already hold inputs (U divides t+1); row t is y_t
#pragma unroll
    for (int k = 0; k < U - 1; ++k) yb[k] = row(1 - U + k);
    // output j uses lags U+j-k, k < U: for j in [j0, j0+UJ) that is j0+1 .. j0+UJ+U-1
#pragma unroll
    for (int l = 1; l < UJ + U; ++l) {
      const int lag = j0 + l;
      const float v = at(hc + (size_t)(FULL || lag < lags ? lag : lags - 1) * D);
      hh[l] = FULL || lag < lags ? v : 0.f;
    }
#pragma unroll
    for (int jj = 0; jj < UJ; ++jj) {
      const int r = 1 + j0 + jj;
      zo[jj] = row(FULL || r <= rows ? r : rows);
    }
  }
  // Pin every loaded value here, after the last load (an empty statement
  // that reads and writes each register): no load is sunk into the
  // conditional red-cell or tile blocks below, and all of them are in flight
  // together.  The tile's values only up to U = 16: with the 80 and more
  // values of the larger tiles held at once the compiler issues the loads in
  // small groups instead.
  constexpr bool PIN = U <= 16;
  // y_t as well without the red cell: with nothing pinned there, the tile of
  // U = 32 issued its lag loads one round trip each
  if constexpr (RED)
    asm volatile("" : "+v"(acc), "+v"(h0), "+v"(yt));
  else
    asm volatile("" : "+v"(yt));
  if constexpr (U > 0 && PIN) {
#pragma unroll
    for (int l = 1; l < UJ + U; ++l) asm volatile("" : "+v"(hh[l]));
#pragma unroll
    for (int jj = 0; jj < UJ; ++jj) asm volatile("" : "+v"(zo[jj]));
#pragma unroll
    for (int k = 0; k < U - 1; ++k) asm volatile("" : "+v"(yb[k]));
  }
  if (!live) return;
  if (red) {
    at(z + slab) = fmaf(h0, yt, acc);
    row(0) = yt;
  }
  if constexpr (U > 0) {
    yb[U - 1] = yt;
#pragma unroll
    for (int jj = 0; jj < UJ; ++jj) {
      if (FULL || j0 + jj < rows) {
        float o = 0.f;
#pragma unroll
        for (int k = 0; k < U; ++k) o = fmaf(yb[k], hh[U + jj - k], o);
        row(1 + j0 + jj) = zo[jj] + o;
      }
    }
  }
}

// The chain's input rule y = x + 0.5 tanh(z), evaluated as (x + 1/2) - r,
// r = 1/(1 + e^{2z}) (the same function: 0.5 tanh(z) = 1/2 - r), from the
// hardware base-2 exponential and reciprocal (each within about one ulp): no
// branch, and x + 1/2 is off the serial chain.  Absolute error of y below 3.3e-7
// for |x| <= 3 (an fp32 model of these steps with both hardware results off by
// one ulp either way, against fp64, on 1.2M points with z over [-20, 20] and 1e-8
// .. 32 of either sign); z = +inf gives x + 1/2, z = -inf x - 1/2, NaN stays NaN.
// What runs from layer to layer and position to position is the rounded z that is
// handed out: carrying 2 log2(e) z = B y + A with scaled taps and accumulators
// saves the chain one multiplication (1.515 against 1.524 ms for 1024 positions
// of 18 layers x 3072 columns), but rounds each term by itself: y was off by 3e-6
// from the z handed out where h_0 y and the accumulator cancel from 100, by 1.7e-4
// from 10^4, and not a number where only the scaled sum overflows (as it is: below
// 1.5e-7 in all of them).  At t = 0 layer 0's input is x itself: x in place of
// x + 1/2 and r = 0.
__device__ __forceinline__ float chain_r(float z) {
  return __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(2.8853900817779268f * z));  // e^{2z}
}
__device__ __forceinline__ float chain_xh(float x, bool first) { return first ? x : x + 0.5f; }

template <int U>
struct ChainChunk {
  static constexpr int value = U <= 2 ? 8 : (U <= 8 ? 4 : (U <= 16 ? 2 : 1));
};

template <int U, int K>
__global__ __launch_bounds__(kThreads) void k_chain_fused(const float* __restrict__ x,
                                                         float* __restrict__ z,
                                                         float* __restrict__ S,
                                                         const float* __restrict__ Hf,
                                                         float* __restrict__ prev, int M, int L,
                                                         int SL, int BD, int D, int t,
                                                         int dst_len) {
  constexpr int NY = U > 0 ? U : 1;
  constexpr int NH = U > 0 ? 2 * U : 1;
  constexpr int NZ = U > 0 ? U : 1;
  const int d = (int)blockIdx.x * kThreads + (int)threadIdx.x;
  if (d >= D) return;
  const int c = (int)blockIdx.y * D + d;
  const size_t rs = (size_t)BD;
  const bool tile = (U > 0) && (dst_len > 0);
  float zl = 0.f;  // z^{M-1}_{t-1} (loaded with the first chunk), then z^{m-1}_t
  for (int m0 = 0; m0 < M; m0 += K) {
    float xv[K], acc[K], h0[K];
    float yb[K][NY], hh[K][NH], zo[K][NZ];
    // loads of the chunk's layers (past the last layer: layer M-1 again,
    // unused; rows and lags clamped into range)
#pragma unroll
    for (int kk = 0; kk < K; ++kk) {
      const int m = m0 + kk < M ? m0 + kk : M - 1;
      const float* col = S + (size_t)m * SL * BD + c;
      const float* hc = Hf + (size_t)m * L * D + d;
      xv[kk] = x[(size_t)m * BD + c];
      acc[kk] = col[(size_t)t * rs];
      h0[kk] = hc[0];
      if constexpr (U > 0) {
#pragma unroll
        for (int k = 0; k < U - 1; ++k) yb[kk][k] = col[(size_t)(t + 1 - U + k) * rs];
#pragma unroll
        for (int l = 1; l < 2 * U; ++l) {
          const float v = hc[(size_t)(l < L ? l : L - 1) * D];
          hh[kk][l] = l < L ? v : 0.f;
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
          const int row = t + 1 + j;
          zo[kk][j] = col[(size_t)(row < L ? row : L - 1) * rs];
        }
      }
    }
    if (m0 == 0) zl = prev[c];  // unused at t = 0
    // the chain through the chunk, then its stores
#pragma unroll
    for (int kk = 0; kk < K; ++kk) {
      const int m = m0 + kk;
      if (m < M) {
        float* col = S + (size_t)m * SL * BD + c;
        const float yv = (m == 0 && t == 0) ? xv[kk] : (xv[kk] + 0.5f) - chain_r(zl);
        zl = fmaf(h0[kk], yv, acc[kk]);
        z[(size_t)m * BD + c] = zl;
        col[(size_t)t * rs] = yv;
        if constexpr (U > 0) {
          if (tile) {
            yb[kk][U - 1] = yv;
#pragma unroll
            for (int j = 0; j < U; ++j) {
              if (j < dst_len) {
                float o = 0.f;
#pragma unroll
                for (int k = 0; k < U; ++k) o = fmaf(yb[kk][k], hh[kk][U + j - k], o);
                col[(size_t)(t + 1 + j) * rs] = zo[kk][j] + o;
              }
            }
          }
        }
      }
    }
  }
  prev[c] = zl;
}

// The chained steps (lcsm_step_chain) of the positions [t0, t1) of one
// aligned block of kChainBlockW positions (b = t0 rounded down to it), in
// one launch, when every gray tile of the stretch is direct with
// U <= kChainBlockW / 2 (the tile of the last position only when
// tile_last).  Such a tile, of i = b + r + 1 with r + 1 < kChainBlockW,
// reads y rows [i - U, i) and adds into rows [i, i + U), all inside
// [b, b + kChainBlockW): the block's rows of a column stay in that column's
// registers from the first position to the last, and no position of the
// stretch moves a tile's operands through memory.
//
// Every lane that holds a column's block keeps v[k] = state row b + k (y for
// positions already taken, the accumulator otherwise) and the lags 1 ..
// kChainBlockW - 1 of its channel in registers.  The tile arithmetic is that
// of k_step_fused<U, false> (per output, the fmaf chain over the U inputs in
// increasing order, then added to the accumulator), so the results equal the
// per-position steps bit for bit.  At the end the accumulator rows at and
// after t1 (a stretch cut before its block ends) go back to the state.
//
// k_chain_lane, up to kChainLaneMaxM layers: a lane owns one column of every
// layer and walks chain, red cells and tiles alone; nothing is exchanged.
//
// k_chain_block, above: a workgroup owns NC columns.  Wave 0 walks the chain,
// the other waves hold 64 / NC layers each.  What bounds it is the chain, M
// dependent layers per position and nothing beside it, so the layers are cut
// into two halves and a position into two phases: while wave 0 walks one
// half, the waves of the other half take the y it left them, store y and z,
// add the tile's first row (the next accumulator) and hand it over, so that
// wave 0 finds it ready when it comes back.  A phase ends with a
// barrier that orders LDS only (no wave reads global memory another wave of
// the launch writes).  A tile's other rows and the part of the next first row
// that does not need the newest input follow in the phase after, and x is
// loaded kChainXAhead positions ahead.  18 layers x 3072 columns: 49.5 us per
// 32 positions when each position's layer work ran between the chain's end
// and its next start, 28.7 with the phases.
// f(std::integral_constant<int, 0>{}), ..., f(std::integral_constant<int, N-1>{}).
template <class F, int... R>
__device__ __forceinline__ void static_for_impl(F& f, std::integer_sequence<int, R...>) {
  (f(std::integral_constant<int, R>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

__device__ __forceinline__ void chain_block_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The tile of i = b + R + 1 (U = lowbit(R + 1)) on the register rows v, in
// three parts: of its first output row (R + 1, the accumulator the next
// position's chain needs) the sum without the newest input, then that input's
// term, and the rest (rows R + 2 .. R + U).  rem = L - i clips the rows past
// the end.
template <int R>
__device__ __forceinline__ float chain_block_first_part(const float (&v)[kChainBlockW],
                                                        const float (&hh)[kChainBlockW]) {
  constexpr int U = (R + 1) & -(R + 1);
  float o = 0.f;
#pragma unroll
  for (int k = 0; k < U - 1; ++k) o = fmaf(v[R + 1 - U + k], hh[U - k], o);
  return o;
}

template <int R>
__device__ __forceinline__ void chain_block_rest_rows(float (&v)[kChainBlockW],
                                                      const float (&hh)[kChainBlockW], int rem) {
  constexpr int U = (R + 1) & -(R + 1);
#pragma unroll
  for (int j = 1; j < U; ++j) {
    if (j < rem) {
      float o = 0.f;
#pragma unroll
      for (int k = 0; k < U; ++k) o = fmaf(v[R + 1 - U + k], hh[U + j - k], o);
      v[R + 1 + j] = v[R + 1 + j] + o;
    }
  }
}

// Block rows and lags of one column of layer m (column c of the layer, rows
// and lags past the end clamped, the lags zero).
__device__ __forceinline__ void chain_block_load(const float* Sc, const float* hc, size_t rs,
                                                 int D, int L, int b, float (&v)[kChainBlockW],
                                                 float (&hh)[kChainBlockW], float& h0) {
  constexpr int W = kChainBlockW;
#pragma unroll
  for (int k = 0; k < W; ++k) v[k] = Sc[(size_t)(b + k < L ? b + k : L - 1) * rs];
  h0 = hc[0];
  hh[0] = 0.f;
#pragma unroll
  for (int l = 1; l < W; ++l) {
    const float hv = hc[(size_t)(l < L ? l : L - 1) * D];
    hh[l] = l < L ? hv : 0.f;
  }
}

template <int ML>
__global__ __launch_bounds__(64) void k_chain_lane(
    const float* __restrict__ x, size_t xst, int xring, int xs0, float* __restrict__ z,
    size_t zst, int zring, int zs0, float* __restrict__ S, const float* __restrict__ Hf,
    float* __restrict__ prev, int L, int SL, int BD, int D, int t0, int t1, int tile_last) {
  constexpr int W = kChainBlockW;
  const int c = (int)blockIdx.x * 64 + (int)threadIdx.x;
  if (c >= BD) return;
  const int d = c % D;
  const size_t rs = (size_t)BD;
  const int b = t0 & ~(W - 1);
  const int r0 = t0 - b, r1 = t1 - b;
  float v[ML][W], hh[ML][W], h0[ML], xv[ML][W];
  // the block's inputs too, all at once: a position takes less than a load
  {
    int xs = xs0 % xring;
#pragma unroll
    for (int r = 0; r < W; ++r) {
      const bool in = r >= r0 && r < r1;
#pragma unroll
      for (int m = 0; m < ML; ++m) xv[m][r] = x[(size_t)xs * xst + (size_t)m * BD + c];
      if (in && r + 1 < r1) xs = xs + 1 == xring ? 0 : xs + 1;
    }
  }
#pragma unroll
  for (int m = 0; m < ML; ++m)
    chain_block_load(S + (size_t)m * SL * BD + c, Hf + (size_t)m * L * D + d, rs, D, L, b, v[m],
                     hh[m], h0[m]);
  float zl = prev[c];  // z^{M-1}_{t-1}, unused at t = 0
  int zs = zs0 % zring;
  auto position = [&](auto rc) {
    constexpr int r = decltype(rc)::value;
    if (r < r0 || r >= r1) return;
    const int t = b + r;
    const bool tile = r + 1 < W && t + 1 < L && (r + 1 < r1 || tile_last);
#pragma unroll
    for (int m = 0; m < ML; ++m) {
      const bool first = m == 0 && t == 0;
      const float xh = chain_xh(xv[m][r], first);
      const float rr = first ? 0.f : chain_r(zl);
      const float yv = xh - rr;
      zl = fmaf(h0[m], yv, v[m][r]);
      z[(size_t)zs * zst + (size_t)m * BD + c] = zl;
      S[((size_t)m * SL + t) * rs + c] = yv;
      v[m][r] = yv;
      if constexpr (r + 1 < W) {
        if (tile) {
          const float o = fmaf(yv, hh[m][1], chain_block_first_part<r>(v[m], hh[m]));
          v[m][r + 1] = v[m][r + 1] + o;
          chain_block_rest_rows<r>(v[m], hh[m], L - (t + 1));
        }
      }
    }
    zs = zs + 1 == zring ? 0 : zs + 1;
  };
  static_for<W>(position);
  prev[c] = zl;
#pragma unroll
  for (int m = 0; m < ML; ++m)
#pragma unroll
    for (int k = 0; k < W; ++k)
      if (k >= r1 && b + k < L) S[((size_t)m * SL + b + k) * rs + c] = v[m][k];
}

// Layers of the first half: whole waves of LPW layers, at least one in each half.
template <int LPW>
constexpr int chain_half(int M) {
  return (M + LPW) / (2 * LPW) * LPW;
}

// Wave 0 of k_chain_block for M layers known at compile time: the dependent
// chain without a branch in it (with the layer count in a register, a jump per
// layer and half made it 1.3 times slower).  Phase h: half h's layers in order,
// then the barrier.
template <int M, int NC, int HM>
__device__ __forceinline__ float chain_walk(const float2 (*abuf)[NC], const float (*hbuf)[NC],
                                            float (*ybuf)[NC], int col, float zl, bool first,
                                            int n) {
  constexpr int H = chain_half<64 / NC>(M);
  float h0[M];
#pragma unroll
  for (int m = 0; m < M; ++m) h0[m] = hbuf[m < H ? m : HM + m - H][col];
  for (; n > 0; --n) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int m0 = h ? H : 0, m1 = h ? M : H;
      float2 av[HM];
#pragma unroll
      for (int m = m0; m < m1; ++m) av[m - m0] = abuf[h * HM + m - m0][col];
#pragma unroll
      for (int m = m0; m < m1; ++m) {
        float rr = chain_r(zl);
        if (m == 0) rr = first ? 0.f : rr;
        const float yv = av[m - m0].x - rr;
        ybuf[h * HM + m - m0][col] = yv;  // lanes of one column write the same value
        zl = fmaf(h0[m], yv, av[m - m0].y);
      }
      chain_block_sync();
    }
    first = false;
  }
  return zl;
}

// HM: layers of the larger half at most; ML0 .. ML1 the layer counts.
template <int NC, int HM, int ML0, int ML1>
__global__ __launch_bounds__(64 * (1 + (ML1 + 64 / NC - 1) / (64 / NC))) void k_chain_block(
    const float* __restrict__ x, size_t xst, int xring, int xs0, float* __restrict__ z,
    size_t zst, int zring, int zs0, float* __restrict__ S, const float* __restrict__ Hf,
    float* __restrict__ prev, int M, int L, int SL, int BD, int D, int t0, int t1,
    int tile_last) {
  constexpr int W = kChainBlockW, LPW = 64 / NC, XA = kChainXAhead;
  // x + 1/2 and the accumulator of the next position, by half and layer in it
  __shared__ float2 abuf[2 * HM][NC];
  __shared__ float hbuf[2 * HM][NC];   // h_0
  __shared__ float ybuf[2 * HM][NC];   // y of the position taken last
  const int lane = (int)threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int col = lane & (NC - 1);
  const int c = (int)blockIdx.x * NC + col;
  const bool live = c < BD;
  const int cc = live ? c : BD - 1;
  const int b = t0 & ~(W - 1);
  const int r0 = t0 - b, r1 = t1 - b;
  const int H = chain_half<LPW>(M);
  if (wv == 0) {
    __builtin_amdgcn_s_setprio(3);
    float zl = prev[cc];  // z^{M-1}_{t-1}; unused at t = 0
    chain_block_sync();
    auto walk = [&](auto mc) {
      constexpr int MM = ML0 + decltype(mc)::value;
      if (M == MM) zl = chain_walk<MM, NC, HM>(abuf, hbuf, ybuf, col, zl, t0 == 0, r1 - r0);
    };
    static_for<ML1 - ML0 + 1>(walk);
    if (lane < NC && live) prev[c] = zl;
    return;
  }
  const int m = LPW * (wv - 1) + lane / NC;
  const int half = LPW * (wv - 1) >= H ? 1 : 0;  // a wave's layers lie in one half
  const bool has = m < M;
  const int mc = has ? m : M - 1;
  const int slot = half * HM + (mc - (half ? H : 0));
  const int d = cc % D;
  const size_t rs = (size_t)BD;
  float* Sc = S + (size_t)mc * SL * BD + cc;
  const float* xc = x + (size_t)mc * BD + cc;
  float* zc = z + (size_t)mc * BD + cc;
  const bool store = has && live;
  float v[W], hh[W], h0, xq[XA];
  // x of the next XA positions (past the stretch: its last one, unused)
  int xs = xs0 % xring, xt = t0, zs = zs0 % zring;
  auto next_x = [&]() {
    const float xv = xc[(size_t)xs * xst];
    if (++xt < t1) xs = xs + 1 == xring ? 0 : xs + 1;
    return xv;
  };
#pragma unroll
  for (int k = 0; k < XA; ++k) xq[k] = next_x();
  chain_block_load(Sc, Hf + (size_t)mc * L * D + d, rs, D, L, b, v, hh, h0);
  float part = 0.f;
  // what wave 0 needs of position t, its accumulator complete
  auto prepare = [&](int t, float acc, float xv) {
    if (has) abuf[slot][col] = make_float2(chain_xh(xv, mc == 0 && t == 0), acc);
  };
  auto tile_of = [&](int r) { return r + 1 < W && b + r + 1 < L && (r + 1 < r1 || tile_last); };
  auto begin = [&](auto rc) {
    constexpr int r = decltype(rc)::value;
    if (r != r0) return;
    prepare(t0, v[r], xq[0]);
    part = chain_block_first_part<r>(v, hh);
  };
  static_for<W>(begin);
  if (has) hbuf[slot][col] = h0;
  chain_block_sync();
  chain_block_sync();
  if (half) chain_block_sync();
  auto position = [&](auto rc) {
    constexpr int r = decltype(rc)::value;
    if (r < r0 || r >= r1) return;
    const int t = b + r;
    const float yv = ybuf[slot][col];
    const float zv = fmaf(h0, yv, v[r]);
    v[r] = yv;
    if constexpr (r + 1 < W) {
      if (tile_of(r)) v[r + 1] = v[r + 1] + fmaf(yv, hh[1], part);
#pragma unroll
      for (int k = 0; k + 1 < XA; ++k) xq[k] = xq[k + 1];
      prepare(t + 1, v[r + 1], xq[0]);
    }
    if (store) {
      zc[(size_t)zs * zst] = zv;
      Sc[(size_t)t * rs] = yv;
    }
    zs = zs + 1 == zring ? 0 : zs + 1;
    if (r + 1 < r1) {
      xq[XA - 1] = next_x();
      chain_block_sync();
    }
    if constexpr (r + 1 < W) {
      if (tile_of(r)) chain_block_rest_rows<r>(v, hh, L - (t + 1));
      part = chain_block_first_part<r + 1>(v, hh);
    }
    if (r + 1 < r1) chain_block_sync();
  };
  static_for<W>(position);
  if (!half) chain_block_sync();
  if (store) {
#pragma unroll
    for (int k = 0; k < W; ++k)
      if (k >= r1 && b + k < L) Sc[(size_t)(b + k) * rs] = v[k];
  }
}

// Red cell of one layer.
__global__ __launch_bounds__(kThreads) void k_red_layer(const float* __restrict__ y,
                                                       float* __restrict__ z,
                                                       float* __restrict__ Sm,
                                                       const float* __restrict__ Hm, int BD, int D,
                                                       int t) {
  const int c = blockIdx.x * kThreads + threadIdx.x;
  if (c >= BD) return;
  float* p = Sm + (size_t)t * BD + c;
  const float yt = y[c];
  z[c] = fmaf(Hm[c % D], yt, *p);
  *p = yt;
}

// Direct gray tile for U >= J (U a multiple of J): thread = (column c,
// output chunk j0 .. j0+J-1, layer m).  The J lags needed at input k form a
// window that slides down by one per k, so each step loads one input and one
// new lag.
template <int J>
__global__ __launch_bounds__(kThreads) void k_direct_tile(float* __restrict__ S,
                                                         const float* __restrict__ Hf, int L,
                                                         int SL, int BD, int D, int i, int U,
                                                         int dst_len) {
  const int c = blockIdx.x * kThreads + threadIdx.x;
  const int j0 = blockIdx.y * J;
  const int m = blockIdx.z;
  if (c >= BD || j0 >= dst_len) return;
  const int d = c % D;
  const size_t rs = (size_t)BD;
  float* col = S + (size_t)m * SL * BD + c;
  const float* hc = Hf + (size_t)m * L * D + d;

  float acc[J];
  float w[J];  // w[jj] = h[U + j0 + jj - k] at input k
#pragma unroll
  for (int jj = 0; jj < J; ++jj) {
    acc[jj] = 0.f;
    const int lag = U + j0 + jj;
    w[jj] = (lag < L) ? hc[(size_t)lag * D] : 0.f;
  }
  const float* ysrc = col + (size_t)(i - U) * rs;
  for (int k = 0; k < U; ++k) {
    const float yk = ysrc[(size_t)k * rs];
#pragma unroll
    for (int jj = 0; jj < J; ++jj) acc[jj] = fmaf(yk, w[jj], acc[jj]);
#pragma unroll
    for (int jj = J - 1; jj > 0; --jj) w[jj] = w[jj - 1];
    const int lag = U + j0 - k - 1;  // >= j0 >= 0
    w[0] = (k + 1 < U) ? hc[(size_t)lag * D] : 0.f;
  }
  float* dst = col + (size_t)(i + j0) * rs;
#pragma unroll
  for (int jj = 0; jj < J; ++jj)
    if (j0 + jj < dst_len) dst[(size_t)jj * rs] += acc[jj];
}

__global__ __launch_bounds__(kThreads) void k_transpose(const float* __restrict__ src,
                                                       float* __restrict__ dst, int D, int L) {
  // src [D][L] -> dst [L][D] for layer blockIdx.z; 32x32 tiles, padded LDS.
  // Channel tiles on x (up to 2^31 blocks), lag tiles on y (L <= 2^19 gives
  // at most 16384, inside the 65536-block limit of y and z).
  __shared__ float tile[32][33];
  const size_t off = (size_t)blockIdx.z * D * L;
  const int d0 = blockIdx.x * 32, l0 = blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
  for (int r = ty; r < 32; r += 8) {
    const int d = d0 + r, l = l0 + tx;
    if (d < D && l < L) tile[r][tx] = src[off + (size_t)d * L + l];
  }
  __syncthreads();
  for (int r = ty; r < 32; r += 8) {
    const int l = l0 + r, d = d0 + tx;
    if (d < D && l < L) dst[off + (size_t)l * D + d] = tile[tx][r];
  }
}

// Prompt rows in: S[m][t][c] = y[t * ys + m * BD + c] for t < P (grid-stride
// over P * M * BD, consecutive threads on consecutive c).
__global__ __launch_bounds__(kThreads) void k_rows_in(const float* __restrict__ y, size_t ys,
                                                     float* __restrict__ S, int M, int SL, int BD,
                                                     int P) {
  const size_t n = (size_t)P * M * BD, stride = (size_t)gridDim.x * kThreads;
  for (size_t e = (size_t)blockIdx.x * kThreads + threadIdx.x; e < n; e += stride) {
    const size_t tm = e / BD;
    const int c = (int)(e - tm * BD);
    const int m = (int)(tm % M), t = (int)(tm / M);
    S[((size_t)m * SL + t) * BD + c] = y[t * ys + (size_t)m * BD + c];
  }
}

// State rows out: z[t * zs + m * BD + c] = S[m][row0 + t][c], then the state
// entry is cleared, for t < P.
__global__ __launch_bounds__(kThreads) void k_rows_out_clear(float* __restrict__ S, int M, int SL,
                                                            int BD, int row0, int P,
                                                            float* __restrict__ z, size_t zs) {
  const size_t n = (size_t)P * M * BD, stride = (size_t)gridDim.x * kThreads;
  for (size_t e = (size_t)blockIdx.x * kThreads + threadIdx.x; e < n; e += stride) {
    const size_t tm = e / BD;
    const int c = (int)(e - tm * BD);
    const int m = (int)(tm % M), t = (int)(tm / M);
    float* p = S + ((size_t)m * SL + row0 + t) * BD + c;
    z[t * zs + (size_t)m * BD + c] = *p;
    *p = 0.f;
  }
}

__global__ __launch_bounds__(kThreads) void k_zero(float* __restrict__ p, size_t n) {
  const size_t stride = (size_t)gridDim.x * kThreads;
  for (size_t k = (size_t)blockIdx.x * kThreads + threadIdx.x; k < n; k += stride) p[k] = 0.f;
}

// Zero the first n floats of each layer (grid y = layers, grid-stride on x).
__global__ __launch_bounds__(kThreads) void k_zero_rows(float* __restrict__ p, size_t stride,
                                                       size_t n) {
  float* q = p + (size_t)blockIdx.y * stride;
  const size_t step = (size_t)gridDim.x * kThreads;
  for (size_t k = (size_t)blockIdx.x * kThreads + threadIdx.x; k < n; k += step) q[k] = 0.f;
}

inline unsigned blocks_for(int64_t n) { return (unsigned)((n + kThreads - 1) / kThreads); }

// Layers go on grid z (times the output split); launches are chunked over
// layers so that z stays within the 65536-block limit of y and z.
template <bool RED>
hipError_t dispatch_fused(int U, const float* y, float* z, float* S, const float* Hf,
                          const Shape& s, int t, int dst_len, hipStream_t st) {
  const dim3 block(step_threads(s.D));
  const size_t ls = (size_t)s.SL * s.BD, hls = (size_t)s.L * s.D;
  // with half-state storage S lies outside its allocation: integer arithmetic
  float* St = (float*)((uintptr_t)S + sizeof(float) * (size_t)t * s.BD);
#define LCSM_FUSED(UU, FULL)                                                                     \
  hipLaunchKernelGGL((k_step_fused<UU, RED, FULL>),                                              \
                     dim3(blocks_for(s.D), (unsigned)s.B, (unsigned)(mc * SP)), block, 0, st,    \
                     y + (RED ? (size_t)m0 * s.BD : 0), z + (RED ? (size_t)m0 * s.BD : 0),       \
                     St + m0 * ls, Hf + m0 * hls, ls, hls, s.BD, s.D, s.L - 1 - t, s.L)
#define LCSM_FUSED_CASE(UU)                                                                      \
  case UU: {                                                                                     \
    constexpr int SP = UU > 0 ? Split<UU>::value : 1;                                            \
    constexpr int MC = 65535 / SP;                                                               \
    for (int m0 = 0; m0 < s.M; m0 += MC) {                                                       \
      const int mc = s.M - m0 < MC ? s.M - m0 : MC;                                              \
      if (UU == 0 || dst_len == UU)                                                              \
        LCSM_FUSED(UU, true);                                                                    \
      else                                                                                       \
        LCSM_FUSED(UU, false);                                                                   \
    }                                                                                            \
    break;                                                                                       \
  }
  switch (U) {
    LCSM_FUSED_CASE(0)
    LCSM_FUSED_CASE(1)
    LCSM_FUSED_CASE(2)
    LCSM_FUSED_CASE(4)
    LCSM_FUSED_CASE(8)
    LCSM_FUSED_CASE(16)
    LCSM_FUSED_CASE(32)
    LCSM_FUSED_CASE(64)
    default:
      return hipErrorInvalidValue;
  }
#undef LCSM_FUSED_CASE
#undef LCSM_FUSED
  return hipGetLastError();
}

}  // namespace

hipError_t launch_transpose_filters(const float* src, float* dst, const Shape& s, hipStream_t st) {
  const dim3 grid((s.D + 31) / 32, (s.L + 31) / 32, s.M);
  hipLaunchKernelGGL(k_transpose, grid, dim3(kThreads), 0, st, src, dst, s.D, s.L);
  return hipGetLastError();
}

hipError_t launch_step_fused(const float* y, float* z, float* S, const float* Hf, const Shape& s,
                             int t, int U, int dst_len, hipStream_t st) {
  return dispatch_fused<true>(U, y, z, S, Hf, s, t, dst_len, st);
}

hipError_t launch_chain_fused(const float* x, float* z, float* S, const float* Hf, float* prev,
                              const Shape& s, int t, int U, int dst_len, hipStream_t st) {
  const dim3 grid(blocks_for(s.D), (unsigned)s.B), block(kThreads);
#define LCSM_CHAIN_K(UU, KK)                                                                      \
  hipLaunchKernelGGL((k_chain_fused<UU, KK>), grid, block, 0, st, x, z, S, Hf, prev, s.M, s.L,   \
                     s.SL, s.BD, s.D, t, dst_len)
#define LCSM_CHAIN_CASE(UU)                                                                       \
  case UU: {                                                                                      \
    constexpr int KM = ChainChunk<UU>::value;                                                     \
    if (KM >= 8 && s.M >= 8) {                                                                    \
      LCSM_CHAIN_K(UU, (KM >= 8 ? 8 : 1));                                                        \
    } else if (KM >= 4 && s.M >= 4) {                                                             \
      LCSM_CHAIN_K(UU, (KM >= 4 ? 4 : 1));                                                        \
    } else if (KM >= 2 && s.M >= 2) {                                                             \
      LCSM_CHAIN_K(UU, (KM >= 2 ? 2 : 1));                                                        \
    } else {                                                                                      \
      LCSM_CHAIN_K(UU, 1);                                                                        \
    }                                                                                             \
    break;                                                                                        \
  }
  switch (U) {
    LCSM_CHAIN_CASE(0)
    LCSM_CHAIN_CASE(1)
    LCSM_CHAIN_CASE(2)
    LCSM_CHAIN_CASE(4)
    LCSM_CHAIN_CASE(8)
    LCSM_CHAIN_CASE(16)
    LCSM_CHAIN_CASE(32)
    default:
      return hipErrorInvalidValue;
  }
#undef LCSM_CHAIN_CASE
#undef LCSM_CHAIN_K
  return hipGetLastError();
}

hipError_t launch_chain_block(const float* x, size_t xst, int xring, int xs0, float* z,
                              size_t zst, int zring, int zs0, float* S, const float* Hf,
                              float* prev, const Shape& s, int t0, int t1, bool tile_last,
                              hipStream_t st) {
  if (s.M > kChainBlockMaxM || t1 <= t0 || (t0 & ~(kChainBlockW - 1)) != ((t1 - 1) & ~(kChainBlockW - 1)))
    return hipErrorInvalidValue;
  const int tl = tile_last ? 1 : 0;
  static_assert(kChainLaneMaxM == 2, "one k_chain_lane per layer count");
#define LCSM_CHAIN_LANE(ML)                                                                        \
  hipLaunchKernelGGL((k_chain_lane<ML>), dim3((unsigned)((s.BD + 63) / 64)), dim3(64), 0, st, x,   \
                     xst, xring, xs0, z, zst, zring, zs0, S, Hf, prev, s.L, s.SL, s.BD, s.D, t0, t1, \
                     tl)
  if (s.M <= kChainLaneMaxM) {
    if (s.M == 1) LCSM_CHAIN_LANE(1); else LCSM_CHAIN_LANE(2);
    return hipGetLastError();
  }
#undef LCSM_CHAIN_LANE
#define LCSM_CHAIN_BLOCK(NC, HM, ML0, ML1)                                                        \
  hipLaunchKernelGGL((k_chain_block<NC, HM, ML0, ML1>), dim3((unsigned)((s.BD + NC - 1) / NC)),   \
                     dim3((unsigned)(64 * (1 + (s.M * NC + 63) / 64))), 0, st, x, xst, xring, xs0, \
                     z, zst, zring, zs0, S, Hf, prev, s.M, s.L, s.SL, s.BD, s.D, t0, t1, tl)
  // 16 columns per workgroup (half the waves, so the chain wave meets less
  // company on its SIMD) while a workgroup per CU holds them all
  const bool narrow = s.M >= 8 && (s.BD + 15) / 16 <= kChainBlockMaxGroups;
  if (s.M <= 8 && !narrow)
    LCSM_CHAIN_BLOCK(32, 4, 3, 8);
  else if (s.M <= 16)
    if (narrow) LCSM_CHAIN_BLOCK(16, 8, 8, 16); else LCSM_CHAIN_BLOCK(32, 8, 9, 16);
  else if (s.M <= 22)
    if (narrow) LCSM_CHAIN_BLOCK(16, 12, 17, 22); else LCSM_CHAIN_BLOCK(32, 12, 17, 22);
  else
    if (narrow) LCSM_CHAIN_BLOCK(16, 16, 23, 30); else LCSM_CHAIN_BLOCK(32, 16, 23, 30);
#undef LCSM_CHAIN_BLOCK
  return hipGetLastError();
}

hipError_t launch_red_layer(const float* y, float* z, float* S, const float* Hf, const Shape& s,
                            int layer, int t, hipStream_t st) {
  float* Sm = S + (size_t)layer * s.SL * s.BD;
  const float* Hm = Hf + (size_t)layer * s.L * s.D;
  hipLaunchKernelGGL(k_red_layer, dim3(blocks_for(s.BD)), dim3(kThreads), 0, st, y, z, Sm, Hm,
                     s.BD, s.D, t);
  return hipGetLastError();
}

hipError_t launch_direct_tile(float* S, const float* Hf, const Shape& s, int i, int U, int dst_len,
                              hipStream_t st) {
  if (dst_len <= 0) return hipSuccess;
  if (U <= kFusedMaxU) {
    // small tiles: whole tile per thread; position t = i-1 already holds y
    return dispatch_fused<false>(U, nullptr, nullptr, S, Hf, s, i - 1, dst_len, st);
  }
  const dim3 grid(blocks_for(s.BD), (dst_len + kDirectJ - 1) / kDirectJ, s.M);
  hipLaunchKernelGGL(k_direct_tile<kDirectJ>, grid, dim3(kThreads), 0, st, S, Hf, s.L, s.SL, s.BD,
                     s.D, i, U, dst_len);
  return hipGetLastError();
}

hipError_t launch_rows_in(const float* y, size_t y_stride, float* S, const Shape& s, int P,
                          hipStream_t st) {
  const size_t n = (size_t)P * s.M * s.BD;
  if (n == 0) return hipSuccess;
  size_t blocks = (n + kThreads - 1) / kThreads;
  if (blocks > 8192) blocks = 8192;
  hipLaunchKernelGGL(k_rows_in, dim3((unsigned)blocks), dim3(kThreads), 0, st, y, y_stride, S, s.M,
                     s.SL, s.BD, P);
  return hipGetLastError();
}

hipError_t launch_rows_out_clear(float* S, const Shape& s, int row0, int P, float* z,
                                 size_t z_stride, hipStream_t st) {
  const size_t n = (size_t)P * s.M * s.BD;
  if (n == 0) return hipSuccess;
  size_t blocks = (n + kThreads - 1) / kThreads;
  if (blocks > 8192) blocks = 8192;
  hipLaunchKernelGGL(k_rows_out_clear, dim3((unsigned)blocks), dim3(kThreads), 0, st, S, s.M, s.SL,
                     s.BD, row0, P, z, z_stride);
  return hipGetLastError();
}

hipError_t launch_zero_rows(float* p, int M, size_t stride, size_t n, hipStream_t st) {
  if (n == 0 || M <= 0) return hipSuccess;
  size_t bx = (n + kThreads - 1) / kThreads;
  const size_t cap = (8192 + (size_t)M - 1) / (size_t)M;  // about 8192 workgroups in all
  if (bx > cap) bx = cap;
  for (int m0 = 0; m0 < M; m0 += 65535) {
    const int mc = M - m0 < 65535 ? M - m0 : 65535;
    hipLaunchKernelGGL(k_zero_rows, dim3((unsigned)bx, (unsigned)mc), dim3(kThreads), 0, st,
                       p + (size_t)m0 * stride, stride, n);
  }
  return hipGetLastError();
}

hipError_t launch_zero(float* p, size_t n, hipStream_t st) {
  if (n == 0) return hipSuccess;
  size_t blocks = (n + kThreads - 1) / kThreads;
  if (blocks > 8192) blocks = 8192;
  hipLaunchKernelGGL(k_zero, dim3((unsigned)blocks), dim3(kThreads), 0, st, p, n);
  return hipGetLastError();
}

}  // namespace lcsm
