// The synthetic end-to-end model of the experiments (Sec. 5): per layer a
// long-convolution mixer and an MLP block of hidden width 2D with the exact
// GELU; the next token's input is the last layer's output plus noise (the
// sampler of Alg. 3).
//
// Per position t the work is (all on the mixer context's stream):
//   k_synth_red0            y^0_t = eps_t (+ a^M_{t-1}); layer 0's red cell
//   for each layer m:
//     k_prod<UP>            hid = gelu(W_up[m] z^m_t + b_up[m])        [B][2D]
//     k_prod<DOWN>          a^{m+1}_t = W_down[m] hid + b_down[m] -> act[m];
//                           its epilogue is layer m+1's red cell (y^{m+1}_t =
//                           a^{m+1}_t), or keeps a^M_t for the sampler
//   the gray tiles of i = t+1 for all layers (the mixer's batched launch).
//
// The products are matrix-vector products over B <= 16 rows at a time (k_prod):
// their time is the weight read (4 bytes per weight, 2B flops) plus what every
// dependent launch costs, so a workgroup puts its whole share of the weights
// in flight at once and nothing follows the sums but the stores.
#include <math.h>
#include <stdio.h>
#include <string.h>

#include <new>
#include <type_traits>

#include "lcsm_internal.h"
#include "lcsm_synth.h"

namespace lcsm {
namespace {

constexpr int kProdMaxThreads = 1024;
constexpr int kProdCus = 256;    // compute units to fill
constexpr int kMaxRows = 16;     // batch rows per product launch

enum { kUp = 0, kDown = 1 };

// Arguments of the DOWN epilogue: the next layer's red cell, or the copy of
// a^M_t for the sampler (S == nullptr).
struct RedNext {
  float* S;          // state slot row of position t, layer m+1: S + (m+1)*SL*BD + t*BD
  const float* h0;   // filter taps h[m+1, d, 0] (lag-0 row of layer m+1)
  float* z;          // the next layer's mixer output, quad layout
  float* last;       // [B][D] a^M_t (last layer only)
};

// Quad layout of a matrix of rows of K values (K a multiple of 4): four rows
// at a time, four consecutive values of each in turn, [row / 4][k / 4][row % 4][4].
// 16 consecutive lanes of k_prod then read one 256-byte run; with rows of K
// floats they met four lines, and the products were bound by that (16 rows,
// 2048 x 4096: 14.5 us, of which 4.5 us for the inputs' loads alone).
__device__ __forceinline__ size_t quad_at(int row, int k, int K) {
  return (size_t)(row >> 2) * 4 * K + (size_t)(k >> 2) * 16 + (row & 3) * 4 + (k & 3);
}

__device__ __forceinline__ float gelu(float v) {
  return 0.5f * v * (1.0f + erff(v * 0.70710678118654752f));
}

// out rows r < nrows of the product W [N][K] x^T with x [nrows][K] (row
// stride K): MODE kUp -> out[r][n] = gelu(sum + bias[n]) (row stride N);
// MODE kDown -> a = sum + bias[n], out[r][n] = a (row stride N = D), then the
// red cell of the next layer or the sampler copy.  nrows <= 4 RG.  The rows past
// nrows are those of the last quad, which init zeroes and nothing writes; units
// past N are computed from the last quad of units; neither is stored.  K must be
// a multiple of 4.  W, and x of kUp and kDown alike, are in the quad layout
// (quad_at); kUp writes out in it, kDown row by row.
//
// A workgroup takes 4 UG output units; its waves split K into chunks of 64
// (wave w: chunks w, w + nw, ...).  One v_mfma_f32_4x4x1_16b multiplies, in
// each of its 16 blocks, one k of 4 rows with the same k of 4 units, so lane
// 4 b + j holds four consecutive k of block b of unit j (and of row j) in one
// 16-byte load and feeds four of them: a load of the wave is 256 contiguous
// bytes of 4 rows, an input row is read once per 4 UG units, and a quad of
// rows fills the matrix operand (a 16x16 block would be three quarters empty
// at 4 rows).  The 16 blocks of a wave are summed with permlane swaps, each
// halving the registers that still have to be summed, and two rotations in
// the rows of 16 lanes; the waves' sums meet in LDS and are added in a fixed
// order (deterministic).  The epilogue's operands (bias, next red cell) are
// loaded first, under the weights.
//
// In a chain of launches over matrices out of the caches: 4 rows against 768 x
// 1536 3.5 us (1.3 TB/s; a bare read of it, launch included, takes 2.4), 16
// rows against 2048 x 4096 11.0 us (3.0 TB/s; bare read 6.7).  The model of 18
// layers, 4 rows, 768 channels went from 168 to 123 us per position, that of 32
// layers, 16 rows, 2048 channels from 1016 to 717 us.  What is left above the
// reads is the inputs' traffic from L2 (16 rows of K per workgroup) and the
// serial end: sums, barrier, epilogue, store.
typedef float v4f __attribute__((ext_vector_type(4)));

template <int CTRL>
__device__ __forceinline__ float dpp_add(float v) {
  const int o = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false);
  return v + __builtin_bit_cast(float, o);
}

// a + b after exchanging a's upper with b's lower 32 lanes: lanes 0..31 hold
// a's two halves summed, lanes 32..63 b's.
__device__ __forceinline__ float swap_add32(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, a),
                                                  __builtin_bit_cast(unsigned, b), false, false);
  const unsigned lo = r[0], hi = r[1];
  return __builtin_bit_cast(float, lo) + __builtin_bit_cast(float, hi);
}
// The same with the odd rows of 16 lanes of a and the even ones of b.
__device__ __forceinline__ float swap_add16(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, a),
                                                  __builtin_bit_cast(unsigned, b), false, false);
  const unsigned lo = r[0], hi = r[1];
  return __builtin_bit_cast(float, lo) + __builtin_bit_cast(float, hi);
}

template <int RG, int UG, int MODE>
__global__ __launch_bounds__(kProdMaxThreads) void k_prod(const float* __restrict__ x,
                                                          const float* __restrict__ W,
                                                          const float* __restrict__ bias,
                                                          float* __restrict__ out, int N, int K,
                                                          int nrows, RedNext rn) {
  constexpr int NU = 4 * UG, NO = NU * 4 * RG;  // units, outputs of a workgroup
  constexpr int R = 4 * RG * UG;                // partial sums per lane
  constexpr int NA = RG * UG <= 2 ? 4 : 2;      // sums side by side: shorter chains
  __shared__ float part[kProdMaxThreads / 64][NO];
  const int tid = (int)threadIdx.x;
  const int lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nw = (int)blockDim.x >> 6;
  const int n0 = (int)blockIdx.x * NU;
  const int k4 = (lane >> 2) * 4;  // the lane's k in a chunk; its unit and row of a quad: lane % 4

  // output of this thread: for kUp in the order of the quads it writes
  const int orow = MODE == kUp ? tid / (4 * NU) * 4 + tid / 4 % 4 : tid / NU;
  const int ou = MODE == kUp ? tid / 16 % UG * 4 + tid % 4 : tid % NU;
  const int on = n0 + ou;
  const bool ohas = tid < NO && orow < nrows && on < N;
  const size_t oe = (size_t)orow * N + on;
  float obias = 0.f, oh0 = 0.f, oslot = 0.f;
  if (ohas) {
    obias = bias[on];
    if constexpr (MODE == kDown) {
      if (rn.S) {
        oh0 = rn.h0[on];
        oslot = rn.S[oe];
      }
    }
  }

  const float* wp[UG];
  const float* xp[RG];
#pragma unroll
  for (int u = 0; u < UG; ++u) {
    const int q = n0 / 4 + u;
    wp[u] = W + (size_t)(4 * q < N ? q : N / 4 - 1) * 4 * K + 4 * lane;
  }
#pragma unroll
  for (int g = 0; g < RG; ++g) xp[g] = x + (size_t)g * 4 * K + 4 * lane;
  v4f acc[NA][UG][RG];
#pragma unroll
  for (int n = 0; n < NA; ++n)
#pragma unroll
    for (int u = 0; u < UG; ++u)
#pragma unroll
      for (int g = 0; g < RG; ++g) acc[n][u][g] = v4f{0.f, 0.f, 0.f, 0.f};

  auto chunk = [&](int c, auto tail) {
    constexpr bool TAIL = decltype(tail)::value;  // some k are past K: zeros on both sides
    const bool in = !TAIL || 64 * c + k4 < K;
    auto load = [&](const float* p) -> v4f {
      const v4f v = *reinterpret_cast<const v4f*>(in ? p + 256 * c : p - 4 * lane);
      return in ? v : v4f{0.f, 0.f, 0.f, 0.f};
    };
    v4f w[UG], xv[RG];
#pragma unroll
    for (int g = 0; g < RG; ++g) xv[g] = load(xp[g]);
#pragma unroll
    for (int u = 0; u < UG; ++u) w[u] = load(wp[u]);
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int u = 0; u < UG; ++u)
#pragma unroll
        for (int g = 0; g < RG; ++g) {
          v4f& a = acc[e % NA][u][g];
          a = __builtin_amdgcn_mfma_f32_4x4x1f32(xv[g][e], w[u][e], a, 0, 0, 0);
        }
  };
  int c = wv;
  for (; 64 * (c + 1) <= K; c += nw) chunk(c, std::false_type{});
  if (64 * c < K) chunk(c, std::true_type{});
  // the epilogue's operands have arrived with the weights: not loaded later
  asm volatile("" : "+v"(obias), "+v"(oh0), "+v"(oslot));

  // sum i of the lane: unit 4 (i / (4 RG)) + j, row i % (4 RG)
  float s[R];
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const int u = i / (4 * RG), g = i / 4 % RG, e = i % 4;
    s[i] = acc[0][u][g][e];
    s[i] += acc[1][u][g][e];
    if constexpr (NA == 4) s[i] += acc[2][u][g][e] + acc[3][u][g][e];
  }
#pragma unroll
  for (int i = 0; i < R / 2; ++i) s[i] = swap_add32(s[i], s[i + R / 2]);
#pragma unroll
  for (int i = 0; i < R / 4; ++i) s[i] = swap_add16(s[i], s[i + R / 4]);
#pragma unroll
  for (int i = 0; i < R / 4; ++i) s[i] = dpp_add<0x128>(dpp_add<0x124>(s[i]));
  if ((lane & 12) == 0) {
    const int i0 = ((lane >> 4) & 1) * (R / 4) + (lane >> 5) * (R / 2);
#pragma unroll
    for (int i = 0; i < R / 4; ++i) {
      const int si = i0 + i;
      part[wv][(si % (4 * RG)) * NU + 4 * (si / (4 * RG)) + (lane & 3)] = s[i];
    }
  }
  __syncthreads();
  if (!ohas) return;
  float ps[4] = {0.f, 0.f, 0.f, 0.f};
  const float* po = &part[0][orow * NU + ou];
  int w = 0;
  for (; w + 4 <= nw; w += 4)
#pragma unroll
    for (int i = 0; i < 4; ++i) ps[i] += po[(w + i) * NO];
  for (; w < nw; ++w) ps[0] += po[w * NO];
  const float sum = ((ps[0] + ps[1]) + (ps[2] + ps[3])) + obias;
  if constexpr (MODE == kUp) {
    out[quad_at(orow, on, N)] = gelu(sum);
  } else {
    out[oe] = sum;
    if (rn.S) {
      rn.z[quad_at(orow, on, N)] = fmaf(oh0, sum, oslot);
      rn.S[oe] = sum;
    } else {
      rn.last[oe] = sum;
    }
  }
}

// dst = src [rows][K] in the quad layout (rows and K multiples of 4), one
// thread per four values of a row.  src is the caller's: aligned as a float is.
typedef float v4f_any __attribute__((ext_vector_type(4), aligned(4)));

__global__ __launch_bounds__(256) void k_quads(const float* __restrict__ src,
                                               float* __restrict__ dst, size_t rows, int K) {
  const size_t n = rows * (size_t)(K / 4), step = (size_t)gridDim.x * 256;
  for (size_t q = (size_t)blockIdx.x * 256 + threadIdx.x; q < n; q += step) {
    // q counts the destination's quads: [row / 4][k / 4][row % 4]
    const size_t g = q / K, r = q - g * K;  // K quads per four rows
    const v4f v = *reinterpret_cast<const v4f_any*>(src + (4 * g + (r & 3)) * K + (r & ~(size_t)3));
    *reinterpret_cast<v4f*>(dst + 4 * q) = v;
  }
}

// Sampler and layer 0's red cell at position t: y = eps (+ last for t > 0),
// z = fmaf(h0[d], y, slot) in the quad layout, slot = y.
__global__ __launch_bounds__(256) void k_synth_red0(const float* __restrict__ eps,
                                                    const float* __restrict__ last,
                                                    float* __restrict__ slot_row,
                                                    const float* __restrict__ h0,
                                                    float* __restrict__ z, int BD, int D, int t) {
  const int c = (int)blockIdx.x * 256 + (int)threadIdx.x;
  if (c >= BD) return;
  const float y = t > 0 ? last[c] + eps[c] : eps[c];
  const int b = c / D, d = c - b * D;
  z[quad_at(b, d, D)] = fmaf(h0[d], y, slot_row[c]);
  slot_row[c] = y;
}

hipError_t launch_quads(const float* src, float* dst, size_t rows, int K, hipStream_t st) {
  size_t blocks = (rows * (size_t)(K / 4) + 255) / 256;
  if (blocks > 16384) blocks = 16384;
  hipLaunchKernelGGL(k_quads, dim3((unsigned)blocks), dim3(256), 0, st, src, dst, rows, K);
  return hipGetLastError();
}

template <int RG, int MODE>
hipError_t prod_rows(const float* x, const float* W, const float* bias, float* out, int N, int K,
                     int nrows, const RedNext& rn, hipStream_t st) {
  // 8 units per workgroup while that leaves three workgroups for every four
  // CUs (the inputs are then read half as often), else 4: 16 rows against
  // 2048 x 4096 take 11.4 against 13.5 us, 4 rows against 768 x 1536 3.6
  // either way
  const bool two = N >= 6 * kProdCus;
  const int nch = (K + 63) / 64, outs = 16 * RG * (two ? 2 : 1);
  // at most 16 waves, chunks shared evenly; 8 for the long rows, whose 16
  // waves only compete (16 rows, 4096 x 2048: 10.3 against 11.4 us).  One row
  // takes 16 throughout: a model of 18 layers, 1024 channels, one row 149.1 us per
  // position against 159.4 with 8 (158.6 with a unit's row per workgroup on the
  // vector ALU), 2048 channels 283.6 against 291.9, 8 layers of 1024 channels,
  // whose weights stay in the caches, 61.8 against 61.6
  const int most = nch <= 24 || nrows == 1 ? kProdMaxThreads / 64 : 8;
  const int rounds = (nch + most - 1) / most;
  int threads = 64 * ((nch + rounds - 1) / rounds);
  if (threads < outs) threads = (outs + 63) / 64 * 64;  // a thread per output
  if (two)
    hipLaunchKernelGGL((k_prod<RG, 2, MODE>), dim3((unsigned)((N + 7) / 8)), dim3(threads), 0, st, x,
                       W, bias, out, N, K, nrows, rn);
  else
    hipLaunchKernelGGL((k_prod<RG, 1, MODE>), dim3((unsigned)((N + 3) / 4)), dim3(threads), 0, st, x,
                       W, bias, out, N, K, nrows, rn);
  return hipGetLastError();
}

template <int MODE>
hipError_t prod(const float* x, const float* W, const float* bias, float* out, int N, int K,
                int nrows, const RedNext& rn, hipStream_t st) {
  switch ((nrows + 3) / 4) {
    case 1: return prod_rows<1, MODE>(x, W, bias, out, N, K, nrows, rn, st);
    case 2: return prod_rows<2, MODE>(x, W, bias, out, N, K, nrows, rn, st);
    case 3: return prod_rows<3, MODE>(x, W, bias, out, N, K, nrows, rn, st);
    default: return prod_rows<4, MODE>(x, W, bias, out, N, K, nrows, rn, st);
  }
}

}  // namespace
}  // namespace lcsm

struct lcsm_synth {
  lcsm_ctx* mixer;
  int M, B, D, L;
  hipStream_t stream;
  char* mem;
  float *w_up, *b_up, *w_down, *b_down;
  float *z, *hid, *last;
  bool faulted;
  char msg[256];
};

namespace {

int synth_fail(lcsm_synth* s, int code, const char* what, hipError_t e) {
  if (e != hipSuccess) {
    snprintf(s->msg, sizeof(s->msg), "%s: %s", what, hipGetErrorString(e));
    s->faulted = true;
    return LCSM_EDEVICE;
  }
  snprintf(s->msg, sizeof(s->msg), "%s", what);
  return code;
}

size_t align256(size_t v) { return (v + 255) / 256 * 256; }

}  // namespace

extern "C" {

int lcsm_synth_init(lcsm_synth** out, const float* filters, const float* w_up, const float* b_up,
                    const float* w_down, const float* b_down, int M, int B, int D, int L,
                    void* stream, const lcsm_options* opt) {
  if (!out) return LCSM_EINVAL;
  *out = nullptr;
  if (!filters || !w_up || !b_up || !w_down || !b_down) return LCSM_EINVAL;
  if (D < 4 || D % 4 != 0) return LCSM_EINVAL;
  size_t need = 0;
  int r = lcsm_workspace_bytes(M, B, D, L, opt, &need);  // validates shape and options
  if (r) return r;
  lcsm_synth* s = new (std::nothrow) lcsm_synth();
  if (!s) return LCSM_ENOMEM;
  s->M = M;
  s->B = B;
  s->D = D;
  s->L = L;
  s->stream = (hipStream_t)stream;
  s->msg[0] = 0;
  const size_t D2 = 2 * (size_t)D, BD = (size_t)B * D;
  const size_t n_wup = (size_t)M * D2 * D, n_bup = (size_t)M * D2, n_wdn = (size_t)M * D * D2,
               n_bdn = (size_t)M * D;
  const size_t B4 = ((size_t)B + 3) / 4 * 4;  // rows of the quad layout
  size_t off[7], total = 0;
  const size_t sizes[7] = {n_wup, n_bup, n_wdn, n_bdn, B4 * D, B4 * D2, BD};
  for (int k = 0; k < 7; ++k) {
    off[k] = total;
    total = align256(total + sizeof(float) * sizes[k]);
  }
  void* p = nullptr;
  if (hipMalloc(&p, total) != hipSuccess) {
    (void)hipGetLastError();
    delete s;
    return LCSM_ENOMEM;
  }
  s->mem = (char*)p;
  float* f[7];
  for (int k = 0; k < 7; ++k) f[k] = (float*)(s->mem + off[k]);
  s->w_up = f[0];
  s->b_up = f[1];
  s->w_down = f[2];
  s->b_down = f[3];
  s->z = f[4];
  s->hid = f[5];
  s->last = f[6];
  r = lcsm_init(&s->mixer, filters, M, B, D, L, stream, nullptr, 0, opt);
  if (r) {
    (void)hipFree(s->mem);
    delete s;
    return r;
  }
  const float* src[4] = {w_up, b_up, w_down, b_down};
  hipError_t e = hipSuccess;
  for (int k = 1; k < 4 && e == hipSuccess; k += 2)  // the biases
    e = hipMemcpyAsync(f[k], src[k], sizeof(float) * sizes[k], hipMemcpyDeviceToDevice, s->stream);
  if (e == hipSuccess) e = lcsm::launch_quads(w_up, s->w_up, (size_t)M * D2, D, s->stream);
  if (e == hipSuccess) e = lcsm::launch_quads(w_down, s->w_down, (size_t)M * D, (int)D2, s->stream);
  // z, hid and last (the rows past B of the last quad stay zero)
  if (e == hipSuccess) e = lcsm::launch_zero(s->z, (total - off[4]) / sizeof(float), s->stream);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    lcsm_destroy(s->mixer);
    (void)hipFree(s->mem);
    delete s;
    return LCSM_EDEVICE;
  }
  s->faulted = false;
  *out = s;
  return LCSM_OK;
}

int lcsm_synth_step(lcsm_synth* s, const float* eps_t, float* act_t) {
  if (!s) return LCSM_EINVAL;
  if (!eps_t || !act_t) return synth_fail(s, LCSM_EINVAL, "null input or output pointer", hipSuccess);
  if (s->faulted) return LCSM_ESTATE;
  lcsm::StepView v;
  int r = lcsm::begin_external_step(s->mixer, &v);
  if (r) return r == LCSM_EDONE ? r : synth_fail(s, r, lcsm_last_error(s->mixer), hipSuccess);
  const int M = s->M, B = s->B, D = s->D, D2 = 2 * D, BD = B * D;
  const size_t lstride = (size_t)v.s.SL * BD;  // state floats per layer
  const size_t hstride = (size_t)v.s.L * D;    // filter floats per layer
  hipStream_t st = v.stream;
  // sampler + layer 0's red cell (state slot row of position t, layer 0)
  hipLaunchKernelGGL(lcsm::k_synth_red0, dim3((unsigned)((BD + 255) / 256)), dim3(256), 0, st,
                     eps_t, s->last, v.S + (size_t)v.t * BD, v.Hf, s->z, BD, D, v.t);
  hipError_t e = hipGetLastError();
  for (int m = 0; m < M && e == hipSuccess; ++m) {
    for (int r0 = 0; r0 < B && e == hipSuccess; r0 += lcsm::kMaxRows) {
      const int nr = B - r0 < lcsm::kMaxRows ? B - r0 : lcsm::kMaxRows;
      lcsm::RedNext none{nullptr, nullptr, nullptr, nullptr};
      e = lcsm::prod<lcsm::kUp>(s->z + (size_t)r0 * D, s->w_up + (size_t)m * D2 * D,
                                s->b_up + (size_t)m * D2, s->hid + (size_t)r0 * D2, D2, D, nr,
                                none, st);
      lcsm::RedNext rn{nullptr, nullptr, nullptr, nullptr};
      if (m + 1 < M) {
        rn.S = v.S + (size_t)(m + 1) * lstride + (size_t)v.t * BD + (size_t)r0 * D;
        rn.h0 = v.Hf + (size_t)(m + 1) * hstride;
        rn.z = s->z + (size_t)r0 * D;
      } else {
        rn.last = s->last + (size_t)r0 * D;
      }
      if (e == hipSuccess)
        e = lcsm::prod<lcsm::kDown>(s->hid + (size_t)r0 * D2, s->w_down + (size_t)m * D * D2,
                                    s->b_down + (size_t)m * D,
                                    act_t + (size_t)m * BD + (size_t)r0 * D, D, D2, nr, rn, st);
    }
  }
  if (e != hipSuccess) return synth_fail(s, LCSM_EDEVICE, "model kernel launch", e);
  r = lcsm::end_external_step(s->mixer);
  if (r) return synth_fail(s, r, lcsm_last_error(s->mixer), hipSuccess);
  return LCSM_OK;
}

int lcsm_synth_reset(lcsm_synth* s) {
  if (!s) return LCSM_EINVAL;
  int r = lcsm_reset(s->mixer);
  if (r) return synth_fail(s, r, lcsm_last_error(s->mixer), hipSuccess);
  s->faulted = false;
  s->msg[0] = 0;
  return LCSM_OK;
}

int lcsm_synth_position(const lcsm_synth* s, int* t) {
  if (!s || !t) return LCSM_EINVAL;
  return lcsm_position(s->mixer, t);
}

void lcsm_synth_destroy(lcsm_synth* s) {
  if (!s) return;
  lcsm_destroy(s->mixer);  // waits for the stream
  (void)hipFree(s->mem);
  delete s;
}

const char* lcsm_synth_last_error(const lcsm_synth* s) { return s ? s->msg : ""; }

}  // extern "C"
