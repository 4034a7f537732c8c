// Kernels of the learned support proposal (an extension of the paper's
// method): a multilayer perceptron maps the magnitude of the normalised first
// correlation of a signal, f_n = sqrt(M) |a_n^T y| / (||a_n|| ||y||) (Algorithm
// 1's first selection statistic, scaled to unit size),
// to one score per atom; the S best-scored atoms are checked by one
// least-squares solve (Eq. 2, by the Cholesky factorisation of the Gram
// block, Section 2.2), and plain OMP handles the signals whose residual misses
// the tolerance.
//
// Network: h1 = relu(W1 f + b1), h2 = relu(W2 h1 + b2), z = W3 h2 + b3, with
// BF16 operands and FP32 accumulation; W_l is stored [out][in]. Training
// minimises binary cross-entropy with logits against the multi-hot OMP
// support, averaged over the batch, with Adam (Kingma and Ba, 2015).
//
// All matrix products are the "NT" BF16 MFMA product of mfma_tile.h with a
// fused epilogue; every layout below keeps the reduction index contiguous:
//   forward   H1[b][o]  = F[b][:]   . W1[o][:]          (+ b1, relu)
//   backward  dH2[b][i] = dZ[b][:]  . W3T[i][:]         (x (H2 > 0))
//   weights   dW3[o][i] = dZT[o][:] . H2T[i][:]         (one launch for the three layers)
// with W_lT the transposed BF16 copy kept by the optimiser and the activation
// transposes made per step.

#include <cmath>
#include <type_traits>
#include <utility>

#include "../../include/batched_omp.h"
#include "lds_limit.h"
#include "mfma_tile.h"
#include "mlp_internal.h"
#include "omp_internal.h"
#include "wave_ops.h"

namespace bomp {
namespace {

// Tiles of the products: 256 x 256 (8 wavefronts of 128 x 64), 128 x 128 (4 of 64 x 64)
// and 64 x 64 (4 of 32 x 32). Every tile sums K in the same order, so the choice changes
// no product; it follows the number of workgroups (gemm_tile).
using GT256 = Tile<256, 256, 2, 4>;
using GT128 = Tile<128, 128, 2, 2>;
using GT64 = Tile<64, 64, 2, 2>;

__device__ inline uint16_t bf16_rne(float f) {
  const uint32_t u = __float_as_uint(f);
  return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}
__device__ inline float bf16_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// sigmoid(z) and softplus(z) from e = exp(-|z|).
__device__ inline float sigmoid_of(float z, float e) { return (z >= 0.f ? 1.f : e) / (1.f + e); }
__device__ inline float softplus_of(float z, float e) { return fmaxf(z, 0.f) + log1pf(e); }

// ---------------------------------------------------------------------------
// BF16 "NT" product C[m][n] = sum_k P[m][k] Q[n][k] with a fused epilogue.
// P: [rows][ldp] BF16, Q: [cols][ldq] BF16, K a multiple of 64. The grid is
// (M / T::TN) x (N / T::TB) tiles times `splits` slices of K (EPI_PARTIAL only).
// ---------------------------------------------------------------------------
constexpr int GT64_STAGES = 4;  // LDS buffers of the 64 x 64 tiles' main loop (64 KiB)
template <class T>
constexpr size_t gemm_lds() {
  return T::TN == 64 ? (size_t)GT64_STAGES * T::STAGE * 16 : T::LDS_BYTES;
}

template <int EPI, class T>
__device__ inline void gemm_nt_tile(const uint16_t *__restrict__ P, int64_t ldp, const uint16_t *__restrict__ Q,
                                    int64_t ldq, int64_t Mrows, int64_t Ncols, int64_t K, int splits, int64_t block,
                                    const GemmEpi &e) {
  extern __shared__ u32x4 lds[];
  const int64_t ntm = Mrows / T::TN, ntn = Ncols / T::TB;
  const int64_t tile = block % (ntm * ntn);
  const int split = (int)(block / (ntm * ntn));
  const int64_t tm = tile % ntm, tn = tile / ntm;
  const int64_t kc = K / splits;  // elements of K per split (a multiple of 64)
  const int64_t prs = ldp / 8, qrs = ldq / 8;
  const u32x4 *Pp = reinterpret_cast<const u32x4 *>(P) + tm * T::TN * prs + (split * kc) / 8;
  const u32x4 *Qp = reinterpret_cast<const u32x4 *>(Q) + tn * T::TB * qrs + (split * kc) / 8;
  f32x16 acc[T::FN][T::FB];
  if constexpr (T::TN == 64)
    mainloop_staged<OpBF16, T, GT64_STAGES>(Pp, prs, Qp, qrs, (int)(kc / 64), lds, acc);
  else
    mainloop<OpBF16, T>(Pp, prs, Qp, qrs, (int)(kc / 64), lds, acc);

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wn = wave % T::WN, wb = wave / T::WN;
  float lsum = 0.f;
#pragma unroll
  for (int i = 0; i < T::FN; ++i)
#pragma unroll
    for (int j = 0; j < T::FB; ++j) {
      const int64_t n = tn * T::TB + wb * T::FB * 32 + j * 32 + (lane & 31);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int64_t m = tm * T::TN + wn * T::FN * 32 + i * 32 + frag_row(lane, r);
        const float c = acc[i][j][r];
        const int64_t o = m * e.ldo + n;
        if (EPI == EPI_FEATURES) {
          reinterpret_cast<uint16_t *>(e.out)[o] = bf16_rne(fabsf(c) * e.colscale[n] * e.rowscale[m] * e.scale);
        } else if (EPI == EPI_BIAS_RELU) {
          reinterpret_cast<uint16_t *>(e.out)[o] = bf16_rne(fmaxf(c + e.bias[n], 0.f));
        } else if (EPI == EPI_BIAS) {
          reinterpret_cast<float *>(e.out)[o] = c + e.bias[n];
        } else if (EPI == EPI_BCE) {
          // rows at or beyond the batch are padding: no gradient, no loss
          float dz = 0.f;
          if (m < e.mvalid) {
            const float z = c + e.bias[n];
            const float t = (float)((e.labels[m * e.ldl + (n >> 5)] >> (n & 31)) & 1u);
            const float ez = expf(-fabsf(z));
            dz = (sigmoid_of(z, ez) - t) * e.scale;
            lsum += softplus_of(z, ez) - t * z;
          }
          reinterpret_cast<uint16_t *>(e.out)[o] = bf16_rne(dz);
        } else if (EPI == EPI_RELU_MASK) {
          const bool on = bf16_to_f32(e.mask[o]) > 0.f;
          reinterpret_cast<uint16_t *>(e.out)[o] = bf16_rne(on ? c : 0.f);
        } else {  // EPI_PARTIAL: split-K partial sums, summed by the optimiser
          reinterpret_cast<float *>(e.out)[(int64_t)split * Mrows * e.ldo + o] = c;
        }
      }
    }
  if (EPI == EPI_BCE) {
    // block sum of the loss terms, one partial per block (summed in block order)
    __shared__ float red[T::NTHR / 64];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) lsum += __shfl_xor(lsum, off);
    if (lane == 0) red[wave] = lsum;
    __syncthreads();
    if (threadIdx.x == 0) {
      float s = 0.f;
      for (int i = 0; i < T::NTHR / 64; ++i) s += red[i];
      e.loss_part[block] = s;
    }
  }
}

template <int EPI, class T>
__global__ __launch_bounds__(T::NTHR) void k_gemm_nt(const uint16_t *__restrict__ P, int64_t ldp,
                                                    const uint16_t *__restrict__ Q, int64_t ldq, int64_t Mrows,
                                                    int64_t Ncols, int64_t K, GemmEpi e) {
  gemm_nt_tile<EPI, T>(P, ldp, Q, ldq, Mrows, Ncols, K, 1, blockIdx.x, e);
}

// The weight gradients of all three layers, dW_l = dOutT_l InT_l^T, in one launch: block
// ranges of the layers one after another, so the small products of a layer share the chip.
template <class T>
__global__ __launch_bounds__(T::NTHR) void k_wgrad(WgradBatch g, int64_t K, int splits) {
  int l = 0;
  while (l < 2 && (int64_t)blockIdx.x >= g.end[l]) ++l;
  GemmEpi e = {};
  e.out = g.out[l];
  e.ldo = g.in[l];
  gemm_nt_tile<EPI_PARTIAL, T>(g.dOutT[l], K, g.InT[l], K, g.rows[l], g.in[l], K, splits,
                               blockIdx.x - (l ? g.end[l - 1] : 0), e);
}

// ---------------------------------------------------------------------------
// Signals to BF16 (padded) and 1/||y|| (0 for a zero or non-finite signal).
// One wavefront per padded signal.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(64) void k_prep_signals(const float *__restrict__ Y, int64_t ldy, int64_t B, int64_t M,
                                                     int64_t Mp, uint16_t *__restrict__ Y16,
                                                     float *__restrict__ yinv) {
  const int64_t b = blockIdx.x;
  const int lane = threadIdx.x;
  double s = 0.0;
  int finite = 1;
  for (int64_t m = lane; m < Mp; m += 64) {
    const float v = (b < B && m < M) ? Y[b * ldy + m] : 0.f;
    finite &= isfinite(v) ? 1 : 0;
    const float vz = isfinite(v) ? v : 0.f;
    Y16[b * Mp + m] = bf16_rne(vz);
    s += (double)vz * (double)vz;
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
  const bool ok = __all(finite) && s > 0.0;
  if (lane == 0) yinv[b] = ok ? (float)(1.0 / sqrt(s)) : 0.f;
}

// Zero-padded copy of B rows of a BF16 matrix into [Bp][cols]; row b is source
// row rows[b] when `rows` is given. With `sup` also the rows' multi-hot labels from
// supports [.][S] (-1 padded; the same row map): bits [Bp][words], gathered in LDS.
__global__ __launch_bounds__(256) void k_pad_rows16(const uint16_t *__restrict__ src, int64_t lds_,
                                                    const int32_t *__restrict__ rows, int64_t B, int64_t cols,
                                                    uint16_t *__restrict__ dst, const int32_t *__restrict__ sup, int S,
                                                    int64_t words, uint32_t *__restrict__ bits) {
  extern __shared__ uint32_t lab[];
  const int64_t b = blockIdx.x;
  const int64_t sb = b < B ? (rows ? (int64_t)rows[b] : b) : 0;
  const uint16_t *s = src + sb * lds_;
  uint16_t *o = dst + b * cols;
  if (((cols | lds_) & 7) == 0 && ((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) & 15) == 0) {
    for (int64_t c = threadIdx.x; c < cols / 8; c += blockDim.x)
      reinterpret_cast<uint4 *>(o)[c] = b < B ? reinterpret_cast<const uint4 *>(s)[c] : make_uint4(0, 0, 0, 0);
  } else {
    for (int64_t c = threadIdx.x; c < cols; c += blockDim.x) o[c] = b < B ? s[c] : 0;
  }
  if (!sup) return;
  for (int64_t t = threadIdx.x; t < words; t += blockDim.x) lab[t] = 0u;
  __syncthreads();
  if (b < B)
    for (int j = threadIdx.x; j < S; j += blockDim.x) {
      const int n = sup[sb * S + j];
      if (n >= 0 && n < words * 32) atomicOr(&lab[n >> 5], 1u << (n & 31));
    }
  __syncthreads();
  for (int64_t t = threadIdx.x; t < words; t += blockDim.x) bits[b * words + t] = lab[t];
}

// BF16 transposes dst[c][r] = src[r][c] of all matrices of a batch (R rows, a multiple of
// 64; C a multiple of 64) in one launch, and of the matrices with `part` the column sums
// of every group of `rpc` rows (a multiple of 64): part[group][c]. A block takes 64 columns
// of one group, 64 x 64 tiles through LDS, so the sums cost no pass of their own: 10 us
// for a batch of 1024 on 1024-wide layers, where six transposes of 4.4 us and three column
// sums of 16.5 us (64 threads' serial loads per column) took 75.
__global__ __launch_bounds__(256) void k_transposes16(TransposeBatch g, int64_t R, int64_t rpc) {
  // rows of nine 16-byte pieces: a row is written by pieces and read by columns
  struct alignas(16) Row {
    uint16_t v[72];
  };
  static_assert(sizeof(Row) == 144, "every row starts at a 16-byte piece");
  __shared__ Row t[64];
  __shared__ float red[8][64];
  int m = 0;
  while (m < 5 && (int64_t)blockIdx.x >= g.end[m]) ++m;
  const int64_t blk = blockIdx.x - (m ? g.end[m - 1] : 0), C = g.cols[m];
  const int64_t tc = blk % (C / 64), grp = blk / (C / 64);
  const int64_t r0 = grp * rpc, r1 = min(R, r0 + rpc);
  const int tid = threadIdx.x;
  float sum = 0.f;
  for (int64_t r = r0; r < r1; r += 64) {
    // 64 rows of 8 chunks of 16 bytes: two chunks per thread
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int f = tid + 256 * q, row = f >> 3, c8 = f & 7;
      *reinterpret_cast<uint4 *>(&t[row].v[c8 * 8]) =
          *reinterpret_cast<const uint4 *>(g.src[m] + (r + row) * C + tc * 64 + c8 * 8);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int f = tid + 256 * q, col = f & 63, r8 = f >> 6;  // eight rows of one column
      uint16_t v[8];
      float s8 = 0.f;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        v[i] = t[r8 * 8 + i].v[col];
        s8 += bf16_to_f32(v[i]);
      }
      red[r8][col] = s8;
      uint4 o;
      o.x = v[0] | ((uint32_t)v[1] << 16);
      o.y = v[2] | ((uint32_t)v[3] << 16);
      o.z = v[4] | ((uint32_t)v[5] << 16);
      o.w = v[6] | ((uint32_t)v[7] << 16);
      *reinterpret_cast<uint4 *>(g.dst[m] + (tc * 64 + col) * R + r + r8 * 8) = o;
    }
    __syncthreads();
    if (g.part[m] && tid < 64) {
#pragma unroll
      for (int i = 0; i < 8; ++i) sum += red[i][tid];
    }
  }
  if (g.part[m] && tid < 64) g.part[m][grp * C + tc * 64 + tid] = sum;
}

// The sums that end a gradient, in one launch: block 0 adds the loss partials in block
// order, the others the split or group partials of up to six arrays.
__global__ __launch_bounds__(256) void k_grad_sums(SumBatch g, const float *__restrict__ loss_part, int64_t nloss,
                                                   float scale, float *__restrict__ loss_out) {
  if (blockIdx.x == 0) {
    if (threadIdx.x >= 64 || !loss_out) return;
    double s = 0.0;
    for (int64_t i = threadIdx.x; i < nloss; i += 64) s += loss_part[i];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
    if (threadIdx.x == 0) loss_out[0] = (float)(s * scale);
    return;
  }
  const int64_t blk = blockIdx.x - 1;
  int m = 0;
  while (m < 5 && blk >= g.end[m]) ++m;
  const int64_t i = (blk - (m ? g.end[m - 1] : 0)) * 256 + threadIdx.x;
  if (i >= g.n[m]) return;
  float v[16];
#pragma unroll
  for (int s = 0; s < 16; ++s) v[s] = s < g.parts[m] ? g.part[m][(int64_t)s * g.n[m] + i] : 0.f;
  float sum = 0.f;
#pragma unroll
  for (int s = 0; s < 16; ++s) sum += v[s];
  g.out[m][i] = sum;
}

// ---------------------------------------------------------------------------
// Adam on one weight matrix W [out][in] (64 x 64 tiles): gradient = sum of the
// split-K partials; moments, master weights, the BF16 copy and its transpose.
// c1 = 1/(1 - beta1^t), c2 = 1/(1 - beta2^t). lr = 0 only copies (no update).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_adam_w(LayerView L, const float *__restrict__ gpart, int splits,
                                                float lr, float b1, float b2, float eps, float c1, float c2,
                                                int update) {
  __shared__ uint16_t t[64][66];
  const int64_t nin = L.n_in, nout = L.n_out;
  const int64_t ti = blockIdx.x % (nin / 64), to = blockIdx.x / (nin / 64);
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  for (int i = ty; i < 64; i += 4) {
    const int64_t o = to * 64 + i, in = ti * 64 + tx, idx = o * nin + in;
    float w = L.W32[idx];
    if (update) {
      float g = 0.f;
      for (int s = 0; s < splits; ++s) g += gpart[(int64_t)s * nout * nin + idx];
      const float m = b1 * L.mW[idx] + (1.f - b1) * g;
      const float v = b2 * L.vW[idx] + (1.f - b2) * g * g;
      L.mW[idx] = m;
      L.vW[idx] = v;
      w -= lr * (m * c1) / (sqrtf(v * c2) + eps);
      L.W32[idx] = w;
    }
    const uint16_t h = bf16_rne(w);
    L.W16[idx] = h;
    t[i][tx] = h;
  }
  __syncthreads();
  for (int i = ty; i < 64; i += 4) L.W16T[(ti * 64 + i) * nout + to * 64 + tx] = t[tx][i];
}

__global__ __launch_bounds__(256) void k_adam_b(LayerView L, const float *__restrict__ gpart, int chunks, float lr,
                                                float b1, float b2, float eps, float c1, float c2) {
  const int64_t o = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (o >= L.n_out) return;
  float g = 0.f;
  for (int s = 0; s < chunks; ++s) g += gpart[(int64_t)s * L.n_out + o];
  const float m = b1 * L.mb[o] + (1.f - b1) * g;
  const float v = b2 * L.vb[o] + (1.f - b2) * g * g;
  L.mb[o] = m;
  L.vb[o] = v;
  L.b32[o] -= lr * (m * c1) / (sqrtf(v * c2) + eps);
}

// Plain FP32 copies and zero fills (kernels, so that captured graphs hold no memset).
__global__ __launch_bounds__(256) void k_copy32(const float *__restrict__ src, int64_t n, float *__restrict__ dst) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) dst[i] = src ? src[i] : 0.f;
}

// ---------------------------------------------------------------------------
// Top-S of N scores per signal (one wavefront; NPL = N / 64 scores per lane, S <= 64),
// in descending order, ties to the lowest index. The S-th largest score is found bit by
// bit on orderable 32-bit keys: each bit costs one compare per score, its count taken
// from the ballot on the scalar unit, and the search ends as soon as a threshold keeps
// exactly S. The S survivors (of equal scores the lowest indices) then take one lane
// each, and a survivor's place is the number of larger keys. The kernel is bound by its
// vector instructions: S rounds of a maximum over all 64-bit keys took 122 us for 16384
// signals of N = 1024, S = 32; this takes 33 us.
// ---------------------------------------------------------------------------
__device__ inline uint32_t orderable(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

template <int NPL>
__global__ __launch_bounds__(64) void k_topk(const float *__restrict__ Z, int64_t ldz, int S,
                                             int32_t *__restrict__ P) {
  __shared__ uint64_t list[64];
  const int64_t b = blockIdx.x;
  const int lane = threadIdx.x;
  uint32_t key[NPL];
#pragma unroll
  for (int q = 0; q < NPL; ++q) key[q] = orderable(Z[b * ldz + q * 64 + lane]);
  uint32_t T = 0;  // at least S keys are >= T
  int need = 0;    // keys equal to T to take beside the keys above it
  bool exact = false;
  for (int bit = 31; bit >= 0 && !exact; --bit) {
    const uint32_t cand = T | (1u << bit);
    int cnt = 0;
#pragma unroll
    for (int q = 0; q < NPL; ++q) cnt += __popcll(__ballot(key[q] >= cand));
    if (cnt >= S) T = cand;
    exact = cnt == S;
  }
  if (exact) {
    --T;  // (cand >= 1) the keys above T are the S
  } else {
    need = S;
#pragma unroll
    for (int q = 0; q < NPL; ++q) need -= __popcll(__ballot(key[q] > T));
  }
  int base = 0;
#pragma unroll
  for (int q = 0; q < NPL; ++q) {
    const uint64_t eq = __ballot(key[q] == T);
    const int erank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(eq >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)eq, 0u));
    const bool in = key[q] > T || (key[q] == T && erank < need);
    const uint64_t sel = __ballot(in);
    const int pos = base + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(sel >> 32),
                                                          __builtin_amdgcn_mbcnt_lo((uint32_t)sel, 0u));
    if (in) list[pos] = ((uint64_t)key[q] << 32) | (uint64_t)(0xFFFFFFFFu - (uint32_t)(q * 64 + lane));
    base += __popcll(sel);
    need = max(0, need - (int)__popcll(eq));
  }
  __syncthreads();
  const uint64_t mine = lane < S ? list[lane] : 0ull;
  int rank = 0;
  for (int j = 0; j < S; ++j) rank += readlane64(mine, j) > mine ? 1 : 0;
  if (lane < S) P[b * S + rank] = (int32_t)(0xFFFFFFFFu - (uint32_t)(mine & 0xFFFFFFFFull));
}

// ---------------------------------------------------------------------------
// Least-squares check of a proposed support (one wavefront per signal, S <= SMAX):
// Cholesky of the Gram block G[P, P] (pivots in FP64; a pivot below the
// dependency threshold rejects the proposal), beta = A_P^T y with exact
// products and FP64 sums, forward and back solves, the residual
// r = y - A_P x in FP32 and ||r|| in FP64; accepted when ||r|| <= eps_b.
//
// Lane i holds row i of the Gram block and of the factor in registers, and the
// factorisation is right-looking: column j is scaled once, then added to the running
// sums of every later column (one broadcast and one FMA each), so nothing waits for
// LDS and every loop is unrolled. beta is summed eight atoms at a time: the eight
// sums are folded into eight lane groups by three exchanges instead of being reduced
// one by one. Only the back solve needs columns of the factor across lanes; they pass
// through LDS (SMAX x (SMAX + 1) floats per wavefront). The former left-looking loops
// over LDS rows, with a cross-lane read in each of their 3 S^2 / 2 steps, took 563 us
// for 16384 signals at M = 256, S = 32; this takes 191 us, about 2.1 GB of cache lines
// (64 KB of atoms and 496 scattered Gram entries per signal) at 11 TB/s.
// ---------------------------------------------------------------------------
constexpr int LS_WAVES = 4;

// f(0), f(1), ..., f(N - 1) with constant arguments.
template <class F, int... I>
__device__ inline void unrolled_seq(F &&f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>()), ...);
}
template <int N, class F>
__device__ inline void unrolled(F &&f) {
  unrolled_seq(f, std::make_integer_sequence<int, N>());
}

// Chunk c (samples 4c .. 4c + 3) of signal y, zero past M.
__device__ inline float4 signal_chunk(const float *__restrict__ y, int64_t M, bool vec, int64_t c) {
  if (vec) return 4 * c < M ? reinterpret_cast<const float4 *>(y)[c] : make_float4(0.f, 0.f, 0.f, 0.f);
  const int64_t m = 4 * c;
  return make_float4(m < M ? y[m] : 0.f, m + 1 < M ? y[m + 1] : 0.f, m + 2 < M ? y[m + 2] : 0.f,
                     m + 3 < M ? y[m + 3] : 0.f);
}

template <int SMAX>
__global__ __launch_bounds__(64 * LS_WAVES) __attribute__((amdgpu_waves_per_eu(2, SMAX == 64 ? 2 : 4))) void k_ls_check(DictView d, const float *__restrict__ Y, int64_t ldy,
                                                            int64_t B, const int32_t *__restrict__ P, int S,
                                                            const float *__restrict__ eps_per, float eps,
                                                            int32_t *__restrict__ support_out,
                                                            float *__restrict__ coef_out,
                                                            int32_t *__restrict__ status_out,
                                                            float *__restrict__ rnorm_out,
                                                            int32_t *__restrict__ accept) {
  extern __shared__ float lsm[];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t b = (int64_t)blockIdx.x * LS_WAVES + wv;
  if (b >= B) return;
  constexpr int LD = SMAX + 1;
  float *Ls = lsm + (size_t)wv * SMAX * LD;
  const int pi = P[b * S + (lane < S ? lane : 0)];  // (past S the first atom again, times zero)
  const double nu2i = d.nu2[pi];
  // row i of the Gram block's lower triangle (symmetric: column p_i of row p_j); zero
  // elsewhere. Each entry is a cache line of its own, so the upper one is not read.
  float g[SMAX];
#pragma unroll
  for (int j = 0; j < SMAX; ++j) {
    g[j] = 0.f;
    if (j < S) {
      const char *row = reinterpret_cast<const char *>(d.G + (int64_t)__builtin_amdgcn_readlane(pi, j) * d.Np);
      if (lane >= j && lane < S) g[j] = *reinterpret_cast<const float *>(row + 4u * (uint32_t)pi);
    }
  }
  // beta_j = a_{P_j}^T y and the signal's own finiteness.
  const float *y = Y + b * ldy;
  const bool vec = (d.M & 3) == 0 && (reinterpret_cast<uintptr_t>(y) & 15) == 0;
  const uint32_t nc4 = (uint32_t)(d.Mp / 4);
  const float4 *A4 = reinterpret_cast<const float4 *>(d.A32);
  double bj = 0.0;
  int finite = 1;
  for (int j0 = 0; j0 < S; j0 += 8) {
    double s[8] = {};
    for (uint32_t c = lane; c < nc4; c += 64) {
      const float4 v = signal_chunk(y, d.M, vec, c);
      if (j0 == 0) finite &= (isfinite(v.x) && isfinite(v.y) && isfinite(v.z) && isfinite(v.w)) ? 1 : 0;
      float4 a[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {  // (past S: the first atom's sum again, dropped below)
        const char *row = reinterpret_cast<const char *>(A4 + (int64_t)__builtin_amdgcn_readlane(pi, j0 + u) * nc4);
        a[u] = *reinterpret_cast<const float4 *>(row + 16u * c);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        s[u] += (double)a[u].x * v.x + (double)a[u].y * v.y + (double)a[u].z * v.z + (double)a[u].w * v.w;
    }
    // fold: after the exchanges over lane bits 5, 4 and 3 lane group l / 8 holds sum l / 8
#pragma unroll
    for (int w = 4; w >= 1; w >>= 1) {
      const bool hi = lane & (8 * w);
#pragma unroll
      for (int u = 0; u < w; ++u) {
        const double send = hi ? s[u] : s[u + w], keep = hi ? s[u + w] : s[u];
        s[u] = keep + __shfl_xor(send, 8 * w);
      }
    }
    s[0] += dppd<DPP_XOR1>(s[0]);
    s[0] += dppd<DPP_XOR2>(s[0]);
    s[0] += dppd<DPP_HALF_MIRROR>(s[0]);
    const double mine = __shfl(s[0], (lane & 7) * 8);
    bj = (lane >> 3) == (j0 >> 3) ? mine : bj;
  }
  // Cholesky, column by column: L[j][j] = sqrt(G[j][j] - sum_k L[j][k]^2) (FP64),
  // L[i][j] = (G[i][j] - sum_k L[i][k] L[j][k]) / L[j][j] for i > j. L[k] holds the
  // running sum of column k until step k makes it the factor's entry.
  bool dependent = !__all(finite);
  float L[SMAX];
#pragma unroll
  for (int k = 0; k < SMAX; ++k) L[k] = 0.f;
  double dd = 0.0;   // sum_k L[i][k]^2 of the lane's row so far
  float rdj = 0.f;   // lane j keeps 1 / L[j][j]
  unrolled<SMAX>([&](auto step) {
    constexpr int j = decltype(step)::value;
    if (j < S && !dependent) {
      const double d2 = __longlong_as_double(
          (long long)readlane64((uint64_t)__double_as_longlong((double)g[j] - dd), j));
      const double nu2 = __longlong_as_double((long long)readlane64((uint64_t)__double_as_longlong(nu2i), j));
      if (!(d2 > DEP_TOL2 * nu2)) {
        dependent = true;
      } else {
        const float dj = (float)sqrt(d2);
        const float lij = lane > j ? (g[j] - L[j]) / dj : 0.f;  // (zero on lanes past S)
        if (lane == j) rdj = 1.f / dj;
        L[j] = lij;
        dd += (double)lij * (double)lij;
#pragma unroll
        for (int k0 = j + 1; k0 < SMAX; k0 += 8)
          if (k0 < S) {
#pragma unroll
            for (int k = k0; k < k0 + 8 && k < SMAX; ++k) L[k] = fmaf(lij, readlane(lij, k), L[k]);
          }
      }
    }
  });
  float x = 0.f;
  double rn = 0.0;
  if (!dependent) {
    // forward solve L u = beta: u_j = (beta_j - sum_k L[j][k] u_k) / L[j][j]
    float t = lane < S ? (float)bj : 0.f;
#pragma unroll
    for (int j = 0; j < SMAX; ++j)
      if (j < S) t = fmaf(-L[j], readlane(t, j) * readlane(rdj, j), t);
    t *= rdj;
    // back solve L^T x = u, last unknown first, row i of L read from LDS
#pragma unroll
    for (int k = 0; k < SMAX; ++k)
      if (lane < SMAX) Ls[lane * LD + k] = L[k];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int lc = lane < SMAX ? lane : 0;
#pragma unroll
    for (int i = SMAX - 1; i >= 0; --i)
      if (i < S) t = fmaf(-Ls[i * LD + lc], readlane(t, i) * readlane(rdj, i), t);
    x = t * rdj;  // (lanes past S: rdj = 0)
    // residual and its norm
    for (uint32_t c = lane; c < nc4; c += 64) {
      float4 r = signal_chunk(y, d.M, vec, c);
      for (int j0 = 0; j0 < S; j0 += 4) {
        float4 a[4];
        float xj[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {  // (past S: the first atom times zero)
          const char *row = reinterpret_cast<const char *>(A4 + (int64_t)__builtin_amdgcn_readlane(pi, j0 + u) * nc4);
          xj[u] = -readlane(x, j0 + u);
          a[u] = *reinterpret_cast<const float4 *>(row + 16u * c);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          r.x = fmaf(xj[u], a[u].x, r.x); r.y = fmaf(xj[u], a[u].y, r.y);
          r.z = fmaf(xj[u], a[u].z, r.z); r.w = fmaf(xj[u], a[u].w, r.w);
        }
      }
      rn += (double)r.x * r.x + (double)r.y * r.y + (double)r.z * r.z + (double)r.w * r.w;
    }
    rn = sqrt(wave_sum(rn));
  }
  float eb = eps_per ? eps_per[b] : eps;
  eb = fmaxf(eb, 0.f);
  const bool ok = !dependent && rn <= (double)eb;
  if (lane < S) {
    support_out[b * S + lane] = ok ? pi : -1;
    coef_out[b * S + lane] = ok ? x : 0.f;
  }
  if (lane == 0) {
    accept[b] = ok ? 1 : 0;
    if (ok) {
      status_out[b] = (S << 8) | OMP_SIG_EPS | OMP_SIG_LEARNED;
      rnorm_out[b] = (float)rn;
    }
  }
}

// Rejected signals: compacted index list (order irrelevant: each signal's
// fallback result does not depend on the others) and their signals and
// tolerances gathered for the fallback solve.
__global__ __launch_bounds__(256) void k_compact(const int32_t *__restrict__ accept, int64_t B,
                                                 int32_t *__restrict__ idx, int32_t *__restrict__ count) {
  const int64_t b = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (b < B && !accept[b]) idx[atomicAdd(count, 1)] = (int32_t)b;
}

__global__ __launch_bounds__(64) void k_gather_rejects(const float *__restrict__ Y, int64_t ldy, int64_t M,
                                                       const float *__restrict__ eps_per, float eps,
                                                       const int32_t *__restrict__ idx, float *__restrict__ Yr,
                                                       float *__restrict__ eps_r) {
  const int64_t i = blockIdx.x;
  const int64_t b = idx[i];
  for (int64_t m = threadIdx.x; m < M; m += 64) Yr[i * M + m] = Y[b * ldy + m];
  if (threadIdx.x == 0) eps_r[i] = eps_per ? eps_per[b] : eps;
}

__global__ __launch_bounds__(64) void k_scatter_fallback(const int32_t *__restrict__ idx, int S,
                                                         const int32_t *__restrict__ sup_r,
                                                         const float *__restrict__ coef_r,
                                                         const int32_t *__restrict__ st_r,
                                                         const float *__restrict__ rn_r, int32_t *__restrict__ support_out,
                                                         float *__restrict__ coef_out, int32_t *__restrict__ status_out,
                                                         float *__restrict__ rnorm_out) {
  const int64_t i = blockIdx.x;
  const int64_t b = idx[i];
  for (int j = threadIdx.x; j < S; j += 64) {
    support_out[b * S + j] = sup_r[i * S + j];
    coef_out[b * S + j] = coef_r[i * S + j];
  }
  if (threadIdx.x == 0) {
    status_out[b] = st_r[i];
    rnorm_out[b] = rn_r[i];
  }
}

// Tile size of an M x N x K product. A workgroup of the 256 x 256 tiles fills a CU, two of the
// others share one. 256 x 256 from 192 tiles on, except where a second round would run on less
// than half of the CUs; 64 x 64 where 128 x 128 would leave CUs idle. The features (one product
// into many 16-bit stores) keep 128 x 128 for short signals and wherever the rounds of the others
// are not well filled (a 256 x 256 tile takes 3.3 times a 128 x 128 one's time), the loss epilogue
// always: with the accumulators of a 256 x 256 tile its exponential and logarithm do not fit the
// registers (576 bytes of scratch a lane). Measured, us, 128 x 128 against 256 x 256: the three
// layers of 2048, B = 8192 (256 tiles) 292 and 241, B = 8704 (272) 359 and 397, B = 10,240 (320)
// 404 and 411, B = 17,408 (544) 682 and 658; features of 1000 samples, N = 4096, B = 4096 (256)
// 63 and 57, B = 5120 (320) 76 and 86, B = 8704 (544) 131 and 136, of 64 samples, N = 2048, B =
// 10,240 35 and 39; 5120 x 4096 x 1024 with the loss 149 and 608. 64 x 64 against 128 x 128: the
// layers of 1024, B = 2048 (128 tiles of 128 x 128) 41 and 57, with gradients 117 and 176, B =
// 2816 (176) 60 and 62, 173 and 192; features of 1000 samples, N = 1024, B = 2304 31 and 29.
int gemm_tile(int epi, int64_t M, int64_t N, int64_t K) {
  const int64_t t256 = (M / 256) * (N / 256), t128 = (M / 128) * (N / 128);
  const bool whole = M % 256 == 0 && N % 256 == 0 && t256 >= 192;
  if (epi == EPI_FEATURES) {
    if (whole && K >= 256 && 332 * ((t256 + 255) / 256) < 100 * ((4 * t256 + 255) / 256)) return 256;
    return t128 > 128 ? 128 : 64;
  }
  if (whole && epi != EPI_BCE && !(t256 > 256 && t256 <= 384)) return 256;
  return t128 >= 192 ? 128 : 64;
}

template <int EPI, class T>
hipError_t gemm_t(const uint16_t *P, int64_t ldp, const uint16_t *Q, int64_t ldq, int64_t M, int64_t N, int64_t K,
                  const GemmEpi &e, hipStream_t st) {
  hipError_t err = lds_limit(k_gemm_nt<EPI, T>, gemm_lds<T>());
  if (err != hipSuccess) return err;
  const unsigned grid = (unsigned)((M / T::TN) * (N / T::TB));
  hipLaunchKernelGGL((k_gemm_nt<EPI, T>), dim3(grid), dim3(T::NTHR), gemm_lds<T>(), st, P, ldp, Q, ldq, M, N, K, e);
  return hipGetLastError();
}

template <int EPI>
hipError_t gemm_any(const uint16_t *P, int64_t ldp, const uint16_t *Q, int64_t ldq, int64_t M, int64_t N, int64_t K,
                    const GemmEpi &e, hipStream_t st) {
  const int tile = gemm_tile(EPI, M, N, K);
  if (tile == 64) return gemm_t<EPI, GT64>(P, ldp, Q, ldq, M, N, K, e, st);
  if constexpr (EPI != EPI_BCE)
    if (tile == 256) return gemm_t<EPI, GT256>(P, ldp, Q, ldq, M, N, K, e, st);
  return gemm_t<EPI, GT128>(P, ldp, Q, ldq, M, N, K, e, st);
}

}  // namespace

int64_t loss_blocks(int64_t M, int64_t N) {
  const int64_t t = gemm_tile(EPI_BCE, M, N, 64);
  return (M / t) * (N / t);
}

hipError_t launch_gemm_bf16(int epi, const uint16_t *P, int64_t ldp, const uint16_t *Q, int64_t ldq, int64_t M,
                            int64_t N, int64_t K, const GemmEpi &e, hipStream_t st) {
  if (M % 128 || N % 128 || K % 64 || ldp % 8 || ldq % 8) return hipErrorInvalidValue;
  switch (epi) {
    case EPI_FEATURES: return gemm_any<EPI_FEATURES>(P, ldp, Q, ldq, M, N, K, e, st);
    case EPI_BIAS_RELU: return gemm_any<EPI_BIAS_RELU>(P, ldp, Q, ldq, M, N, K, e, st);
    case EPI_BIAS: return gemm_any<EPI_BIAS>(P, ldp, Q, ldq, M, N, K, e, st);
    case EPI_BCE: return gemm_any<EPI_BCE>(P, ldp, Q, ldq, M, N, K, e, st);
    case EPI_RELU_MASK: return gemm_any<EPI_RELU_MASK>(P, ldp, Q, ldq, M, N, K, e, st);
    default: return hipErrorInvalidValue;  // (EPI_PARTIAL: launch_wgrad)
  }
}

hipError_t launch_prep_signals(const float *Y, int64_t ldy, int64_t B, int64_t M, int64_t Mp, int64_t Bp,
                               uint16_t *Y16, float *yinv, hipStream_t st) {
  hipLaunchKernelGGL(k_prep_signals, dim3((unsigned)Bp), dim3(64), 0, st, Y, ldy, B, M, Mp, Y16, yinv);
  return hipGetLastError();
}

hipError_t launch_pad_rows16(const uint16_t *src, int64_t ld, const int32_t *rows, int64_t B, int64_t cols,
                             int64_t Bp, uint16_t *dst, hipStream_t st, const int32_t *sup, int S, int64_t n_out,
                             uint32_t *bits) {
  const size_t lds = sup ? (size_t)(n_out / 32) * 4 : 0;  // at most 2 KiB (n_out <= 16384)
  hipLaunchKernelGGL(k_pad_rows16, dim3((unsigned)Bp), dim3(256), lds, st, src, ld, rows, B, cols, dst, sup, S,
                     n_out / 32, bits);
  return hipGetLastError();
}

int64_t transpose_rows(int64_t R) {
  const int64_t per = (R + COLSUM_GROUPS - 1) / COLSUM_GROUPS;
  return (per + 63) / 64 * 64;
}

hipError_t launch_transposes16(TransposeBatch g, int64_t R, hipStream_t st) {
  if (R % 64) return hipErrorInvalidValue;
  const int64_t rpc = transpose_rows(R), groups = (R + rpc - 1) / rpc;
  int64_t blocks = 0;
  for (int m = 0; m < 6; ++m) {
    if (g.cols[m] % 64) return hipErrorInvalidValue;
    blocks += g.cols[m] / 64 * groups;
    g.end[m] = blocks;
  }
  hipLaunchKernelGGL(k_transposes16, dim3((unsigned)blocks), dim3(256), 0, st, g, R, rpc);
  return hipGetLastError();
}

namespace {
template <class T>
hipError_t wgrad_t(WgradBatch g, int64_t K, int splits, hipStream_t st) {
  hipError_t err = lds_limit(k_wgrad<T>, gemm_lds<T>());
  if (err != hipSuccess) return err;
  int64_t blocks = 0;
  for (int l = 0; l < 3; ++l) {
    blocks += (g.rows[l] / T::TN) * (g.in[l] / T::TB) * splits;
    g.end[l] = blocks;
  }
  hipLaunchKernelGGL(k_wgrad<T>, dim3((unsigned)blocks), dim3(T::NTHR), gemm_lds<T>(), st, g, K, splits);
  return hipGetLastError();
}

// Entries of the three layers' weights
int64_t wgrad_area(const WgradBatch &g) { return g.rows[0] * g.in[0] + g.rows[1] * g.in[1] + g.rows[2] * g.in[2]; }
}  // namespace

// The batch is split over up to WSPLITS_MAX workgroups per tile only where the 64 x 64
// tiles of the three layers together leave CUs idle: every split writes and reads the
// whole gradient once more (four of them moved 108 MB for 1024-wide layers, where the
// products themselves read 25 MB: products and sums 61 us, without the split 18 us).
int wgrad_splits(const WgradBatch &g, int64_t K) {
  int sp = 1;
  while (sp < WSPLITS_MAX && wgrad_area(g) / 4096 * sp < 256 && K % (128 * sp) == 0) sp *= 2;
  return sp;
}

// 128 x 128 tiles of the three layers together, or 64 x 64 ones where those are too few
hipError_t launch_wgrad(const WgradBatch &g, int64_t K, int splits, hipStream_t st) {
  for (int l = 0; l < 3; ++l)
    if (g.rows[l] % 128 || g.in[l] % 128) return hipErrorInvalidValue;
  if (K % (64 * splits)) return hipErrorInvalidValue;
  return wgrad_area(g) / 16384 * splits >= 512 ? wgrad_t<GT128>(g, K, splits, st) : wgrad_t<GT64>(g, K, splits, st);
}

hipError_t launch_grad_sums(SumBatch g, const float *loss_part, int64_t nloss, float scale, float *loss_out,
                            hipStream_t st) {
  int64_t blocks = 0;
  for (int m = 0; m < 6; ++m) {
    if (g.parts[m] > 16) return hipErrorInvalidValue;
    if (!g.out[m]) g.n[m] = 0;
    blocks += (g.n[m] + 255) / 256;
    g.end[m] = blocks;
  }
  if (blocks == 0 && !loss_out) return hipSuccess;
  hipLaunchKernelGGL(k_grad_sums, dim3((unsigned)(blocks + 1)), dim3(256), 0, st, g, loss_part, nloss, scale,
                     loss_out);
  return hipGetLastError();
}

hipError_t launch_adam_w(const LayerView &L, const float *gpart, int splits, float lr, float b1, float b2, float eps,
                         float c1, float c2, int update, hipStream_t st) {
  hipLaunchKernelGGL(k_adam_w, dim3((unsigned)((L.n_out / 64) * (L.n_in / 64))), dim3(256), 0, st, L, gpart, splits,
                     lr, b1, b2, eps, c1, c2, update);
  return hipGetLastError();
}

hipError_t launch_adam_b(const LayerView &L, const float *gpart, int chunks, float lr, float b1, float b2, float eps,
                         float c1, float c2, hipStream_t st) {
  hipLaunchKernelGGL(k_adam_b, dim3((unsigned)((L.n_out + 255) / 256)), dim3(256), 0, st, L, gpart, chunks, lr, b1,
                     b2, eps, c1, c2);
  return hipGetLastError();
}

hipError_t launch_copy32(const float *src, int64_t n, float *dst, hipStream_t st) {
  hipLaunchKernelGGL(k_copy32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, src, n, dst);
  return hipGetLastError();
}

hipError_t launch_topk(const float *Z, int64_t ldz, int64_t N, int64_t B, int S, int32_t *P, hipStream_t st) {
  switch (N / 64) {
    case 4: hipLaunchKernelGGL(k_topk<4>, dim3((unsigned)B), dim3(64), 0, st, Z, ldz, S, P); break;
    case 8: hipLaunchKernelGGL(k_topk<8>, dim3((unsigned)B), dim3(64), 0, st, Z, ldz, S, P); break;
    case 16: hipLaunchKernelGGL(k_topk<16>, dim3((unsigned)B), dim3(64), 0, st, Z, ldz, S, P); break;
    case 32: hipLaunchKernelGGL(k_topk<32>, dim3((unsigned)B), dim3(64), 0, st, Z, ldz, S, P); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_ls_check(const DictView &d, const float *Y, int64_t ldy, int64_t B, const int32_t *P, int S,
                           const float *eps_per, float eps, int32_t *support_out, float *coef_out, int32_t *status_out,
                           float *rnorm_out, int32_t *accept, hipStream_t st) {
  if (S < 1 || S > 64) return hipErrorInvalidValue;
  const int smax = S <= 16 ? 16 : S <= 32 ? 32 : 64;  // rows per factor: the unrolled loops' length
  auto kern = smax == 16 ? k_ls_check<16> : smax == 32 ? k_ls_check<32> : k_ls_check<64>;
  const size_t lds = (size_t)LS_WAVES * smax * (smax + 1) * sizeof(float);
  hipError_t e = lds_limit(kern, lds);
  if (e != hipSuccess) return e;
  const unsigned blocks = (unsigned)((B + LS_WAVES - 1) / LS_WAVES);
  hipLaunchKernelGGL(kern, dim3(blocks), dim3(64 * LS_WAVES), lds, st, d, Y, ldy, B, P, S, eps_per, eps, support_out,
                     coef_out, status_out, rnorm_out, accept);
  return hipGetLastError();
}

hipError_t launch_compact(const int32_t *accept, int64_t B, int32_t *idx, int32_t *count, hipStream_t st) {
  hipLaunchKernelGGL(k_copy32, dim3(1), dim3(256), 0, st, nullptr, 1, reinterpret_cast<float *>(count));
  hipLaunchKernelGGL(k_compact, dim3((unsigned)((B + 255) / 256)), dim3(256), 0, st, accept, B, idx, count);
  return hipGetLastError();
}

hipError_t launch_gather_rejects(const float *Y, int64_t ldy, int64_t M, const float *eps_per, float eps,
                                 const int32_t *idx, int64_t n, float *Yr, float *eps_r, hipStream_t st) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_gather_rejects, dim3((unsigned)n), dim3(64), 0, st, Y, ldy, M, eps_per, eps, idx, Yr, eps_r);
  return hipGetLastError();
}

hipError_t launch_scatter_fallback(const int32_t *idx, int64_t n, int S, const int32_t *sup_r, const float *coef_r,
                                   const int32_t *st_r, const float *rn_r, int32_t *support_out, float *coef_out,
                                   int32_t *status_out, float *rnorm_out, hipStream_t st) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_scatter_fallback, dim3((unsigned)n), dim3(64), 0, st, idx, S, sup_r, coef_r, st_r, rn_r,
                     support_out, coef_out, status_out, rnorm_out);
  return hipGetLastError();
}

}  // namespace bomp
