// Warm-start network: forward, loss gradient and Adam on gfx950.
//
// Three dense layers over the spots of one patient (rows of X, B x F):
//   h1 = relu(X W1^T + b1), h2 = relu(h1 W2^T + b2), y = softplus(h2 . w3 + b3)
// and a penalty head lr = mean_b(h2) . wr + br.  Loss
//   L = mean_b (y_b - t_b)^2 + lam (lr - lr_t)^2.
// Flat parameter order W1, b1, W2, b2, w3, b3, wr, br (float32).
//
// A training step is five launches: k_mlp_forward (both layers, the intensity
// head and the block's share of mean(h2) and of the loss), k_mlp_scalars
// (penalty head, loss, dL/dlr), k_mlp_backward (dz3, dz2 and, through W2, dz1),
// k_mlp_wgrad (every weight and bias gradient, row ranges apart) and
// k_mlp_grads (their sums).  The layer products run on the fp32 16x16x4 MFMA,
// the sums over rows (weight gradients, mean, loss) in fp64 in a fixed order,
// so gradients are deterministic.  The sizes are small (B about 3 000, H =
// 128: 0.3 GFLOP a step), so launches and dependent loads bound a step, not
// arithmetic: with one thread walking all B rows of every weight gradient,
// mean and loss sum, a step took 3.2 ms at B = 2 981, H = 128 (2.9 ms in those
// sums); now 0.147 ms with its copies and the Adam step: forward 18 us, scalars
// 6, backward 11, weight gradients 15, their sums 5.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <exception>
#include <new>
#include <string>
#include <vector>

#include "../../include/admmbb.h"
#include "scalars.h"

namespace {

using admmbb::group_allsum;

typedef float v4f __attribute__((ext_vector_type(4)));
typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int kRows = 16;  // rows per block of the layer kernels: one MFMA tile
constexpr int kNt = 256;   // threads of every kernel but k_mlp_scalars

struct HipErr {
  hipError_t e;
};
inline void ck(hipError_t e) {
  if (e != hipSuccess) throw HipErr{e};
}

__device__ __forceinline__ float bf16_round(float x) {
  uint32_t u = __float_as_uint(x);
  u += 0x7fffu + ((u >> 16) & 1u);
  return __uint_as_float(u & 0xffff0000u);
}

// LDS row stride (floats) of an activation tile with n columns: whole
// four-column steps (zero beyond n) and four more, so that for n a multiple of
// 64 the 16 rows that one load instruction reads start in different banks.
__host__ __device__ __forceinline__ int lds_stride(int n) { return ((n + 3) & ~3) + 4; }

// Everything the kernels address, by value.
struct MlpArgs {
  const float* X;  // B x F
  const float* t;  // B, or nullptr (no loss)
  float *z1, *z2;  // B x H pre-activations kept for the backward pass (nullptr: inference)
  float *z3, *y, *dz3, *dz2, *dz1, *pooled;
  const float* th;   // parameters
  double* blk;       // per forward block: H sums of h2 over its rows, then its sum of (y - t)^2
  double* sc;        // lr, L, dL/dlr
  double* part;      // per row range: np gradient sums
  float* g;          // gradient
  int64_t oW1, ob1, oW2, ob2, ow3, ob3, owr, obr, np;
  int B, F, H, nblk, splits, rows_per_split;
  float lr_t, lam;
};

// One layer of a block: dst[r][k] = bias[k] + sum_i src[r][i] W[k][i] for its 16
// rows, columns k in 16-wide groups dealt to the four waves.  Each MFMA step
// takes four consecutive i in ascending order (lane l: row or column l % 16,
// i = l / 16 of the four), which gives the sums of a plain ascending fma chain.
// src is zero beyond nin.  fin(r, k, v) receives every entry.
template <class Fin>
__device__ __forceinline__ void layer_rows(const float* src, int ss, int nin, const float* __restrict__ W,
                                           const float* __restrict__ bias, int H, Fin fin) {
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63, m = l & 15, kk = l >> 4;
  for (int k0 = 16 * w; k0 < H; k0 += 64) {
    const int k = k0 + m;
    const float* wk = W + static_cast<int64_t>(k < H ? k : H - 1) * nin + kk;
    const float* sm = src + m * ss + kk;
    v4f acc = {0.0f, 0.0f, 0.0f, 0.0f};
    int i0 = 0;
    for (; i0 + 64 <= nin; i0 += 64) {
      float b[16];
#pragma unroll
      for (int q = 0; q < 16; ++q) b[q] = wk[i0 + 4 * q];
#pragma unroll
      for (int q = 0; q < 16; ++q) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(sm[i0 + 4 * q], b[q], acc, 0, 0, 0);
    }
    for (; i0 < nin; i0 += 4)
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(sm[i0], i0 + kk < nin ? wk[i0] : 0.0f, acc, 0, 0, 0);
    // item r of the lane: row 4 (l / 16) + r, column k0 + l % 16
    if (k < H) {
      const float bk = bias[k];
#pragma unroll
      for (int r = 0; r < 4; ++r) fin(4 * kk + r, k, acc[r] + bk);
    }
  }
}

// Both layers and the intensity head of 16 rows.  BF16 (inference): the hidden
// activations rounded to bf16 as they are stored in LDS, weights and sums fp32.
// LDS: the input tile, later h2 (the input is dead by then), and h1.
template <bool BF16>
__global__ __launch_bounds__(kNt) void k_mlp_forward(MlpArgs a) {
  extern __shared__ __align__(16) float smem[];
  __shared__ float ysh[kRows];
  const int H = a.H, F = a.F, B = a.B;
  const int sF = lds_stride(F), sH = lds_stride(H);
  float* h1 = smem;               // kRows x sH
  float* xs = smem + kRows * sH;  // kRows x max(sF, sH)
  const int b0 = static_cast<int>(blockIdx.x) * kRows;
  const int nr = B - b0 < kRows ? B - b0 : kRows;
  const int tid = threadIdx.x;
  for (int e = tid; e < kRows * sF; e += kNt) {
    const int r = e / sF, i = e - r * sF;
    xs[e] = (r < nr && i < F) ? a.X[static_cast<int64_t>(b0 + r) * F + i] : 0.0f;
  }
  // zero columns H .. of the hidden tiles: the next product reads whole groups
  for (int e = tid; e < kRows * (sH - H); e += kNt) h1[(e / (sH - H)) * sH + H + e % (sH - H)] = 0.0f;
  __syncthreads();
  auto act = [](float v) {
    v = fmaxf(v, 0.0f);
    return BF16 ? bf16_round(v) : v;
  };
  layer_rows(xs, sF, F, a.th + a.oW1, a.th + a.ob1, H, [&](int r, int k, float v) {
    h1[r * sH + k] = act(v);
    if (!BF16 && a.z1 != nullptr && r < nr) a.z1[static_cast<int64_t>(b0 + r) * H + k] = v;
  });
  __syncthreads();
  float* h2 = xs;
  layer_rows(h1, sH, H, a.th + a.oW2, a.th + a.ob2, H, [&](int r, int k, float v) {
    h2[r * sH + k] = act(v);
    if (!BF16 && a.z2 != nullptr && r < nr) a.z2[static_cast<int64_t>(b0 + r) * H + k] = v;
  });
  __syncthreads();
  {
    // 16 lanes a row
    const int r = tid >> 4, c = tid & 15;
    const float* w3 = a.th + a.ow3;
    float s = 0.0f;
    for (int k = c; k < H; k += 16) s = fmaf(h2[r * sH + k], w3[k], s);
    s = group_allsum<16>(s);
    if (c == 0) {
      const float z = s + a.th[a.ob3];
      const float y = fmaxf(z, 0.0f) + log1pf(expf(-fabsf(z)));
      ysh[r] = y;
      if (r < nr) {
        if (a.z3 != nullptr) a.z3[b0 + r] = z;
        a.y[b0 + r] = y;
      }
    }
  }
  double* bp = a.blk + static_cast<int64_t>(blockIdx.x) * (H + 1);
  for (int k = tid; k < H; k += kNt) {
    double s = 0.0;
    for (int r = 0; r < nr; ++r) s += static_cast<double>(h2[r * sH + k]);
    bp[k] = s;
  }
  __syncthreads();
  if (tid == 0) {
    double se = 0.0;
    if (a.t != nullptr)
      for (int r = 0; r < nr; ++r) {
        const double d = static_cast<double>(ysh[r]) - static_cast<double>(a.t[b0 + r]);
        se += d * d;
      }
    bp[H] = se;
  }
}

// pooled = mean_b(h2), lr, the loss and dL/dlr from the forward blocks' sums:
// one workgroup; column k's blocks are dealt to nsl threads (as many as 1024
// threads give every column), their sums added in order, so nothing depends on
// timing.
__global__ __launch_bounds__(1024) void k_mlp_scalars(MlpArgs a) {
  __shared__ double sh[1024];
  __shared__ double wsum[16];
  __shared__ double se;  // sum of squared errors (the last column)
  const int tid = threadIdx.x, H = a.H, C = H + 1;
  const int w = C < 1024 ? C : 1024;
  const int nsl = 1024 / w;
  double lr = 0.0;
  for (int c0 = 0; c0 < C; c0 += w) {
    const int c = c0 + tid % w, sl = tid / w;
    double s = 0.0;
    if (sl < nsl && c < C) {
      int b = sl;
      for (; b + 7 * nsl < a.nblk; b += 8 * nsl) {
        double q[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) q[u] = a.blk[static_cast<int64_t>(b + u * nsl) * C + c];
#pragma unroll
        for (int u = 0; u < 8; ++u) s += q[u];
      }
      for (; b < a.nblk; b += nsl) s += a.blk[static_cast<int64_t>(b) * C + c];
    }
    sh[tid] = s;
    __syncthreads();
    if (sl == 0 && c < C) {
      for (int u = 1; u < nsl; ++u) s += sh[u * w + tid];
      if (c < H) {
        const float p = static_cast<float>(s / a.B);
        a.pooled[c] = p;
        lr += static_cast<double>(p) * static_cast<double>(a.th[a.owr + c]);
      } else {
        se = s;
      }
    }
    __syncthreads();
  }
  lr = group_allsum<64>(lr);
  if ((tid & 63) == 0) wsum[tid >> 6] = lr;
  __syncthreads();
  if (tid == 0) {
    double s = static_cast<double>(a.th[a.obr]);
    for (int q = 0; q < 16; ++q) s += wsum[q];
    const double d = s - static_cast<double>(a.lr_t), lam = static_cast<double>(a.lam);
    a.sc[0] = s;
    a.sc[1] = se / a.B + lam * d * d;
    a.sc[2] = 2.0 * lam * d;
  }
}

// Of 16 rows: dz3 = 2 (y - t) / B sigmoid(z3), dz2 = (dz3 w3 + dL/dlr wr / B)
// [z2 > 0] and dz1 = (dz2 W2) [z1 > 0] by the MFMA, operands as in layer_rows
// with W2 read down its columns (64 contiguous bytes per row and load).
__global__ __launch_bounds__(kNt) void k_mlp_backward(MlpArgs a) {
  extern __shared__ __align__(16) float smem[];
  __shared__ float d3[kRows];
  const int H = a.H, B = a.B, sH = lds_stride(H);
  const int b0 = static_cast<int>(blockIdx.x) * kRows;
  const int nr = B - b0 < kRows ? B - b0 : kRows;
  const int tid = threadIdx.x;
  if (tid < kRows) {
    float d = 0.0f;
    if (tid < nr) {
      const float s = 1.0f / (1.0f + expf(-a.z3[b0 + tid]));
      d = 2.0f * (a.y[b0 + tid] - a.t[b0 + tid]) / B * s;
      a.dz3[b0 + tid] = d;
    }
    d3[tid] = d;
  }
  __syncthreads();
  const float dlr = static_cast<float>(a.sc[2]);
  for (int e = tid; e < kRows * sH; e += kNt) {
    const int r = e / sH, k = e - r * sH;
    float v = 0.0f;
    if (r < nr && k < H) {
      const int64_t o = static_cast<int64_t>(b0 + r) * H + k;
      const float g = d3[r] * a.th[a.ow3 + k] + dlr * a.th[a.owr + k] / B;
      v = a.z2[o] > 0.0f ? g : 0.0f;
      a.dz2[o] = v;
    }
    smem[e] = v;
  }
  __syncthreads();
  const int w = tid >> 6, l = tid & 63, m = l & 15, kk = l >> 4;
  const float* W2 = a.th + a.oW2;
  for (int i0 = 16 * w; i0 < H; i0 += 64) {
    const int i = i0 + m, ic = i < H ? i : H - 1;
    v4f acc = {0.0f, 0.0f, 0.0f, 0.0f};
    const float* sm = smem + m * sH + kk;
    const float* wp = W2 + static_cast<int64_t>(kk) * H + ic;
    int k0 = 0;
    for (; k0 + 64 <= H; k0 += 64) {
      float b[16];
#pragma unroll
      for (int q = 0; q < 16; ++q) b[q] = wp[static_cast<int64_t>(k0 + 4 * q) * H];
#pragma unroll
      for (int q = 0; q < 16; ++q) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(sm[k0 + 4 * q], b[q], acc, 0, 0, 0);
    }
    for (; k0 < H; k0 += 4)
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(sm[k0], k0 + kk < H ? wp[static_cast<int64_t>(k0) * H] : 0.0f, acc, 0,
                                                 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 4 * kk + r;
      if (i < H && row < nr) {
        const int64_t o = static_cast<int64_t>(b0 + row) * H + i;
        a.dz1[o] = a.z1[o] > 0.0f ? acc[r] : 0.0f;
      }
    }
  }
}

// Weight and bias gradients of one layer as one product over rows:
// gW[k][i] = sum_b dz[b][k] act(in[b][i]), gb[k] with a column of ones at
// i = nin.  Three layers: (dz1, X), (dz2, relu z1) and (dz3, relu z2; one k).
struct Layer {
  const float *dz, *in;
  int K, nin, relu;
  int64_t oW, ob;
};
__device__ __forceinline__ Layer layer_of(const MlpArgs& a, int which) {
  if (which == 0) return Layer{a.dz2, a.z1, a.H, a.H, 1, a.oW2, a.ob2};
  if (which == 1) return Layer{a.dz1, a.X, a.H, a.F, 0, a.oW1, a.ob1};
  return Layer{a.dz3, a.z2, 1, a.H, 1, a.ow3, a.ob3};
}
__host__ __device__ __forceinline__ int wgrad_tiles(int K, int nin) { return ((K + 63) / 64) * ((nin + 64) / 64); }

// One 64 x 64 tile of one layer's gradient over one range of rows: wave w takes
// 16 k and up to four 16-column groups on the fp64 16x16x4 MFMA, four rows a
// step, operands straight from memory (64 contiguous bytes per row; the
// activations are L2-resident).  Row ranges make enough blocks to fill the
// chip (see admm_mlp::plan); their sums go to part, one slice per range.
__global__ __launch_bounds__(kNt) void k_mlp_wgrad(MlpArgs a) {
  int tile = static_cast<int>(blockIdx.x), which = 0;
  for (; which < 2; ++which) {
    const Layer q = layer_of(a, which);
    const int n = wgrad_tiles(q.K, q.nin);
    if (tile < n) break;
    tile -= n;
  }
  const Layer L = layer_of(a, which);
  const int ni = (L.nin + 64) / 64;
  const int k0 = (tile / ni) * 64 + 16 * static_cast<int>(threadIdx.x >> 6), i0 = (tile % ni) * 64;
  if (k0 >= L.K) return;
  const int l = threadIdx.x & 63, m = l & 15, kk = l >> 4;
  const int k = k0 + m;
  int ng = (L.nin + 1 - i0 + 15) / 16;  // column groups of the tile, the ones column included
  if (ng > 4) ng = 4;
  const int s = static_cast<int>(blockIdx.y);
  const int r0 = s * a.rows_per_split;
  const int r1 = r0 + a.rows_per_split < a.B ? r0 + a.rows_per_split : a.B;
  v4d acc[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) acc[g] = v4d{0.0, 0.0, 0.0, 0.0};
  // addresses: a wave-uniform base per step and the lane's offset within four
  // rows, fixed over the loop; columns clamped into the arrays
  bool one[4];
  int off[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int i = i0 + 16 * g + m;
    one[g] = i >= L.nin;  // the ones column (and, beyond it, columns not written)
    off[g] = kk * L.nin + (one[g] ? L.nin - 1 : i);
  }
  const int offz = kk * L.K + (k < L.K ? k : L.K - 1);
  auto step = [&](float av, const float* bv) {
#pragma unroll
    for (int g = 0; g < 4; ++g)
      if (g < ng) {
        const float v = one[g] ? 1.0f : (L.relu ? fmaxf(bv[g], 0.0f) : bv[g]);
        acc[g] =
            __builtin_amdgcn_mfma_f64_16x16x4f64(static_cast<double>(av), static_cast<double>(v), acc[g], 0, 0, 0);
      }
  };
  constexpr int U = 8;  // steps of a round, whose loads are in flight together
  int b = r0;
  for (; b + 4 * U <= r1; b += 4 * U) {
    float av[U], bv[U][4];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      av[u] = (L.dz + static_cast<int64_t>(b + 4 * u) * L.K)[offz];
      const float* in = L.in + static_cast<int64_t>(b + 4 * u) * L.nin;
#pragma unroll
      for (int g = 0; g < 4; ++g) bv[u][g] = in[off[g]];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) step(av[u], bv[u]);
  }
  for (; b < r1; b += 4) {
    // rows past the range: a valid row's data, and dz = 0
    const int up = b + kk < r1 ? 0 : b + kk - (r1 - 1);
    float av = (L.dz + static_cast<int64_t>(b) * L.K)[offz - up * L.K], bv[4];
    if (up > 0) av = 0.0f;
    const float* in = L.in + static_cast<int64_t>(b) * L.nin;
#pragma unroll
    for (int g = 0; g < 4; ++g) bv[g] = in[off[g] - up * L.nin];
    step(av, bv);
  }
  // item r of the lane: k index l / 16 + 4 r, column l % 16
  double* out = a.part + static_cast<int64_t>(s) * a.np;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int i = i0 + 16 * g + m;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int ko = k0 + kk + 4 * r;
      if (ko >= L.K || i > L.nin) continue;
      if (i < L.nin)
        out[L.oW + static_cast<int64_t>(ko) * L.nin + i] = acc[g][r];
      else
        out[L.ob + ko] = acc[g][r];
    }
  }
}

// g = sum of the row ranges' parts in order; the penalty head's gradients
__global__ __launch_bounds__(kNt) void k_mlp_grads(MlpArgs a) {
  const int64_t j = static_cast<int64_t>(blockIdx.x) * kNt + threadIdx.x;
  if (j >= a.np) return;
  if (j >= a.owr) {
    const float dlr = static_cast<float>(a.sc[2]);
    a.g[j] = j < a.obr ? dlr * a.pooled[j - a.owr] : dlr;
    return;
  }
  double s = 0.0;
  int p = 0;
  for (; p + 8 <= a.splits; p += 8) {
    double q[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) q[u] = a.part[(p + u) * a.np + j];
#pragma unroll
    for (int u = 0; u < 8; ++u) s += q[u];
  }
  for (; p < a.splits; ++p) s += a.part[p * a.np + j];
  a.g[j] = static_cast<float>(s);
}

__global__ void k_adam(float* __restrict__ th, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, int64_t n, float lr, float b1, float b2, float eps, float c1, float c2) {
  const int64_t j = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (j >= n) return;
  const float gj = g[j];
  const float mj = b1 * m[j] + (1.0f - b1) * gj;
  const float vj = b2 * v[j] + (1.0f - b2) * gj * gj;
  m[j] = mj;
  v[j] = vj;
  th[j] -= lr * (mj / c1) / (sqrtf(vj / c2) + eps);
}

uint64_t splitmix64(uint64_t& s) {
  uint64_t z = (s += 0x9E3779B97F4A7C15ull);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

thread_local std::string g_mlp_error;

}  // namespace

struct admm_mlp {
  int F = 0, H = 0;
  int64_t np = 0;
  hipStream_t stream = nullptr;
  bool own_stream = false;
  float *th = nullptr, *g = nullptr, *m = nullptr, *v = nullptr;
  int cap = 0;  // rows the activation buffers hold
  float *X = nullptr, *t = nullptr, *z1 = nullptr, *z2 = nullptr, *z3 = nullptr, *y = nullptr, *dz3 = nullptr;
  float *dz2 = nullptr, *dz1 = nullptr, *pooled = nullptr;
  double *blk = nullptr, *part = nullptr;
  double* sc = nullptr;
  double* h_sc = nullptr;
  int64_t step = 0;
  // parameter offsets
  int64_t oW1, ob1, oW2, ob2, ow3, ob3, owr, obr;

  ~admm_mlp() {
    if (stream) (void)hipStreamSynchronize(stream);
    for (void* p : {static_cast<void*>(th), static_cast<void*>(g), static_cast<void*>(m), static_cast<void*>(v)})
      if (p) (void)hipFree(p);
    free_rows();
    if (part) (void)hipFree(part);
    if (sc) (void)hipFree(sc);
    if (h_sc) (void)hipHostFree(h_sc);
    if (own_stream && stream) (void)hipStreamDestroy(stream);
  }
  void free_rows() {
    for (float* p : {X, t, z1, z2, z3, y, dz3, dz2, dz1, pooled})
      if (p) (void)hipFree(p);
    if (blk) (void)hipFree(blk);
    X = t = z1 = z2 = z3 = y = dz3 = dz2 = dz1 = pooled = nullptr;
    blk = nullptr;
    cap = 0;
  }
  void ensure(int B) {
    if (B <= cap) return;
    free_rows();
    const int c = std::max(B, 1024);
    auto a = [&](float** p, int64_t n) { ck(hipMalloc(reinterpret_cast<void**>(p), sizeof(float) * n)); };
    a(&X, static_cast<int64_t>(c) * F);
    a(&t, c);
    a(&z1, static_cast<int64_t>(c) * H);
    a(&z2, static_cast<int64_t>(c) * H);
    a(&z3, c);
    a(&y, c);
    a(&dz3, c);
    a(&dz2, static_cast<int64_t>(c) * H);
    a(&dz1, static_cast<int64_t>(c) * H);
    a(&pooled, H);
    ck(hipMalloc(reinterpret_cast<void**>(&blk), sizeof(double) * ((c + kRows - 1) / kRows) * (H + 1)));
    cap = c;
  }
  // Row ranges of the weight gradients, whole rounds of 32 rows: the tiles of
  // all three layers times the ranges make up to 640 blocks (B = 2 981, H = 128:
  // 11 tiles, 47 ranges of 64 rows).  Longer ranges leave the chip idle behind
  // the rounds' load latency, shorter ones only write more parts.
  int max_splits() const {
    const int tiles = wgrad_tiles(H, H) + wgrad_tiles(H, F) + wgrad_tiles(1, H);
    return std::max(1, 640 / tiles);
  }
  MlpArgs plan(int B) const {
    MlpArgs a{};
    a.X = X;
    a.t = t;
    a.z1 = z1;
    a.z2 = z2;
    a.z3 = z3;
    a.y = y;
    a.dz3 = dz3;
    a.dz2 = dz2;
    a.dz1 = dz1;
    a.pooled = pooled;
    a.th = th;
    a.blk = blk;
    a.sc = sc;
    a.part = part;
    a.g = g;
    a.oW1 = oW1;
    a.ob1 = ob1;
    a.oW2 = oW2;
    a.ob2 = ob2;
    a.ow3 = ow3;
    a.ob3 = ob3;
    a.owr = owr;
    a.obr = obr;
    a.np = np;
    a.B = B;
    a.F = F;
    a.H = H;
    a.nblk = (B + kRows - 1) / kRows;
    const int want = std::min(max_splits(), std::max(1, B / 64));
    a.rows_per_split = ((B + want - 1) / want + 31) & ~31;
    a.splits = (B + a.rows_per_split - 1) / a.rows_per_split;
    return a;
  }
  // on the net's own stream, which the null stream does not wait for, nor it for that
  void clear_moments() {
    admmbb::launch_fill_f32(m, 0.0f, np, stream);
    admmbb::launch_fill_f32(v, 0.0f, np, stream);
  }
  // the layers and the scalars
  void forward(const MlpArgs& a, bool bf16) {
    const int smem = 4 * kRows * (lds_stride(H) + std::max(lds_stride(F), lds_stride(H)));
    auto kern = bf16 ? k_mlp_forward<true> : k_mlp_forward<false>;
    if (smem > 65536)
      ck(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, smem));
    hipLaunchKernelGGL(kern, dim3(a.nblk), dim3(kNt), smem, stream, a);
    hipLaunchKernelGGL(k_mlp_scalars, dim3(1), dim3(1024), 0, stream, a);
  }
  void backward(const MlpArgs& a) {
    const int smem = 4 * kRows * lds_stride(H);
    if (smem > 65536)
      ck(hipFuncSetAttribute(reinterpret_cast<const void*>(k_mlp_backward), hipFuncAttributeMaxDynamicSharedMemorySize,
                             smem));
    hipLaunchKernelGGL(k_mlp_backward, dim3(a.nblk), dim3(kNt), smem, stream, a);
    const int tiles = wgrad_tiles(H, H) + wgrad_tiles(H, F) + wgrad_tiles(1, H);
    hipLaunchKernelGGL(k_mlp_wgrad, dim3(tiles, a.splits), dim3(kNt), 0, stream, a);
    hipLaunchKernelGGL(k_mlp_grads, dim3(static_cast<unsigned>((np + kNt - 1) / kNt)), dim3(kNt), 0, stream, a);
  }
};

namespace {
admm_status mlp_fail(admm_mlp* n, const char* what, hipError_t e) {
  (void)n;
  g_mlp_error = std::string(what) + ": " + hipGetErrorString(e);
  return e == hipErrorOutOfMemory ? ADMM_E_OOM : ADMM_E_HIP;
}
}  // namespace

extern "C" {

const char* mlp_last_error(void) { return g_mlp_error.c_str(); }

admm_status mlp_create(int32_t nin, int32_t hidden, uint64_t seed, void* stream, admm_mlp** out) {
  if (!out) return ADMM_E_ARG;
  *out = nullptr;
  if (nin < 1 || nin > 1024 || hidden < 1 || hidden > 1024) {
    g_mlp_error = "nin and hidden must be in 1..1024";
    return ADMM_E_ARG;
  }
  admm_mlp* n = new (std::nothrow) admm_mlp();
  if (!n) return ADMM_E_OOM;
  try {
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev <= 0) {
      delete n;
      g_mlp_error = "no HIP device available";
      return ADMM_E_HIP;
    }
    n->F = nin;
    n->H = hidden;
    const int F = nin, H = hidden;
    n->oW1 = 0;
    n->ob1 = n->oW1 + static_cast<int64_t>(H) * F;
    n->oW2 = n->ob1 + H;
    n->ob2 = n->oW2 + static_cast<int64_t>(H) * H;
    n->ow3 = n->ob2 + H;
    n->ob3 = n->ow3 + H;
    n->owr = n->ob3 + 1;
    n->obr = n->owr + H;
    n->np = n->obr + 1;
    if (stream) {
      n->stream = static_cast<hipStream_t>(stream);
    } else {
      ck(hipStreamCreateWithFlags(&n->stream, hipStreamNonBlocking));
      n->own_stream = true;
    }
    for (float** p : {&n->th, &n->g, &n->m, &n->v}) ck(hipMalloc(reinterpret_cast<void**>(p), sizeof(float) * n->np));
    ck(hipMalloc(reinterpret_cast<void**>(&n->sc), sizeof(double) * 4));
    ck(hipMalloc(reinterpret_cast<void**>(&n->part), sizeof(double) * n->max_splits() * n->np));
    ck(hipHostMalloc(reinterpret_cast<void**>(&n->h_sc), sizeof(double) * 4, hipHostMallocDefault));
    // He-uniform weights from a splitmix64 stream, zero biases
    std::vector<float> th(static_cast<size_t>(n->np), 0.0f);
    uint64_t s = seed;
    auto uni = [&](double lim) {
      const double u = (splitmix64(s) >> 11) * (1.0 / 9007199254740992.0);
      return static_cast<float>((2.0 * u - 1.0) * lim);
    };
    for (int64_t j = 0; j < static_cast<int64_t>(H) * F; ++j) th[n->oW1 + j] = uni(std::sqrt(6.0 / F));
    for (int64_t j = 0; j < static_cast<int64_t>(H) * H; ++j) th[n->oW2 + j] = uni(std::sqrt(6.0 / H));
    for (int j = 0; j < H; ++j) th[n->ow3 + j] = uni(std::sqrt(3.0 / H));
    for (int j = 0; j < H; ++j) th[n->owr + j] = uni(std::sqrt(3.0 / H)) * 0.1f;
    ck(hipMemcpy(n->th, th.data(), sizeof(float) * n->np, hipMemcpyHostToDevice));
    n->clear_moments();
    admmbb::launch_fill_f32(n->g, 0.0f, n->np, n->stream);
    ck(hipGetLastError());
    ck(hipStreamSynchronize(n->stream));
  } catch (const HipErr& e) {
    delete n;
    return mlp_fail(nullptr, "mlp_create", e.e);
  } catch (const std::exception&) {
    delete n;
    return mlp_fail(nullptr, "mlp_create", hipErrorOutOfMemory);
  }
  *out = n;
  return ADMM_OK;
}

void mlp_destroy(admm_mlp* n) { delete n; }

int64_t mlp_num_params(const admm_mlp* n) { return n ? n->np : 0; }

admm_status mlp_get_params(admm_mlp* n, float* out) {
  if (!n || !out) return ADMM_E_ARG;
  try {
    ck(hipStreamSynchronize(n->stream));
    ck(hipMemcpy(out, n->th, sizeof(float) * n->np, hipMemcpyDeviceToHost));
  } catch (const HipErr& e) {
    return mlp_fail(n, "mlp_get_params", e.e);
  } catch (const std::exception&) {  // host allocation: nothing crosses the C boundary
    return mlp_fail(n, "mlp_get_params", hipErrorOutOfMemory);
  }
  return ADMM_OK;
}

admm_status mlp_set_params(admm_mlp* n, const float* in) {
  if (!n || !in) return ADMM_E_ARG;
  for (int64_t j = 0; j < n->np; ++j)
    if (!std::isfinite(in[j])) {
      g_mlp_error = "parameters not finite";
      return ADMM_E_NONFINITE;
    }
  try {
    ck(hipStreamSynchronize(n->stream));
    ck(hipMemcpy(n->th, in, sizeof(float) * n->np, hipMemcpyHostToDevice));
    n->clear_moments();
    ck(hipGetLastError());
    ck(hipStreamSynchronize(n->stream));
    n->step = 0;
  } catch (const HipErr& e) {
    return mlp_fail(n, "mlp_set_params", e.e);
  } catch (const std::exception&) {  // host allocation: nothing crosses the C boundary
    return mlp_fail(n, "mlp_set_params", hipErrorOutOfMemory);
  }
  return ADMM_OK;
}

admm_status mlp_forward(admm_mlp* n, const float* X, int32_t rows, int32_t precision, float* y_out,
                        float* log_rho_out) {
  (void)hipGetLastError();  // report only this call's errors
  if (!n || !X || rows < 1 || (precision != ADMM_PREC_FP32 && precision != ADMM_PREC_BF16)) return ADMM_E_ARG;
  try {
    n->ensure(rows);
    ck(hipMemcpyAsync(n->X, X, sizeof(float) * rows * n->F, hipMemcpyHostToDevice, n->stream));
    MlpArgs a = n->plan(rows);
    a.t = nullptr;
    a.z1 = a.z2 = a.z3 = nullptr;
    n->forward(a, precision == ADMM_PREC_BF16);
    ck(hipGetLastError());
    if (y_out) ck(hipMemcpyAsync(y_out, n->y, sizeof(float) * rows, hipMemcpyDeviceToHost, n->stream));
    ck(hipMemcpyAsync(n->h_sc, n->sc, sizeof(double) * 3, hipMemcpyDeviceToHost, n->stream));
    ck(hipStreamSynchronize(n->stream));
    if (log_rho_out) *log_rho_out = static_cast<float>(n->h_sc[0]);
  } catch (const HipErr& e) {
    return mlp_fail(n, "mlp_forward", e.e);
  } catch (const std::exception&) {  // host allocation: nothing crosses the C boundary
    return mlp_fail(n, "mlp_forward", hipErrorOutOfMemory);
  }
  return ADMM_OK;
}

admm_status mlp_loss_grad(admm_mlp* n, const float* X, const float* target, int32_t rows, float target_log_rho,
                          float lam, double* loss_out, float* grad_out) {
  (void)hipGetLastError();  // report only this call's errors
  if (!n || !X || !target || rows < 1 || !std::isfinite(target_log_rho) || !(lam >= 0)) return ADMM_E_ARG;
  try {
    const int B = rows, F = n->F;
    n->ensure(B);
    ck(hipMemcpyAsync(n->X, X, sizeof(float) * B * F, hipMemcpyHostToDevice, n->stream));
    ck(hipMemcpyAsync(n->t, target, sizeof(float) * B, hipMemcpyHostToDevice, n->stream));
    MlpArgs a = n->plan(B);
    a.lr_t = target_log_rho;
    a.lam = lam;
    n->forward(a, false);
    n->backward(a);
    ck(hipGetLastError());
    ck(hipMemcpyAsync(n->h_sc, n->sc, sizeof(double) * 3, hipMemcpyDeviceToHost, n->stream));
    if (grad_out) ck(hipMemcpyAsync(grad_out, n->g, sizeof(float) * n->np, hipMemcpyDeviceToHost, n->stream));
    ck(hipStreamSynchronize(n->stream));
    if (loss_out) *loss_out = n->h_sc[1];
  } catch (const HipErr& e) {
    return mlp_fail(n, "mlp_loss_grad", e.e);
  } catch (const std::exception&) {  // host allocation: nothing crosses the C boundary
    return mlp_fail(n, "mlp_loss_grad", hipErrorOutOfMemory);
  }
  return ADMM_OK;
}

admm_status mlp_adam_step(admm_mlp* n, float lr, float beta1, float beta2, float eps) {
  (void)hipGetLastError();  // report only this call's errors
  if (!n || !(lr > 0) || !(beta1 >= 0 && beta1 < 1) || !(beta2 >= 0 && beta2 < 1) || !(eps > 0)) return ADMM_E_ARG;
  try {
    n->step += 1;
    const float c1 = 1.0f - std::pow(beta1, static_cast<float>(n->step));
    const float c2 = 1.0f - std::pow(beta2, static_cast<float>(n->step));
    hipLaunchKernelGGL(k_adam, dim3(static_cast<unsigned>((n->np + 255) / 256)), dim3(256), 0, n->stream, n->th, n->g,
                       n->m, n->v, n->np, lr, beta1, beta2, eps, c1, c2);
    ck(hipGetLastError());
    ck(hipStreamSynchronize(n->stream));
  } catch (const HipErr& e) {
    return mlp_fail(n, "mlp_adam_step", e.e);
  } catch (const std::exception&) {  // host allocation: nothing crosses the C boundary
    return mlp_fail(n, "mlp_adam_step", hipErrorOutOfMemory);
  }
  return ADMM_OK;
}

}  // extern "C"
