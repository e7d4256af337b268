// Projected gradient descent with Armijo backtracking (Sec. 2.1) on the cached
// dense Gram sum of the dense x-update, driven on the device.
//
// With S = sum_s G_s (packed upper 64 x 64 tiles, fp64) the objective and its
// gradient are f(x) = x^T S x - g0^T x + const and grad f(x) = 2 S x - g0.
// One round evaluates kPgdK backtracking steps at once, in two launches:
//   k_pgd_tiles   the decision about the last round's trial points: the first k
//                 (largest step) with f(x_k) <= f(x) + beta g^T (x_k - x) is
//                 accepted (stopping tests), x = x_k with gradient 2 u_k - g0;
//                 the next trial points x_k = P(x - t_k g), t_k = t_base
//                 gamma^k; and for every tile T of S and every k the products
//                 T x_k,J and T^T x_k,I, one read of S for all trial points
//   k_pgd_rows    u_k = S x_k from the tile products, and f(x_k) partial sums
// so an iteration whose step is found within kPgdK trials reads S once.
// A round that accepts nothing retries from the same x with the next kPgdK
// steps.  Every workgroup of k_pgd_tiles takes the decision itself, from the
// same sums in the same order, and forms the trial points of its two blocks
// while its tile is on the way; the workgroup of a diagonal tile also writes its
// block's (in a launch of its own between the rows and the tiles, decision and
// trial points took 6.8 us of a 30 us round at 2 981 spots; a round now takes
// 15.5 + 4.5 us).  The host queues rounds ahead of the state it reads.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "internal.h"
#include "scalars.h"

namespace admmbb {

namespace {

constexpr int kT = 64;  // tile size

typedef double v4d __attribute__((ext_vector_type(4)));

__device__ __forceinline__ int64_t ptile(int I, int J, int nb) {
  return static_cast<int64_t>(I) * nb - static_cast<int64_t>(I) * (I - 1) / 2 + (J - I);
}

// the upper tile number t = ptile(I, J, nb), I <= J, without a table read
__device__ __forceinline__ void tile_place(int t, int nb, int& I, int& J) {
  const float b = static_cast<float>(2 * nb + 1);
  I = static_cast<int>(0.5f * (b - sqrtf(fmaxf(b * b - 8.0f * static_cast<float>(t), 0.0f))));
  I = I < 0 ? 0 : (I >= nb ? nb - 1 : I);
  while (I > 0 && ptile(I, I, nb) > t) --I;  // the root is within one of the row
  while (I + 1 < nb && ptile(I + 1, I + 1, nb) <= t) ++I;
  J = I + static_cast<int>(t - ptile(I, I, nb));
}

// LDS written by some lanes of a wave and then read by others of the same wave
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// LDS of a tile workgroup: the trial points of its two blocks, per wave a 16 x 16
// block on its way to the transposed operand, and (in the same place, later) the
// waves' sums of the transposed product.
constexpr int kTrLd = 17;
constexpr int kVLd = kT + 4;  // the eight vectors' entries that one load reads lie in different banks
template <int KC>
struct TileLds {
  double vJ[KC][kVLd], vI[KC][kVLd];
  union {
    double tr[4][16 * kTrLd];
    double red[4][KC][kT];
  };
};

// The products of one tile T (rows of block I, columns of block J) with KC <= 8
// vectors of each block, on the fp64 16x16x4 MFMA with the vectors as the rows of
// the first operand (16 rows, zero beyond KC).  Wave w holds rows 16 w .. 16 w +
// 15 of T in t[c][q]: row 16 w + l / 16 + 4 q, column 16 c + l % 16 of lane l,
// which is the second operand of v_I T as loaded; for v_J T^T each 16 x 16 block
// is transposed through the wave's own LDS.  v_I T is summed over the waves.
// (The whole tile in LDS for both products left five workgroups per CU; 25 KB
// leave six, and no barrier between the loads and the products.)
// part[(tile * KC + k) * 128 + i]      = (T v_k,J)_i
// part[(tile * KC + k) * 128 + 64 + i] = (T^T v_k,I)_i   (off-diagonal tiles)
template <int KC>
__device__ __forceinline__ void tile_products(TileLds<KC>& s, const double (&t)[4][4], bool diag,
                                              double* __restrict__ out) {
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63, m = l & 15, kk = l >> 4;
  const bool live = m < KC;
  const int mc = live ? m : 0;
  v4d a1 = {0.0, 0.0, 0.0, 0.0}, a2[4];
  double* tr = s.tr[w];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    a2[c] = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < 4; ++q) tr[(kk + 4 * q) * kTrLd + m] = t[c][q];
    wave_lds_sync();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      // column 16 c + 4 q + kk of row 16 w + m
      const double vj = s.vJ[mc][16 * c + 4 * q + kk];
      a1 = __builtin_amdgcn_mfma_f64_16x16x4f64(live ? vj : 0.0, tr[m * kTrLd + 4 * q + kk], a1, 0, 0, 0);
    }
    wave_lds_sync();
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const double vi = s.vI[mc][16 * w + 4 * q + kk];
#pragma unroll
    for (int c = 0; c < 4; ++c)
      a2[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(live ? vi : 0.0, t[c][q], a2[c], 0, 0, 0);
  }
  // item r of a lane: vector l / 16 + 4 r, column l % 16
#pragma unroll
  for (int r = 0; r < (KC + 3) / 4; ++r)
    if (kk + 4 * r < KC) out[(kk + 4 * r) * 2 * kT + 16 * w + m] = a1[r];
  if (diag) return;
  __syncthreads();  // the transposed blocks have been read
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int r = 0; r < (KC + 3) / 4; ++r)
      if (kk + 4 * r < KC) s.red[w][kk + 4 * r][16 * c + m] = a2[c][r];
  __syncthreads();
  for (int e = tid; e < KC * kT; e += 256) {
    const int k = e / kT, i = e % kT;
    out[k * 2 * kT + kT + i] = (s.red[0][k][i] + s.red[1][k][i]) + (s.red[2][k][i] + s.red[3][k][i]);
  }
}

// the wave's rows of tile `tile`, requested (in bounds whatever the state)
__device__ __forceinline__ void load_tile(const PgdArgs& a, int64_t tile, double (&t)[4][4]) {
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63, m = l & 15, kk = l >> 4;
  const double* T = a.Gp + tile * kT * kT + (16 * w + kk) * kT + m;
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int q = 0; q < 4; ++q) t[c][q] = T[4 * q * kT + 16 * c];
}

// One round's decision, trial points and tile products.  State, x, g, trial
// points and partial sums of g^T (x_k - x) are double-buffered by the round's
// parity: this launch reads slot par and writes slot par ^ 1.
// mode kPgdRound; kPgdFirst: every trial point was x, record f(x) and take its
// gradient; kPgdPrime: no decision, every trial point is x (with `power`, alpha
// from the power iteration's last norm).
enum { kPgdRound = 0, kPgdFirst = 1, kPgdPrime = 2 };
__global__ __launch_bounds__(256, 5) void k_pgd_tiles(PgdArgs a, int mode, int power, int par, uint32_t seq) {
  __shared__ TileLds<kPgdK> s;
  __shared__ double fk[kPgdK], gd[kPgdK];
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int64_t tile = blockIdx.x;  // in packed order
  int I, J;
  tile_place(static_cast<int>(tile), a.nb, I, J);
  const PgdDevState cur = a.st[par];
  PgdDevState nxt = cur;
  const bool diag = I == J, first = blockIdx.x == 0;
  // threads 0 .. 63 take the spots of block I, 64 .. 127 those of block J
  const bool mine = tid < (diag ? 64 : 128);
  const int j = (tid < 64 ? I : J) * kT + lane;
  const bool in = mine && j < a.n;
  const int jc = in ? j : 0;
  const int64_t np = a.np;
  const double* x0 = a.x + par * np;
  const double* g0v = a.g + par * np;
  const double* xc = a.xc + par * kPgdK * np;
  double* x1 = a.x + (par ^ 1) * np;
  double* g1 = a.g + (par ^ 1) * np;
  double* xc1 = a.xc + (par ^ 1) * kPgdK * np;
  // the decision's sums: wave w takes k = w and w + 4, at most 128 block rows
  double fp[2][2], gp[2][2];
  if (mode == kPgdPrime) {
    if (power)
      for (int h = 0; h < 2; ++h) fp[0][h] = lane + 64 * h < a.nb ? a.fpart[lane + 64 * h] : 0.0;
  } else {
    const double* gdin = a.gdpart + static_cast<int64_t>(par) * kPgdK * a.nb;
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int b = lane + 64 * h, at = (w + 4 * q) * a.nb + b;
        fp[q][h] = b < a.nb ? a.fpart[at] : 0.0;
        gp[q][h] = b < a.nb ? gdin[at] : 0.0;
      }
  }
  double xj = 0.0, gj = 0.0, g0j = 0.0, lo = 0.0, hi = 0.0;
  if (mine) {
    xj = x0[jc];
    gj = g0v[jc];
    g0j = a.g0[jc];
    lo = a.lb[jc];
    hi = a.ub[jc];
  }
  // the tile last: loads return in order, and the decision (the other loads) is
  // formed while it is on the way.  The picked trial point and its product are
  // read after the decision: all eight beforehand are as many bytes as the tile
  // (19.3 instead of 17.0 us)
  __builtin_amdgcn_sched_barrier(0);
  double t[4][4];
  load_tile(a, tile, t);
  __builtin_amdgcn_sched_barrier(0);
  if (cur.done) {
    if (first && tid == 0) {
      a.st[par ^ 1] = cur;
      __hip_atomic_store(a.progress, seq << 1 | 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    if (diag && tid < 64) x1[j] = in ? xj : 0.0;
    return;
  }
  int p = -1;
  if (mode == kPgdPrime) {
    nxt.t_base = 0.0;
    if (power) {
      const double nrm = sqrt(group_allsum<64>(fp[0][0] + fp[0][1]));
      nxt.alpha = nrm > 0 ? 10.0 / nrm : 1.0;
    }
  } else {
    // f(x_k) and g^T (x_k - x), fixed order
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const double fs = group_allsum<64>(fp[q][0] + fp[q][1]);
      const double ds = group_allsum<64>(gp[q][0] + gp[q][1]);
      if (lane == 0) {
        fk[w + 4 * q] = a.fconst + fs;
        gd[w + 4 * q] = ds;
      }
    }
    __syncthreads();
    bool stop = false;
    if (mode == kPgdFirst) {
      p = 0;
      nxt.f = fk[0];
      nxt.t_base = cur.alpha;
      if (a.max_iter <= 0) {
        stop = true;
        nxt.status = 3;
      }
    } else {
      for (int k = 0; k < kPgdK; ++k)
        if (cur.trials + k < a.max_trials && fk[k] <= cur.f + a.beta * gd[k]) {
          p = k;
          break;
        }
      if (p >= 0) {
        nxt.f = fk[p];
        nxt.iter = cur.iter + 1;
        nxt.trials = 0;
        nxt.t_base = cur.alpha;
        if (fabs(cur.f - fk[p]) <= a.tol * fabs(cur.f)) {
          stop = true;
          nxt.status = 1;
        } else if (nxt.iter >= a.max_iter) {
          stop = true;
          nxt.status = 3;
        }
      } else {
        nxt.trials = cur.trials + kPgdK;
        double tb = cur.t_base;
        for (int k = 0; k < kPgdK; ++k) tb *= a.gamma;
        nxt.t_base = tb;
        if (nxt.trials >= a.max_trials) {
          stop = true;
          nxt.status = 2;
        }
      }
    }
    if (stop) nxt.done = 1;
  }
  nxt.pick = p;
  if (first && tid == 0) {
    a.st[par ^ 1] = nxt;
    __hip_atomic_store(a.progress, seq << 1 | (nxt.done ? 1u : 0u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
  if (mine) {
    if (p >= 0) {
      xj = xc[p * np + jc];
      gj = 2.0 * a.u[p * np + jc] - g0j;
    }
    if (!in) xj = gj = 0.0;
    if (diag) {
      x1[j] = xj;
      g1[j] = gj;
    }
  }
  if (nxt.done) return;
  if (mine) {
    double tk = nxt.t_base;
    double* gdout = a.gdpart + static_cast<int64_t>(par ^ 1) * kPgdK * a.nb;
#pragma unroll
    for (int k = 0; k < kPgdK; ++k) {
      const double v = in ? fmin(fmax(xj - tk * gj, lo), hi) : 0.0;
      if (tid < 64) s.vI[k][lane] = v;
      if (tid >= 64 || diag) s.vJ[k][lane] = v;
      if (diag) {
        xc1[k * np + j] = v;
        const double d = group_allsum<64>(gj * (v - xj));
        if (lane == 0) gdout[k * a.nb + I] = d;
      }
      tk *= a.gamma;
    }
  }
  __syncthreads();
  tile_products<kPgdK>(s, t, diag, a.part + tile * (kPgdK * 2 * kT));
}

// Power iteration on H = 2 S: v = u / ||u|| with u = 2 S v_old from the last
// products (their squares' sums in fpart), or v0 everywhere at the start, and the
// tile products of v.
__global__ __launch_bounds__(256, 5) void k_pgd_power_tiles(PgdArgs a, int start, double v0) {
  __shared__ TileLds<1> s;
  const int tid = threadIdx.x, lane = tid & 63;
  const int64_t tile = blockIdx.x;
  int I, J;
  tile_place(static_cast<int>(tile), a.nb, I, J);
  const int jv = (tid < 64 ? I : J) * kT + lane;
  double q = 0.0, uj = 0.0;
  if (!start && tid < 128) {
    for (int b = lane; b < a.nb; b += 64) q += a.fpart[b];
    uj = a.u[jv < a.n ? jv : 0];
  }
  __builtin_amdgcn_sched_barrier(0);
  double t[4][4];
  load_tile(a, tile, t);
  __builtin_amdgcn_sched_barrier(0);
  const bool diag = I == J;
  if (tid < 128) {
    double v = v0;
    if (!start) {
      const double nrm = sqrt(group_allsum<64>(q));
      v = nrm > 0 ? 2.0 * uj / nrm : 0.0;
    }
    if (jv >= a.n) v = 0.0;
    if (tid < 64)
      s.vI[0][lane] = v;
    else
      s.vJ[0][lane] = v;
  }
  __syncthreads();
  tile_products<1>(s, t, diag, a.part + tile * (2 * kT));
}

// Block row I of u_k = S v_k (workgroup (I, k)) from the tile products, and
// fpart[k * nb + I] = sum over the block's rows of v_k (u_k - g0); POWER: of
// (2 u)^2.  Four waves take every fourth tile of the block row; fixed summation
// order.
template <int KC, bool POWER>
__global__ __launch_bounds__(256) void k_pgd_rows(PgdArgs a, int par) {
  __shared__ double red[4][kT];
  const int I = static_cast<int>(blockIdx.x), k = static_cast<int>(blockIdx.y);
  const int i = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int row = I * kT + i;
  // four independent loads in flight per lane, then a fixed-order sum
  double s = 0.0;
  for (int J0 = w; J0 < a.nb; J0 += 16) {
    double e[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int J = J0 + 4 * q;
      const int64_t t = J < I ? ptile(J, I, a.nb) : ptile(I, J, a.nb);
      e[q] = J < a.nb ? a.part[(t * KC + k) * (2 * kT) + (J < I ? kT : 0) + i] : 0.0;
    }
    s += (e[0] + e[1]) + (e[2] + e[3]);
  }
  double v = 0.0, g0 = 0.0;
  if (!POWER) {
    v = a.xc[(static_cast<int64_t>(par) * kPgdK + k) * a.np + row];
    g0 = row < a.n ? a.g0[row] : 0.0;
    if (a.st[par].done) return;  // checked after the (in-bounds) loads are under way
  }
  red[w][i] = s;
  __syncthreads();
  if (w != 0) return;
  s = (red[0][i] + red[1][i]) + (red[2][i] + red[3][i]);
  double d = 0.0;
  if (row < a.n) {
    a.u[static_cast<int64_t>(k) * a.np + row] = s;
    d = POWER ? (2.0 * s) * (2.0 * s) : v * (s - g0);
  }
  d = group_allsum<64>(d);
  if (i == 0) a.fpart[static_cast<int64_t>(k) * a.nb + I] = d;
}

}  // namespace

void launch_pgd_power(const PgdArgs& a, int start, double v0, hipStream_t st) {
  hipLaunchKernelGGL(k_pgd_power_tiles, dim3(a.njobs), dim3(256), 0, st, a, start, v0);
  hipLaunchKernelGGL((k_pgd_rows<1, true>), dim3(a.nb, 1), dim3(256), 0, st, a, 0);
}

void launch_pgd_prime(const PgdArgs& a, int power, int par, uint32_t seq, hipStream_t st) {
  hipLaunchKernelGGL(k_pgd_tiles, dim3(a.njobs), dim3(256), 0, st, a, static_cast<int>(kPgdPrime), power, par, seq);
  hipLaunchKernelGGL((k_pgd_rows<kPgdK, false>), dim3(a.nb, kPgdK), dim3(256), 0, st, a, par ^ 1);
}

void launch_pgd_round(const PgdArgs& a, int first, int par, uint32_t seq, hipStream_t st) {
  hipLaunchKernelGGL(k_pgd_tiles, dim3(a.njobs), dim3(256), 0, st, a,
                     static_cast<int>(first ? kPgdFirst : kPgdRound), 0, par, seq);
  hipLaunchKernelGGL((k_pgd_rows<kPgdK, false>), dim3(a.nb, kPgdK), dim3(256), 0, st, a, par ^ 1);
}

}  // namespace admmbb
