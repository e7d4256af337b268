// Dense x-update: the exact solve of every scenario subproblem through a
// cached inverse of its system matrix (Appendix A factors B_s = A_s^T W~_s A_s
// + rho/2 I once and reuses the factor in every iteration; here the factor is
// the inverse itself, so that each x-update is one bandwidth-bound GEMV).
//
//  1. G_s = A_s^T diag(c_s w) A_s, upper 64 x 64 tiles: lists of the rows
//     that reach each tile (k_gram_rows, k_gram_scan), then one workgroup per
//     tile multiplies its rows on the fp64 MFMA and adds them up without loss
//     (k_gram_tiles).  k_gram (one fp64
//     atomic per product, one wave per stored row) is the fallback when the
//     lists do not fit in device memory.
//  2. k_gram_finish: the upper tiles of the sweep work matrix
//     A = G_s + rho/2 I (identity on the padding to npad) and sum_s G_s.
//     Steps 1-3 run on chunks of scenarios, so that only a chunk's fp64
//     set-up matrices occupy device memory at a time.
//  3. block sweep (Gauss-Jordan on 128-blocks, no pivoting: the pivot blocks
//     are Schur complements of an SPD matrix): for each block K,
//        P = A_KK^-1, U = A_:K P, R = A_K: (old),
//        A_ij -= U_i R_j off the block row and column,
//        A_:K = U, A_K: = U^T, A_KK = -P;
//     after the last block A = -B_s^-1.  The sweep matrix stays symmetric, so
//     only its upper 64 x 64 tiles are updated (half the work).  The last
//     step stores M_s = B_s^-1 in fp32.
//  4. k_gq_pack: sum_s G_s rounded to 48 bits for the objective tiles.
//  5. every iteration, three launches: k_dense_x (x_s = M_s c_s tile by tile,
//     the previous iteration's stopping test in one workgroup per patient), k_xzres (the
//     partial sums of x_s with the z-update), k_dense_tail_dual (residual
//     norms and dual step, the dual
//     update with the next right-hand sides c_s, the objective at the new z
//     from the quadratic form).  k_fheadobj forms the right-hand sides and the
//     objective of the state a run starts from.
// The symmetric matrices used in every iteration (M_s and sum_s G_s) are stored
// as their upper 64 x 64 tiles only, which halves the bytes each iteration reads.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "internal.h"
#include "scalars.h"

namespace admmbb {

namespace {

typedef double v2d __attribute__((ext_vector_type(2)));
typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int kFb = 64;  // packed tile size

__host__ __device__ __forceinline__ int64_t tile_index(int I, int J, int nb) {
  return static_cast<int64_t>(I) * nb - static_cast<int64_t>(I) * (I - 1) / 2 + (J - I);
}

__device__ __forceinline__ double wave_sum_d(double v) { return group_allsum<64>(v); }

// ---------------------------------------------------------------------------
// Gram matrix
// ---------------------------------------------------------------------------

template <bool C16>
__global__ __launch_bounds__(256) void k_gram(MatDev mat, const double* __restrict__ rw64, Scen sc,
                                              double* __restrict__ G, int ld) {
  const int row = static_cast<int>(blockIdx.x) * 4 + static_cast<int>(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= sc.rows) return;
  const uint32_t c0 = mat.rp[sc.rp_base + row], c1 = mat.rp[sc.rp_base + row + 1];
  const int64_t e0 = sc.nnz_base + 4 * static_cast<int64_t>(c0);
  const int k = 4 * static_cast<int>(c1 - c0);
  const double rw = rw64[sc.row_base + row];
  const float* val = static_cast<const float*>(mat.val);
  auto colat = [&](int64_t e) -> int {
    if constexpr (C16)
      return static_cast<const uint16_t*>(mat.col)[e];
    else
      return static_cast<const int32_t*>(mat.col)[e];
  };
  for (int base = 0; base < k; base += 64) {
    const int kk = base + lane;
    const bool valid = kk < k;
    const int ck = valid ? colat(e0 + kk) : 0;
    const double vk = valid ? rw * static_cast<double>(val[e0 + kk]) : 0.0;
    const int jend = base + 64 < k ? base + 64 : k;
    for (int jj = 0; jj < jend; ++jj) {
      const float vj = val[e0 + jj];
      if (vj == 0.0f) continue;  // chunk padding
      const int cj = colat(e0 + jj);
      // columns increase along a stored row, so jj <= kk gives cj <= ck
      if (valid && jj <= kk && vk != 0.0)
        unsafeAtomicAdd(&G[static_cast<int64_t>(cj) * ld + ck], vk * static_cast<double>(vj));
    }
  }
}

// Gram matrix by output tiles.  Every stored row adds w_i a_i a_i^T to the
// 64 x 64 tiles (I, J), I <= J, of the blocks its nonzeros fall in.  Lists of
// the rows that reach each tile are built first, then one workgroup per tile
// adds its rows' products and writes the tile once.
//
// The lists: the voxels of a scenario, in groups of 64, are dealt to `nchunk`
// waves (group i to wave i mod nchunk).  Each wave counts its rows' entries per
// tile in LDS (k_gram_rows<false>), k_gram_prefix turns the counts of a tile
// into each wave's first slot, k_gram_scan the totals into tile offsets, and the
// same waves write the entries (k_gram_rows<true>).  One launch each covers
// every scenario of the chunk, no counter is shared between waves (counting and
// filling with one global atomic per entry and a launch per scenario took 6.2
// ms for 13 scenarios of 1 700 spots, against 0.5 ms), and a list's order is
// fixed: the sums below repeat bit for bit, and neighbouring voxels, which the
// same spots reach, stand together.

// row_of[s * ms + voxel] = the stored row of the voxel (preset to -1: no nonzero)
__global__ __launch_bounds__(256) void k_gram_order(MatDev mat, const Scen* __restrict__ scen, int g0, int ms,
                                                    int32_t* __restrict__ row_of) {
  const Scen sc = scen[g0 + static_cast<int>(blockIdx.y)];
  int32_t* to = row_of + static_cast<int64_t>(blockIdx.y) * ms;
  for (int r = static_cast<int>(blockIdx.x) * 256 + threadIdx.x; r < sc.rows; r += static_cast<int>(gridDim.x) * 256)
    to[mat.rorig[sc.row_base + r]] = r;
}

// Columns are uint16 in every dense context (n <= 8128).
__device__ __forceinline__ int col_at(const MatDev& mat, int64_t e) { return static_cast<const uint16_t*>(mat.col)[e]; }

// LDS written by some lanes of a wave and then read by others of the same wave
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

constexpr int kMaxBlocks = 128;  // 64-column blocks of a patient (n <= 8192)

// One wave per workgroup: blockIdx.x the chunk, blockIdx.y the scenario.
// cnt[(s * nchunk + chunk) * nt + tile]: FILL = false writes the wave's entries
// per tile, FILL = true reads its first slot in the tile's list.
template <bool FILL>
__global__ __launch_bounds__(64) void k_gram_rows(MatDev mat, const Scen* __restrict__ scen, int g0, int nb,
                                                  const int32_t* __restrict__ row_of, int ms, int nchunk,
                                                  uint32_t* __restrict__ cnt,
                                                  const int64_t* __restrict__ off, GramEntry* __restrict__ list) {
  extern __shared__ __align__(16) uint32_t slot[];  // one per tile
  __shared__ int bl[kMaxBlocks], st[kMaxBlocks + 1];  // the row's blocks, and where each starts
  const int lane = threadIdx.x;
  const int chunk = static_cast<int>(blockIdx.x), s = static_cast<int>(blockIdx.y);
  const Scen sc = scen[g0 + s];
  const int nt = nb * (nb + 1) / 2;
  uint32_t* mine = cnt + (static_cast<int64_t>(s) * nchunk + chunk) * nt;
  for (int t = lane; t < nt; t += 64) slot[t] = FILL ? mine[t] : 0u;
  wave_lds_sync();
  const uint32_t* rp = mat.rp + sc.rp_base;
  const int32_t* rows = row_of + static_cast<int64_t>(s) * ms;
  for (int64_t v0 = 64 * chunk; v0 < sc.m; v0 += 64 * nchunk) {
    // the extents of the group's rows, one per lane
    const int myrow = v0 + lane < sc.m ? rows[v0 + lane] : -1;
    uint32_t myc0 = 0, myc1 = 0;
    if (myrow >= 0) {
      myc0 = rp[myrow];
      myc1 = rp[myrow + 1];
    }
    for (uint64_t left = __ballot(myrow >= 0); left != 0; left &= left - 1) {
      const int from = __ffsll(static_cast<unsigned long long>(left)) - 1;
      const int row = __builtin_amdgcn_readlane(myrow, from);
      const uint32_t c0 = __builtin_amdgcn_readlane(myc0, from), c1 = __builtin_amdgcn_readlane(myc1, from);
      const int64_t e0 = sc.nnz_base + 4 * static_cast<int64_t>(c0);
      const int k = 4 * static_cast<int>(c1 - c0);
      int r = 0, last = -1;
      for (int base = 0; base < k; base += 64) {
        const int kk = base + lane;
        const int b = kk < k ? col_at(mat, e0 + kk) >> 6 : -1;
        const int up = __shfl_up(b, 1, 64);
        const bool start = kk < k && b != (lane == 0 ? last : up);  // columns are non-decreasing along a row
        const uint64_t m = __ballot(start);
        const int at = r + __popcll(m & ((uint64_t{1} << lane) - 1));
        if (start && at < kMaxBlocks) {
          bl[at] = b;
          st[at] = kk;
        }
        r += __popcll(m);
        last = __shfl(b, 63, 64);
      }
      if (r > kMaxBlocks) r = kMaxBlocks;  // cannot happen for n <= 8192
      if (lane == 0) st[r] = k;
      wave_lds_sync();
      for (int t = lane; t < r * r; t += 64) {
        const int p = t / r, q = t - p * r;
        if (p > q) continue;
        const int ti = static_cast<int>(tile_index(bl[p], bl[q], nb));
        const uint32_t at = slot[ti];  // the row's tiles are distinct: no two lanes share one
        slot[ti] = at + 1;
        if constexpr (FILL)
          list[off[static_cast<int64_t>(s) * nt + ti] + at] =
              GramEntry{row, c0, static_cast<uint32_t>(st[p]) | static_cast<uint32_t>(st[p + 1] - st[p]) << 16,
                        static_cast<uint32_t>(st[q]) | static_cast<uint32_t>(st[q + 1] - st[q]) << 16};
      }
      wave_lds_sync();
    }
  }
  if constexpr (!FILL) {
    wave_lds_sync();
    for (int t = lane; t < nt; t += 64) mine[t] = slot[t];
  }
}

// Per tile: cnt of every chunk replaced by the sum of the chunks before it, the
// total to tot.  Workgroup: 64 tiles (lanes) of one scenario, eight waves an
// eighth of the chunks each.
constexpr int kPrefixWaves = 8;
__global__ __launch_bounds__(64 * kPrefixWaves) void k_gram_prefix(uint32_t* __restrict__ cnt, int nt, int nchunk,
                                                                   int32_t* __restrict__ tot) {
  __shared__ uint32_t part[kPrefixWaves][64];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int t = static_cast<int>(blockIdx.x) * 64 + lane, s = static_cast<int>(blockIdx.y);
  const int per = (nchunk + kPrefixWaves - 1) / kPrefixWaves;
  const int b = w * per < nchunk ? w * per : nchunk, e = b + per < nchunk ? b + per : nchunk;
  uint32_t* c = cnt + static_cast<int64_t>(s) * nchunk * nt + t;
  uint32_t sum = 0;
  if (t < nt)
    for (int i = b; i < e; ++i) sum += c[static_cast<int64_t>(i) * nt];
  part[w][lane] = sum;
  __syncthreads();
  if (t >= nt) return;
  uint32_t run = 0;
  for (int q = 0; q < w; ++q) run += part[q][lane];
  for (int i = b; i < e; ++i) {
    const uint32_t v = c[static_cast<int64_t>(i) * nt];
    c[static_cast<int64_t>(i) * nt] = run;
    run += v;
  }
  if (w == kPrefixWaves - 1) tot[static_cast<int64_t>(s) * nt + t] = static_cast<int32_t>(run);
}

// off[i] = cnt[0] + ... + cnt[i - 1] for i <= nt (one workgroup)
__global__ __launch_bounds__(1024) void k_gram_scan(const int32_t* __restrict__ cnt, int64_t nt,
                                                    int64_t* __restrict__ off) {
  __shared__ int64_t part[1024];
  const int t = threadIdx.x;
  const int64_t per = (nt + 1023) / 1024;
  const int64_t b = t * per < nt ? t * per : nt, e = b + per < nt ? b + per : nt;
  int64_t sum = 0;
  for (int64_t i = b; i < e; ++i) sum += cnt[i];
  part[t] = sum;
  __syncthreads();
  for (int d = 1; d < 1024; d <<= 1) {
    const int64_t v = t >= d ? part[t - d] : 0;
    __syncthreads();
    part[t] += v;
    __syncthreads();
  }
  int64_t run = part[t] - sum;
  for (int64_t i = b; i < e; ++i) {
    off[i] = run;
    run += cnt[i];
  }
  if (t == 1023) off[nt] = part[1023];
}

// One workgroup per tile (I, J) of scenario g0 + blockIdx.y: sum over the rows
// of its list of (c_s w_i a_i,I) a_i,J^T, a 64 x rows x 64 product on the fp64
// 16x16x4 MFMA.  32 listed rows at a time, each wave expands eight: their
// segments of the two blocks (13 of 64 columns on average, contiguous, two
// 16-byte loads of four elements per lane) go to zeroed LDS rows, the first
// block's times its weight in fp64; then each wave adds all 32 rows to its 32 x
// 32 quarter of the tile, leaving out the 16-column groups that no row of a
// step uses (listed in voxel order, four rows need a third of the products; in
// the order of the stored rows, four fifths).
//
// The products of four rows start from zero, and their sums are added without
// loss: `hi` starts from gbig[s], a power of two above every entry of G_s, so
// t = hi + d rounds once and d - (t - hi) is exactly what it dropped, which `lo`
// collects (hi - big is exact at the end).  An entry is then one rounding from
// its four-row sums, however many rows it has: the diagonal of a patient's matrix
// (1 500 to 2 300 rows) is 4.8e-17 off (relative, root mean square), where 64-bit
// fixed-point sums of one product at a time through LDS atomics (17.7 ms at 13
// scenarios of 2 981 spots) leave 6e-17 to 9e-17 and a running fp64 sum over the
// list 1.2e-15 to 1.5e-15.  The residuals and their registers (three workgroups
// per CU instead of four) cost 8.8 instead of 5.3 ms there, 3.7 instead of 2.3 ms
// at 1 700 spots; four workgroups with spills (12 ms) or eight waves with an
// eighth of the tile each (9 to 12 ms) are no faster.
//
// The next rows are requested before the products of the current ones.  Padding
// (value 0, the last column repeated) is left out.
constexpr int kGramWaves = 4;
constexpr int kGramRows = 8;       // listed rows a wave expands at a time
constexpr int kGramLd = kFb + 16;  // row stride: four rows that one load reads start 32 (16) banks apart

__global__ __launch_bounds__(64 * kGramWaves, 3) void k_gram_tiles(MatDev mat, const double* __restrict__ rw64,
                                                                const Scen* __restrict__ scen, int g0, int nb,
                                                                const int64_t* __restrict__ off,
                                                                const GramEntry* __restrict__ list,
                                                                const double* __restrict__ gbig,
                                                                double* __restrict__ G, int ld) {
  constexpr int kStep = kGramWaves * kGramRows;
  __shared__ __align__(16) double bufI[kStep * kGramLd];
  __shared__ __align__(16) float bufJ[kStep * kGramLd];
  __shared__ uint32_t occ[kStep / 4];  // per four rows: 16-column groups in use, block I in bits 0-3, J in 4-7
  const int64_t ntiles = static_cast<int64_t>(nb) * (nb + 1) / 2;
  const int64_t t = blockIdx.x;
  const int s = static_cast<int>(blockIdx.y);
  int I = 0;
  int64_t rem = t;
  while (rem >= nb - I) {
    rem -= nb - I;
    ++I;
  }
  const int J = I + static_cast<int>(rem);
  const Scen sc = scen[g0 + s];
  const float* val = static_cast<const float*>(mat.val);
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int g = tid >> 3, sub = lane & 7;  // eight lanes expand row g of the 32
  const int m = lane & 15, kk = lane >> 4;
  const int wu = __builtin_amdgcn_readfirstlane(w);
  const int qi = 32 * (wu >> 1), qj = 32 * (wu & 1);  // the wave's quarter
  const int64_t l0 = off[s * ntiles + t], le = off[s * ntiles + t + 1];
  const double big = gbig[s];
  v4d hi[2][2], lo[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      hi[a][b] = v4d{big, big, big, big};
      lo[a][b] = v4d{0.0, 0.0, 0.0, 0.0};
    }
  // one row's share of a lane: of either segment, the chunk (four elements,
  // aligned, so a neighbouring block's may be among them) at its place of the
  // eight, and the one eight further on
  struct Row {
    uint32_t cI, cJ;  // the segments' first chunks
    int nI, nJ;       // their chunks
    double rw;
    float4 vI[2], vJ[2];
    uint2 kI[2], kJ[2];
  };
  const float4* valc = reinterpret_cast<const float4*>(val + sc.nnz_base);
  const uint2* colc = reinterpret_cast<const uint2*>(static_cast<const uint16_t*>(mat.col) + sc.nnz_base);
  auto entry = [&](int64_t li, GramEntry& e) {
    e = GramEntry{0, 0, 0, 0};  // no row: empty segments
    if (li < le) e = list[li];
  };
  auto chunks = [](uint32_t c0, uint32_t seg, uint32_t& first, int& n) {
    const uint32_t st = seg & 0xffffu, len = seg >> 16;
    first = c0 + (st >> 2);
    n = len ? static_cast<int>(((st + len + 3) >> 2) - (st >> 2)) : 0;
  };
  auto request = [&](const GramEntry& e, Row& r) {
    chunks(e.c0, e.segI, r.cI, r.nI);
    chunks(e.c0, e.segJ, r.cJ, r.nJ);
    r.rw = r.nI > 0 ? rw64[sc.row_base + e.row] : 0.0;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int p = sub + 8 * u;
      r.vI[u] = r.vJ[u] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);  // value 0: nothing is placed
      r.kI[u] = r.kJ[u] = make_uint2(0u, 0u);
      if (p < r.nI) {
        r.vI[u] = valc[r.cI + p];
        r.kI[u] = colc[r.cI + p];
      }
      if (p < r.nJ) {
        r.vJ[u] = valc[r.cJ + p];
        r.kJ[u] = colc[r.cJ + p];
      }
    }
  };
  double* rI = bufI + g * kGramLd;
  float* rJ = bufJ + g * kGramLd;
  auto put = [&](auto* dst, int blk, const float4& v, const uint2& c, auto scale, uint32_t& used) {
    const float vv[4] = {v.x, v.y, v.z, v.w};
    const uint32_t cc[4] = {c.x & 0xffffu, c.x >> 16, c.y & 0xffffu, c.y >> 16};
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (vv[q] != 0.0f && static_cast<int>(cc[q] >> 6) == blk) {
        dst[cc[q] & (kFb - 1)] = scale * vv[q];
        used |= 1u << ((cc[q] >> 4) & 3);
      }
  };
  GramEntry e1;
  Row cur;
  entry(l0 + g, e1);
  request(e1, cur);
  entry(l0 + kStep + g, e1);
  for (int64_t li = l0; li < le; li += kStep) {
    // zero the row (its 64 columns, eight lanes), then place the segments
#pragma unroll
    for (int q = 0; q < 4; ++q) *reinterpret_cast<double2*>(rI + 16 * q + 2 * sub) = make_double2(0.0, 0.0);
#pragma unroll
    for (int q = 0; q < 2; ++q)
      *reinterpret_cast<float4*>(rJ + 32 * q + 4 * sub) = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    wave_lds_sync();
    uint32_t uI = 0, uJ = 0;
    put(rI, I, cur.vI[0], cur.kI[0], cur.rw, uI);
    put(rJ, J, cur.vJ[0], cur.kJ[0], 1.0f, uJ);
    if (sub + 8 < cur.nI) put(rI, I, cur.vI[1], cur.kI[1], cur.rw, uI);
    if (sub + 8 < cur.nJ) put(rJ, J, cur.vJ[1], cur.kJ[1], 1.0f, uJ);
    for (int p = sub + 16; p < cur.nI; p += 8) put(rI, I, valc[cur.cI + p], colc[cur.cI + p], cur.rw, uI);
    for (int p = sub + 16; p < cur.nJ; p += 8) put(rJ, J, valc[cur.cJ + p], colc[cur.cJ + p], 1.0f, uJ);
    {
      // over the 32 lanes of four rows
      uint32_t u = uI | uJ << 4;
#pragma unroll
      for (int d = 1; d < 32; d <<= 1) u |= __shfl_xor(u, d, 64);
      if ((lane & 31) == 0) occ[tid >> 5] = u;
    }
    request(e1, cur);  // the next row's, in flight over the products
    entry(li + 2 * kStep + g, e1);
    __syncthreads();
    uint32_t use[kStep / 4];
#pragma unroll
    for (int h = 0; h < kStep / 4; ++h) use[h] = __builtin_amdgcn_readfirstlane(occ[h]);
#pragma unroll
    for (int h = 0; h < kStep / 4; ++h) {
      const uint32_t ui = (use[h] >> (qi / 16)) & 3u, uj = (use[h] >> (4 + qj / 16)) & 3u;
      if (ui == 0 || uj == 0) continue;
      double av[2], bv[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        av[q] = bufI[(4 * h + kk) * kGramLd + qi + 16 * q + m];
        bv[q] = static_cast<double>(bufJ[(4 * h + kk) * kGramLd + qj + 16 * q + m]);
      }
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
          if ((ui >> a & 1u) && (uj >> b & 1u)) {
            const v4d d = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a], bv[b], v4d{0.0, 0.0, 0.0, 0.0}, 0, 0, 0);
            const v4d t = hi[a][b] + d;
            lo[a][b] += d - (t - hi[a][b]);  // exact: hi >= big >= d
            hi[a][b] = t;
          }
    }
    __syncthreads();  // the next rows overwrite the buffers
  }
  // item r of a lane is row l / 16 + 4 r and column l % 16 of its 16 x 16 block
  double* Gs = G + static_cast<int64_t>(s) * ld * ld;
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = qi + 16 * a + kk + 4 * r, col = qj + 16 * b + m;
        if (I != J || row <= col)
          Gs[static_cast<int64_t>(I * kFb + row) * ld + J * kFb + col] = (hi[a][b][r] - big) + lo[a][b][r];
      }
}

// For the chunk of scenarios [scen_begin, scen_begin + nscen) of one patient
// (chunk buffers, npad x npad per scenario, upper triangle of G accumulated):
// the upper tiles of A = G + rho/2 I (identity on the padding; inside a
// diagonal tile both triangles, the lower one read from the upper), and, when
// accumulate_gsum, their sum over the chunk added to the packed sum_s G_s.
__global__ __launch_bounds__(256) void k_gram_finish(FactorArgs f, int patient, int scen_begin, int nscen,
                                                     int npad, int n, double rho, int accumulate_gsum) {
  const Pat pt = f.pat[patient];
  const int64_t nn = static_cast<int64_t>(npad) * npad;
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  (void)scen_begin;
  for (int64_t idx = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; idx < nn; idx += stride) {
    const int i = static_cast<int>(idx / npad), j = static_cast<int>(idx % npad);
    const int I = i / kFb, J = j / kFb;
    if (I > J) continue;  // only the upper tiles are used from here on
    const int64_t src = (i <= j) ? idx : static_cast<int64_t>(j) * npad + i;
    double sum = 0.0;
    for (int s = 0; s < nscen; ++s) {
      const double gv = f.G[s * nn + src];
      sum += gv;
      double a = gv;
      if (i == j) a += (i < n) ? 0.5 * rho : 1.0;
      f.A[s * nn + idx] = a;
    }
    if (accumulate_gsum)
      f.Gp[pt.gpack_off + tile_index(I, J, pt.nbk) * kFb * kFb + (i % kFb) * kFb + (j % kFb)] += sum;
  }
}

// ---------------------------------------------------------------------------
// block sweep
// ---------------------------------------------------------------------------

// The sweep takes pivot blocks of kKb = 128 (a last one of 64 where npad / 64 is
// odd), so that every tile of the matrix is read and written once per 128
// columns: at 13 scenarios of 2 981 spots one pass over the upper tiles moves
// 0.96 GB, which bounded the rank-64 update (275 us a step, twice as many
// steps); the rank-128 products run on the fp64 MFMA.
constexpr int kKb = 128;

// Value of lane t of the lane's row of 16, in every lane of the row.
template <int t>
__device__ __forceinline__ double row_bcast(double x) {
  return dpp_move<0x150 + t>(x);  // row_newbcast
}

// In place, the sweep of a 16 x 16 matrix held by one wave in the MFMA's output
// layout (item q of lane l: row l / 16 + 4 q, column l % 16): -inverse.
template <int t>
__device__ __forceinline__ void sweep16_steps(double (&r)[4], int m, int kk) {
  constexpr int tk = t & 3, tq = t >> 2;
  const double rowv = __shfl(r[tq], 16 * tk + m, 64);  // pivot row
  const double inv = 1.0 / row_bcast<t>(rowv);
  const double w = m == t ? -inv : rowv * inv;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const double c = row_bcast<t>(r[q]);  // pivot column
    r[q] = fma(-c, w, m == t ? 0.0 : r[q]);
  }
  if (kk == tk) r[tq] = w;
  if constexpr (t < 15) sweep16_steps<t + 1>(r, m, kk);
}

// P = A_KK^-1 for a pivot block of KB = 128 or 64 (one workgroup of eight waves
// per scenario): the same block sweep on 16-blocks, the upper 16 x 16 tiles kept
// in LDS.  Per 16-block b: U_i^T = P16 M_bi (one wave per i), then M_ij -= U_i
// M_bj by the MFMA; the wave that owns the next pivot tile updates it first and
// inverts it in registers while the others work, so the chain is eight times 16
// scalar steps of about 0.2 us.  A scalar sweep of 64 columns, two barriers a
// step, took 65 us; this takes 32 us for 128 and 14 for 64.
template <int KB>
__global__ __launch_bounds__(512) void k_sweep_pivot(FactorArgs f, int npad, int k0) {
  constexpr int NB = KB / 16, NT = NB * (NB + 1) / 2;
  __shared__ double M[NT * 256];      // tile (i, j), i <= j, row-major
  __shared__ double U[NB * 256];      // U_i^T
  __shared__ double V[NB * 256];      // M_bi before the step
  __shared__ double P16[2][256];
  const int g = static_cast<int>(blockIdx.x);  // place in the chunk
  const double* A = f.A + static_cast<int64_t>(blockIdx.x) * npad * npad;  // chunk buffer
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, m = lane & 15, kk = lane >> 4;
  auto tile = [](int i, int j) { return 256 * (i * NB - i * (i - 1) / 2 + (j - i)); };
  // upper 16 x 16 tile t -> (i, j)
  auto place = [](int t, int& i, int& j) {
    i = 0;
    while (t >= NB - i) {
      t -= NB - i;
      ++i;
    }
    j = i + t;
  };
  const int wu = __builtin_amdgcn_readfirstlane(w);
  constexpr int kPer = (NT + 7) / 8;  // tiles of a wave, all requested at once
  double x[kPer][4];
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    int i, j;
    place(wu + 8 * u < NT ? wu + 8 * u : 0, i, j);
    const double* T = A + static_cast<int64_t>(k0 + 16 * i) * npad + k0 + 16 * j;
#pragma unroll
    for (int q = 0; q < 4; ++q) x[u][q] = T[static_cast<int64_t>(kk + 4 * q) * npad + m];
  }
#pragma unroll
  for (int u = 0; u < kPer; ++u)
    if (wu + 8 * u < NT) {
#pragma unroll
      for (int q = 0; q < 4; ++q) M[256 * (wu + 8 * u) + (kk + 4 * q) * 16 + m] = x[u][q];
    }
  __syncthreads();
  auto invert = [&](double (&r)[4], double* out) {
    sweep16_steps<0>(r, m, kk);
#pragma unroll
    for (int q = 0; q < 4; ++q) out[(kk + 4 * q) * 16 + m] = -r[q];
  };
  if (w == 0) {
    double r[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) r[q] = M[(kk + 4 * q) * 16 + m];
    invert(r, P16[0]);
  }
  __syncthreads();
  for (int b = 0; b < NB; ++b) {
    const double* P = P16[b & 1];
    // panel: wave i
    if (w < NB && w != b) {
      double v[4];
      v4d d = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        // M_bi [kk + 4 q][m]
        v[q] = b < w ? M[tile(b, w) + (kk + 4 * q) * 16 + m] : M[tile(w, b) + m * 16 + kk + 4 * q];
        d = __builtin_amdgcn_mfma_f64_16x16x4f64(P[(kk + 4 * q) * 16 + m], v[q], d, 0, 0, 0);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        V[w * 256 + (kk + 4 * q) * 16 + m] = v[q];
        U[w * 256 + (kk + 4 * q) * 16 + m] = d[q];
      }
    }
    __syncthreads();
    auto update = [&](int i, int j, double (&r)[4]) {
      double* T = M + tile(i, j);
      v4d d;
#pragma unroll
      for (int q = 0; q < 4; ++q) d[q] = -T[(kk + 4 * q) * 16 + m];
#pragma unroll
      for (int q = 0; q < 4; ++q)
        d = __builtin_amdgcn_mfma_f64_16x16x4f64(U[i * 256 + (kk + 4 * q) * 16 + m], V[j * 256 + (kk + 4 * q) * 16 + m], d,
                                                 0, 0, 0);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        r[q] = -d[q];
        T[(kk + 4 * q) * 16 + m] = r[q];
      }
    };
    double r[4];
    if (w == 0 && b + 1 < NB) {
      update(b + 1, b + 1, r);
      invert(r, P16[(b + 1) & 1]);
    } else {
      // the other tiles, dealt to the other waves (to all of them in the last step)
      const int first = b + 1 < NB ? 1 : 0, nw = 8 - first;
      for (int t = wu - first; t < NT; t += nw) {
          int i, j;
          place(t, i, j);
          if (i == b + 1 && j == b + 1) continue;
          double* T = M + tile(i, j);
          if (i != b && j != b) {
            update(i, j, r);
          } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const int row = kk + 4 * q;
              T[row * 16 + m] = i == j ? -P[row * 16 + m] : (i == b ? U[j * 256 + row * 16 + m] : U[i * 256 + m * 16 + row]);
            }
          }
      }
    }
    __syncthreads();
  }
  // the swept block is -A_KK^-1; both triangles of P
  double* P = f.P + static_cast<int64_t>(g) * kKb * kKb;
  for (int t = wu; t < NT; t += 8) {
    int i, j;
    place(t, i, j);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = kk + 4 * q;
      P[(16 * i + r) * kKb + 16 * j + m] = -M[256 * t + r * 16 + m];
      if (i != j) P[(16 * j + r) * kKb + 16 * i + m] = -M[256 * t + m * 16 + r];
    }
  }
}

// Element at a wave-uniform base and a byte offset per lane: one scalar pointer
// and one 32-bit register address it.
template <class T>
__device__ __forceinline__ T* at_bytes(T* base, uint32_t bytes) {
  return reinterpret_cast<T*>(reinterpret_cast<std::conditional_t<std::is_const_v<T>, const char*, char*>>(base) + bytes);
}

// The 16 x 16 tiles (i, j), i <= j, of a pivot block of KB columns, in the
// registers of four waves: wave 0 has the diagonal ones (tile (s, s) in slot s)
// and, of 128 columns, the last of the others, which waves 1 to 3 take in turn.
template <int KB>
struct PivotTiles {
  static constexpr int NB = KB / 16, kOff = NB * (NB - 1) / 2, kPer = NB == 8 ? 9 : 4;
  v4d T[kPer];  // item q: row kk + 4 q, column m
  int ij[kPer];  // 16 i + j, -1: none
  __device__ __forceinline__ explicit PivotTiles(int wu) {
#pragma unroll
    for (int s = 0; s < kPer; ++s) {
      int t = wu == 0 ? 27 : 3 * s + wu - 1;
      ij[s] = -1;
      if (wu == 0 && s < NB) {
        ij[s] = 17 * s;
      } else if (t < kOff && (wu == 0 || t != 27)) {
        int i = 0;
        while (t >= NB - 1 - i) {
          t -= NB - 1 - i;
          ++i;
        }
        ij[s] = 16 * i + i + 1 + t;
      }
    }
  }
};

constexpr int kPivotLds = 8 * 256 * 2 + 2 * 256;  // doubles

// k_sweep_pivot on a block held in PivotTiles, within the threads, registers and
// LDS of k_sweep_update, with the same results bit for bit: the owners of row and
// column b form V_i and U_i, wave 0 inverts.  With four waves the chain takes
// 53 us for 128 columns, beside other work.
template <int KB>
__device__ __forceinline__ void sweep_pivot_block(PivotTiles<KB>& pt, double* lds, double* P) {
  using PT = PivotTiles<KB>;
  constexpr int NB = PT::NB, kPer = PT::kPer;
  double* U = lds;              // U_i^T
  double* V = lds + 8 * 256;    // M_bi before the step
  double* P16 = lds + 16 * 256;  // two of 256
  const int tid = threadIdx.x, lane = tid & 63, m = lane & 15, kk = lane >> 4;
  const int wu = __builtin_amdgcn_readfirstlane(tid >> 6);
  auto invert = [&](const v4d& t, double* out) {
    double r[4] = {t[0], t[1], t[2], t[3]};
    sweep16_steps<0>(r, m, kk);
#pragma unroll
    for (int q = 0; q < 4; ++q) out[(kk + 4 * q) * 16 + m] = -r[q];
  };
  auto update = [&](int i, int j, v4d t) {
    v4d d = -t;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      d = __builtin_amdgcn_mfma_f64_16x16x4f64(U[i * 256 + (kk + 4 * q) * 16 + m], V[j * 256 + (kk + 4 * q) * 16 + m], d, 0,
                                               0, 0);
    return -d;
  };
  if (wu == 0) invert(pt.T[0], P16);
  __syncthreads();
#pragma unroll 1
  for (int b = 0; b < NB; ++b) {
    const double* Pb = P16 + 256 * (b & 1);
#pragma unroll
    for (int s = 0; s < kPer; ++s) {
      __builtin_amdgcn_sched_barrier(0);  // a tile at a time: the registers are those of the update
      int ij = pt.ij[s];
      asm volatile("" : "+s"(ij));  // no address kept over the rounds
      const int i = ij >> 4, j = ij & 15;
      if (ij < 0 || (i == b) == (j == b)) continue;
      const int o = i == b ? j : i;
      double v[4];
      if (i == b) {
#pragma unroll
        for (int q = 0; q < 4; ++q) V[o * 256 + (kk + 4 * q) * 16 + m] = v[q] = pt.T[s][q];
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) V[o * 256 + m * 16 + kk + 4 * q] = pt.T[s][q];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = V[o * 256 + (kk + 4 * q) * 16 + m];
      }
      v4d d = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int q = 0; q < 4; ++q) d = __builtin_amdgcn_mfma_f64_16x16x4f64(Pb[(kk + 4 * q) * 16 + m], v[q], d, 0, 0, 0);
#pragma unroll
      for (int q = 0; q < 4; ++q) U[o * 256 + (kk + 4 * q) * 16 + m] = d[q];
    }
    __syncthreads();
    if (wu == 0 && b + 1 < NB) {
      v4d t = pt.T[0];
#pragma unroll
      for (int s = 1; s < NB; ++s)
#pragma unroll
        for (int q = 0; q < 4; ++q) t[q] = s == b + 1 ? pt.T[s][q] : t[q];
      t = update(b + 1, b + 1, t);
#pragma unroll
      for (int s = 1; s < NB; ++s)
#pragma unroll
        for (int q = 0; q < 4; ++q) pt.T[s][q] = s == b + 1 ? t[q] : pt.T[s][q];
      invert(t, P16 + 256 * ((b + 1) & 1));
    }
#pragma unroll
    for (int s = 0; s < kPer; ++s) {
      __builtin_amdgcn_sched_barrier(0);
      int ij = pt.ij[s];
      asm volatile("" : "+s"(ij));
      const int i = ij >> 4, j = ij & 15;
      if (ij < 0 || (i == b + 1 && j == b + 1)) continue;
      if (i != b && j != b) {
        pt.T[s] = update(i, j, pt.T[s]);
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int row = kk + 4 * q;
          pt.T[s][q] = i == j ? -Pb[row * 16 + m] : (i == b ? U[j * 256 + row * 16 + m] : U[i * 256 + m * 16 + row]);
        }
      }
    }
    __syncthreads();
  }
  // the swept block is -A_KK^-1; both triangles of P
#pragma unroll
  for (int s = 0; s < kPer; ++s) {
    __builtin_amdgcn_sched_barrier(0);
    if (pt.ij[s] < 0) continue;
    const int i = pt.ij[s] >> 4, j = pt.ij[s] & 15;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = kk + 4 * q;
      P[(16 * i + r) * kKb + 16 * j + m] = -pt.T[s][q];
      if (i != j) P[(16 * j + m) * kKb + 16 * i + r] = -pt.T[s][q];
    }
  }
}

// Panels of a pivot block for 64 columns i of the matrix: R = A_K,i (old values)
// and Ut = U^T = P A_K,i.  Only the upper tiles (I <= J) of the sweep matrix are
// kept up to date (it stays symmetric), so blocks before the pivot are read from
// the mirrored tile, transposed.  The columns of A_K,i go through LDS 32 rows at
// a time; wave w forms KB / 4 rows of Ut, its operand P read by columns (P is
// symmetric) straight from memory.  The columns of the pivot block itself have
// no panels: there the block is replaced by -P.
template <int KB>
__global__ __launch_bounds__(256) void k_sweep_panel(FactorArgs f, int npad, int k0) {
  constexpr int kLd = kFb + 16;
  __shared__ double ks[32][kLd];
  const int g = static_cast<int>(blockIdx.y);  // place in the chunk
  double* A = f.A + static_cast<int64_t>(blockIdx.y) * npad * npad;  // chunk buffer
  const int i0 = static_cast<int>(blockIdx.x) * kFb;
  const double* Pg = f.P + static_cast<int64_t>(g) * kKb * kKb;
  if (i0 / kKb == k0 / kKb) {
    for (int e = threadIdx.x; e < (i0 + kFb - k0) * kFb; e += 256) {
      const int r = e / kFb, c = i0 - k0 + e % kFb;
      A[static_cast<int64_t>(k0 + r) * npad + k0 + c] = -Pg[r * kKb + c];
    }
    return;
  }
  double* Ut = f.U + static_cast<int64_t>(g) * npad * kKb;
  double* R = f.R + static_cast<int64_t>(g) * npad * kKb;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, m = lane & 15, kk = lane >> 4;
  constexpr int NC = KB / 64;  // 16-row groups of Ut per wave
  v4d acc[NC][4];
#pragma unroll
  for (int a = 0; a < NC; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = v4d{0.0, 0.0, 0.0, 0.0};
  for (int s0 = 0; s0 < KB; s0 += 32) {
    double x[8];
    const bool stored = i0 / kFb >= (k0 + s0) / kFb;  // tile (K, I) of the upper tiles
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int e = tid + 256 * q;
      if (stored)
        x[q] = A[static_cast<int64_t>(k0 + s0 + e / kFb) * npad + i0 + e % kFb];
      else
        x[q] = A[static_cast<int64_t>(i0 + e / 32) * npad + k0 + s0 + e % 32];
    }
    __syncthreads();  // the last slab has been read
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int e = tid + 256 * q;
      if (stored)
        ks[e / kFb][e % kFb] = x[q];
      else
        ks[e % 32][e / 32] = x[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int e = tid + 256 * q;
      R[static_cast<int64_t>(s0 + e / kFb) * npad + i0 + e % kFb] = ks[e / kFb][e % kFb];
    }
#pragma unroll
    for (int h = 0; h < 8; ++h) {
      double av[NC], bv[4];
#pragma unroll
      for (int a = 0; a < NC; ++a) av[a] = Pg[(s0 + 4 * h + kk) * kKb + (w * NC + a) * 16 + m];
#pragma unroll
      for (int b = 0; b < 4; ++b) bv[b] = ks[4 * h + kk][16 * b + m];
#pragma unroll
      for (int a = 0; a < NC; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a], bv[b], acc[a][b], 0, 0, 0);
    }
  }
#pragma unroll
  for (int a = 0; a < NC; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        Ut[static_cast<int64_t>((w * NC + a) * 16 + kk + 4 * r) * npad + i0 + 16 * b + m] = acc[a][b][r];
}

// Rank-KB update of the next pivot block (at k1, KBN columns) of scenario g, and
// its inverse: the accumulators start from -A_ij, the panels' columns pass
// through LDS in slabs of 8 rows, the next slab's loads in flight over the
// current one's products.
template <int KB, int KBN>
__device__ __forceinline__ void sweep_next_pivot(const FactorArgs& f, int npad, int k1, int g, double* lds) {
  constexpr int kLd = KBN + 16, kSlab = 8, kQ = (kSlab * KBN / 2 + 255) / 256;
  constexpr int kPer = PivotTiles<KBN>::kPer;
  static_assert(4 * kSlab * kLd <= 4 * 16 * 80 && kPivotLds <= 4 * 16 * 80 && kSlab * KBN / 2 % 256 == 0);
  const double* A = f.A + static_cast<int64_t>(g) * npad * npad + static_cast<int64_t>(k1) * npad + k1;
  const double* Ut = f.U + static_cast<int64_t>(g) * npad * kKb + k1;
  const double* R = f.R + static_cast<int64_t>(g) * npad * kKb + k1;
  const int tid = threadIdx.x, lane = tid & 63, m = lane & 15, kk = lane >> 4;
  PivotTiles<KBN> pt(__builtin_amdgcn_readfirstlane(tid >> 6));
  uint32_t o[kQ];
#pragma unroll
  for (int q = 0; q < kQ; ++q) {
    const int e = tid + 256 * q, r = e / (KBN / 2), c = 2 * (e % (KBN / 2));
    o[q] = 8u * static_cast<uint32_t>(r * npad + c);
  }
  v2d ub[kQ], rb[kQ];
  auto fetch = [&](int s) {
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      ub[q] = *reinterpret_cast<const v2d*>(at_bytes(Ut + static_cast<int64_t>(s) * kSlab * npad, o[q]));
      rb[q] = *reinterpret_cast<const v2d*>(at_bytes(R + static_cast<int64_t>(s) * kSlab * npad, o[q]));
    }
  };
  auto stage = [&](int buf) {
    double* u = lds + buf * kSlab * kLd;
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      const int e = tid + 256 * q, r = e / (KBN / 2), c = 2 * (e % (KBN / 2));
      *reinterpret_cast<v2d*>(&u[r * kLd + c]) = ub[q];
      *reinterpret_cast<v2d*>(&u[2 * kSlab * kLd + r * kLd + c]) = rb[q];
    }
  };
  fetch(0);
#pragma unroll
  for (int s = 0; s < kPer; ++s) {
    const int ij = pt.ij[s] < 0 ? 0 : pt.ij[s];
#pragma unroll
    for (int q = 0; q < 4; ++q)
      pt.T[s][q] = -*at_bytes(A + static_cast<int64_t>(16 * (ij >> 4) + 4 * q) * npad + 16 * (ij & 15),
                              8u * static_cast<uint32_t>(kk * npad + m));
  }
  stage(0);
  __syncthreads();
  constexpr int ns = KB / kSlab;
#pragma unroll 1
  for (int s = 0; s < ns; ++s) {
    fetch(s + 1 < ns ? s + 1 : 0);  // the last round's is not used
    __builtin_amdgcn_sched_barrier(0);
    const double* u = lds + (s & 1) * kSlab * kLd;
    const double* v = u + 2 * kSlab * kLd;
#pragma unroll
    for (int t = 0; t < kPer; ++t) {
      if (t % 3 == 0) __builtin_amdgcn_sched_barrier(0);
      int ij = pt.ij[t] < 0 ? 0 : pt.ij[t];
      asm volatile("" : "+s"(ij));
#pragma unroll
      for (int h = 0; h < kSlab / 4; ++h)
        pt.T[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(u[(4 * h + kk) * kLd + 16 * (ij >> 4) + m],
                                                       v[(4 * h + kk) * kLd + 16 * (ij & 15) + m], pt.T[t], 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    stage((s + 1) & 1);
    __syncthreads();
  }
#pragma unroll
  for (int s = 0; s < kPer; ++s) pt.T[s] = -pt.T[s];
  sweep_pivot_block<KBN>(pt, lds, f.P + static_cast<int64_t>(g) * kKb * kKb);
}

// A 64 x 64 tile of M_s in LDS (rows kLdM apart) to its stored order.  Thread t of
// the x-update holds the 4 x 4 block of rows 4 (t / 16) .. + 3 and columns
// 4 (t % 16) .. + 3 as four float4 (row k = 0..3 of the block); float4 k of
// thread t is stored at k * 256 + t, so that every wave load instruction of
// the x-update reads 1 KiB contiguous.
constexpr int kLdM = kFb + 4;
__device__ __forceinline__ void store_xtile(float* __restrict__ dst, const float* tile) {
  const int t = threadIdx.x;
#pragma unroll
  for (int k = 0; k < 4; ++k)
    *reinterpret_cast<float4*>(dst + 4 * (k * 256 + t)) =
        *reinterpret_cast<const float4*>(tile + (4 * (t >> 4) + k) * kLdM + 4 * (t & 15));
}

// Rank-KB update A_ij -= U_i R_j of one upper 64 x 64 tile off the pivot row and
// column, whose tiles are replaced by the panels.  Waves 2 x 2, 32 rows and
// columns each, on the fp64 MFMA: the accumulators start from -A_ij, the panels
// pass through LDS in slabs of 16 columns, the next slab's loads in flight over
// the current one's products.  13 scenarios of 2 981 spots: 328 us a step of 128
// (47 TFLOP/s, the products' issue; the rank-64 vector form took 2 x 275 us),
// 351 us with blocks of 128 x 128 (at 1 700 spots 129 against 104 us: too few
// blocks), and the same with an XCD's tiles next to each other.
//
// The first workgroups, one per scenario, instead update the next pivot block
// (KBN columns; 0: none) in registers, in the same order of products, and invert
// it beside the other tiles' work: two inversions of 13 scenarios of 2 003 spots
// and a warm start's other work 9.57 -> 8.74 ms.
//
// LAST: the last step's tiles are the inverse's, rounded to fp32 and stored in the
// x-update's order instead of going back to A (a kernel that did so afterwards
// took 109 us at 13 scenarios of 2 003 spots; the step itself 149 -> 140).
template <int KB, int KBN, bool LAST>
__global__ __launch_bounds__(256, 4) void k_sweep_update(FactorArgs f, int npad, int k0, int nscen, int patient,
                                                         int scen_begin) {
  constexpr int MT = kFb, kLd = MT + 16, kSlab = 16;
  constexpr int W = MT / 32;                 // 16-wide groups of a wave
  constexpr int kQ = kSlab * MT / 2 / 256;   // double2 per thread, slab and panel
  __shared__ __align__(16) double lds[4 * kSlab * kLd];
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, m = lane & 15, kk = lane >> 4;
  const int wu = __builtin_amdgcn_readfirstlane(w);
  const int k1 = k0 + KB;  // the next pivot block
  int x = static_cast<int>(blockIdx.x);
  if constexpr (KBN != 0) {
    if (x < nscen) {
      __builtin_amdgcn_s_setprio(2);  // the chain goes before the tiles that share its CU
      sweep_next_pivot<KB, KBN>(f, npad, k1, x, lds);
      return;
    }
    x -= nscen;
  }
  const int nm = npad / MT, nt = nm * (nm + 1) / 2;
  const int g = x / nt;  // place in the chunk
  // upper tile number -> (bi, bj), bi <= bj
  int t0 = x - g * nt, bi = 0;
  while (t0 >= nm - bi) {
    t0 -= nm - bi;
    ++bi;
  }
  const int bj = bi + t0;
  double* A = f.A + static_cast<int64_t>(g) * npad * npad;  // chunk buffer
  const int i0 = bi * MT, j0 = bj * MT;
  const double* Ut = f.U + static_cast<int64_t>(g) * npad * kKb;
  const double* R = f.R + static_cast<int64_t>(g) * npad * kKb;
  const bool rowK = i0 / kKb == k0 / kKb, colK = j0 / kKb == k0 / kKb;
  float* Mt = nullptr;  // the stored tile, formed in LDS first
  float* mt = reinterpret_cast<float*>(lds);
  if constexpr (LAST) {
    Mt = f.Mp + f.scen[scen_begin + g].mpack_off + tile_index(bi, bj, f.pat[patient].nbk) * kFb * kFb;
    if (colK) {  // M = -A: P, or -U
      const double* Pg = f.P + static_cast<int64_t>(g) * kKb * kKb;
      for (int q = 0; q < kFb / 4; ++q) {
        const int r = tid & 63, c = (tid >> 6) + 4 * q;
        mt[r * kLdM + c] = static_cast<float>(rowK ? Pg[(j0 - k0 + c) * kKb + i0 - k0 + r]
                                                   : -Ut[static_cast<int64_t>(j0 - k0 + c) * npad + i0 + r]);
      }
      __syncthreads();
      store_xtile(Mt, mt);
      return;
    }
  }
  if (rowK && colK) return;  // already -P
  if (KBN != 0 && i0 / kKb == k1 / kKb && j0 / kKb == k1 / kKb) return;
  if (rowK || colK) {
    double* tr = lds;  // 32 x 33, for the transposed copies
    for (int sub = 0; sub < MT / 32 * (MT / 32); ++sub) {
      const int r0 = i0 + 32 * (sub / (MT / 32)), c0 = j0 + 32 * (sub % (MT / 32));
      if (rowK) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int r = r0 + (tid >> 5) + 8 * q, c = c0 + (tid & 31);
          A[static_cast<int64_t>(r) * npad + c] = Ut[static_cast<int64_t>(r - k0) * npad + c];
        }
      } else {
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int c = c0 + (tid >> 5) + 8 * q, r = r0 + (tid & 31);
          tr[((tid >> 5) + 8 * q) * 33 + (tid & 31)] = Ut[static_cast<int64_t>(c - k0) * npad + r];
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int r = r0 + (tid >> 5) + 8 * q, c = c0 + (tid & 31);
          A[static_cast<int64_t>(r) * npad + c] = tr[(tid & 31) * 33 + (tid >> 5) + 8 * q];
        }
      }
    }
    return;
  }
  double (*us)[kSlab * kLd] = reinterpret_cast<double (*)[kSlab * kLd]>(lds);
  double (*rs)[kSlab * kLd] = us + 2;
  const int wi = (MT / 2) * (wu >> 1), wj = (MT / 2) * (wu & 1);
  // every address: a wave-uniform base and a 32-bit byte offset per lane
  uint32_t oi[kQ], oj[kQ];
#pragma unroll
  for (int q = 0; q < kQ; ++q) {
    const int e = tid + 256 * q, r = e / (MT / 2), c = 2 * (e % (MT / 2));
    oi[q] = 8u * static_cast<uint32_t>(r * npad + i0 + c);
    oj[q] = 8u * static_cast<uint32_t>(r * npad + j0 + c);
  }
  v2d ub[kQ], rb[kQ];
  auto fetch = [&](int s) {
    const double* u = Ut + static_cast<int64_t>(s) * kSlab * npad;
    const double* r = R + static_cast<int64_t>(s) * kSlab * npad;
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      ub[q] = *reinterpret_cast<const v2d*>(at_bytes(u, oi[q]));
      rb[q] = *reinterpret_cast<const v2d*>(at_bytes(r, oj[q]));
    }
  };
  auto stage = [&](int buf) {
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      const int e = tid + 256 * q, r = e / (MT / 2), c = 2 * (e % (MT / 2));
      *reinterpret_cast<v2d*>(&us[buf][r * kLd + c]) = ub[q];
      *reinterpret_cast<v2d*>(&rs[buf][r * kLd + c]) = rb[q];
    }
  };
  fetch(0);
  v4d acc[W][W];
  double* Aw = A + static_cast<int64_t>(i0 + wi) * npad + j0 + wj;
  const uint32_t oa = 8u * static_cast<uint32_t>(kk * npad + m);
#pragma unroll
  for (int a = 0; a < W; ++a)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const double* row = Aw + static_cast<int64_t>(16 * a + 4 * r) * npad;
#pragma unroll
      for (int b = 0; b < W; ++b) acc[a][b][r] = -*at_bytes(row + 16 * b, oa);
    }
  stage(0);
  __syncthreads();
  constexpr int ns = KB / kSlab;
#pragma unroll 2
  for (int s = 0; s < ns; ++s) {
    fetch(s + 1 < ns ? s + 1 : 0);  // the last round's is not used
    __builtin_amdgcn_sched_barrier(0);  // requested before the products, waited for after them
    const double* u = &us[s & 1][kk * kLd + wi + m];
    const double* v = &rs[s & 1][kk * kLd + wj + m];
#pragma unroll
    for (int h = 0; h < kSlab / 4; ++h) {
      double av[W], bv[W];
#pragma unroll
      for (int q = 0; q < W; ++q) {
        av[q] = u[4 * h * kLd + 16 * q];
        bv[q] = v[4 * h * kLd + 16 * q];
      }
#pragma unroll
      for (int a = 0; a < W; ++a)
#pragma unroll
        for (int b = 0; b < W; ++b) acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a], bv[b], acc[a][b], 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    stage((s + 1) & 1);
    __syncthreads();
  }
  if constexpr (LAST) {
#pragma unroll
    for (int a = 0; a < W; ++a)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int b = 0; b < W; ++b)
          mt[(wi + 16 * a + kk + 4 * r) * kLdM + wj + 16 * b + m] = static_cast<float>(acc[a][b][r]);
    __syncthreads();
    store_xtile(Mt, mt);
    return;
  }
#pragma unroll
  for (int a = 0; a < W; ++a)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      double* row = Aw + static_cast<int64_t>(16 * a + 4 * r) * npad;
#pragma unroll
      for (int b = 0; b < W; ++b) *at_bytes(row + 16 * b, oa) = -acc[a][b][r];
    }
}

// ---------------------------------------------------------------------------
// per-iteration kernels
// ---------------------------------------------------------------------------

// Row rotations by DPP for the x-update's row sums (the pair and quad
// exchanges are those of scalars.h).
constexpr int kDppRor4 = 0x124;
constexpr int kDppRor8 = 0x128;

// One packed tile T = M_s[I, J] (I <= J) per workgroup: a = T c_J and, off
// the diagonal, b = T^T c_I (the tile's contribution to the rows of block J).
// Thread t holds the 4 x 4 block at rows 4 rb, columns 4 cb (rb = t / 16,
// cb = t % 16; four float4 loads, each a 1 KiB contiguous read per wave in
// the stored order of store_xtile), so both products use the registers as
// loaded: the row sums are reduced over the 16 lanes of a DPP row, the column
// sums over the wave's four rows by shuffles and over the four waves in
// shared memory.  The tile table entry carries every address, so the tile
// load depends on one table read only.  The right-hand side and all sums are
// fp64: the inverse has entries of both signs and |M| |c| exceeds |M c| by two
// orders of magnitude, so fp32 sums would put a floor of about 1e-5 relative
// under every x-update; the fp32 storage of M itself contributes about 1e-6.
// kLoadsFirst (a context of one patient): the tile's 16 KB (tile idx of the
// table is stored at Mp + 4096 idx) are requested before the table and
// stop-flag reads, and the empty statement keeps the compiler from moving the
// loads below the early exit (a stopped patient ends the run within an
// iteration).  Otherwise (a batch, whose other patients go on iterating) the
// flag is read first and a stopped patient's tiles are not loaded at all.
template <bool kLoadsFirst>
__device__ __forceinline__ void xsym_tile(const FactorArgs& f, const double* __restrict__ c, int idx) {
  __shared__ double2 cI[kFb / 2], cJ[kFb / 2];
  __shared__ double bpart[4][kFb];  // column sums of each wave
  const int tid = threadIdx.x;
  const int rb = tid >> 4, cb = tid & 15, lane = tid & 63;
  const float4* T = reinterpret_cast<const float4*>(f.Mp) + static_cast<int64_t>(idx) * 1024;
  float4 m[4];
  XTile tj;
  if constexpr (kLoadsFirst) {
#pragma unroll
    for (int k = 0; k < 4; ++k) m[k] = T[k * 256 + tid];
    tj = f.xtiles[idx];
    const bool stopped = f.ps[tj.patient].stopped != 0;
    asm volatile("" ::: "memory");
    if (stopped) return;
  } else {
    tj = f.xtiles[idx];
    if (f.ps[tj.patient].stopped) return;
#pragma unroll
    for (int k = 0; k < 4; ++k) m[k] = T[k * 256 + tid];
  }
  if (tid < kFb) {
    const int jc = tj.J * kFb + tid, ic = tj.I * kFb + tid;
    reinterpret_cast<double*>(cJ)[tid] = jc < tj.n ? c[tj.vbase + jc] : 0.0;
    reinterpret_cast<double*>(cI)[tid] = ic < tj.n ? c[tj.vbase + ic] : 0.0;
  }
  __syncthreads();
  // a: row 4 rb + k over this block's four columns
  const double2 j01 = cJ[2 * cb], j23 = cJ[2 * cb + 1];
  double a[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    double v = static_cast<double>(m[k].x) * j01.x;
    v = fma(static_cast<double>(m[k].y), j01.y, v);
    v = fma(static_cast<double>(m[k].z), j23.x, v);
    a[k] = fma(static_cast<double>(m[k].w), j23.y, v);
  }
  // sum over the 16 column blocks (the lanes of one DPP row), scattered so
  // that lane cb ends with row 4 rb + (cb % 4): lane pairs (xor 1) keep rows of
  // their own parity, quad pairs (xor 2) one row each, then the four lanes of
  // a row add up by rotations of 4 and 8
  const bool b0 = (cb & 1) != 0, b1 = (cb & 2) != 0;
  double k0 = b0 ? a[1] : a[0], k1 = b0 ? a[3] : a[2];
  k0 += dpp_move<kDppXor1>(b0 ? a[0] : a[1]);
  k1 += dpp_move<kDppXor1>(b0 ? a[2] : a[3]);
  double r = (b1 ? k1 : k0) + dpp_move<kDppXor2>(b1 ? k0 : k1);
  r += dpp_move<kDppRor8>(r);
  r += dpp_move<kDppRor4>(r);
  double* out = f.xpart + static_cast<int64_t>(idx) * (2 * kFb);
  if (cb < 4) out[4 * rb + cb] = r;
  if (tj.I == tj.J) return;
  // b: column 4 cb + j over this block's four rows
  const double2 i01 = cI[2 * rb], i23 = cI[2 * rb + 1];
  double bv[4];
  {
    const float* m0 = reinterpret_cast<const float*>(&m[0]);
    const float* m1 = reinterpret_cast<const float*>(&m[1]);
    const float* m2 = reinterpret_cast<const float*>(&m[2]);
    const float* m3 = reinterpret_cast<const float*>(&m[3]);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      double v = static_cast<double>(m0[j]) * i01.x;
      v = fma(static_cast<double>(m1[j]), i01.y, v);
      v = fma(static_cast<double>(m2[j]), i23.x, v);
      bv[j] = fma(static_cast<double>(m3[j]), i23.y, v);
    }
  }
  // sum over the wave's four row blocks (lane bits 4 and 5), scattered so
  // that the lane ends with column 4 cb + lane / 16
  const bool g0 = (lane & 16) != 0, g1 = (lane & 32) != 0;
  double h0 = g0 ? bv[1] : bv[0], h1 = g0 ? bv[3] : bv[2];
  h0 += __shfl_xor(g0 ? bv[0] : bv[1], 16, 64);
  h1 += __shfl_xor(g0 ? bv[2] : bv[3], 16, 64);
  const double u = (g1 ? h1 : h0) + __shfl_xor(g1 ? h0 : h1, 32, 64);
  bpart[tid >> 6][4 * cb + (lane >> 4)] = u;
  __syncthreads();
  if (tid < kFb) out[kFb + tid] = (bpart[0][tid] + bpart[1][tid]) + (bpart[2][tid] + bpart[3][tid]);
}

// Table index of the tile that workgroup b of an x-update launch takes: the
// order reverses from one iteration to the next (by the parity of the first
// patient's iteration count, which only the previous launches write), so that
// an iteration starts on the tiles the last one read most recently, while
// they may still sit in the memory-side cache.  Every tile is taken once
// either way, and the results do not depend on the order.
__device__ __forceinline__ int xsym_order(const FactorArgs& f, int b) {
  return (f.ps[0].iter & 1) ? f.nxtiles - 1 - b : b;
}

template <bool kLoadsFirst>
__global__ __launch_bounds__(256) void k_xsym(FactorArgs f, const double* __restrict__ c) {
  xsym_tile<kLoadsFirst>(f, c, xsym_order(f, static_cast<int>(blockIdx.x)));
}

// The reduction of the x-update partials fused with the z-update (the dense
// x-update's iteration, both launch orders): one workgroup per 16 spots of a
// patient (a quarter of a column block, the z-update's job), one wave per
// scenario (waves w, w + 16, ... for more than 16).  For the wave's scenario
// its four 16-lane groups g add the partials of the tiles J = g, g + 4, ...
// of the spots' row block I (T_IJ c_J for J >= I, T_JI^T c_J below), each
// lane one spot, then across the groups by lane swaps: x_s of the 16 spots,
// rounded to fp32 as stored.  Then the z-update of k_zres on the same spots:
// z = P(mean_s(x_s + y_s / rho)) in a fixed order over the waves, d = x_s - z
// and the eight fp64 partial sums of the residuals and the dual step.
constexpr int kXzWaves = 16;
constexpr int kXzCols = 16;
__global__ __launch_bounds__(64 * kXzWaves) void k_xzres(FactorArgs f, VecArgs a) {
  __shared__ double sacc[kXzWaves][kXzCols];
  __shared__ float zsh[kXzCols];
  __shared__ double sred[kXzWaves][8];
  const int bi4 = static_cast<int>(blockIdx.x);
  const ZJob pt = a.zjobs[bi4 >> 2];
  const PatState* ps = a.ps + pt.patient;
  const int stopped = ps->stopped;  // read beside the loads below; checked before any write
  const double rho = ps->rho;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, g = lane >> 4, c = lane & 15;
  const int r = (bi4 & 3) * kXzCols + c;  // row within the block of 64 spots
  const int j = pt.col0 + r;
  const bool valid = j < pt.n;
  const int I = pt.col0 / kFb, nb = (pt.n + kFb - 1) / kFb;
  const int64_t ntile = static_cast<int64_t>(nb) * (nb + 1) / 2;
  const int64_t zi = pt.zvec_base + j;
  // the first scenario's vectors and the projection's inputs, requested first
  float y0 = 0.0f, lbv = 0.0f, ubv = 0.0f, zold = 0.0f;
  double dp0 = 0.0;
  if (valid && g == 0 && w < pt.N) {
    const int64_t vi = pt.vec_base + static_cast<int64_t>(w) * pt.n + j;
    y0 = a.y[vi];
    dp0 = a.dprev[vi];
  }
  if (valid && tid < kXzCols) {
    lbv = a.lb[zi];
    ubv = a.ub[zi];
    zold = a.z[zi];
  }
  // x_s of the wave's scenarios and their sum with y_s / rho
  float x0 = 0.0f;
  double zacc = 0.0;
  const int wu = __builtin_amdgcn_readfirstlane(w);  // the wave's index, as a scalar
  for (int s = wu; s < pt.N; s += kXzWaves) {
    // the scenario's partials (a scalar base) and 32-bit offsets per lane
    const double* xp = f.xpart + (pt.xtile0 + static_cast<int64_t>(s) * ntile) * (2 * kFb);
    // the group's tiles J = g + 4k, twelve loads in flight per lane, added in
    // the order of k
    double acc = 0.0;
    if (valid) {
      for (int J0 = g; J0 < nb; J0 += 48) {
        double q[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) {
          const int J = J0 + 4 * k;
          const int off = J < I ? static_cast<int>(tile_index(J, I, nb)) * (2 * kFb) + kFb + r
                                : static_cast<int>(tile_index(I, J, nb)) * (2 * kFb) + r;
          q[k] = J >= nb ? 0.0 : xp[off];
        }
#pragma unroll
        for (int k = 0; k < 12; ++k) acc += q[k];
      }
    }
    const double xs = swap_sum<32>(swap_sum<16>(acc));
    const float xf = static_cast<float>(xs);
    const int64_t vi = pt.vec_base + static_cast<int64_t>(s) * pt.n + j;
    if (g == 0 && valid) {
      const float yv = s == wu ? y0 : a.y[vi];
      if (!stopped) a.x[vi] = xf;
      zacc += static_cast<double>(xf);
      if (a.prm.z_mode == 0) zacc += static_cast<double>(yv) / rho;
    }
    if (s == wu) x0 = xf;
  }
  if (stopped) return;  // the whole workgroup: one patient
  if (g == 0) sacc[w][c] = zacc;
  __syncthreads();
  // ||dz||^2, ||z||^2, ||d||^2, <dd,d_prev>, ||dd||^2, ||x||^2, <y,d>, ||y||^2
  double v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  if (tid < kXzCols) {
    float znf = 0.0f;
    if (valid) {
      double sum = 0.0;
      for (int q = 0; q < kXzWaves; ++q) sum += sacc[q][c];
      double zn = sum / pt.N;
      zn = fmin(fmax(zn, static_cast<double>(lbv)), static_cast<double>(ubv));
      znf = static_cast<float>(zn);
      const double dz = static_cast<double>(znf) - static_cast<double>(zold);
      a.z[zi] = znf;
      v[0] = dz * dz;
      v[1] = static_cast<double>(znf) * znf;
    }
    zsh[c] = znf;
  }
  __syncthreads();
  if (valid && g == 0) {
    const double znd = static_cast<double>(zsh[c]);
    for (int s = w; s < pt.N; s += kXzWaves) {
      const int64_t vi = pt.vec_base + static_cast<int64_t>(s) * pt.n + j;
      const double xv = static_cast<double>(s == w ? x0 : a.x[vi]);
      const double yv = static_cast<double>(s == w ? y0 : a.y[vi]);
      const double d = xv - znd;
      const double dp = s == w ? dp0 : a.dprev[vi];
      const double dd = d - dp;
      v[2] += d * d;
      v[3] += dd * dp;
      v[4] += dd * dd;
      v[5] += xv * xv;
      v[6] += yv * d;
      v[7] += yv * yv;
      a.dprev[vi] = d;
    }
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) v[k] = group_allsum<64>(v[k]);
  if (lane == 0)
    for (int k = 0; k < 8; ++k) sred[w][k] = v[k];
  __syncthreads();
  if (tid < 8) {
    auto q4 = [&](int b) { return (sred[b][tid] + sred[b + 1][tid]) + (sred[b + 2][tid] + sred[b + 3][tid]); };
    a.bpartp[static_cast<int64_t>(bi4) * 8 + tid] = (q4(0) + q4(4)) + (q4(8) + q4(12));
  }
}

// The dual update y_s += tau d_s at one spot (when `update`) and the
// right-hand side c_s = b_s + rho/2 z - y_s/2 of the next x-update there, with
// the roundings written out, so that every launch order that applies them
// gives the same bits.  Returns y_s at the spot.
__device__ __forceinline__ float dual_rhs_at(const VecArgs& a, int64_t vi, bool update, float yv, double dp,
                                             double bv, float zj, double tau, double rho) {
  if (update) {
    yv = static_cast<float>(fma(tau, dp, static_cast<double>(yv)));
    a.y[vi] = yv;
  }
  a.c64[vi] = fma(-0.5, static_cast<double>(yv), fma(0.5 * rho, static_cast<double>(zj), bv));
  return yv;
}

// completion of the pending dual update and the right-hand side
// c_s = b_s + rho/2 z - y_s/2 (one scenario column block of 64 per workgroup)
// one wave: column block bi of one scenario, lane = column within the block
__device__ __forceinline__ void fhead_block(const VecArgs& a, int bi, int lane) {
  const Blk bk = a.blk[bi];
  const Scen sc = a.scen[bk.owner];
  const int j = bk.col0 + lane;
  const bool in = j < sc.n;
  const int64_t vi = sc.vec_base + j;
  // the scenario's vectors are requested beside the patient's entries
  float yv = 0.0f;
  double dp = 0.0, bv = 0.0;
  if (in) {
    yv = a.y[vi];
    dp = a.dprev[vi];
    bv = a.b64[vi];
  }
  const Pat pt = a.pat[sc.patient];
  const PatState* ps = a.ps + sc.patient;
  const float zj = in ? a.z[pt.zvec_base + j] : 0.0f;
  if (ps->stopped) return;
  double yy = 0.0;
  if (in) {
    yv = dual_rhs_at(a, vi, ps->pending != 0, yv, dp, bv, zj, ps->tau, ps->rho);
    yy = static_cast<double>(yv) * yv;
  }
  yy = wave_sum_d(yy);
  if (lane == 0) {
    double* bp = a.bpart + static_cast<int64_t>(bi) * 8;
    bp[0] = 0.0;
    bp[1] = 0.0;
    bp[2] = yy;
  }
}

// The objective tiles read sum_s G_s rounded to 48 bits (sign, exponent and
// the leading 36 of the 52 fraction bits, to nearest): 24 KB a tile instead of
// 32 KB, relative error at most 2^-37 per entry.  Thread t of fobj_tile takes
// the 16 entries e = 0..15 at (row 8 (e / 2) + t / 32, column 2 (t % 32) +
// e % 2) of the tile; their upper 32 bits are four 16-byte words at
// 256 k + t (k = 0..3, entries 4k .. 4k + 3) of the tile's first 16 KB, their
// next 16 bits two 16-byte words at 256 k + t (k = 0..1, entries 8k .. 8k + 7)
// of its last 8 KB, so every wave load reads 1 KiB contiguous.
constexpr int kGqWords = 6144;  // 32-bit words of one tile
__global__ __launch_bounds__(256) void k_gq_pack(const double* __restrict__ Gp, uint32_t* __restrict__ Gq,
                                                 int64_t n) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t idx = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; idx < n; idx += stride) {
    const int64_t tile = idx >> 12;
    const int L = static_cast<int>(idx & 4095);  // row-major within the tile: 512 (e / 2) + 2 t + e % 2
    const int t = (L & 511) >> 1, e = 2 * (L >> 9) + (L & 1);
    const unsigned long long r = static_cast<unsigned long long>(__double_as_longlong(Gp[idx])) + 0x8000ull;
    uint32_t* q = Gq + tile * kGqWords;
    q[((e >> 2) * 256 + t) * 4 + (e & 3)] = static_cast<uint32_t>(r >> 32);
    reinterpret_cast<uint16_t*>(q + 4096)[((e >> 3) * 256 + t) * 8 + (e & 7)] =
        static_cast<uint16_t>((r >> 16) & 0xffffu);
  }
}

__device__ __forceinline__ uint32_t word_of(const uint4& v, int i) {
  return i == 0 ? v.x : (i == 1 ? v.y : (i == 2 ? v.z : v.w));
}

// objective partial of one packed tile T of sum_s G_s: z_I^T T z_J, doubled off
// the diagonal; a diagonal tile also carries -g0_I^T z_I.  fp64 arithmetic on
// the 48-bit entries above.  The tile's 24 KB are requested first, from its
// list index alone.
__device__ __forceinline__ void fobj_tile(const FactorArgs& f, const float* __restrict__ z, int jb) {
  __shared__ double zI[kFb], zJ[kFb], red[4];
  const int tid = threadIdx.x;
  const uint4* Q = reinterpret_cast<const uint4*>(f.Gq + static_cast<int64_t>(jb) * kGqWords);
  uint4 hi[4], lo[2];
#pragma unroll
  for (int k = 0; k < 4; ++k) hi[k] = Q[k * 256 + tid];
#pragma unroll
  for (int k = 0; k < 2; ++k) lo[k] = Q[1024 + k * 256 + tid];
  const XJob job = f.fjobs[jb];
  if (f.ps[job.g].stopped) return;
  const Pat pt = f.pat[job.g];
  const int I = job.ij >> 16, J = job.ij & 0xffff;
  if (tid < kFb) {
    const int jc = J * kFb + tid, ic = I * kFb + tid;
    zJ[tid] = jc < pt.n ? static_cast<double>(z[pt.zvec_base + jc]) : 0.0;
    zI[tid] = ic < pt.n ? static_cast<double>(z[pt.zvec_base + ic]) : 0.0;
  }
  __syncthreads();
  auto entry = [&](int e) {
    const uint32_t h = word_of(hi[e >> 2], e & 3);
    const uint32_t l2 = word_of(lo[e >> 3], (e & 7) >> 1);
    const uint32_t l = (e & 1) ? (l2 >> 16) : (l2 & 0xffffu);
    return __longlong_as_double(static_cast<long long>((static_cast<unsigned long long>(h) << 32) |
                                                       (static_cast<unsigned long long>(l) << 16)));
  };
  const int c = 2 * (tid & 31), r0 = tid >> 5;
  double a = 0.0;
#pragma unroll
  for (int k = 0; k < 8; ++k) a = fma(zI[8 * k + r0], fma(entry(2 * k), zJ[c], entry(2 * k + 1) * zJ[c + 1]), a);
  double v = (I == J ? 1.0 : 2.0) * a;
  if (I == J && tid < kFb) {
    const int row = I * kFb + tid;
    if (row < pt.n) v -= f.g0[pt.zvec_base + row] * zI[tid];
  }
  v = wave_sum_d(v);
  if ((tid & 63) == 0) red[tid >> 6] = v;
  __syncthreads();
  if (tid == 0) f.fpart[jb] = (red[0] + red[1]) + (red[2] + red[3]);
}

// The four-launch dense iteration ends with two launches that each pair one
// scalar workgroup per patient (the first workgroups) with independent wide work:
//   tail: the residual norms, tolerances and BB step (body_scalars_run), the
//         other workgroups the objective tiles at the new z;
//   head: the objective sums and stopping tests
//         (head_scalars_run), the others the dual update y_s += tau d_s and
//         the right-hand sides c_s of the next x-update, gated by dual_go,
//         which the tail set (the stopping test of the same launch does not
//         gate them: as in the six-launch order, the dual update of an
//         iteration precedes its stopping test).
__device__ __forceinline__ void dense_head_block(const VecArgs& a, int bi, int lane) {
  const Blk bk = a.blk[bi];
  const Scen sc = a.scen[bk.owner];
  const int j = bk.col0 + lane;
  const bool in = j < sc.n;
  const int64_t vi = sc.vec_base + j;
  float yv = 0.0f;
  double dp = 0.0, bv = 0.0;
  if (in) {
    yv = a.y[vi];
    dp = a.dprev[vi];
    bv = a.b64[vi];
  }
  const Pat pt = a.pat[sc.patient];
  const PatState* ps = a.ps + sc.patient;
  const float zj = in ? a.z[pt.zvec_base + j] : 0.0f;
  if (!ps->dual_go) return;
  if (in) (void)dual_rhs_at(a, vi, true, yv, dp, bv, zj, ps->tau, ps->rho);
}

// The same update in the launch that forms tau: every wave forms its
// patient's tau itself, from the z-update's partial sums in the order of
// wave_strided_sums and the inputs the last head recorded, which gives the
// bits the scalar workgroup of that launch (body_scalars_run) stores.
__device__ __forceinline__ void dense_dual_block(const VecArgs& a, int bi, int lane) {
  const Blk bk = a.blk[bi];
  const Scen sc = a.scen[bk.owner];
  const int j = bk.col0 + lane;
  const bool in = j < sc.n;
  const int64_t vi = sc.vec_base + j;
  float yv = 0.0f;
  double dp = 0.0, bv = 0.0;
  if (in) {
    yv = a.y[vi];
    dp = a.dprev[vi];
    bv = a.b64[vi];
  }
  const Pat pt = a.pat[sc.patient];
  const PatState* ps = a.ps + sc.patient;
  const float zj = in ? a.z[pt.zvec_base + j] : 0.0f;
  const int stopped = ps->stopped;
  const double rho = ps->rho, tau0 = ps->bb_tau0;
  const int it0 = ps->bb_iter0;
  double v[2];
  wave_strided_sums<2>(a.bpartp + static_cast<int64_t>(4 * pt.blk_begin) * 8, 4 * pt.nblk, 3, v);
  if (stopped) return;
  const double tau = bb_dual_step(a.prm, rho, tau0, it0, v[0], v[1]);
  if (in) (void)dual_rhs_at(a, vi, true, yv, dp, bv, zj, tau, rho);
}

__global__ __launch_bounds__(256) void k_dense_tail(FactorArgs f, VecArgs a, int nfobj) {
  const int b = static_cast<int>(blockIdx.x) - f.npat;
  if (b < 0) {
    body_scalars_run<true>(a, static_cast<int>(blockIdx.x));
    return;
  }
  if (b < nfobj) fobj_tile(f, a.z, b);
}

__global__ __launch_bounds__(256) void k_dense_head(VecArgs a, int nblk) {
  const int b = static_cast<int>(blockIdx.x) - a.prm.num_pat;
  if (b < 0) {
    head_scalars_run<true>(a, static_cast<int>(blockIdx.x), 0);
    return;
  }
  const int bi = 4 * b + static_cast<int>(threadIdx.x >> 6);
  if (bi < nblk) dense_head_block(a, bi, threadIdx.x & 63);
}

// The three-launch dense iteration (the reduction and the z-update between them):
//   x:    one workgroup per patient the objective sum and stopping test of the
//         previous iteration (head_scalars_run), the others the x-update tiles.
//         The tiles read the stop flag that it may be setting: a tile of
//         a patient that stops there writes partial sums that nothing reads
//         (the reduction and the z-update read the flag after the launch),
//         and none writes the iteration count that orders the tiles;
//   tail: one workgroup per patient the residual norms, tolerances and dual
//         step (body_scalars_run), then the dual update with the next right-hand
//         sides (each wave forms tau itself, dense_dual_block), then the
//         objective tiles at the new z.
// Every value equals the four-launch order's; the stopping test of the last
// iteration of a run follows in a launch of its own.
template <bool kLoadsFirst>
__global__ __launch_bounds__(256) void k_dense_x(FactorArgs f, VecArgs a, const double* __restrict__ c) {
  const int b = static_cast<int>(blockIdx.x) - f.npat;
  if (b < 0) {
    head_scalars_run<true>(a, static_cast<int>(blockIdx.x), 0);
    return;
  }
  xsym_tile<kLoadsFirst>(f, c, xsym_order(f, b));
}

__global__ __launch_bounds__(256) void k_dense_tail_dual(FactorArgs f, VecArgs a, int nfobj, int nblk) {
  const int b = static_cast<int>(blockIdx.x) - f.npat;
  if (b < 0) {
    body_scalars_run<true>(a, static_cast<int>(blockIdx.x));
    return;
  }
  const int ndual = (nblk + 3) / 4;
  if (b < ndual) {
    const int bi = 4 * b + static_cast<int>(threadIdx.x >> 6);
    if (bi < nblk) dense_dual_block(a, bi, threadIdx.x & 63);
    return;
  }
  if (b - ndual < nfobj) fobj_tile(f, a.z, b - ndual);
}

// The head of a dense iteration in one launch: workgroups [0, nfobj) take the
// objective tiles, the rest four column blocks each of the pending dual update
// and right-hand sides (the two parts are independent).
__global__ __launch_bounds__(256) void k_fheadobj(FactorArgs f, VecArgs a, int nfobj, int nblk) {
  const int b = static_cast<int>(blockIdx.x);
  if (b < nfobj) {
    fobj_tile(f, a.z, b);
    return;
  }
  const int bi = 4 * (b - nfobj) + static_cast<int>(threadIdx.x >> 6);
  if (bi < nblk) fhead_block(a, bi, threadIdx.x & 63);
}

}  // namespace

void launch_gram(const MatDev& m, const double* rw64, const Scen& sc, double* G, int ld, hipStream_t st) {
  if (sc.rows <= 0) return;
  const unsigned nb = static_cast<unsigned>((sc.rows + 3) / 4);
  if (m.col16)
    hipLaunchKernelGGL(k_gram<true>, dim3(nb), dim3(256), 0, st, m, rw64, sc, G, ld);
  else
    hipLaunchKernelGGL(k_gram<false>, dim3(nb), dim3(256), 0, st, m, rw64, sc, G, ld);
}

void launch_gram_lists(const MatDev& m, const Scen* scen, int g0, int nscen, int nb, int ms, int32_t* row_of,
                       int nchunk, uint32_t* cnt, int32_t* tot, int64_t* off, hipStream_t st) {
  const int nt = nb * (nb + 1) / 2;
  launch_fill_f32(reinterpret_cast<float*>(row_of), __builtin_bit_cast(float, -1), static_cast<int64_t>(ms) * nscen, st);
  hipLaunchKernelGGL(k_gram_order, dim3(64, nscen), dim3(256), 0, st, m, scen, g0, ms, row_of);
  hipLaunchKernelGGL(k_gram_rows<false>, dim3(nchunk, nscen), dim3(64), 4 * nt, st, m, scen, g0, nb, row_of, ms, nchunk,
                     cnt, static_cast<const int64_t*>(nullptr), static_cast<GramEntry*>(nullptr));
  hipLaunchKernelGGL(k_gram_prefix, dim3((nt + 63) / 64, nscen), dim3(64 * kPrefixWaves), 0, st, cnt, nt, nchunk, tot);
  hipLaunchKernelGGL(k_gram_scan, dim3(1), dim3(1024), 0, st, tot, static_cast<int64_t>(nt) * nscen, off);
}

void launch_gram_tiles(const MatDev& m, const double* rw64, const Scen* scen, int g0, int nscen, int nb, int ms,
                       const int32_t* row_of, int nchunk, uint32_t* cnt, const int64_t* off, GramEntry* list,
                       const double* gbig, double* G, int ld, hipStream_t st) {
  const int nt = nb * (nb + 1) / 2;
  hipLaunchKernelGGL(k_gram_rows<true>, dim3(nchunk, nscen), dim3(64), 4 * nt, st, m, scen, g0, nb, row_of, ms, nchunk,
                     cnt, off, list);
  hipLaunchKernelGGL(k_gram_tiles, dim3(nt, nscen), dim3(64 * kGramWaves), 0, st, m, rw64, scen, g0, nb, off, list,
                     gbig, G, ld);
}

void launch_gram_finish(FactorArgs f, int patient, int scen_begin, int nscen, int npad, int n, double rho,
                        int accumulate_gsum, hipStream_t st) {
  int64_t nb = (static_cast<int64_t>(npad) * npad + 255) / 256;
  if (nb > 8192) nb = 8192;
  hipLaunchKernelGGL(k_gram_finish, dim3(static_cast<unsigned>(nb)), dim3(256), 0, st, f, patient, scen_begin,
                     nscen, npad, n, rho, accumulate_gsum);
}

void launch_sweep(FactorArgs f, int patient, int scen_begin, int nscen, int npad, hipStream_t st) {
  const int n64 = npad / 64, nt = n64 * (n64 + 1) / 2;
  // The next pivot block goes beside the update where the update takes longer
  // than the pivot's chain within it (85 to 105 us, against 32 in a launch of its
  // own): per step, update and pivot 64 + 31 against 103 us with 2 730 tiles over
  // the scenarios, 104 + 31 against 127 us with 4 914, 147 + 32 against 157 us
  // with 6 864.  A whole new penalty from 4 096 tiles on, apart against beside, over
  // other numbers of scenarios: 715 against 700 us at 192 spots x 700, 1 175 against
  // 1 095 at 707 x 63, 1 390 against 1 290 at 1 000 x 31, 3 410 against 3 000 at
  // 2 003 x 13, 3 340 against 3 230 at 2 981 x 4, 6 180 against 6 060 at 5 762 x 1.
  const bool beside = static_cast<int64_t>(nt) * nscen >= 4096;
  auto step = [&](auto kbc, auto kbn, auto last, int k0) {
    constexpr int KB = decltype(kbc)::value, KBN = decltype(kbn)::value;
    if (k0 == 0 || !beside) hipLaunchKernelGGL(k_sweep_pivot<KB>, dim3(nscen), dim3(512), 0, st, f, npad, k0);
    hipLaunchKernelGGL(k_sweep_panel<KB>, dim3(n64, nscen), dim3(256), 0, st, f, npad, k0);
    hipLaunchKernelGGL((k_sweep_update<KB, KBN, decltype(last)::value>), dim3((nt + (KBN != 0 ? 1 : 0)) * nscen), dim3(256),
                       0, st, f, npad, k0, nscen, patient, scen_begin);
  };
  constexpr std::integral_constant<int, kKb> full{};
  constexpr std::integral_constant<int, 64> half{};
  constexpr std::integral_constant<int, 0> none{};
  for (int k0 = 0; k0 < npad; k0 += kKb) {
    const int left = npad - k0;
    if (left >= 2 * kKb && beside)
      step(full, full, std::false_type{}, k0);
    else if (left > kKb && beside)
      step(full, half, std::false_type{}, k0);
    else if (left > kKb)
      step(full, none, std::false_type{}, k0);
    else if (left == kKb)
      step(full, none, std::true_type{}, k0);
    else
      step(half, none, std::true_type{}, k0);
  }
}

void launch_gq_pack(const double* Gp, uint32_t* Gq, int64_t ntiles, hipStream_t st) {
  if (ntiles <= 0) return;
  const int64_t n = ntiles * 4096;
  const unsigned grid = static_cast<unsigned>(std::min<int64_t>((n + 255) / 256, 65536));
  hipLaunchKernelGGL(k_gq_pack, dim3(grid), dim3(256), 0, st, Gp, Gq, n);
}

void launch_xsym(const FactorArgs& f, const double* c, int njobs, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
  if (njobs <= 0) return;
  const int grid = njobs;
  auto kern = f.npat == 1 ? k_xsym<true> : k_xsym<false>;
  if (e0 != nullptr)
    hipExtLaunchKernelGGL(kern, dim3(grid), dim3(256), 0, st, e0, e1, 0, f, c);
  else
    hipLaunchKernelGGL(kern, dim3(grid), dim3(256), 0, st, f, c);
}

void launch_xzres(const FactorArgs& f, const VecArgs& a, int npblk, hipStream_t st) {
  if (npblk <= 0) return;
  hipLaunchKernelGGL(k_xzres, dim3(static_cast<unsigned>(4 * npblk)), dim3(64 * kXzWaves), 0, st, f, a);
}

void launch_dense_tail(const FactorArgs& f, const VecArgs& a, int nfobj, hipStream_t st) {
  hipLaunchKernelGGL(k_dense_tail, dim3(f.npat + nfobj), dim3(256), 0, st, f, a, nfobj);
}

void launch_dense_head(const VecArgs& a, int nblk, hipStream_t st) {
  hipLaunchKernelGGL(k_dense_head, dim3(a.prm.num_pat + (nblk + 3) / 4), dim3(256), 0, st, a, nblk);
}

void launch_dense_x(const FactorArgs& f, const VecArgs& a, const double* c, int njobs, hipStream_t st, hipEvent_t e0,
                    hipEvent_t e1) {
  const dim3 grid(static_cast<unsigned>(f.npat + njobs));
  auto kern = f.npat == 1 ? k_dense_x<true> : k_dense_x<false>;
  if (e0 != nullptr)
    hipExtLaunchKernelGGL(kern, grid, dim3(256), 0, st, e0, e1, 0, f, a, c);
  else
    hipLaunchKernelGGL(kern, grid, dim3(256), 0, st, f, a, c);
}

void launch_dense_tail_dual(const FactorArgs& f, const VecArgs& a, int nfobj, int nblk, hipStream_t st) {
  const int grid = f.npat + (nblk + 3) / 4 + nfobj;
  hipLaunchKernelGGL(k_dense_tail_dual, dim3(static_cast<unsigned>(grid)), dim3(256), 0, st, f, a, nfobj, nblk);
}

void launch_fheadobj(const FactorArgs& f, const VecArgs& a, int nfobj, int nblk, hipStream_t st) {
  const int grid = nfobj + (nblk + 3) / 4;
  if (grid <= 0) return;
  hipLaunchKernelGGL(k_fheadobj, dim3(grid), dim3(256), 0, st, f, a, nfobj, nblk);
}

}  // namespace admmbb
