// Element-wise and reduction kernels of the residual, the energy and the Jacobi/DIIS update.
//
// Reductions are deterministic: a fixed grid, a fixed per-thread stride pattern, a fixed
// wave64 shuffle tree and a fixed second stage, with no floating-point atomics, so the same
// inputs always give bitwise the same energy, norms and DIIS coefficients.
#include <algorithm>
#include <cmath>

#include <type_traits>

#include "internal.h"
#include "lowp.h"

namespace ascc {
namespace {

constexpr int kThreads = 256;
constexpr int kRedBlocks = 1024;  // first-stage blocks of a reduction at most

struct P4 {
  double* out;
  long os[4];
  int d[4];
  double c0;
  int nin;
  const double* in[4];
  long s[4][4];
  double coef[4];
};

__global__ __launch_bounds__(kThreads) void permute4_kernel(P4 p, long total) {
  for (long idx = blockIdx.x * (long)blockDim.x + threadIdx.x; idx < total; idx += (long)gridDim.x * blockDim.x) {
    long r = idx;
    const int i3 = r % p.d[3];
    r /= p.d[3];
    const int i2 = r % p.d[2];
    r /= p.d[2];
    const int i1 = r % p.d[1];
    const int i0 = r / p.d[1];
    double* o = p.out + i0 * p.os[0] + i1 * p.os[1] + i2 * p.os[2] + i3 * p.os[3];
    double v = (p.c0 == 0.0) ? 0.0 : p.c0 * *o;
#pragma unroll
    for (int t = 0; t < 4; ++t)
      if (t < p.nin) v += p.coef[t] * p.in[t][i0 * p.s[t][0] + i1 * p.s[t][1] + i2 * p.s[t][2] + i3 * p.s[t][3]];
    *o = v;
  }
}

// Same operation when the output is contiguous along i3 and some inputs are contiguous along
// another index t instead (a transposition): 32 x 32 tiles over (i_t, i3) for fixed (i_u, i_w);
// the transposed inputs (bit q of tmask) are summed into an LDS tile with reads along i_t, the
// others are read along i3 with the output row, so reads and writes are coalesced.
__global__ __launch_bounds__(kThreads) void permute4_tiled_kernel(P4 p, int t, int u, int w, int tiles3, int tmask) {
  __shared__ double tile[32][33];
  const int it0 = (blockIdx.x / tiles3) * 32, i30 = (blockIdx.x % tiles3) * 32;
  const long iu = blockIdx.y, iw = blockIdx.z;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
  const int dt = p.d[t], d3 = p.d[3];
#pragma unroll
  for (int k = 0; k < 4; ++k) {  // tile[i3 - i30][it - it0], reads along it
    const long i3 = i30 + ty + 8 * k, it = it0 + tx;
    double acc = 0.0;
    if (i3 < d3 && it < dt)
      for (int q = 0; q < p.nin; ++q)
        if ((tmask >> q) & 1)
          acc += p.coef[q] * p.in[q][iu * p.s[q][u] + iw * p.s[q][w] + it * p.s[q][t] + i3 * p.s[q][3]];
    tile[ty + 8 * k][tx] = acc;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 4; ++k) {  // output along i3
    const long it = it0 + ty + 8 * k, i3 = i30 + tx;
    if (it < dt && i3 < d3) {
      double* o = p.out + iu * p.os[u] + iw * p.os[w] + it * p.os[t] + i3 * p.os[3];
      double v = (p.c0 == 0.0) ? 0.0 : p.c0 * *o;
      for (int q = 0; q < p.nin; ++q)
        if (!((tmask >> q) & 1)) v += p.coef[q] * p.in[q][iu * p.s[q][u] + iw * p.s[q][w] + it * p.s[q][t] + i3 * p.s[q][3]];
      *o = v + tile[tx][ty + 8 * k];
    }
  }
}

// Doubles residual, element (i,j,a,b) of the [o][o][v][v] output:
//   R = 1/2 (G1[iajb] + G1[jbia]) + 1/2 (RL[ijab] + RL[jiba]) + EM[ijab] + EM[jiba]
//       - 1/2 (P1[jbia] + P1[iajb]) + 1/2 (P2[jbia] + P2[iajb]) - (P1[ibja] + P1[jaib])
// (ovov arrays are [o][v][o][v]).  G1 and RL are pair-symmetric in exact arithmetic; taking their
// symmetric parts makes R[ijab] = R[jiba] whatever the rounding of the products behind them (a
// low-precision ladder is not), so amplitudes that start pair-symmetric stay so.  The part of t2
// odd under the joint (ij)(ab) swap is outside the closed-shell equations and barely damped by
// the Jacobi step; fed by rounding, it stalls the DIIS iteration of excited (ASCC) states.
// R2[ij][ab] = X(i,j,a,b) + X(j,i,b,a) with
//   X(i,j,a,b) = EM[ijab] + (RL[ijab] + G1[iajb]) / 2 - P1[iajb] / 2 + P2[iajb] / 2 - P1[jaib].
// One workgroup per pair i <= j and 32 x 32 blocks (A, B) of (a, b): it forms X(i,j) on A x B with
// reads along b and X(j,i) on B x A with reads along a (every term is contiguous in the index read
// along), keeps both tiles in LDS and writes R2[ij] on A x B and R2[ji] on B x A, so each input
// element is read once.  For i = j only A <= B runs; with A = B both tiles are the same block and
// the two writes of an element carry the same value.
__device__ __forceinline__ double assemble_x(const double* __restrict__ g1, const double* __restrict__ em,
                                             const double* __restrict__ p1, const double* __restrict__ p2, double rl,
                                             long x, long iajb, long jaib) {
  return 0.5 * (g1[iajb] + rl) + em[x] - 0.5 * p1[iajb] + 0.5 * p2[iajb] - p1[jaib];
}

// Pair index of i <= j among n: pidx(i, j) = i*n - i*(i-1)/2 + (j - i)  (row-major upper triangle).
__device__ __forceinline__ long pidx(long i, long j, long n) { return i * n - i * (i - 1) / 2 + (j - i); }

// PAIRS: the ladders come as pair rows R+-[p(i,j)][p(a,b)] (rows at stride ldr; RL_ij^ab = R+ + R- for
// a <= b, R+ - R- for a > b) instead of RL[i][j][a][b]: each block reads its 32 x 32 pair elements once,
// along the row, and the transposed block takes them through LDS, so no pass unpacks them.
template <bool PAIRS>
__global__ __launch_bounds__(kThreads) void assemble_r2_kernel(double* __restrict__ r2, const double* __restrict__ g1,
                                                              const double* __restrict__ rl,
                                                              const double* __restrict__ rminus, long ldr,
                                                              const double* __restrict__ em,
                                                              const double* __restrict__ p1,
                                                              const double* __restrict__ p2, int o, int v) {
  __shared__ double t1[32][33], t2[32][33];  // t1[a - a0][b - b0] = X(i,j,a,b), t2[b - b0][a - a0] = X(j,i,b,a)
  __shared__ double up[PAIRS ? 32 : 1][33], um[PAIRS ? 32 : 1][33];  // R+ + R-, R+ - R- of the block's pairs
  const int tv = (v + 31) / 32;
  const int ta = blockIdx.y / tv, tb = blockIdx.y % tv;
  // pair p = j (j + 1) / 2 + i, i <= j
  const long p = blockIdx.x;
  int j = (int)((sqrt(8.0 * (double)p + 1.0) - 1.0) * 0.5);
  while ((long)j * (j + 1) / 2 > p) --j;
  while ((long)(j + 1) * (j + 2) / 2 <= p) ++j;
  const int i = (int)(p - (long)j * (j + 1) / 2);
  if (i == j && ta > tb) return;
  const int a0 = ta * 32, b0 = tb * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
  auto ov = [&](int q, int x, int r, int y) -> long { return ((long)(q * v + x) * o + r) * v + y; };
  const long ij = ((long)i * o + j) * v * v, ji = ((long)j * o + i) * v * v;
  if constexpr (PAIRS) {
    const long row = pidx(i, j, o) * ldr;
    const int c0 = min(a0, b0), d0 = max(a0, b0);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int r = ty + 8 * k, c = c0 + r, d = d0 + tx;
      if (c <= d && d < v) {
        const long q = row + pidx(c, d, v);
        const double x = rl[q], y = rminus[q];
        up[r][tx] = x + y;
        um[r][tx] = x - y;
      }
    }
    __syncthreads();
  }
  // RL_ij^ab of a = a0 + x, b = b0 + y
  auto ladder = [&](int x, int y, long idx) -> double {
    if constexpr (PAIRS) {
      if (a0 < b0 || (a0 == b0 && x <= y)) return up[x][y];
      return um[y][x];
    } else {
      return rl[idx];
    }
  };
  double x1[4], x2[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int r = ty + 8 * k;
    {  // X(i,j,a,b), a = a0 + r, b = b0 + tx: along b
      const int a = a0 + r, b = b0 + tx;
      const long x = ij + (long)a * v + b;
      x1[k] = (a < v && b < v) ? assemble_x(g1, em, p1, p2, ladder(r, tx, x), x, ov(i, a, j, b), ov(j, a, i, b)) : 0.0;
      t1[r][tx] = x1[k];
    }
    {  // X(j,i,b,a), b = b0 + r, a = a0 + tx: along a
      const int b = b0 + r, a = a0 + tx;
      const long x = ji + (long)b * v + a;
      x2[k] = (a < v && b < v) ? assemble_x(g1, em, p1, p2, ladder(tx, r, x), x, ov(j, b, i, a), ov(i, b, j, a)) : 0.0;
      t2[r][tx] = x2[k];
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int r = ty + 8 * k;
    {  // R2[ij][a][b] = X(i,j,a,b) + X(j,i,b,a)
      const int a = a0 + r, b = b0 + tx;
      if (a < v && b < v) r2[ij + (long)a * v + b] = x1[k] + t2[tx][r];
    }
    {  // R2[ji][b][a] = X(j,i,b,a) + X(i,j,a,b)
      const int b = b0 + r, a = a0 + tx;
      if (a < v && b < v) r2[ji + (long)b * v + a] = x2[k] + t1[tx][r];
    }
  }
}

// ---------------------------------------------------------------------------------------
// T1 dressing B^ = X B Y^T with X = 1 - t1 (virtual-occupied block) and Y^T = 1 + t1 (virtual-occupied), every
// array with the fitting index Q last (rows of ldq values, zero past naux), so that the dressed blocks are
// written in the layout that the contractions over Q read, in two passes over B (o20 v180 Q600, with the Fock
// matrix: 0.53 ms as products, block copies and traces of [Q][p][q] arrays, 0.2 ms so).
//
// Both sides are products with the fitting index as their columns, on v_mfma_f64_16x16x4 (lane l supplies A(l%16, l/16) and
// B(l/16, l%16) and holds rows l/16 + 4r of column l%16): fragments of B come straight from its rows (four pieces of
// 128 bytes a load), and no value has to reach all lanes (with t1 broadcast from LDS the reads of it took four times as
// long as the products).  Bound by the reads of B.
//
// Right side: D[k][p] = B[p][k] + sum_c B[p][o + c] t1[k][c], all p, k < o.  A workgroup holds 64 Q of one p and
// 16 MT values of k; its four waves share the columns c and their sums are added through LDS.  One Q column a
// thread and its chain over c took o8 v72 27, o13 v117 80, o20 v180 82 us, now 7, 17 and 69 (2.8 TB/s).
typedef double dress_d4 __attribute__((ext_vector_type(4)));
template <int MT>
__global__ __launch_bounds__(kThreads) void dress_right_kernel(double* __restrict__ D, const double* __restrict__ B,
                                                              const double* __restrict__ t1, int o, int v, long ldq) {
  __shared__ dress_d4 sh[2][MT * 4][64];  // two waves' sums
  const int n = o + v, p = blockIdx.y, k0 = blockIdx.z * 16 * MT, lane = threadIdx.x & 63, l16 = lane & 15, lq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const double* Bp = B + (long)p * n * ldq;
  // this lane's columns j of the four tiles: q + j, four values side by side (rows are a multiple of 16 long; columns past the
  // row's end repeat its first ones and are not stored)
  const long q0 = blockIdx.x * 64L + 4 * l16, q = q0 < ldq ? q0 : 0;
  dress_d4 acc[MT][4];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[m][j] = dress_d4{0.0, 0.0, 0.0, 0.0};
  constexpr int UN = 2;  // groups of four c in flight
  const int ng = (v + 3) / 4;
  for (int g = wave; g < ng; g += 4 * UN) {
    double a[UN][MT];
    dress_d4 x[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int c = 4 * (g + 4 * u) + lq, cc = min(c, v - 1);
      const dress_d4 y = *reinterpret_cast<const dress_d4*>(Bp + (o + cc) * ldq + q);
      x[u] = c < v ? y : dress_d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        const int k = k0 + 16 * m + l16;
        const double y = t1[(long)min(k, o - 1) * v + cc];
        a[u][m] = c < v ? y : 0.0;
      }
    }
#pragma unroll
    for (int u = 0; u < UN; ++u)
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[m][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u][m], x[u][j], acc[m][j], 0, 0, 0);
  }
  // (wave 0 + wave 2) + (wave 1 + wave 3)
#pragma unroll
  for (int half = 2; half > 0; half >>= 1) {
    if (half == 1) __syncthreads();
    if (wave >= half && wave < 2 * half) {
#pragma unroll
      for (int y = 0; y < 4 * MT; ++y) sh[wave - half][y][lane] = acc[y / 4][y % 4];
    }
    __syncthreads();
    if (wave < half) {
#pragma unroll
      for (int y = 0; y < 4 * MT; ++y) acc[y / 4][y % 4] += sh[wave][y][lane];
    }
  }
  if (wave != 0 || q0 >= ldq) return;
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int k = k0 + 16 * m + lq + 4 * r;
      if (k >= o) continue;
      const dress_d4 y = *reinterpret_cast<const dress_d4*>(Bp + k * ldq + q);
      *reinterpret_cast<dress_d4*>(D + ((long)k * n + p) * ldq + q) =
          y + dress_d4{acc[m][0][r], acc[m][1][r], acc[m][2][r], acc[m][3][r]};
    }
}

// Wave sum over the 64 lanes, every lane gets it (a fixed order).
__device__ __forceinline__ double wave_all(double x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
  return x;
}
__device__ __forceinline__ double wave_max(double x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x = fmax(x, __shfl_xor(x, off, 64));
  return x;
}

// Left side: out[a][x] = in[a][x] - sum_k t1[k][a] w[k][x] for the columns x
//   x = c < v:       bvv[a][c] = B[o+a][o+c] - sum_k t1[k][a] B[k][o+c]
//   x = v + i:       bvo[i][a] = D[i][o+a]   - sum_k t1[k][a] D[i][k],  and boo[k][i] = D[i][k]
// and the Coulomb part of the Fock matrix, f[p][q] = h[p][q] + 2 sum_Q J_Q B[p][q], J_Q = sum_k D[k][k]: its
// virtual-virtual rows from the same reads, the others by the workgroups behind the columns.
// A workgroup holds one column x and 32 values of a; each wave takes every fourth chunk of 64 Q by itself (with a chunk
// shared through LDS, each waited for its reads and three barriers: o8 v72 20, o13 v117 45, o20 v180 150 us, now 12, 37 and 112).
constexpr int kDressA = 32;
struct DressP {
  const double *B, *D, *t1, *h;
  double *bvv, *bvo, *boo, *f;
  int o, v;
  long ldq;
  Shadow svv, svo, soo;  // of bvv, bvo and boo, or none
};
template <bool SHADOW>
__global__ __launch_bounds__(kThreads, 2) void dress_left_kernel(DressP p) {
  __shared__ double part[kDressA][4][17];  // sums of J B over a wave's chunks, by row and column of a tile
  const int o = p.o, v = p.v, n = o + v, lane = threadIdx.x & 63, l16 = lane & 15, lq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const long ldq = p.ldq;
  const int x = blockIdx.x, a0 = blockIdx.y * kDressA, i = x - v;
  const bool vv = x < v, coul = x >= n, dots = vv || coul;
  const int nrow = n * n - v * v, y0 = ((x - n) * (int)gridDim.y + (int)blockIdx.y) * 32;
  if (coul && y0 >= nrow) return;
  const int valid = coul ? min(32, nrow - y0) : min(32, v - a0);  // rows past it repeat the last one and are not stored
  // row of the block: of the a of column x or, behind the columns, of the pairs (p, q) with p or q occupied (rows of
  // the occupied p first, then (o + a, k))
  auto row_of = [&](int z) -> int {
    z = min(z, valid - 1);
    if (!coul) return vv ? (o + a0 + z) * n + o + x : i * n + o + a0 + z;
    const int y = y0 + z;
    return y < o * n ? y : (o + (y - o * n) / o) * n + (y - o * n) % o;
  };
  const double* in = vv || coul ? p.B : p.D;
  const double* w = vv ? p.B + (long)(o + x) * ldq : p.D + (long)i * n * ldq;  // of k = 0
  const long sw = vv ? n * ldq : ldq;
  double* out = vv ? p.bvv + ((long)a0 * v + x) * ldq : p.bvo + ((long)i * v + a0) * ldq;
  const long sout = vv ? v * ldq : ldq;
  long row[2][4];
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int r = 0; r < 4; ++r) row[m][r] = row_of(16 * m + lq + 4 * r) * ldq;
  double dot[2][4] = {};
  for (long qc = 64 * wave; qc < ldq; qc += 256) {
    const long q0 = qc + 4 * l16, q = q0 < ldq ? q0 : 0;
    const bool inq = q0 < ldq;
    auto load = [](const double* x) { return *reinterpret_cast<const dress_d4*>(x); };
    // this lane's four columns of a shadow's row; past ldq (less than a chunk) zeros
    auto shadow = [&](const Shadow& s, long srow, double y0, double y1, double y2, double y3) {
      if (q0 >= s.ld) return;
      const double d[4] = {inq ? y0 : 0.0, inq ? y1 : 0.0, inq ? y2 : 0.0, inq ? y3 : 0.0};
      put_lowp4(s, srow, q0, d);
    };
    dress_d4 acc[2][4];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const dress_d4 y = load(in + row[m][r] + q);
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[m][j][r] = y[j];
      }
    if (dots) {  // J: every fourth k per lane group
      dress_d4 J{0.0, 0.0, 0.0, 0.0};
      for (int k = lq; k < o; k += 4) J += load(p.D + (long)k * (n + 1) * ldq + q);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        double y = J[j];
        y += __shfl_xor(y, 16, 64);
        y += __shfl_xor(y, 32, 64);
        if (inq)
#pragma unroll
          for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r) dot[m][r] += y * acc[m][j][r];
      }
    }
    if (coul) continue;
#pragma unroll 2
    for (int kg = 0; kg < o; kg += 4) {
      const int k = kg + lq, kk = min(k, o - 1);
      double t[2];
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        const double y = p.t1[(long)kk * v + min(a0 + 16 * m + l16, v - 1)];
        t[m] = k < o ? -y : 0.0;
      }
      dress_d4 z = load(w + kk * sw + q);
      if (!vv && blockIdx.y == 0 && k < o) {
        if (inq) *reinterpret_cast<dress_d4*>(p.boo + ((long)k * o + i) * ldq + q) = z;
        if constexpr (SHADOW) shadow(p.soo, (long)k * o + i, z[0], z[1], z[2], z[3]);
      }
      z = k < o ? z : dress_d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[m][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(t[m], z[j], acc[m][j], 0, 0, 0);
    }
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int z = 16 * m + lq + 4 * r;
        if (z >= valid) continue;
        if (inq)
          *reinterpret_cast<dress_d4*>(out + z * sout + q) = dress_d4{acc[m][0][r], acc[m][1][r], acc[m][2][r], acc[m][3][r]};
        if constexpr (SHADOW)
          shadow(vv ? p.svv : p.svo, vv ? (long)(a0 + z) * v + x : (long)i * v + a0 + z, acc[m][0][r], acc[m][1][r], acc[m][2][r],
                 acc[m][3][r]);
      }
  }
  if (!dots) return;
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int r = 0; r < 4; ++r) part[16 * m + lq + 4 * r][wave][l16] = dot[m][r];
  __syncthreads();
  // eight lanes per row, eight of its 64 sums each
  const int z = threadIdx.x >> 3, e = threadIdx.x & 7;
  double s = 0.0;
#pragma unroll
  for (int y = 0; y < 8; ++y) s += part[z][e >> 1][8 * (e & 1) + y];
#pragma unroll
  for (int off = 4; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  if (e == 0 && z < valid) {
    const int f = row_of(z);
    p.f[f] = p.h[f] + 2.0 * s;
  }
}

// f[row] = f0[row] + alpha sum_Q J_Q B[row], J_Q = sum_k B[k][k], for all n^2 rows, 32 per workgroup.
__global__ __launch_bounds__(kThreads) void coulomb_kernel(double* __restrict__ f, const double* __restrict__ f0,
                                                          const double* __restrict__ B, double alpha, int o, int n,
                                                          long ldq) {
  __shared__ double J[64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const long nn = (long)n * n, row = blockIdx.x * 32L + wave * 8;
  double dot[8] = {};
  for (long q0 = 0; q0 < ldq; q0 += 64) {
    const long q = q0 + lane;
    __syncthreads();
    if (wave == 0) {
      double s = 0.0;
      if (q < ldq)
        for (int k = 0; k < o; ++k) s += B[((long)k * n + k) * ldq + q];
      J[lane] = s;
    }
    __syncthreads();
    if (q < ldq) {
#pragma unroll
      for (int r = 0; r < 8; ++r)
        if (row + r < nn) dot[r] += J[lane] * B[(row + r) * ldq + q];
    }
  }
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const double s = wave_all(dot[r]);
    if (lane == 0 && row + r < nn) f[row + r] = f0[row + r] + alpha * s;
  }
}

// Dressed Fock blocks F^ = X f Y^T: fvv [v][v], foo [o][o], fvo as r1[i][a] = F^_ai, fov [o][v] = f_ov (zero to ldf).  The
// first v workgroups form the rows b of fvv, the others the columns j < o (g(x) = f[x][j] + sum_c f[x][o+c] t1[j][c]).
__global__ __launch_bounds__(512) void fock_finish_kernel(double* __restrict__ fvv, double* __restrict__ foo,
                                                         double* __restrict__ r1, double* __restrict__ fov, long ldf,
                                                         const double* __restrict__ f, const double* __restrict__ t1,
                                                         int o, int v) {
  extern __shared__ double g[];  // [o + v]
  const int n = o + v;
  if ((int)blockIdx.x < v) {
    const int b = blockIdx.x;
    for (int k = threadIdx.x; k < o; k += 512) g[k] = t1[(long)k * v + b];
    __syncthreads();
    for (int c = threadIdx.x; c < v; c += 512) {
      double s = f[(long)(o + b) * n + o + c];
      for (int k = 0; k < o; ++k) s -= g[k] * f[(long)k * n + o + c];
      fvv[(long)b * v + c] = s;
    }
    return;
  }
  const int j = blockIdx.x - v, lane = threadIdx.x & 63;
  for (int x = threadIdx.x >> 6; x < n; x += 8) {
    double s = 0.0;
    for (int c = lane; c < v; c += 64) s += f[(long)x * n + o + c] * t1[(long)j * v + c];
    s = wave_all(s);
    if (lane == 0) g[x] = f[(long)x * n + j] + s;
  }
  __syncthreads();
  for (int k = threadIdx.x; k < o; k += 512) foo[(long)k * o + j] = g[k];
  for (int a = threadIdx.x; a < v; a += 512) {
    double s = g[o + a];
    for (int k = 0; k < o; ++k) s -= t1[(long)k * v + a] * g[k];
    r1[(long)j * v + a] = s;
    fov[(long)j * v + a] = f[(long)j * n + o + a];
  }
  if (j == 0)
    for (long x = (long)o * v + threadIdx.x; x < ldf; x += 512) fov[x] = 0.0;
}

// x -> (1 + c E_hp) x (1 - c E_hp) on an n x n matrix of rows of len values (stride ld): row h += c row p, then
// column p -= c column h of the result; element (r, s) of either step is one workgroup row of len values.
__global__ __launch_bounds__(kThreads) void onebody_row_kernel(double* __restrict__ X, int n, long ld, long len, int h,
                                                               int p, double c) {
  double* d = X + ((long)h * n + blockIdx.x) * ld;
  const double* s = X + ((long)p * n + blockIdx.x) * ld;
  for (long q = threadIdx.x; q < len; q += kThreads) d[q] += c * s[q];
}
__global__ __launch_bounds__(kThreads) void onebody_col_kernel(double* __restrict__ X, int n, long ld, long len, int h,
                                                               int p, double c) {
  double* d = X + ((long)blockIdx.x * n + p) * ld;
  const double* s = X + ((long)blockIdx.x * n + h) * ld;
  for (long q = threadIdx.x; q < len; q += kThreads) d[q] -= c * s[q];
}

// t1 = 0 except t1[h][a] = s1; t2 = 0 except t2[h][h][a][a] = s2.
__global__ __launch_bounds__(kThreads) void initial_guess_kernel(double* __restrict__ t1, double* __restrict__ t2,
                                                                 long len1, long len2, long k1, long k2, double s1,
                                                                 double s2) {
  for (long x = blockIdx.x * (long)kThreads + threadIdx.x; x < len1 + len2; x += (long)gridDim.x * kThreads) {
    if (x < len1)
      t1[x] = (x == k1) ? s1 : 0.0;
    else
      t2[x - len1] = (x - len1 == k2) ? s2 : 0.0;
  }
}

__device__ __forceinline__ double wave_sum(double x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x += __shfl_down(x, off, 64);
  return x;
}

// Block sum of one value per thread; result valid in thread 0.
__device__ double block_sum(double x, double* sh) {
  x = wave_sum(x);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) sh[w] = x;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0)
    for (int k = 0; k < (int)(blockDim.x >> 6); ++k) s += sh[k];
  return s;
}
__global__ __launch_bounds__(kThreads) void energy_stage1(double* partial, const double* __restrict__ t1,
                                                         const double* __restrict__ t2,
                                                         const double* __restrict__ L, int o, int v, long total) {
  __shared__ double sh[kThreads / 64];
  double acc = 0.0;
  const long vv = (long)v * v, ovv = (long)o * vv;
  for (long idx = blockIdx.x * (long)blockDim.x + threadIdx.x; idx < total; idx += (long)gridDim.x * blockDim.x) {
    const int i = idx / ovv;
    const int j = (idx / vv) % o;
    const int a = (idx / v) % v;
    const int b = idx % v;
    acc += (t2[idx] + t1[i * v + a] * t1[j * v + b]) * L[idx];
  }
  const double s = block_sum(acc, sh);
  if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

__global__ __launch_bounds__(kThreads) void energy_stage2(double* e, const double* partial, int nblk,
                                                         const double* t1, const double* fov, int nov) {
  __shared__ double sh[kThreads / 64];
  double acc = 0.0;
  for (int k = threadIdx.x; k < nblk; k += blockDim.x) acc += partial[k];
  for (int k = threadIdx.x; k < nov; k += blockDim.x) acc += 2.0 * fov[k] * t1[k];
  const double s = block_sum(acc, sh);
  if (threadIdx.x == 0) *e = s;
}

// ---------------------------------------------------------------------------------------
// Jacobi step + DIIS.
//
// Element x of the amplitude vector t1 (+) t2 gets s = R/D, t_new = t + s.  When the call
// stores a DIIS pair, (t_new, s) go to history slot `head`, and the overlaps <s, e_k> with
// every stored error vector are accumulated (the new slot's own entry is <s, s>).
// Partial sums per block: [0] sum R^2, [1] max|R|, [2] non-finite count, [3 + k] <s, e_k>.

__device__ __forceinline__ double denom(long x, int o, int v, const double* eps, double shift) {
  const long ov = (long)o * v;
  if (x < ov) {
    const int i = x / v, a = x % v;
    return eps[i] - eps[o + a] - shift;
  }
  const long y = x - ov, vv = (long)v * v, ovv = (long)o * vv;
  const int i = y / ovv, j = (y / vv) % o, a = (y / v) % v, b = y % v;
  return eps[i] + eps[j] - eps[o + a] - eps[o + b] - shift;
}

struct UK {
  const double* t1i;  // the amplitudes the step starts from (t1, t2 themselves in place)
  const double* t2i;
  double* t1;
  double* t2;
  const double* r1;
  const double* r2;
  const double* eps;
  double* hist_t;
  double* hist_e;
  double* partial;
  const DiisState* st;
  int o, v, m, start, nstat;
  long len;
  double shift;
  long ss;         // byte stride between the slots of a batched update (0: one slot)
  const int* tab;  // slot of grid row blockIdx.y (nullptr: blockIdx.y)
};

// The same pointer in slot k of a batched update (slots at a fixed byte stride).
template <class T>
__device__ __forceinline__ T* in_slot(T* p, long k, long ss) {
  return reinterpret_cast<T*>(reinterpret_cast<char*>(const_cast<typename std::remove_const<T>::type*>(p)) + k * ss);
}

__global__ __launch_bounds__(kThreads) void update_stage1(UK p) {
  if (p.ss) {  // this grid row's slot
    const long k = p.tab ? p.tab[blockIdx.y] : blockIdx.y;
    p.t1i = in_slot(p.t1i, k, p.ss);
    p.t2i = in_slot(p.t2i, k, p.ss);
    p.t1 = in_slot(p.t1, k, p.ss);
    p.t2 = in_slot(p.t2, k, p.ss);
    p.r1 = in_slot(p.r1, k, p.ss);
    p.r2 = in_slot(p.r2, k, p.ss);
    p.eps = in_slot(p.eps, k, p.ss);
    p.hist_t = in_slot(p.hist_t, k, p.ss);
    p.hist_e = in_slot(p.hist_e, k, p.ss);
    p.partial = in_slot(p.partial, k, p.ss);
    p.st = in_slot(p.st, k, p.ss);
  }
  __shared__ double sh[kThreads / 64][3 + kMaxDiis];
  const int head = p.st->head;
  const bool store = p.st->calls >= p.start;  // decided on the device, so a captured graph replays it
  bool valid[kMaxDiis];
  for (int k = 0; k < kMaxDiis; ++k) valid[k] = store && k < p.m && (k == head || p.st->slot_age[k] >= 0);
  double dots[kMaxDiis];
  for (int k = 0; k < kMaxDiis; ++k) dots[k] = 0.0;
  double rr = 0.0, rmax = 0.0, bad = 0.0;
  const long ov = (long)p.o * p.v;
  for (long x = blockIdx.x * (long)blockDim.x + threadIdx.x; x < p.len; x += (long)gridDim.x * blockDim.x) {
    const double r = (x < ov) ? p.r1[x] : p.r2[x - ov];
    const double s = r / denom(x, p.o, p.v, p.eps, p.shift);
    const double tn = ((x < ov) ? p.t1i[x] : p.t2i[x - ov]) + s;
    *((x < ov) ? (p.t1 + x) : (p.t2 + (x - ov))) = tn;
    rr += r * r;
    rmax = fmax(rmax, fabs(r));
    if (!isfinite(r)) bad += 1.0;
    if (store) {
      for (int k = 0; k < kMaxDiis; ++k)
        if (valid[k]) dots[k] += s * ((k == head) ? s : p.hist_e[(long)k * p.len + x]);
      p.hist_t[(long)head * p.len + x] = tn;
      p.hist_e[(long)head * p.len + x] = s;
    }
  }
  // per-wave results side by side, then one thread per statistic adds the block's four: one barrier for all of them
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  auto put = [&](int k, double v) {
    if (lane == 0) sh[w][k] = v;
  };
  put(0, wave_all(rr));
  put(1, wave_max(rmax));
  put(2, wave_all(bad));
  if (store)
    for (int k = 0; k < p.m; ++k) put(3 + k, wave_all(dots[k]));
  __syncthreads();
  const int k = threadIdx.x;
  if (k >= 3 + p.m) return;
  double v = 0.0;
  if (k < 3 || store) {
    v = sh[0][k];
    for (int x = 1; x < kThreads / 64; ++x) v = k == 1 ? fmax(v, sh[x][k]) : v + sh[x][k];
  }
  p.partial[(long)blockIdx.x * p.nstat + k] = v;
}

// Orders this wave's LDS accesses as written (they execute in order; the compiler is kept from moving them).
__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Bordered DIIS system over the valid slots (ages age[k] >= 0), oldest first, from the overlaps Bm; returns false if a
// pivot is tiny, else leaves the coefficients in coef by slot.  One wave: rows and columns of an elimination
// step over its lanes (as a chain of one thread the 9 x 9 system took 25 of the update's 45 us at o5 v20).
__device__ bool diis_solve(const int* age, const double* Bm, int m, double* A, double* xs, int* order, double* coef) {
  constexpr int W = kMaxDiis + 2;
  const int lane = threadIdx.x & 63;
  int nv = 0, rank = 0;
  for (int k = 0; k < m; ++k) {
    if (age[k] < 0) continue;
    ++nv;
    if (lane < m && age[k] < age[lane]) ++rank;
  }
  if (lane < m && age[lane] >= 0) order[rank] = lane;
  wave_fence();
  const int nn = nv + 1;
  double scale = 0.0;
  for (int x = lane; x < nn * (nn + 1); x += 64) {
    const int r = x / (nn + 1), c = x % (nn + 1);
    double y = -1.0;
    if (c == nn)
      y = (r == nv) ? -1.0 : 0.0;
    else if (r < nv && c < nv)
      scale = fmax(scale, fabs(y = Bm[order[r] * kMaxDiis + order[c]]));
    else if (r == nv && c == nv)
      y = 0.0;
    A[r * W + c] = y;
  }
  scale = wave_max(scale);
  wave_fence();
  for (int c = 0; c < nn; ++c) {
    int piv = c + lane;  // the first of the largest entries at or below the diagonal
    double best = piv < nn ? fabs(A[piv * W + c]) : -1.0;
    if (lane > 0 && !(best >= 0.0)) best = -1.0;  // a NaN is not larger than the diagonal
    for (int off = 16; off > 0; off >>= 1) {
      const double y = __shfl_xor(best, off, 64);
      const int q = __shfl_xor(piv, off, 64);
      if (y > best || (y == best && q < piv)) {
        best = y;
        piv = q;
      }
    }
    piv = __shfl(piv, 0, 64);
    const bool ok = fabs(A[piv * W + c]) >= 1e-14 * scale;
    if (!ok) return false;
    if (piv != c && lane <= nn) {
      const double t = A[c * W + lane];
      A[c * W + lane] = A[piv * W + lane];
      A[piv * W + lane] = t;
    }
    wave_fence();
    // columns past c only: the lower triangle is not read again
    for (int x = lane; x < (nn - 1 - c) * (nn - c); x += 64) {
      const int r = c + 1 + x / (nn - c), k = c + 1 + x % (nn - c);
      A[r * W + k] -= A[r * W + c] / A[c * W + c] * A[c * W + k];
    }
    wave_fence();
  }
  double acc = lane < nn ? A[lane * W + nn] : 0.0;
  for (int r = nn - 1; r >= 0; --r) {
    if (lane == r) xs[r] = acc / A[r * W + r];
    wave_fence();
    if (lane < r) acc -= A[lane * W + r] * xs[r];
  }
  if (lane < nv) coef[order[lane]] = xs[lane];
  wave_fence();
  return true;
}

__global__ __launch_bounds__(kThreads) void update_stage2(DiisState* st, const double* partial, int nblk, int nstat,
                                                         int m, int start, const double* e, double* stats,
                                                         double shift, long ss, const int* tab) {
  if (ss) {  // this grid row's slot; its statistics block is row k of stats
    const long k = tab ? tab[blockIdx.y] : blockIdx.y;
    st = in_slot(st, k, ss);
    partial = in_slot(partial, k, ss);
    e = in_slot(e, k, ss);
    stats += 8 * k;
  }
  __shared__ double red[3 + kMaxDiis], Bm[kMaxDiis * kMaxDiis], coef[kMaxDiis];
  __shared__ double A[(kMaxDiis + 1) * (kMaxDiis + 2)], xs[kMaxDiis + 1];
  __shared__ int age[kMaxDiis], order[kMaxDiis];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  // one wave per statistic
  for (int q = w; q < 3 + m; q += kThreads / 64) {
    double a = 0.0;
    for (int k = lane; k < nblk; k += 64) {
      const double y = partial[(long)k * nstat + q];
      a = q == 1 ? fmax(a, y) : a + y;
    }
    a = q == 1 ? wave_max(a) : wave_all(a);
    if (lane == 0) red[q] = a;
  }
  for (int x = threadIdx.x; x < kMaxDiis * kMaxDiis; x += kThreads) Bm[x] = st->Bm[x];
  if (threadIdx.x < kMaxDiis) age[threadIdx.x] = st->slot_age[threadIdx.x];
  __syncthreads();
  if (w != 0) return;

  const double E = *e;
  int flags = 0, nvec = st->nvec;
  if (red[2] > 0.0 || !isfinite(E) || !isfinite(red[0])) flags |= 1;
  const int calls = st->calls;
  if (calls >= start) {
    const int head = st->head, counter = st->counter;
    if (lane < m && (lane == head || age[lane] >= 0)) {
      Bm[head * kMaxDiis + lane] = Bm[lane * kMaxDiis + head] = red[3 + lane];
      st->Bm[head * kMaxDiis + lane] = st->Bm[lane * kMaxDiis + head] = red[3 + lane];
    }
    if (lane == 0) age[head] = counter;
    wave_fence();
    nvec = 0;
    for (int k = 0; k < m; ++k) nvec += (age[k] >= 0);
    for (;;) {
      if (lane < kMaxDiis) coef[lane] = 0.0;
      wave_fence();
      if (nvec < 2 || (flags & 1) || diis_solve(age, Bm, m, A, xs, order, coef)) break;
      int oldest = -1;
      for (int k = 0; k < m; ++k)
        if (age[k] >= 0 && (oldest < 0 || age[k] < age[oldest])) oldest = k;
      wave_fence();
      if (lane == 0) age[oldest] = -1;
      wave_fence();
      nvec -= 1;
      flags |= 2;
    }
    if (lane < kMaxDiis) {
      st->coef[lane] = coef[lane];
      st->slot_age[lane] = age[lane];
    }
    if (lane == 0) {
      st->counter = counter + 1;
      st->head = (head + 1) % m;
      st->nvec = nvec;
    }
  }
  if (lane != 0) return;
  stats[0] = E;
  stats[1] = st->has_prev ? E - st->e_prev : INFINITY;
  stats[2] = red[1];
  stats[3] = sqrt(red[0]);
  stats[4] = nvec;
  stats[5] = flags;
  stats[6] = calls;
  stats[7] = shift;
  st->e_prev = E;
  st->has_prev = 1;
  st->flags = flags;
  st->calls = calls + 1;
}

// t <- sum_k coef[k] hist_t[k] once two or more pairs are stored (no-op otherwise).
__global__ __launch_bounds__(kThreads) void update_stage3(double* t1, double* t2, const double* hist_t,
                                                         const DiisState* st, int m, long ov, long len, long ss,
                                                         const int* tab) {
  if (ss) {
    const long k = tab ? tab[blockIdx.y] : blockIdx.y;
    t1 = in_slot(t1, k, ss);
    t2 = in_slot(t2, k, ss);
    hist_t = in_slot(hist_t, k, ss);
    st = in_slot(st, k, ss);
  }
  if (st->nvec < 2 || (st->flags & 1)) return;
  double c[kMaxDiis];
  for (int k = 0; k < kMaxDiis; ++k) c[k] = (k < m) ? st->coef[k] : 0.0;
  for (long x = blockIdx.x * (long)blockDim.x + threadIdx.x; x < len; x += (long)gridDim.x * blockDim.x) {
    double acc = 0.0;
    for (int k = 0; k < m; ++k)
      if (c[k] != 0.0) acc += c[k] * hist_t[(long)k * len + x];
    if (x < ov)
      t1[x] = acc;
    else
      t2[x - ov] = acc;
  }
}


// ---------------------------------------------------------------------------------------
// Pair packing for the particle-particle ladder.
//
// Rows of symmetric and antisymmetric halves over the pairs c <= d of a v x v block M(c, d) at row stride
// sc: plus[p(c,d)] = f (M(c,d) + M(d,c)), minus[p(c,d)] = f (M(c,d) - M(d,c)) for c < d, and M(c,c), 0 on
// the diagonal; columns T(v) .. ldo - 1 are zeroed.  The block of grid column x and its output row:
//   kPackT   t+-: the pairs i <= j of t2 (f = 1/2), row p(i,j)
//   kPackV   V+-: W[a - a0][c][b - a0][d] of (ac|bd) for a in [a0, a1), b >= a, row p(a,b)
//   kPackG   G+-: (kc|bd) = W[k][c][b][d], row k*v + b of the rows behind V+-
//   kPackGo  G+-: (kc|ld) = W[k][c][l][d], row ov + k*o + l of the same
// One workgroup per block row and 32 x 32 tile pair (C <= D), or all pairs of one C where the rows are many: both
// tiles are read along their rows, the transposed one through LDS, and both outputs written along theirs (o20 v180:
// t+- 48 -> 15 us; all pairs of one C keep the unaligned ends of 32-value pieces in one L2: V+- of o18 v162 2.2 -> 1.7 ms).
enum { kPackT, kPackV, kPackG, kPackGo };
struct PackP {
  double *plus, *minus;
  long ldo;
  const double* src;
  int mode, o, v, a0;
};
__global__ __launch_bounds__(kThreads) void pack_halves_kernel(PackP p) {
  __shared__ double tile[2][32][33];
  const int o = p.o, v = p.v, nblk = (v + 31) / 32;
  const long vv = (long)v * v, Tv = (long)v * (v + 1) / 2, y = blockIdx.x;
  long base, sc = v, row;
  if (p.mode == kPackT) {
    int i = 0;
    long rem = y;
    while (rem >= o - i) {
      rem -= o - i;
      ++i;
    }
    base = ((long)i * o + i + rem) * vv;
    row = y;
  } else if (p.mode == kPackV) {
    const int a = p.a0 + (int)(y / v), b = (int)(y % v);
    if (b < a) return;
    sc = (long)(v - p.a0) * v;
    base = y / v * v * sc + (long)(b - p.a0) * v;
    row = pidx(a, b, v);
  } else if (p.mode == kPackG) {
    base = y / v * v * vv + y % v * v;
    sc = vv;
    row = y;
  } else {
    sc = (long)o * v;
    base = y / o * v * sc + y % o * v;
    row = (long)o * v + y;
  }
  const double* M = p.src + base;
  double* plus = p.plus + row * p.ldo;
  double* minus = p.minus + row * p.ldo;
  if (blockIdx.y == 0)
    for (long x = Tv + threadIdx.x; x < p.ldo; x += kThreads) plus[x] = minus[x] = 0.0;
  int C = blockIdx.y, D0 = C, D1 = nblk;  // tile pairs (C, D), D0 <= D < D1
  if (p.mode == kPackT) {
    int rem = blockIdx.y;
    for (C = 0; rem >= nblk - C; ++C) rem -= nblk - C;
    D0 = C + rem;
    D1 = D0 + 1;
  }
  const int c0 = 32 * C;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
  const double f = p.mode == kPackT ? 0.5 : 1.0;
  for (int D = D0; D < D1; ++D) {
    const int d0 = 32 * D;
    double(*t)[33] = tile[D & 1];  // the other one may still be read
    double x[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int r = ty + 8 * k;
      if (d0 + r < v && c0 + tx < v) t[r][tx] = M[(d0 + r) * sc + c0 + tx];
      x[k] = (c0 + r < v && d0 + tx < v) ? M[(c0 + r) * sc + d0 + tx] : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int c = c0 + ty + 8 * k, d = d0 + tx;
      if (c > d || d >= v) continue;
      const double a = x[k], b = t[tx][ty + 8 * k];
      const long q = pidx(c, d, v);
      plus[q] = (c == d) ? a : f * (a + b);
      minus[q] = (c == d) ? 0.0 : f * (a - b);
    }
  }
}

// The amplitude views of the contractions from t2 (t_ij^ab = t_ji^ba), one pair i <= j and 32 x 32 tile pair
// (C <= D) of (a, b) per workgroup, each element of t2[ij] read once:
//   Tx[ia][jb] = t_ij^ba, U[ia][jb] = 2 t_ij^ab - t_ij^ba (rows at stride ld, zero past o v)
// and, where plus is given, the pair rows t+- (as pack_halves_kernel).  o20 v180: 125 + 36 us as three
// passes, 75 us as one.
__global__ __launch_bounds__(kThreads) void amp_views_kernel(double* __restrict__ Tx, double* __restrict__ U, long ld,
                                                            double* __restrict__ plus, double* __restrict__ minus,
                                                            long ldo, const double* __restrict__ t2, int o, int v) {
  __shared__ double x1[32][33], x2[32][33];  // x1[c - c0][d - d0] = M(c, d), x2[d - d0][c - c0] = M(d, c), M = t2[ij]
  const int nblk = (v + 31) / 32;
  const long vv = (long)v * v, ov = (long)o * v, Tv = (long)v * (v + 1) / 2;
  int i = 0, rem = blockIdx.x;
  while (rem >= o - i) {
    rem -= o - i;
    ++i;
  }
  const int j = i + rem;
  int C = 0, trem = blockIdx.y;
  while (trem >= nblk - C) {
    trem -= nblk - C;
    ++C;
  }
  const int c0 = 32 * C, d0 = 32 * (C + trem);
  const bool diag = trem == 0;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
  const double* M = t2 + ((long)i * o + j) * vv;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int r = ty + 8 * k;
    if (c0 + r < v && d0 + tx < v) x1[r][tx] = M[(long)(c0 + r) * v + d0 + tx];
    if (d0 + r < v && c0 + tx < v) x2[r][tx] = M[(long)(d0 + r) * v + c0 + tx];
  }
  __syncthreads();
  // row p, columns q of the views: m = M(a, b), t = M(b, a) with a the row's and b the column's virtual
  auto put = [&](int p, int a, int q, int b, double m, double t) {
    const long x = ((long)p * v + a) * ld + (long)q * v + b;
    Tx[x] = t;
    U[x] = 2.0 * m - t;
  };
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int r = ty + 8 * k;
    {
      const int c = c0 + r, d = d0 + tx;  // along d
      if (c < v && d < v) {
        const double m = x1[r][tx], t = x2[tx][r];
        put(i, c, j, d, m, t);
        if (i != j) put(j, c, i, d, t, m);
        if (plus && c <= d) {
          const long q = blockIdx.x * ldo + pidx(c, d, v);
          plus[q] = (c == d) ? m : 0.5 * (m + t);
          minus[q] = (c == d) ? 0.0 : 0.5 * (m - t);
        }
      }
    }
    if (!diag) {
      const int d = d0 + r, c = c0 + tx;  // along c
      if (d < v && c < v) {
        const double m = x2[r][tx], t = x1[tx][r];
        put(i, d, j, c, m, t);
        if (i != j) put(j, d, i, c, t, m);
      }
    }
  }
  if (plus && blockIdx.y == 0)
    for (long x = Tv + threadIdx.x; x < ldo; x += kThreads) plus[blockIdx.x * ldo + x] = minus[blockIdx.x * ldo + x] = 0.0;
  // the padding columns of the rows (i, a in C), written once: by the pair (i, i) and the tile pairs (C, C)
  if (i == j && diag) {
    const int pad = (int)(ld - ov);
    for (int x = threadIdx.x; x < 32 * pad; x += kThreads) {
      const int a = c0 + x / pad;
      if (a < v) Tx[((long)i * v + a) * ld + ov + x % pad] = U[((long)i * v + a) * ld + ov + x % pad] = 0.0;
    }
  }
}

// Xc[ia][kc] = g^_kiac - Y1[ia][kc] / 2, Zd[ia][kc] = 2 g^_aikc - g^_kiac + Y2[ia][kc] / 2 (g2[k][i][a][c] = g^_kiac,
// g3[ia][kc] = g^_aikc; Xc, Zd rows at stride ld, zero past o v): one workgroup per row ia, every array along c.
__global__ __launch_bounds__(kThreads) void ring_xz_kernel(double* __restrict__ xc, double* __restrict__ zd, long ld,
                                                          const double* __restrict__ g2, const double* __restrict__ g3,
                                                          const double* __restrict__ y1, const double* __restrict__ y2,
                                                          int o, int v) {
  const long ia = blockIdx.x, ov = (long)o * v, row = ia * ov;
  const double* g = g2 + ia * v;  // [i][a][.] of k = 0; k advances by o v^2
  for (int x = threadIdx.x; x < ld; x += kThreads) {
    double a = 0.0, b = 0.0;
    if (x < ov) {
      const int k = x / v, c = x - k * v;
      const double q = g[(long)k * ov * v + c];
      a = q - 0.5 * y1[row + x];
      b = 2.0 * g3[row + x] - q + 0.5 * y2[row + x];
    }
    xc[ia * ld + x] = a;
    zd[ia * ld + x] = b;
  }
}

// The same, written as low-precision shadows alone (rows ia and, for Zd, o v + ia, zero past o v): four columns per thread, which
// makes the stores 8 or 16 bytes (o20 v180: 132 + 53 us with FP64 rows and their conversion, 144 us as one pass).
__global__ __launch_bounds__(kThreads) void ring_xz_lowp_kernel(Shadow s, const double* __restrict__ g2,
                                                               const double* __restrict__ g3, const double* __restrict__ y1,
                                                               const double* __restrict__ y2, int o, int v) {
  const long ia = blockIdx.x, ov = (long)o * v, row = ia * ov;
  const double* g = g2 + ia * v;
  for (int x = 4 * threadIdx.x; x < s.ld; x += 4 * kThreads) {
    double a[4], b[4];
    int k = x / v, c = x - k * v;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      a[j] = b[j] = 0.0;
      if (x + j < ov) {
        const double q = g[(long)k * ov * v + c];
        a[j] = q - 0.5 * y1[row + x + j];
        b[j] = 2.0 * g3[row + x + j] - q + 0.5 * y2[row + x + j];
      }
      if (++c == v) {
        c = 0;
        ++k;
      }
    }
    put_lowp4(s, ia, x, a);
    put_lowp4(s, ov + ia, x, b);
  }
}

// From the pair rows Rw+-[p(i,j)][m] of W/Z (m = k*v + b: W_ij[k,b] = sum_cd (kc|bd) t_ij^cd, m = ov + k*o + l:
// Z_ij[k,l] = sum_cd (kc|ld) t_ij^cd; X_ij = X+ + X-, X_ji = X+ - X-), with rows at stride ldr:
//   wp[ij][k][b] = W_ij[k,b] - 1/2 sum_l Z_ij[k,l] t1[l][b]   (rows at stride ldw)
//   chi+-[p(i,j)][p(k,l)] = c_kl +- c_lk (k < l), c_kk and 0 (k = l), where
//   c_kl = g^_kilj + Z_ij[k,l] - [k = i] F''_lj - [l = j] F''_ki
// (g4[k][i][l][j] = g^_kilj; the F'' part of the E term joins the hole-hole ladder, which sums c_kl t_kl^ab).
// One workgroup per pair i <= j and eight k; a thread per column b keeps the sixteen sums of ij and ji.
constexpr int kWzRows = 8;
__global__ __launch_bounds__(kThreads) void wz_chi_kernel(double* __restrict__ wp, long ldw, double* __restrict__ chip,
                                                         double* __restrict__ chim, const double* __restrict__ rp,
                                                         const double* __restrict__ rm, long ldr,
                                                         const double* __restrict__ g4, const double* __restrict__ foo,
                                                         const double* __restrict__ t1, int o, int v) {
  extern __shared__ double z[];  // [2][kWzRows][o]: Z_ij and Z_ji of this workgroup's k
  int i = 0, rem = blockIdx.x;
  while (rem >= o - i) {
    rem -= o - i;
    ++i;
  }
  const int j = i + rem, k0 = blockIdx.y * kWzRows, nk = min(kWzRows, o - k0);
  const long ov = (long)o * v, To = (long)o * (o + 1) / 2;
  const double* xp = rp + blockIdx.x * ldr;
  const double* xm = rm + blockIdx.x * ldr;
  for (int x = threadIdx.x; x < kWzRows * o; x += kThreads) {
    double zp = 0.0, zm = 0.0;
    if (x < nk * o) {
      zp = xp[ov + (long)k0 * o + x];
      zm = xm[ov + (long)k0 * o + x];
    }
    z[x] = zp + zm;
    z[kWzRows * o + x] = zp - zm;
  }
  __syncthreads();
  for (int b = threadIdx.x; b < v; b += kThreads) {
    double s1[kWzRows] = {}, s2[kWzRows] = {};
    for (int l = 0; l < o; ++l) {
      const double t = t1[(long)l * v + b];
#pragma unroll
      for (int r = 0; r < kWzRows; ++r) {
        s1[r] += z[r * o + l] * t;
        s2[r] += z[(kWzRows + r) * o + l] * t;
      }
    }
#pragma unroll
    for (int r = 0; r < kWzRows; ++r) {
      if (r >= nk) break;
      const long m = (long)(k0 + r) * v + b;
      const double p = xp[m], q = xm[m];
      wp[((long)i * o + j) * ldw + m] = (p + q) - 0.5 * s1[r];
      if (i != j) wp[((long)j * o + i) * ldw + m] = (p - q) - 0.5 * s2[r];
    }
  }
  for (int x = threadIdx.x; x < nk * o; x += kThreads) {
    const int k = k0 + x / o, l = x % o;
    if (l < k) continue;
    auto c = [&](int kk, int ll) {
      const long m = ov + (long)kk * o + ll;
      double w = g4[(((long)kk * o + i) * o + ll) * o + j] + (xp[m] + xm[m]);
      if (kk == i) w -= foo[(long)ll * o + j];
      if (ll == j) w -= foo[(long)kk * o + i];
      return w;
    };
    const long q = blockIdx.x * To + pidx(k, l, o);
    const double a = c(k, l);
    if (k == l) {
      chip[q] = a;
      chim[q] = 0.0;
    } else {
      const double b = c(l, k);
      chip[q] = a + b;
      chim[q] = a - b;
    }
  }
}

// RL[i][j][a][b] from R+-[p][p(a,b)]: R^ab = R+ + R- (a <= b), R+ - R- (a > b), with R_ij = R_ji^T.
// One workgroup per pair i <= j and 32 x 32 block (A <= B) of (a, b): with u = R+ + R-, w = R+ - R-
// at the packed index p(a, b), a <= b, the four outputs are RL[i][j][a][b] = RL[j][i][b][a] = u and
// RL[i][j][b][a] = RL[j][i][a][b] = w (the residual's pair symmetry; R- vanishes on a = b).  Each
// packed element is read once; the transposed writes go through an LDS tile.
__global__ __launch_bounds__(kThreads) void unpack_rpm_kernel(double* __restrict__ RL, const double* __restrict__ Rplus,
                                                             const double* __restrict__ Rminus, long ldr, int o,
                                                             int v, int nblk) {
  __shared__ double tu[32][33], tw[32][33];
  const long vv = (long)v * v;
  // block pair (A, B), A <= B, from blockIdx.x
  int A = 0, rem = blockIdx.x;
  while (rem >= nblk - A) {
    rem -= nblk - A;
    ++A;
  }
  const int B = A + rem;
  int i = 0, prem = blockIdx.y;  // pair i <= j from blockIdx.y
  while (prem >= o - i) {
    prem -= o - i;
    ++i;
  }
  const int j = i + prem;
  const long p = pidx(i, j, o);
  const double* plus = Rplus + p * ldr;
  const double* minus = Rminus + p * ldr;
  double* dij = RL + ((long)i * o + j) * vv;
  double* dji = RL + ((long)j * o + i) * vv;
  const int a0 = 32 * A, b0 = 32 * B;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
  // read: rows a = a0 + ty + 8r, columns b = b0 + tx (contiguous in the packed row)
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int la = ty + 8 * r, a = a0 + la, b = b0 + tx;
    double u = 0.0, w = 0.0;
    const bool in = a < v && b < v && a <= b;
    if (in) {
      const long k = pidx(a, b, v);
      const double x = plus[k], y = minus[k];
      u = x + y;
      w = x - y;
      dij[(long)a * v + b] = u;
      if (i != j) dji[(long)a * v + b] = (a == b) ? u : w;
    }
    tu[la][tx] = u;
    tw[la][tx] = w;
  }
  __syncthreads();
  // transposed writes: position (b, a), a = a0 + tx contiguous
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int lb = ty + 8 * r, b = b0 + lb, a = a0 + tx;
    if (a < v && b < v && a < b) {
      dij[(long)b * v + a] = tw[tx][lb];
      if (i != j) dji[(long)b * v + a] = tu[tx][lb];
    }
  }
}

// Pair order of the full (ac|bd) storage: R(a,b) = p(a,b) for a <= b, T(v) + strict pair index of
// (b,a) for a > b; pm[n] = R(b,a) for pair n = (a <= b) (n itself when a = b).
__device__ __forceinline__ long pair_order(long a, long b, long v) {
  const long Tv = v * (v + 1) / 2;
  return a <= b ? pidx(a, b, v) : Tv + pidx(b, a, v) - (b + 1);
}

__global__ __launch_bounds__(kThreads) void pair_minus_rows_kernel(int* __restrict__ pm, int v) {
  const int a = blockIdx.x * kThreads + threadIdx.x;
  if (a >= v) return;
  for (int b = a; b < v; ++b) pm[pidx(a, b, v)] = (int)pair_order(b, a, v);
}

// Full (ac|bd) in pair order, rows at stride ldv: V[R(a,b)][R(c,d)] = W[a - a0][c][b][d] for a in [a0, a1),
// the diagonal columns c = d halved, so that V[R(a,b)] +- V[R(b,a)] are the packed halves there too.
__global__ __launch_bounds__(kThreads) void pack_full_kernel(double* __restrict__ V, long ldv,
                                                            const double* __restrict__ W, int a0, int v) {
  const int a = a0 + blockIdx.y / v, b = blockIdx.y % v;
  const long vv = (long)v * v;
  const double* src = W + (long)(a - a0) * v * vv + (long)b * v;
  double* dst = V + pair_order(a, b, v) * ldv;
  if (blockIdx.x == 0)
    for (long x = vv + threadIdx.x; x < ldv; x += kThreads) dst[x] = 0.0;
  for (long x = blockIdx.x * (long)blockDim.x + threadIdx.x; x < vv; x += (long)gridDim.x * blockDim.x) {
    const int c = x / v, d = x % v;
    const double w = src[c * vv + d];
    dst[pair_order(c, d, v)] = (c == d) ? 0.5 * w : w;
  }
}

// First-stage blocks of a reduction over total elements: two of a thread's each, as far as kRedBlocks go (the second stage
// reads one row of partial sums per block).
inline int red_blocks(long total) { return (int)std::clamp<long>((total + 2 * kThreads - 1) / (2 * kThreads), 1, kRedBlocks); }

inline int grid_for(long total) {
  long g = (total + kThreads - 1) / kThreads;
  if (g > 8192) g = 8192;
  if (g < 1) g = 1;
  return (int)g;
}

}  // namespace

static bool p4_in_bounds(const P4& p) {
  const char* names[4] = {"permute input 0", "permute input 1", "permute input 2", "permute input 3"};
  long lo = 0, hi = 0;
  for (int k = 0; k < 4; ++k) {
    const long d = (long)(p.d[k] - 1) * p.os[k];
    if (d < 0) lo += d; else hi += d;
  }
  if (!range_ok(p.out, lo, hi, sizeof(double), "permute output")) return false;
  for (int t = 0; t < p.nin; ++t) {
    lo = hi = 0;
    for (int k = 0; k < 4; ++k) {
      const long d = (long)(p.d[k] - 1) * p.s[t][k];
      if (d < 0) lo += d; else hi += d;
    }
    if (!range_ok(p.in[t], lo, hi, sizeof(double), names[t])) return false;
  }
  return true;
}

// Drops size-1 dimensions (the remaining ones keep their order, right-aligned), then takes the
// tiled kernel when the output is contiguous along its last index and some input is contiguous
// along another index of at least 16.
static hipError_t launch_permute(P4 p, long total, hipStream_t s) {
  P4 c = p;
  int k2 = 3;
  for (int k = 3; k >= 0; --k) {
    if (p.d[k] == 1) continue;
    c.d[k2] = p.d[k];
    c.os[k2] = p.os[k];
    for (int q = 0; q < p.nin; ++q) c.s[q][k2] = p.s[q][k];
    --k2;
  }
  for (; k2 >= 0; --k2) {
    c.d[k2] = 1;
    c.os[k2] = 0;
    for (int q = 0; q < p.nin; ++q) c.s[q][k2] = 0;
  }
  int t = -1, tmask = 0;
  if (c.os[3] == 1 && c.d[3] >= 16) {
    for (int k = 2; k >= 0 && t < 0; --k) {
      if (c.d[k] < 16) continue;
      int m = 0;
      for (int q = 0; q < c.nin; ++q)
        if (c.s[q][k] == 1 && c.s[q][3] != 1) m |= 1 << q;
      if (m) {
        t = k;
        tmask = m;
      }
    }
  }
  if (t >= 0) {
    int u = -1, w = -1;
    for (int k = 0; k < 3; ++k)
      if (k != t) (u < 0 ? u : w) = k;
    const long tiles_t = (c.d[t] + 31) / 32, tiles3 = (c.d[3] + 31) / 32;
    if (tiles_t * tiles3 <= 0x7fffffffL && c.d[u] <= 65535 && c.d[w] <= 65535) {
      hipLaunchKernelGGL(permute4_tiled_kernel, dim3((unsigned)(tiles_t * tiles3), (unsigned)c.d[u], (unsigned)c.d[w]),
                         dim3(kThreads), 0, s, c, t, u, w, (int)tiles3, tmask);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL(permute4_kernel, dim3(grid_for(total)), dim3(kThreads), 0, s, p, total);
  return hipGetLastError();
}

hipError_t permute4(double* out, const int dims[4], double c0, const Perm4In* in, int nin, hipStream_t s) {
  // contiguous output with the given dims
  P4 p{};
  p.out = out;
  p.os[3] = 1;
  p.os[2] = dims[3];
  p.os[1] = (long)dims[3] * dims[2];
  p.os[0] = (long)dims[3] * dims[2] * dims[1];
  for (int k = 0; k < 4; ++k) p.d[k] = dims[k];
  p.c0 = c0;
  p.nin = nin;
  for (int t = 0; t < nin; ++t) {
    p.in[t] = in[t].p;
    p.coef[t] = in[t].coef;
    for (int k = 0; k < 4; ++k) p.s[t][k] = in[t].s[k];
  }
  const long total = (long)dims[0] * dims[1] * dims[2] * dims[3];
  if (total <= 0) return hipSuccess;
  if (bounds_checking() && !p4_in_bounds(p)) return hipErrorInvalidValue;
  if (dry_run()) return hipSuccess;
  return launch_permute(p, total, s);
}

hipError_t permute4_strided(double* out, const long ostr[4], const int dims[4], double c0, const Perm4In* in,
                            int nin, hipStream_t s) {
  P4 p{};
  p.out = out;
  for (int k = 0; k < 4; ++k) {
    p.os[k] = ostr[k];
    p.d[k] = dims[k];
  }
  p.c0 = c0;
  p.nin = nin;
  for (int t = 0; t < nin; ++t) {
    p.in[t] = in[t].p;
    p.coef[t] = in[t].coef;
    for (int k = 0; k < 4; ++k) p.s[t][k] = in[t].s[k];
  }
  const long total = (long)dims[0] * dims[1] * dims[2] * dims[3];
  if (total <= 0) return hipSuccess;
  if (bounds_checking() && !p4_in_bounds(p)) return hipErrorInvalidValue;
  if (dry_run()) return hipSuccess;
  return launch_permute(p, total, s);
}

hipError_t assemble_r2(double* r2, const double* g1, const double* rl, const double* em, const double* p1,
                       const double* p2, int no, int nv, hipStream_t s, const double* rminus, long ldr) {
  const long total = (long)no * no * nv * nv;
  const long ovov = (long)no * nv * no * nv;
  const long tv = (nv + 31) / 32, pairs = (long)no * (no + 1) / 2, Tv = (long)nv * (nv + 1) / 2;
  if (bounds_checking() &&
      !(range_ok(r2, 0, total - 1, 8, "assemble r2") && range_ok(g1, 0, ovov - 1, 8, "assemble g1") &&
        range_ok(rl, 0, rminus ? (pairs - 1) * ldr + Tv - 1 : total - 1, 8, "assemble rl") &&
        (!rminus || range_ok(rminus, 0, (pairs - 1) * ldr + Tv - 1, 8, "assemble R-")) &&
        range_ok(em, 0, total - 1, 8, "assemble em") &&
        range_ok(p1, 0, ovov - 1, 8, "assemble p1") && range_ok(p2, 0, ovov - 1, 8, "assemble p2")))
    return hipErrorInvalidValue;
  if (dry_run()) return hipSuccess;
  if (tv * tv > 65535 || pairs > 0x7fffffffL) return hipErrorInvalidValue;
  const dim3 grid((unsigned)pairs, (unsigned)(tv * tv));
  if (rminus)
    hipLaunchKernelGGL(assemble_r2_kernel<true>, grid, dim3(kThreads), 0, s, r2, g1, rl, rminus, ldr, em, p1, p2, no, nv);
  else
    hipLaunchKernelGGL(assemble_r2_kernel<false>, grid, dim3(kThreads), 0, s, r2, g1, rl, rl, 0L, em, p1, p2, no, nv);
  return hipGetLastError();
}

static bool chk(const void* p, long n, const char* what) { return range_ok(p, 0, n - 1, 8, what); }

hipError_t dress_right(double* D, const double* B, const double* t1, int o, int v, long ldq, hipStream_t s) {
  const long n = o + v;
  if (o < 1 || v < 1 || ldq < 1 || ldq % 4 || n > 65535) return hipErrorInvalidValue;
  if (bounds_checking() && !(chk(D, o * n * ldq, "dress D") && chk(B, n * n * ldq, "dress B") && chk(t1, (long)o * v, "dress t1")))
    return hipErrorInvalidValue;
  if (dry_run()) return hipSuccess;
  // the fewest passes over B with at most 48 values of k each
  const int passes = (o + 47) / 48, mt = ((o + passes - 1) / passes + 15) / 16;
  const dim3 grid((unsigned)((ldq + 63) / 64), (unsigned)n, (unsigned)((o + 16 * mt - 1) / (16 * mt)));
  hipLaunchKernelGGL(mt == 1 ? dress_right_kernel<1> : mt == 2 ? dress_right_kernel<2> : dress_right_kernel<3>, grid, dim3(kThreads), 0,
                     s, D, B, t1, o, v, ldq);
  return hipGetLastError();
}

hipError_t dress_left(double* bvv, double* bvo, double* boo, double* f, const double* B, const double* D,
                      const double* t1, const double* h, int o, int v, long ldq, int prec, float* svv, float* svo, float* soo,
                      hipStream_t s) {
  const long ls = lowp_ld(ldq);  // naux <= ldq <= naux rounded up to 16
  if (svv && bounds_checking() && !(range_ok(svv, 0, (long)v * v * ls - 1, 4, "B^vv shadow") &&
                                    range_ok(svo, 0, (long)o * v * ls - 1, 4, "B^vo shadow") &&
                                    range_ok(soo, 0, (long)o * o * ls - 1, 4, "B^oo shadow")))
    return hipErrorInvalidValue;
  const long n = o + v, oo = (long)o * o, ov = (long)o * v, vv = (long)v * v;
  if (o < 1 || v < 1 || o > 256 || ldq < 1 || ldq % 4) return hipErrorInvalidValue;
  if (bounds_checking() && !(chk(bvv, vv * ldq, "dress B^vv") && chk(bvo, ov * ldq, "dress B^vo") && chk(boo, oo * ldq, "dress B^oo") &&
                             chk(f, n * n, "dress f") && chk(B, n * n * ldq, "dress B") && chk(D, o * n * ldq, "dress D") &&
                             chk(t1, ov, "dress t1") && chk(h, n * n, "dress h")))
    return hipErrorInvalidValue;
  if (dry_run()) return hipSuccess;
  const long ga = (v + kDressA - 1) / kDressA, rest = (n * n - vv + 31) / 32;  // a blocks; Coulomb workgroups
  hipLaunchKernelGGL(svv ? dress_left_kernel<true> : dress_left_kernel<false>, dim3((unsigned)(n + (rest + ga - 1) / ga), (unsigned)ga), dim3(kThreads), 0, s,
                     DressP{B, D, t1, h, bvv, bvo, boo, f, o, v, ldq, {svv, ls, prec}, {svo, ls, prec}, {soo, ls, prec}});
  return hipGetLastError();
}

hipError_t coulomb(double* f, const double* f0, const double* B, double alpha, int o, int n, long ldq, hipStream_t s) {
  const long nn = (long)n * n;
  if (bounds_checking() && !(chk(f, nn, "Coulomb f") && chk(f0, nn, "Coulomb f0") && chk(B, nn * ldq, "Coulomb B")))
    return hipErrorInvalidValue;
  if (dry_run()) return hipSuccess;
  hipLaunchKernelGGL(coulomb_kernel, dim3((unsigned)((nn + 31) / 32)), dim3(kThreads), 0, s, f, f0, B, alpha, o, n, ldq);
  return hipGetLastError();
}

hipError_t fock_finish(double* fvv, double* foo, double* r1, double* fov, long ldf, const double* f, const double* t1,
                       int o, int v, hipStream_t s) {
  const long n = o + v, ov = (long)o * v;
  if (bounds_checking() && !(chk(fvv, (long)v * v, "F^vv") && chk(foo, (long)o * o, "F^oo") && chk(r1, ov, "F^vo") &&
                             chk(fov, std::max(ldf, ov), "F^ov") && chk(f, n * n, "Fock f") && chk(t1, ov, "Fock t1")))
    return hipErrorInvalidValue;
  if (dry_run()) return hipSuccess;
  hipLaunchKernelGGL(fock_finish_kernel, dim3((unsigned)n), dim3(512), n * sizeof(double), s, fvv, foo, r1, fov, ldf, f, t1, o,
                     v);
  return hipGetLastError();
}

hipError_t onebody_transform(double* X, int n, long ld, long len, int h, int p, double c, hipStream_t s) {
  if (n < 1 || len < 1 || ld < len) return hipErrorInvalidValue;
  if (h < 0 || h >= n || p < 0 || p >= n || h == p) return hipErrorInvalidValue;
  if (bounds_checking() && !chk(X, ((long)n * n - 1) * ld + len, "one-body transform")) return hipErrorInvalidValue;
  if (dry_run()) return hipSuccess;
  hipLaunchKernelGGL(onebody_row_kernel, dim3((unsigned)n), dim3(kThreads), 0, s, X, n, ld, len, h, p, c);
  hipLaunchKernelGGL(onebody_col_kernel, dim3((unsigned)n), dim3(kThreads), 0, s, X, n, ld, len, h, p, c);
  return hipGetLastError();
}

hipError_t initial_guess(double* t1, double* t2, int no, int nv, int h, int a, double s1, double s2, hipStream_t s) {
  const long len1 = (long)no * nv, len2 = len1 * len1;
  if (h < 0 || h >= no || a < 0 || a >= nv) return hipErrorInvalidValue;
  if (bounds_checking() && !(range_ok(t1, 0, len1 - 1, 8, "guess t1") && range_ok(t2, 0, len2 - 1, 8, "guess t2")))
    return hipErrorInvalidValue;
  if (dry_run()) return hipSuccess;
  const long k1 = (long)h * nv + a, k2 = (((long)h * no + h) * nv + a) * nv + a;
  hipLaunchKernelGGL(initial_guess_kernel, dim3(grid_for(len1 + len2)), dim3(kThreads), 0, s, t1, t2, len1, len2, k1,
                     k2, s1, s2);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Cross index sets (internal.h): over r = i * nv + a (i < no, a < nv) the members i == h or
// a == pa, m = nv + no - 1 of them in the compact order k < nv -> (h, k), k = nv + q -> (i, pa)
// with i = q (q < h) or q + 1 (q >= h).
__device__ __forceinline__ long cross_row(const Cross& X, long k) {
  if (k < X.nv) return (long)X.h * X.nv + k;
  const long q = k - X.nv;
  return (q < X.h ? q : q + 1) * (long)X.nv + X.pa;
}
__device__ __forceinline__ bool cross_member(const Cross& X, long r) { return r / X.nv == X.h || r % X.nv == X.pa; }

// dst[k][c] = src[cross_row(k)][c] (c < ncols); with zero_diag, the entry whose row and column
// are both the cross's corner r = h * nv + pa is written as 0.
__global__ void cross_gather_rows_kernel(double* __restrict__ dst, long ldd, const double* __restrict__ src, long lds,
                                         long ncols, Cross X, int zero_diag) {
  const long m = X.m(), total = m * ncols, hp = (long)X.h * X.nv + X.pa;
  for (long x = blockIdx.x * (long)blockDim.x + threadIdx.x; x < total; x += (long)gridDim.x * blockDim.x) {
    const long k = x / ncols, c = x - k * ncols;
    const long r = cross_row(X, k);
    dst[k * ldd + c] = (zero_diag && r == hp && c == hp) ? 0.0 : src[r * lds + c];
  }
}

// dst[r][k] = src[r][cross_row(k)] for k < m and 0 for m <= k < ldd (padding); with zero_rows,
// rows r that are members of the row cross R are written as 0.
__global__ void cross_gather_cols_kernel(double* __restrict__ dst, long ldd, const double* __restrict__ src, long lds,
                                         long nrows, Cross X, Cross R, int zero_rows) {
  const long m = X.m(), total = nrows * ldd;
  for (long x = blockIdx.x * (long)blockDim.x + threadIdx.x; x < total; x += (long)gridDim.x * blockDim.x) {
    const long r = x / ldd, k = x - r * ldd;
    dst[x] = (k >= m || (zero_rows && cross_member(R, r))) ? 0.0 : src[r * lds + cross_row(X, k)];
  }
}

// dst[cross_row(k)][c] += alpha * src[k][c] (members are distinct: no two threads share a target).
__global__ void cross_scatter_add_rows_kernel(double* __restrict__ dst, long ldd, const double* __restrict__ src,
                                              long lds, long ncols, double alpha, Cross X) {
  const long m = X.m(), total = m * ncols;
  for (long x = blockIdx.x * (long)blockDim.x + threadIdx.x; x < total; x += (long)gridDim.x * blockDim.x) {
    const long k = x / ncols, c = x - k * ncols;
    dst[cross_row(X, k) * ldd + c] += alpha * src[k * lds + c];
  }
}

// dst[r][cross_row(k)] += alpha * src[r][k]   (r < nrows, k < m).
__global__ void cross_scatter_add_cols_kernel(double* __restrict__ dst, long ldd, const double* __restrict__ src,
                                              long lds, long nrows, double alpha, Cross X) {
  const long m = X.m(), total = nrows * m;
  for (long x = blockIdx.x * (long)blockDim.x + threadIdx.x; x < total; x += (long)gridDim.x * blockDim.x) {
    const long r = x / m, k = x - r * m;
    dst[r * ldd + cross_row(X, k)] += alpha * src[r * lds + k];
  }
}

// dst[cross_row(k1)][cross_row(k2)] += alpha * src[k1][k2].
__global__ void cross_scatter_add_block_kernel(double* __restrict__ dst, long ldd, const double* __restrict__ src,
                                               long lds, double alpha, Cross X) {
  const long m = X.m(), total = m * m;
  for (long x = blockIdx.x * (long)blockDim.x + threadIdx.x; x < total; x += (long)gridDim.x * blockDim.x) {
    const long k1 = x / m, k2 = x - k1 * m;
    dst[cross_row(X, k1) * ldd + cross_row(X, k2)] += alpha * src[k1 * lds + k2];
  }
}

// dst[k][c] = Y[cross_row(k)][c] - [cross_row(k) == hp] T[hp][hp] K[hp][c]  (ld x ld operands, T and K rows at ldk,
// hp = h * nv + pa): the cross rows of (T with its corner entry removed) K, from Y = T K.
__global__ void cross_rows_without_corner_kernel(double* __restrict__ dst, long ldd, const double* __restrict__ Y,
                                                 const double* __restrict__ T, const double* __restrict__ K, long ldk,
                                                 long ld, Cross X) {
  const long m = X.m(), total = m * ld, hp = (long)X.h * X.nv + X.pa;
  const double thp = T[hp * ldk + hp];
  for (long x = blockIdx.x * (long)blockDim.x + threadIdx.x; x < total; x += (long)gridDim.x * blockDim.x) {
    const long k = x / ld, c = x - k * ld;
    const long r = cross_row(X, k);
    dst[k * ldd + c] = Y[r * ld + c] - (r == hp ? thp * K[hp * ldk + c] : 0.0);
  }
}

// EM[ij][a][b] += tc[ij][v + q(a)] * A[b][pa] for a != pa (q(a) = a - [a > pa]): the part of
// sum_c t^M_ij^ac A[b][c] from the entries (a, pa) of rows ij outside the occupied cross, which
// tc holds (compact vv-cross columns, rows of the occupied cross zero).
__global__ void em_cross_column_kernel(double* __restrict__ em, const double* __restrict__ tc, long ldt,
                                       const double* __restrict__ A, int o, int v, int pa) {
  const long vv = (long)v * v, total = (long)o * o * vv;
  for (long x = blockIdx.x * (long)blockDim.x + threadIdx.x; x < total; x += (long)gridDim.x * blockDim.x) {
    const long ij = x / vv, ab = x - ij * vv;
    const int a = (int)(ab / v), b = (int)(ab % v);
    if (a == pa) continue;
    em[x] += tc[ij * ldt + v + (a < pa ? a : a - 1)] * A[(long)b * v + pa];
  }
}

// dst[i][j][a][b] = src[i][j][a][b] where the index set holds h (in i, j) or pa (in a, b) and is
// not all primary (the mixed doubles), else 0.
__global__ void mixed_doubles_kernel(double* __restrict__ dst, const double* __restrict__ src, int o, int v, int h,
                                     int pa) {
  const long vv = (long)v * v, total = (long)o * o * vv;
  for (long x = blockIdx.x * (long)blockDim.x + threadIdx.x; x < total; x += (long)gridDim.x * blockDim.x) {
    const long ij = x / vv, ab = x - ij * vv;
    const int i = (int)(ij / o), j = (int)(ij % o), a = (int)(ab / v), b = (int)(ab % v);
    const bool any = i == h || j == h || a == pa || b == pa;
    const bool all = i == h && j == h && a == pa && b == pa;
    dst[x] = (any && !all) ? src[x] : 0.0;
  }
}

// e0 = sum_{i<o} (h[i * hs] + f[i * fs]): one workgroup, fixed-order tree sum (o <= 256 per thread pass).
__global__ __launch_bounds__(kThreads) void reference_energy_kernel(double* e0, const double* h, long hs,
                                                                   const double* f, long fs, int o) {
  __shared__ double red[kThreads];
  double acc = 0.0;
  for (int i = threadIdx.x; i < o; i += kThreads) acc += h[(long)i * hs] + f[(long)i * fs];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int w = kThreads / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) e0[0] = red[0];
}

hipError_t reference_energy(double* e0, const double* h, long hs, long hlen, const double* f, long fs, long flen,
                            int o, hipStream_t s) {
  if (o < 1 || hs < 0 || fs < 0) return hipErrorInvalidValue;
  if (bounds_checking() && !(range_ok(e0, 0, 0, 8, "reference energy e0") &&
                             range_ok(h, 0, hlen - 1, 8, "reference energy h") && (o - 1) * hs < hlen &&
                             range_ok(f, 0, flen - 1, 8, "reference energy f") && (o - 1) * fs < flen))
    return hipErrorInvalidValue;
  if (dry_run()) return hipSuccess;
  hipLaunchKernelGGL(reference_energy_kernel, dim3(1), dim3(kThreads), 0, s, e0, h, hs, f, fs, o);
  return hipGetLastError();
}

namespace {
bool cross_ok(const Cross& X) { return X.no >= 1 && X.nv >= 1 && X.h >= 0 && X.h < X.no && X.pa >= 0 && X.pa < X.nv; }
unsigned ew_grid(long total) { return (unsigned)std::max<long>(1, std::min<long>((total + 255) / 256, 8192)); }
}  // namespace

hipError_t cross_gather_rows(double* dst, long ldd, const double* src, long lds, long src_rows, long ncols,
                             const Cross& X, bool zero_diag, hipStream_t s) {
  const long m = X.m();
  if (!cross_ok(X) || src_rows < X.n() || ncols < 1 || ncols > lds || ncols > ldd) return hipErrorInvalidValue;
  if (bounds_checking() && !(range_ok(dst, 0, (m - 1) * ldd + ncols - 1, 8, "cross gather rows dst") &&
                             range_ok(src, 0, (src_rows - 1) * lds + ncols - 1, 8, "cross gather rows src")))
    return hipErrorInvalidValue;
  if (dry_run()) return hipSuccess;
  hipLaunchKernelGGL(cross_gather_rows_kernel, dim3(ew_grid(m * ncols)), dim3(256), 0, s, dst, ldd, src, lds, ncols, X,
                     zero_diag ? 1 : 0);
  return hipGetLastError();
}

hipError_t cross_gather_cols(double* dst, long ldd, const double* src, long lds, long nrows, const Cross& X,
                             const Cross* zero_rows, hipStream_t s) {
  const long m = X.m();
  if (!cross_ok(X) || lds < X.n() || nrows < 1 || ldd < m || (zero_rows && (!cross_ok(*zero_rows) || zero_rows->n() < nrows)))
    return hipErrorInvalidValue;
  if (bounds_checking() && !(range_ok(dst, 0, nrows * ldd - 1, 8, "cross gather cols dst") &&
                             range_ok(src, 0, (nrows - 1) * lds + X.n() - 1, 8, "cross gather cols src")))
    return hipErrorInvalidValue;
  if (dry_run()) return hipSuccess;
  const Cross R = zero_rows ? *zero_rows : X;
  hipLaunchKernelGGL(cross_gather_cols_kernel, dim3(ew_grid(nrows * ldd)), dim3(256), 0, s, dst, ldd, src, lds, nrows, X,
                     R, zero_rows ? 1 : 0);
  return hipGetLastError();
}

hipError_t cross_scatter_add_rows(double* dst, long ldd, long dst_rows, const double* src, long lds, long ncols,
                                  double alpha, const Cross& X, hipStream_t s) {
  const long m = X.m();
  if (!cross_ok(X) || dst_rows < X.n() || ncols < 1 || ncols > ldd || ncols > lds) return hipErrorInvalidValue;
  if (bounds_checking() && !(range_ok(dst, 0, (dst_rows - 1) * ldd + ncols - 1, 8, "cross scatter rows dst") &&
                             range_ok(src, 0, (m - 1) * lds + ncols - 1, 8, "cross scatter rows src")))
    return hipErrorInvalidValue;
  if (dry_run()) return hipSuccess;
  hipLaunchKernelGGL(cross_scatter_add_rows_kernel, dim3(ew_grid(m * ncols)), dim3(256), 0, s, dst, ldd, src, lds, ncols,
                     alpha, X);
  return hipGetLastError();
}

hipError_t cross_scatter_add_cols(double* dst, long ldd, long nrows, const double* src, long lds, double alpha,
                                  const Cross& X, hipStream_t s) {
  const long m = X.m();
  if (!cross_ok(X) || ldd < X.n() || nrows < 1 || lds < m) return hipErrorInvalidValue;
  if (bounds_checking() && !(range_ok(dst, 0, (nrows - 1) * ldd + X.n() - 1, 8, "cross scatter cols dst") &&
                             range_ok(src, 0, (nrows - 1) * lds + m - 1, 8, "cross scatter cols src")))
    return hipErrorInvalidValue;
  if (dry_run()) return hipSuccess;
  hipLaunchKernelGGL(cross_scatter_add_cols_kernel, dim3(ew_grid(nrows * m)), dim3(256), 0, s, dst, ldd, src, lds, nrows,
                     alpha, X);
  return hipGetLastError();
}

hipError_t cross_scatter_add_block(double* dst, long ldd, const double* src, long lds, double alpha, const Cross& X,
                                   hipStream_t s) {
  const long m = X.m();
  if (!cross_ok(X) || ldd < X.n() || lds < m) return hipErrorInvalidValue;
  if (bounds_checking() && !(range_ok(dst, 0, (X.n() - 1) * ldd + X.n() - 1, 8, "cross scatter block dst") &&
                             range_ok(src, 0, (m - 1) * lds + m - 1, 8, "cross scatter block src")))
    return hipErrorInvalidValue;
  if (dry_run()) return hipSuccess;
  hipLaunchKernelGGL(cross_scatter_add_block_kernel, dim3(ew_grid(m * m)), dim3(256), 0, s, dst, ldd, src, lds, alpha, X);
  return hipGetLastError();
}

hipError_t cross_rows_without_corner(double* dst, long ldd, const double* Y, const double* T, const double* K,
                                     long ldk, const Cross& X, hipStream_t s) {
  const long m = X.m(), ld = X.n();
  if (!cross_ok(X) || ldd < ld || ldk < ld) return hipErrorInvalidValue;
  if (bounds_checking() && !(range_ok(dst, 0, (m - 1) * ldd + ld - 1, 8, "cross rows dst") &&
                             range_ok(Y, 0, ld * ld - 1, 8, "cross rows Y") &&
                             range_ok(T, 0, (ld - 1) * ldk + ld - 1, 8, "cross rows T") &&
                             range_ok(K, 0, (ld - 1) * ldk + ld - 1, 8, "cross rows K")))
    return hipErrorInvalidValue;
  if (dry_run()) return hipSuccess;
  hipLaunchKernelGGL(cross_rows_without_corner_kernel, dim3(ew_grid(m * ld)), dim3(256), 0, s, dst, ldd, Y, T, K, ldk, ld,
                     X);
  return hipGetLastError();
}

hipError_t em_cross_column(double* em, const double* tc, long ldt, const double* A, int o, int v, int pa,
                           hipStream_t s) {
  const long total = (long)o * o * v * v, mv = 2L * v - 1;
  if (o < 1 || v < 1 || pa < 0 || pa >= v || ldt < mv) return hipErrorInvalidValue;
  if (bounds_checking() && !(range_ok(em, 0, total - 1, 8, "EM cross column em") &&
                             range_ok(tc, 0, ((long)o * o - 1) * ldt + mv - 1, 8, "EM cross column t") &&
                             range_ok(A, 0, (long)v * v - 1, 8, "EM cross column A")))
    return hipErrorInvalidValue;
  if (dry_run()) return hipSuccess;
  hipLaunchKernelGGL(em_cross_column_kernel, dim3(ew_grid(total)), dim3(256), 0, s, em, tc, ldt, A, o, v, pa);
  return hipGetLastError();
}

hipError_t mixed_doubles(double* dst, const double* src, int o, int v, int h, int pa, hipStream_t s) {
  const long total = (long)o * o * v * v;
  if (o < 1 || v < 1 || h < 0 || h >= o || pa < 0 || pa >= v) return hipErrorInvalidValue;
  if (bounds_checking() && !(range_ok(dst, 0, total - 1, 8, "mixed doubles dst") &&
                             range_ok(src, 0, total - 1, 8, "mixed doubles src")))
    return hipErrorInvalidValue;
  if (dry_run()) return hipSuccess;
  hipLaunchKernelGGL(mixed_doubles_kernel, dim3(ew_grid(total)), dim3(256), 0, s, dst, src, o, v, h, pa);
  return hipGetLastError();
}

hipError_t energy(double* e, double* partial, const double* t1, const double* t2, const double* Lijab,
                  const double* fov, int no, int nv, hipStream_t s) {
  const long total = (long)no * no * nv * nv;
  if (bounds_checking() &&
      !(range_ok(e, 0, 0, 8, "energy e") && range_ok(partial, 0, kRedBlocks - 1, 8, "energy partial") &&
        range_ok(t1, 0, (long)no * nv - 1, 8, "energy t1") && range_ok(t2, 0, total - 1, 8, "energy t2") &&
        range_ok(Lijab, 0, total - 1, 8, "energy L") && range_ok(fov, 0, (long)no * nv - 1, 8, "energy fov")))
    return hipErrorInvalidValue;
  if (dry_run()) return hipSuccess;
  hipLaunchKernelGGL(energy_stage1, dim3(red_blocks(total)), dim3(kThreads), 0, s, partial, t1, t2, Lijab, no, nv, total);
  hipLaunchKernelGGL(energy_stage2, dim3(1), dim3(kThreads), 0, s, e, partial, red_blocks(total), t1, fov, no * nv);
  return hipGetLastError();
}


static hipError_t pack_halves(const PackP& p, long rows, long out_lo, long out_hi, long src_len, hipStream_t s) {
  const long Tv = (long)p.v * (p.v + 1) / 2, nblk = (p.v + 31) / 32, ny = p.mode == kPackT ? nblk * (nblk + 1) / 2 : nblk;
  if (rows <= 0) return hipSuccess;
  if (p.ldo < Tv || rows > 0x7fffffffL || ny > 65535) return hipErrorInvalidValue;
  if (bounds_checking() && !(range_ok(p.plus, out_lo * p.ldo, (out_hi + 1) * p.ldo - 1, 8, "pair packing plus") &&
                             range_ok(p.minus, out_lo * p.ldo, (out_hi + 1) * p.ldo - 1, 8, "pair packing minus") &&
                             chk(p.src, src_len, "pair packing input")))
    return hipErrorInvalidValue;
  if (dry_run()) return hipSuccess;
  hipLaunchKernelGGL(pack_halves_kernel, dim3((unsigned)rows, (unsigned)ny), dim3(kThreads), 0, s, p);
  return hipGetLastError();
}

hipError_t pack_tpm(double* tplus, double* tminus, long ldo, const double* t2, int o, int v, hipStream_t s) {
  const long To = (long)o * (o + 1) / 2;
  return pack_halves({tplus, tminus, ldo, t2, kPackT, o, v, 0}, To, 0, To - 1, (long)o * o * v * v, s);
}

hipError_t pack_vvvv(double* vplus, double* vminus, long ldo, const double* W, int a0, int a1, int v, hipStream_t s) {
  if (a1 <= a0) return hipSuccess;
  auto row = [&](long a) { return a * v - a * (a - 1) / 2; };  // p(a, a)
  return pack_halves({vplus, vminus, ldo, W, kPackV, 1, v, a0}, (long)(a1 - a0) * v, row(a0), row(a1) - 1,
                     (long)(a1 - a0) * v * v * (v - a0), s);
}

hipError_t pack_gwz(double* gplus, double* gminus, long ldo, const double* kcbd, const double* kcld, int o, int v,
                    hipStream_t s) {
  const long ov = (long)o * v, oo = (long)o * o;
  const hipError_t e = pack_halves({gplus, gminus, ldo, kcbd, kPackG, o, v, 0}, ov, 0, ov - 1, ov * v * v, s);
  if (e != hipSuccess) return e;
  return pack_halves({gplus, gminus, ldo, kcld, kPackGo, o, v, 0}, oo, ov, ov + oo - 1, ov * ov, s);
}

hipError_t amp_views(double* Tx, double* U, long ld, double* tplus, double* tminus, long ldo, const double* t2, int o,
                     int v, hipStream_t s) {
  const long To = (long)o * (o + 1) / 2, ov = (long)o * v, nblk = (v + 31) / 32;
  if (ld < ov || nblk * (nblk + 1) / 2 > 65535) return hipErrorInvalidValue;
  if (bounds_checking() && !(chk(Tx, ov * ld, "views Tx") && chk(U, ov * ld, "views U") && chk(t2, ov * ov, "views t2") &&
                             (!tplus || (chk(tplus, To * ldo, "views t+") && chk(tminus, To * ldo, "views t-")))))
    return hipErrorInvalidValue;
  if (dry_run()) return hipSuccess;
  hipLaunchKernelGGL(amp_views_kernel, dim3((unsigned)To, (unsigned)(nblk * (nblk + 1) / 2)), dim3(kThreads), 0, s, Tx, U,
                     ld, tplus, tminus, ldo, t2, o, v);
  return hipGetLastError();
}

hipError_t ring_xz_lowp(int prec, float* xz, long ld, const double* g2, const double* g3, const double* y1, const double* y2,
                        int o, int v, hipStream_t s) {
  const long ov = (long)o * v;
  if (ld < ov || ld % 32) return hipErrorInvalidValue;
  if (bounds_checking() && !(range_ok(xz, 0, 2 * ov * ld - 1, 4, "ring Xc|Zd shadow") && chk(g2, ov * ov, "ring g_kiac") &&
                             chk(g3, ov * ov, "ring g_aikc") && chk(y1, ov * ov, "ring Y1") && chk(y2, ov * ov, "ring Y2")))
    return hipErrorInvalidValue;
  if (dry_run()) return hipSuccess;
  hipLaunchKernelGGL(ring_xz_lowp_kernel, dim3((unsigned)ov), dim3(kThreads), 0, s, Shadow{xz, ld, prec}, g2, g3, y1, y2, o, v);
  return hipGetLastError();
}

hipError_t ring_xz(double* xc, double* zd, long ld, const double* g2, const double* g3, const double* y1,
                   const double* y2, int o, int v, hipStream_t s) {
  const long ov = (long)o * v;
  if (ld < ov) return hipErrorInvalidValue;
  if (bounds_checking() && !(chk(xc, ov * ld, "ring Xc") && chk(zd, ov * ld, "ring Zd") && chk(g2, ov * ov, "ring g_kiac") &&
                             chk(g3, ov * ov, "ring g_aikc") && chk(y1, ov * ov, "ring Y1") && chk(y2, ov * ov, "ring Y2")))
    return hipErrorInvalidValue;
  if (dry_run()) return hipSuccess;
  hipLaunchKernelGGL(ring_xz_kernel, dim3((unsigned)ov), dim3(kThreads), 0, s, xc, zd, ld, g2, g3, y1, y2, o, v);
  return hipGetLastError();
}

hipError_t wz_chi(double* wp, long ldw, double* chip, double* chim, const double* rp, const double* rm, long ldr,
                  const double* g4, const double* foo, const double* t1, int o, int v, hipStream_t s) {
  const long To = (long)o * (o + 1) / 2, ov = (long)o * v, oo = (long)o * o, wzl = ov + oo;
  if (o > 256) return hipErrorInvalidValue;
  if (bounds_checking() &&
      !(chk(wp, (oo - 1) * ldw + ov, "W'") && chk(chip, To * To, "chi+") && chk(chim, To * To, "chi-") &&
        chk(rp, (To - 1) * ldr + wzl, "W/Z +") && chk(rm, (To - 1) * ldr + wzl, "W/Z -") && chk(g4, oo * oo, "g_kilj") &&
        chk(foo, oo, "F''") && chk(t1, ov, "W' t1")))
    return hipErrorInvalidValue;
  if (dry_run()) return hipSuccess;
  hipLaunchKernelGGL(wz_chi_kernel, dim3((unsigned)To, (unsigned)((o + kWzRows - 1) / kWzRows)), dim3(kThreads),
                     2 * kWzRows * o * sizeof(double), s, wp, ldw, chip, chim, rp, rm, ldr, g4, foo, t1, o, v);
  return hipGetLastError();
}

hipError_t unpack_rpm(double* RL, const double* Rplus, const double* Rminus, long ldr, int o, int v, hipStream_t s) {
  const long To = (long)o * (o + 1) / 2, Tv = (long)v * (v + 1) / 2, vv = (long)v * v;
  if (bounds_checking() && !(chk(RL, (long)o * o * vv, "unpack_rpm RL") && chk(Rplus, (To - 1) * ldr + Tv, "unpack_rpm plus") &&
                             chk(Rminus, (To - 1) * ldr + Tv, "unpack_rpm minus")))
    return hipErrorInvalidValue;
  if (dry_run()) return hipSuccess;
  const int nblk = (v + 31) / 32;
  dim3 grid((unsigned)(nblk * (nblk + 1) / 2), (unsigned)To);
  hipLaunchKernelGGL(unpack_rpm_kernel, grid, dim3(kThreads), 0, s, RL, Rplus, Rminus, ldr, o, v, nblk);
  return hipGetLastError();
}

hipError_t pair_minus_rows(int* pm, int v, hipStream_t s) {
  const long Tv = (long)v * (v + 1) / 2;
  if (v <= 0) return hipSuccess;
  if (bounds_checking() && !range_ok(pm, 0, Tv - 1, sizeof(int), "pair rows")) return hipErrorInvalidValue;
  if (dry_run()) return hipSuccess;
  hipLaunchKernelGGL(pair_minus_rows_kernel, dim3((v + kThreads - 1) / kThreads), dim3(kThreads), 0, s, pm, v);
  return hipGetLastError();
}

hipError_t pack_full(double* V, long ldv, const double* W, int a0, int a1, int v, hipStream_t s) {
  const long vv = (long)v * v;
  if (a1 <= a0) return hipSuccess;
  if (ldv < vv) return hipErrorInvalidValue;
  if (bounds_checking() && !(chk(V, vv * ldv, "pack_full out") && chk(W, (long)(a1 - a0) * v * vv, "pack_full in")))
    return hipErrorInvalidValue;
  if (dry_run()) return hipSuccess;
  dim3 grid((unsigned)std::min<long>((vv + kThreads - 1) / kThreads, 64), (a1 - a0) * v);
  hipLaunchKernelGGL(pack_full_kernel, grid, dim3(kThreads), 0, s, V, ldv, W, a0, v);
  return hipGetLastError();
}

int update_partial_blocks() { return kRedBlocks; }

hipError_t diis_update(const UpdateArgs& u, hipStream_t s) {
  // Whether this call stores a pair is decided by the caller; the device state decides the
  // slot, which stored pairs are valid and the coefficients.
  UK p;
  p.t1i = u.t1i ? u.t1i : u.t1;
  p.t2i = u.t2i ? u.t2i : u.t2;
  p.t1 = u.t1;
  p.t2 = u.t2;
  p.r1 = u.r1;
  p.r2 = u.r2;
  p.eps = u.eps;
  p.hist_t = u.hist_t;
  p.hist_e = u.hist_e;
  p.partial = u.partial;
  p.st = u.st;
  p.o = u.no;
  p.v = u.nv;
  p.m = u.m;
  p.start = u.start;
  p.nstat = 3 + kMaxDiis;
  p.len = u.len;
  p.shift = u.shift;
  p.ss = u.nslot > 1 || u.tab ? u.ss : 0;
  p.tab = u.tab;
  const long ov = (long)u.no * u.nv;
  if (u.nslot < 1 || u.nslot > 65535 || (p.ss % 8)) return hipErrorInvalidValue;
  if (bounds_checking()) {
    // every slot the table can name (or every grid row), each checked where it lies
    const long nk = u.tab ? u.tab_max + 1 : u.nslot;
    for (long k = 0; k < (p.ss ? nk : 1); ++k) {
      const long o8 = k * p.ss / 8;  // slot offset in doubles
      auto at = [&](const void* q) { return reinterpret_cast<const char*>(q) + k * p.ss; };
      if (!(range_ok(at(p.t1i), 0, ov - 1, 8, "update t1 in") && range_ok(at(p.t2i), 0, u.len - ov - 1, 8, "update t2 in") &&
            range_ok(at(u.t1), 0, ov - 1, 8, "update t1") && range_ok(at(u.t2), 0, u.len - ov - 1, 8, "update t2") &&
            range_ok(at(u.r1), 0, ov - 1, 8, "update r1") && range_ok(at(u.r2), 0, u.len - ov - 1, 8, "update r2") &&
            range_ok(at(u.e), 0, 0, 8, "update e") && range_ok(at(u.eps), 0, u.no + u.nv - 1, 8, "update eps") &&
            range_ok(at(u.hist_t), 0, (long)u.m * u.len - 1, 8, "update hist_t") &&
            range_ok(at(u.hist_e), 0, (long)u.m * u.len - 1, 8, "update hist_e") &&
            range_ok(at(u.partial), 0, (long)kRedBlocks * (3 + kMaxDiis) - 1, 8, "update partial") &&
            range_ok(at(u.st), 0, 0, sizeof(DiisState), "update state") &&
            range_ok(u.stats, 8 * (p.ss ? k : 0), 8 * (p.ss ? k : 0) + 7, 8, "update stats")))
        return hipErrorInvalidValue;
      (void)o8;
    }
  }
  if (u.m < 1 || u.m > kMaxDiis) return hipErrorInvalidValue;
  if (dry_run()) return hipSuccess;
  const int nblk = red_blocks(u.len);
  hipLaunchKernelGGL(update_stage1, dim3(nblk, u.nslot), dim3(kThreads), 0, s, p);
  hipLaunchKernelGGL(update_stage2, dim3(1, u.nslot), dim3(kThreads), 0, s, u.st, u.partial, nblk, 3 + kMaxDiis,
                     u.m, u.start, u.e, u.stats, u.shift, p.ss, u.tab);
  hipLaunchKernelGGL(update_stage3, dim3(grid_for(u.len), u.nslot), dim3(kThreads), 0, s, u.t1, u.t2, u.hist_t, u.st,
                     u.m, (long)u.no * u.nv, u.len, p.ss, u.tab);
  return hipGetLastError();
}

}  // namespace ascc
