// Strided, batched FP64 GEMM on the CDNA4 matrix cores.
//
// C_z(m,n) = alpha * sum_r sum_k A_{z,r}(m,k) B_{z,r}(k,n) + beta * C_z(m,n)
//
// Every contraction of the residual is expressed through this one kernel family: the
// operands are arbitrary strided 2-D views (a permuted slice of T2 or of an integral block
// is just another pair of strides), tiles are staged through LDS, and each wave64 owns a
// (BM/WM) x (BN/WN) block of the output.
//
// The inner product uses v_mfma_f64_16x16x4_f64.  With register operands the 4x4x4 form issues
// more FP64 work per cycle on gfx950, but fed from LDS the 16x16x4 form wins (3-8% on the
// residual's shapes, measured): a 64 x 64 wave tile needs 16 instructions and 8 LDS reads per
// K-step of 4 instead of 64 and 20.  Lane layout (measured): lane l supplies A(l%16, l/16) and
// B(l/16, l%16); register r of the result holds D(l/16 + 4r, l%16).
//
// K-contiguous operands run on a direct-to-LDS kernel in tiles of 32 x 32 to 192 x 192 and 160 x 128 to 256 x 128 (kDmaCfg),
// tile and K slices from a measured cost; small ones of one stage share a launch (gemm_f64_group).  Strided operands
// run on a register-staged kernel: 128 x 128 (4 waves, two workgroups per CU), 256 x 128 and 192 x 192 (8 waves, one
// per CU) by how well whole rounds of 256 workgroups cover the output, 64 x 64 and 32 x 32 for small outputs or a short
// K, 128 x 128 with split-K when a long K meets too few tiles; all with K staged 16 deep.  The particle-particle ladder has
// its own entry point (gemm_f64_ladder) on the direct-to-LDS kernel: tiles of a height that fits the pair dimension, K
// split where one state leaves CUs idle, and optionally the symmetric/antisymmetric vvvv combinations
// formed at the fragment reads from the stored full (ac|bd).
#include <algorithm>
#include <cmath>
#include <cstdint>

#include "internal.h"

namespace ascc {
namespace {


struct GP {
  int M, N, K;
  const double* A;
  long sam, sak, sa1, sa2, sar;
  const double* B;
  long sbk, sbn, sb1, sb2, sbr;
  double* C;
  long scm, scn, sc1, sc2;
  double alpha, beta;
  int nb2, nred;
  int tiles_m, tiles_n;
  int split, it_per_split;  // split-K: slices of the (nred x K-tile) iteration space
  int per;                  // direct-to-LDS: workgroups of one slice
  double* part;             // partial tiles [split][nb2][M][N] when split > 1, of block z1 at stride sp1
  long sp1;
  int seq;                  // split > 1 without partial tiles: a workgroup runs all slices of its tile,
                            // each added to C in turn (the sums of the partial tiles, in slice order)
  const int* pm;            // pair-combined B (ladder): second row of pair n
  const int* tab1;          // batch level 1: operand block of grid index z1 (nullptr: z1 itself)
  int lower;                // symmetric C: tiles on and below the diagonal only (tiles_m == tiles_n), each
                            // stored at its transposed place too
};

// Workgroup-to-tile map.  Workgroups are dispatched to the 8 XCDs round-robin; each XCD gets
// one contiguous range of tiles, walked in groups of kGroupM M-tiles (M fastest inside a group)
// so that the workgroups resident on one XCD at a time cover a compact block of C and share
// both A and B panels in that XCD's L2.
constexpr int kGroupM = 8;
__device__ __forceinline__ void tile_of(int bid, int tiles_m, int tiles_n, int& tm, int& tn) {
  const int total = tiles_m * tiles_n;
  const int q = total >> 3, rem = total & 7;
  const int x = bid & 7, local = bid >> 3;
  const int t = x * q + min(x, rem) + local;
  const int per = kGroupM * tiles_n;
  const int g = t / per, first = g * kGroupM;
  const int gs = min(tiles_m - first, kGroupM);
  const int r = t - g * per;
  tm = first + r % gs;
  tn = r / gs;
}

// The lower-triangle tiles (tn <= tm) of a symmetric product, each XCD a contiguous range of them
// in row order (consecutive tiles share their A rows).
__device__ __forceinline__ void tile_of_lower(int bid, int tiles, int& tm, int& tn) {
  const int total = tiles * (tiles + 1) / 2;
  const int q = total >> 3, rem = total & 7;
  const int x = bid & 7, local = bid >> 3;
  const int t = x * q + min(x, rem) + local;
  int m = (int)((sqrtf(8.f * (float)t + 1.f) - 1.f) * 0.5f);
  while ((m + 1) * (m + 2) / 2 <= t) ++m;
  while (m * (m + 1) / 2 > t) --m;
  tm = m;
  tn = t - m * (m + 1) / 2;
}

// MINB: workgroups per CU the register budget is sized for.
template <int BM, int BN, int BK, int WM, int WN, int MINB, bool AMF, bool BNF>
__global__ __launch_bounds__(WM* WN * 64, MINB) void gemm_f64_kernel(GP p) {
  constexpr int NT = WM * WN * 64;
  constexpr int TM = BM / WM, TN = BN / WN;
  constexpr int RI = TM / 16, RJ = TN / 16;
  constexpr int LA = BM * BK / NT, LB = BK * BN / NT;
  constexpr int PA = BM + 1, PB = BN + 1;  // +1 double: conflict-free transposing stores
  static_assert(RI >= 1 && RJ >= 1 && LA >= 1 && LB >= 1 && TM % 16 == 0 && TN % 16 == 0, "tile config");
  __shared__ double As[2][BK * PA];
  __shared__ double Bs[2][BK * PB];

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;

  int tm, tn;
  const int ntiles = p.tiles_m * p.tiles_n;
  const int bid = blockIdx.x, z2 = blockIdx.y;
  const int slice = bid / ntiles;
  tile_of(bid - slice * ntiles, p.tiles_m, p.tiles_n, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;
  const int z1 = blockIdx.z;
  const int zs = p.tab1 ? p.tab1[z1] : z1;  // operand block of batch level 1
  const double* Ab = p.A + zs * p.sa1 + z2 * p.sa2;
  const double* Bb = p.B + zs * p.sb1 + z2 * p.sb2;
  double* Cb = p.C + zs * p.sc1 + z2 * p.sc2;

  // acc[i][j]: register r of lane l holds C(16i + l/16 + 4r, 16j + l%16) of the wave's tile
  typedef double d4 __attribute__((ext_vector_type(4)));
  d4 acc[RI][RJ];
#pragma unroll
  for (int i = 0; i < RI; ++i)
#pragma unroll
    for (int j = 0; j < RJ; ++j) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};

  const int nkt = (p.K + BK - 1) / BK;
  const int it_begin = slice * p.it_per_split;
  const int it_end = min(nkt * p.nred, it_begin + p.it_per_split);

  double ra[LA], rb[LB];
  auto load = [&](int it) {
    const int r = it / nkt, k0 = (it % nkt) * BK;
    const double* Ar = Ab + r * p.sar;
    const double* Br = Bb + r * p.sbr;
#pragma unroll
    for (int l = 0; l < LA; ++l) {
      const int e = tid + l * NT;
      const int m = AMF ? (e % BM) : (e / BK);
      const int k = AMF ? (e / BM) : (e % BK);
      const int gm = m0 + m, gk = k0 + k;
      ra[l] = (gm < p.M && gk < p.K) ? Ar[gm * p.sam + gk * p.sak] : 0.0;
    }
#pragma unroll
    for (int l = 0; l < LB; ++l) {
      const int e = tid + l * NT;
      const int n = BNF ? (e % BN) : (e / BK);
      const int k = BNF ? (e / BN) : (e % BK);
      const int gn = n0 + n, gk = k0 + k;
      rb[l] = (gn < p.N && gk < p.K) ? Br[gk * p.sbk + gn * p.sbn] : 0.0;
    }
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int l = 0; l < LA; ++l) {
      const int e = tid + l * NT;
      const int m = AMF ? (e % BM) : (e / BK);
      const int k = AMF ? (e / BM) : (e % BK);
      As[buf][k * PA + m] = ra[l];
    }
#pragma unroll
    for (int l = 0; l < LB; ++l) {
      const int e = tid + l * NT;
      const int n = BNF ? (e % BN) : (e / BK);
      const int k = BNF ? (e / BN) : (e % BK);
      Bs[buf][k * PB + n] = rb[l];
    }
  };

  const int lk = lane >> 4, l16 = lane & 15;
  if (it_begin < it_end) {
    load(it_begin);
    store(0);
  }
  __syncthreads();
  for (int it = it_begin; it < it_end; ++it) {
    const int cur = (it - it_begin) & 1;
    if (it + 1 < it_end) load(it + 1);
    const double* as = As[cur] + lk * PA + wm * TM + l16;
    const double* bs = Bs[cur] + lk * PB + wn * TN + l16;
#pragma unroll
    for (int kk = 0; kk < BK; kk += 4) {
      double a[RI], b[RJ];
#pragma unroll
      for (int i = 0; i < RI; ++i) a[i] = as[kk * PA + 16 * i];
#pragma unroll
      for (int j = 0; j < RJ; ++j) b[j] = bs[kk * PB + 16 * j];
#pragma unroll
      for (int i = 0; i < RI; ++i)
#pragma unroll
        for (int j = 0; j < RJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    if (it + 1 < it_end) store(cur ^ 1);
    __syncthreads();
  }

  // epilogue
#pragma unroll
  for (int i = 0; i < RI; ++i)
#pragma unroll
    for (int j = 0; j < RJ; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int gm = m0 + wm * TM + 16 * i + lk + 4 * r;
        const int gn = n0 + wn * TN + 16 * j + l16;
        if (gm < p.M && gn < p.N) {
          const double v = p.alpha * acc[i][j][r];
          if (p.split > 1) {
            p.part[zs * p.sp1 + (((long)slice * gridDim.y + z2) * p.M + gm) * p.N + gn] = v;
          } else {
            double* c = Cb + gm * p.scm + gn * p.scn;
            *c = (p.beta == 0.0) ? v : v + p.beta * *c;
          }
        }
      }
}

// C_z(m,n) = beta * C_z(m,n) + sum_s part[s][z2][m][n] for block z1 = blockIdx.z.  Each workgroup takes 64 consecutive outputs; its
// four waves sum four contiguous slice ranges in slice order, and the four partial sums are added
// in wave order (a fixed order, so the result is deterministic).
__global__ __launch_bounds__(256) void splitk_reduce(GP p, long outs) {
  __shared__ double red[4][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const long x = blockIdx.x * 64L + lane;
  const int s0 = (int)((long)p.split * w / 4), s1 = (int)((long)p.split * (w + 1) / 4);
  const int zs = p.tab1 ? p.tab1[blockIdx.z] : blockIdx.z;
  double acc = 0.0;
  if (x < outs)
    for (int sl = s0; sl < s1; ++sl) acc += p.part[zs * p.sp1 + sl * outs + x];
  red[w][lane] = acc;
  __syncthreads();
  if (w != 0 || x >= outs) return;
  const double sum = ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
  const long mn = (long)p.M * p.N, r = x % mn;
  const int z2 = (int)(x / mn), gm = r / p.N, gn = r % p.N;
  double* c = p.C + zs * p.sc1 + z2 * p.sc2 + gm * p.scm + gn * p.scn;
  *c = (p.beta == 0.0) ? sum : sum + p.beta * *c;
}

// grid of splitk_reduce for `outs` outputs of each of nb1 blocks
inline dim3 splitk_grid(long outs, int nb1) { return dim3((unsigned)((outs + 63) / 64), 1, (unsigned)nb1); }

// The split-K decision is made for one operand block, so that a block's sums take the same order whatever the batch.
template <int BM, int BN, int BK, int WM, int WN, int MINB>
hipError_t launch_cfg(const GP& p0, bool amf, bool bnf, int nb1, double* ws, long ws_elems, hipStream_t s) {
  GP p = p0;
  p.tiles_m = (p.M + BM - 1) / BM;
  p.tiles_n = (p.N + BN - 1) / BN;
  const long tiles = (long)p.tiles_m * p.tiles_n * p.nb2, outs = (long)p.M * p.N * p.nb2;
  const int nit = ((p.K + BK - 1) / BK) * p.nred;
  p.split = 1;
  p.it_per_split = nit;
  p.part = nullptr;
  if (ws && tiles < 192 && nit >= 16) {
    // slices enough for one full round of resident workgroups (MINB per CU)
    int sp = (int)std::min<long>({(256L * MINB + tiles - 1) / tiles, (long)nit / 8, 256L});
    if (ws_elems > 0) sp = (int)std::min<long>(sp, ws_elems / outs);
    if (sp > 1) {
      p.it_per_split = (nit + sp - 1) / sp;
      p.split = (nit + p.it_per_split - 1) / p.it_per_split;
      p.part = ws;
    }
  }
  const dim3 grid(p.tiles_m * p.tiles_n * p.split, p.nb2, nb1), block(WM * WN * 64);
  if (amf && bnf)
    hipLaunchKernelGGL((gemm_f64_kernel<BM, BN, BK, WM, WN, MINB, true, true>), grid, block, 0, s, p);
  else if (amf)
    hipLaunchKernelGGL((gemm_f64_kernel<BM, BN, BK, WM, WN, MINB, true, false>), grid, block, 0, s, p);
  else if (bnf)
    hipLaunchKernelGGL((gemm_f64_kernel<BM, BN, BK, WM, WN, MINB, false, true>), grid, block, 0, s, p);
  else
    hipLaunchKernelGGL((gemm_f64_kernel<BM, BN, BK, WM, WN, MINB, false, false>), grid, block, 0, s, p);
  if (p.split > 1) hipLaunchKernelGGL(splitk_reduce, splitk_grid(outs, nb1), dim3(256), 0, s, p, outs);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Direct-to-LDS path for K-contiguous operands, A(m,k) = A[m*sam + k] and B(k,n) = B[n*sbn + k]:
// rows go from global memory straight into LDS with buffer_load_dwordx4 ... lds (lane l of an
// instruction writes LDS bytes 16l .. 16l + 15), S stages in flight, one barrier per stage and no
// staging registers.  A stage holds 16 K-values of every tile row: whole 128-byte lines, the 16-byte
// chunk c of row r at slot c ^ (r & 7), which makes the fragment reads conflict-free.  Each fragment
// read returns two K-values and feeds two MFMAs: lane group g = l / 16 supplies K = 2g to the first
// and 2g + 1 to the second, identically for A and B; a stage is read as two 8-deep halves in order.
// Rows past M or N and K-values past K read as zero through the descriptor's range check, so every
// load instruction runs on all lanes and the per-wave vmcnt bookkeeping is exact.
//
// Bound: the FP64 matrix pipe (77.9 TFLOP/s from registers, 64 cycles per 16x16x4 product).  What
// keeps it from that rate is the issue of the stage loads, during which a wave issues no product:
// without them the loop runs at 77 TFLOP/s.  Hence (one round of 256 tiles, K = 8192, before and
// after, TFLOP/s): a scalar descriptor and one offset register per load instead of a 64-bit address
// per lane, and the fragment reads one unit ahead of their products with reads and loads issued
// between products instead of in a block after the barrier: 192x192 69.6 -> 71.9 (four rounds),
// 256x128 69.0 -> 71.0, 224x128 66.3 -> 71, 240x128 64.0 -> 72.6, 208x128 63.2 -> 71.6, 128x128
// 65.4 -> 68.8.  Spreading the loads over the whole stage was slower (66-68).
//
// PM: B is pair-combined, V+- = V[n] +- V[pm[n]], both rows of each pair staged and combined once
// read (two B rows per pair leave room for two stages only).  The second rows of a tile's pairs lie
// anywhere in the stored matrix, past a descriptor's range, and are loaded by address.
typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((address_space(1))) const void gbl_void_t;
__device__ __attribute__((aligned(16))) double kZero16[2];
constexpr int kStageK = 16;  // K-values per stage

// This wave's part of a stage has landed (at most N later loads in flight) and its fragment reads so
// far are in registers, then the same for every wave of the workgroup.  A plain s_barrier: no memory
// fence is needed (and __syncthreads would add one that drains all stages in flight).
template <int N>
__device__ __forceinline__ void wait_stage() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x070 | (N & 15) | ((N >> 4) << 14));  // vmcnt(N) lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Descriptor of `rows` rows of a tile at leading dimension ld (elements).  Every component goes
// through readfirstlane, so the loads take it from scalar registers.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_rsrc(const double* base, int rows, long ld) {
  const uint64_t b = reinterpret_cast<uint64_t>(base);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b), hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
  void* ub = reinterpret_cast<void*>(((uint64_t)hi << 32) | lo);
  return __builtin_amdgcn_make_buffer_rsrc(ub, (short)0, __builtin_amdgcn_readfirstlane((int)(rows * ld * 8)), 0x00020000);
}

// One workgroup's tile (and slices): bid numbers the workgroups of p (tiles x slices), z2 and z1 are its batch
// levels.  RED: nred products of K-values each (K a multiple of 16 if there are several)
// run through one K loop, product r at strides sar, sbr.
template <int BM, int BN, int WM, int WN, int S, bool PM, bool RED>
__device__ __forceinline__ void dma_tile(const GP& p, int bid, int z2, const int z1) {
  typedef double dd2 __attribute__((ext_vector_type(2)));
  typedef double d4 __attribute__((ext_vector_type(4)));
  constexpr int NW = WM * WN;
  constexpr int TM = BM / WM, TN = BN / WN, RI = TM / 16, RJ = TN / 16;
  constexpr int NB = PM ? 2 : 1;
  constexpr int KS = kStageK, CPR = KS / 2, RPI = 64 / CPR;  // 16-byte chunks per staged row, rows per load instruction
  constexpr int IA = BM / RPI, IB = BN / RPI, NI = IA + NB * IB;  // 1 KB load instructions per stage
  constexpr int NPW = (NI + NW - 1) / NW, NPWMIN = NI / NW;        // per wave
  constexpr int ROWS = BM + NB * BN;
  static_assert(TM % 16 == 0 && TN % 16 == 0 && S >= 2 && NPWMIN >= 1, "tile config");
  __shared__ __attribute__((aligned(1024))) double T[S][ROWS * KS];
  auto swz = [](int r) { return r & 7; };  // slot of chunk 0 of row r

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int ntiles = p.tiles_m * p.tiles_n;
  const int slice0 = bid / p.per, slice1 = p.seq ? p.split : slice0 + 1;  // split-K slices of this workgroup
  bid -= slice0 * p.per;
  if constexpr (PM) {
    // Both halves of a tile read the same V rows: they are dispatched back to back to the same
    // XCD (workgroups b and b + 8 share an XCD), so the second one finds them in L2.
    const int x = bid & 7, local = bid >> 3;
    z2 = local & 1;
    bid = ((local >> 1) << 3) | x;
    if (bid >= ntiles) return;  // padding of the grid to whole groups of 8
  }
  int tm, tn;
  if (!PM && p.lower)
    tile_of_lower(bid, p.tiles_m, tm, tn);
  else
    tile_of(bid, p.tiles_m, p.tiles_n, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;
  const int zs = p.tab1 ? p.tab1[z1] : z1;  // operand block of batch level 1
  const double* Ab = p.A + zs * p.sa1 + z2 * p.sa2;
  const double* Bb = p.B + zs * p.sb1 + z2 * p.sb2;
  double* Cb = p.C + zs * p.sc1 + z2 * p.sc2;

  // This lane's source in each load instruction its wave issues: rows of A and of B as byte offsets
  // into a buffer descriptor that covers the tile's rows (rows past M or N lie past its range and
  // read as zero; the advance along K is a scalar offset), pair rows of a pair-combined B, which lie
  // anywhere in the stored matrix, as addresses (kZero16 past N).
  constexpr int J2 = (IA + IB) / NW;  // first instruction of a wave that can hold pair rows
  const double* At = Ab + (long)m0 * p.sam;
  const double* Bt = Bb + (long)n0 * p.sbn;
  const int rows_a = min(BM, p.M - m0), rows_b = min(BN, p.N - n0);
  __amdgpu_buffer_rsrc_t ra, rb;
  const int nk1 = (p.K + KS - 1) / KS;  // stages of one product
  int k_red = 0;                         // RED: stages before the current product
  uint32_t off[NPW];
  const double* src2[PM ? NPW - J2 : 1];
  (void)src2;
  const int ck = 2 * ((lane % CPR) ^ swz(lane / CPR));  // the same chunk in every instruction: it starts a group of 8 rows
  static_assert(RPI == 8, "a load instruction covers one period of the swizzle");
#pragma unroll
  for (int j = 0; j < NPW; ++j) {
    const int g = wave + NW * j;
    const int r = RPI * g + lane / CPR;
    off[j] = g < IA ? (uint32_t)(r * p.sam + ck) * 8 : (uint32_t)((r - BM) * p.sbn + ck) * 8;
    if constexpr (PM) {
      if (j >= J2) {
        const int gn = n0 + r - BM - BN;
        src2[j - J2] = (g >= IA + IB && g < NI && gn < p.N) ? Bb + (long)p.pm[gn] * p.sbn + ck : nullptr;
      }
    }
  }
  auto issue1 = [&](int kt, int st, int j) {  // load instruction j of this wave for stage kt
    const int g = wave + NW * j;
    if (NPW * NW == NI || g < NI) {
      lds_void_t* dst = (lds_void_t*)&T[st][g * 128];
      if (!PM || g < IA + IB) {
        const uint32_t o = off[j];
        __builtin_amdgcn_raw_ptr_buffer_load_lds(g < IA ? ra : rb, dst, 16, o, (kt - k_red) * KS * 8, 0, 0);
      } else {
        const double* x = src2[PM && j >= J2 ? j - J2 : 0];
        const double* a = (x && kt * KS + ck < p.K) ? x + kt * KS : kZero16;
        __builtin_amdgcn_global_load_lds((gbl_void_t*)a, dst, 16, 0, 0);
      }
    }
  };
  // before the loads of stage kt (the slice ends before kend): the descriptors, of its product where several are
  // summed; with an empty range past the slice (its loads fetch nothing and write zeros nobody reads), so that
  // the K loop runs without branches and counts the same loads in every stage; on the last stage of an uneven
  // K (no stage follows it) chunks past K read as zero
  int kend = 0;
  auto begin_stage = [&](int kt) {
    const int r = RED && p.nred > 1 ? kt / nk1 : 0;
    if (RED) k_red = r * nk1;
    ra = tile_rsrc(At + r * p.sar, kt < kend ? rows_a : 0, p.sam);
    rb = tile_rsrc(Bt + r * p.sbr, kt < kend ? rows_b : 0, p.sbn);
    if (!(RED && p.nred > 1) && kt < kend && (kt + 1) * KS > p.K && kt * KS + ck >= p.K) {
#pragma unroll
      for (int j = 0; j < NPW; ++j) off[j] = 0x80000000u;  // past the range of every descriptor
    }
  };
  auto issue = [&](int kt, int st) {
    begin_stage(kt);
#pragma unroll
    for (int j = 0; j < NPW; ++j) issue1(kt, st, j);
  };

  d4 acc[RI][RJ];
  const bool minus = PM && z2 == 1;
  const int l16 = lane & 15, q = lane >> 4;
  // Fragments are read one unit ahead of their MFMAs: a unit is one group of A fragment rows of one
  // 8-deep half of a stage (units of a stage: half 0 group 0, half 0 group 1, half 1 group 0, ...).
  constexpr int G = (RI > 8) ? 2 : 1, GI = (RI + G - 1) / G, U = G * (KS / 8);
  static_assert(U % 2 == 0, "the unit parity must be static");
  dd2 fa[2][GI], fb[2][RJ];
  dd2 fw[PM ? RJ : 1];  // pair-combined B: second rows, combined when the unit starts
  (void)fw;
  // read k of unit u's fragments: first the B fragments (unit 0 of a half: they serve all its groups),
  // then the A fragments
  constexpr int RB = NB * RJ, NR = RB + GI;
  auto read1 = [&](const double* Ts, int u, int k) {
    const int kk = u / G, g = u % G;
    if (k < RB) {
      if (g != 0) return;
      const int r = BM + (k / RJ) * BN + wn * TN + 16 * (k % RJ) + l16;
      const dd2 x = *reinterpret_cast<const dd2*>(Ts + r * KS + 2 * ((q + 4 * kk) ^ swz(r)));
      if (k < RJ)
        fb[kk & 1][k] = x;
      else
        fw[k % RJ] = x;
    } else if (g * GI + k - RB < RI) {
      const int r = wm * TM + 16 * (g * GI + k - RB) + l16;
      fa[u & 1][k - RB] = *reinterpret_cast<const dd2*>(Ts + r * KS + 2 * ((q + 4 * kk) ^ swz(r)));
    }
  };
  auto combine = [&](int u) {  // pair-combined B of unit u's half
    if constexpr (PM) {
      const int kk = u / G;
      if (u % G != 0) return;
#pragma unroll
      for (int j = 0; j < RJ; ++j) fb[kk & 1][j] = minus ? fb[kk & 1][j] - fw[j] : fb[kk & 1][j] + fw[j];
    }
  };
  for (int slice = slice0; slice < slice1; ++slice) {
#pragma unroll
    for (int i = 0; i < RI; ++i)
#pragma unroll
      for (int j = 0; j < RJ; ++j) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};
    // stages [kt0, kt0 + nkt) of this slice
    const int kt0 = slice * p.it_per_split;
    const int nkt = min(RED ? nk1 * p.nred : nk1, kt0 + p.it_per_split) - kt0;
    if (slice != slice0) wait_stage<0>();  // every wave is done with the slots of the slice before
    kend = kt0 + nkt;
#pragma unroll
    for (int st = 0; st < S; ++st) issue(kt0 + st, st);
    wait_stage<(S - 1) * NPWMIN>();
#pragma unroll
    for (int k = 0; k < NR; ++k) read1(T[0], 0, k);
    combine(0);
    for (int kt = 0, st = 0; kt < nkt; ++kt) {  // kt counts stages of this slice, st is its slot
      const int st1 = st + 1 == S ? 0 : st + 1;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int kk = u / G, g = u % G;
        const bool last = u + 1 == U;
        const double* Tn = T[last ? st1 : st];
        if (last) {
          // stage kt + 1 has landed once no more than the later stages' loads of this wave are in
          // flight; past the barrier it has for every wave, and every wave holds the last fragments of
          // stage kt in registers, so its slot is refilled from here on
          wait_stage<(S - 2) * NPWMIN>();
          begin_stage(kt0 + kt + S);
        }
        // the unit's products, with a fragment read or a refill load issued behind most of them
        constexpr int NM = 2 * GI * RJ, LS = NR + 2 * NPW <= NM ? 2 : 1;
        constexpr int ML = S == 2 ? 0 : LS == 2 ? NR : NM - NPW;  // two stages: the refill is due soonest
        static_assert(NR <= NM && NPW <= NM, "one read and one load per product at most");
#pragma unroll
        for (int m = 0; m < NM; ++m) {
          const int h = m / (GI * RJ), i = (m / RJ) % GI, j = m % RJ;
          if (g * GI + i < RI)
            acc[g * GI + i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[u & 1][i][h], fb[kk & 1][j][h],
                                                                      acc[g * GI + i][j], 0, 0, 0);
          if (m < NR) read1(Tn, last ? 0 : u + 1, m);
          if (last && m >= ML && m < ML + LS * NPW && (m - ML) % LS == 0) issue1(kt0 + kt + S, st, (m - ML) / LS);
          __builtin_amdgcn_sched_barrier(0);
        }
        combine(last ? 0 : u + 1);
      }
      st = st1;
    }
    __builtin_amdgcn_s_waitcnt(0xF70);  // no load may reach LDS after the workgroup has left
    // the output addresses are formed here: hoisted out of the slice loop they would hold registers
    // across it (a lane index hidden from the optimiser keeps them in place)
    int ol = lane;
    asm volatile("" : "+v"(ol));
    const int oq = ol >> 4, o16 = ol & 15;
#pragma unroll
    for (int i = 0; i < RI; ++i)
#pragma unroll
      for (int j = 0; j < RJ; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int gm = m0 + wm * TM + 16 * i + oq + 4 * r;
          const int gn = n0 + wn * TN + 16 * j + o16;
          if (gm < p.M && gn < p.N) {
            const double v = p.alpha * acc[i][j][r];
            if (p.part) {
              p.part[zs * p.sp1 + (((long)slice * p.nb2 + z2) * p.M + gm) * p.N + gn] = v;
            } else {
              double* c = Cb + (long)gm * p.scm + (long)gn * p.scn;
              *c = (slice != slice0) ? *c + v : (p.beta == 0.0) ? v : v + p.beta * *c;
              if (!PM && BM == BN && p.lower && tm != tn) Cb[(long)gn * p.scm + (long)gm * p.scn] = v;
            }
          }
        }
  }
}

template <int BM, int BN, int WM, int WN, int S, bool PM, bool RED>
__global__ __launch_bounds__(WM* WN * 64, 1) void gemm_f64_dma_kernel(GP p) {
  dma_tile<BM, BN, WM, WN, S, PM, RED>(p, blockIdx.x, blockIdx.y, blockIdx.z);
}

// Several independent contractions as one launch: problem i takes the workgroups start[i] .. start[i + 1] - 1
// (batch level 2, slices and tiles), every problem the same batch level 1 in grid.z.
constexpr int kMaxGroup = 8;
struct GroupP {
  int n, start[kMaxGroup + 1];
  GP p[kMaxGroup];
};
template <int BT, int W>
__global__ __launch_bounds__(W* W * 64, 1) void gemm_f64_group_kernel(GroupP g) {
  int i = 0;
  while (i + 1 < g.n && (int)blockIdx.x >= g.start[i + 1]) ++i;
  const GP& p = g.p[i];
  const int local = (int)blockIdx.x - g.start[i], per2 = p.per * p.split, z2 = local / per2;
  dma_tile<BT, BT, W, W, 3, false, true>(p, local - z2 * per2, z2, blockIdx.z);
}

// The partial tiles of a group: job i sums slices of outs values per operand block (as splitk_reduce) and takes
// the workgroups start[i] .. start[i + 1] - 1.  The slices of several problems with one output follow one another.
struct GroupR {
  int n, start[kMaxGroup + 1];
  int slices[kMaxGroup];
  GP p[kMaxGroup];
};
__global__ __launch_bounds__(256) void group_reduce_kernel(GroupR g) {
  __shared__ double red[4][64];
  int i = 0;
  while (i + 1 < g.n && (int)blockIdx.x >= g.start[i + 1]) ++i;
  const GP& p = g.p[i];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, z1 = blockIdx.z, ns = g.slices[i];
  const int zs = p.tab1 ? p.tab1[z1] : z1;
  const long mn = (long)p.M * p.N, outs = mn * p.nb2, x = ((int)blockIdx.x - g.start[i]) * 64L + lane;
  const int s0 = (int)((long)ns * w / 4), s1 = (int)((long)ns * (w + 1) / 4);
  double acc = 0.0;
  if (x < outs)
    for (int sl = s0; sl < s1; ++sl) acc += p.part[zs * p.sp1 + sl * outs + x];
  red[w][lane] = acc;
  __syncthreads();
  if (w != 0 || x >= outs) return;
  const double sum = ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
  const int z2 = (int)(x / mn), gm = (int)(x % mn / p.N), gn = (int)(x % p.N);
  double* c = p.C + zs * p.sc1 + z2 * p.sc2 + gm * p.scm + gn * p.scn;
  *c = (p.beta == 0.0) ? sum : sum + p.beta * *c;
}

// K-contiguous operands with 16-byte aligned rows and an even K (the loads move K-value pairs; whole
// stages when several products are summed); the rows of a tile do not overlap and lie within the 2 GiB range of a
// buffer descriptor (32 rows here, taller tiles are checked where they are chosen).
bool dma_eligible(const GP& p) {
  auto al = [](const void* x) { return (reinterpret_cast<uintptr_t>(x) & 15) == 0; };
  auto near = [&](long ld) { return ld >= p.K && ld < (1L << 23); };
  return near(p.sam) && near(p.sbn) && p.sak == 1 && p.sbk == 1 && p.K % (p.nred > 1 ? kStageK : 2) == 0 &&
         p.sar % 2 == 0 && p.sbr % 2 == 0 && p.sam % 2 == 0 && p.sbn % 2 == 0 &&
         p.sa1 % 2 == 0 && p.sa2 % 2 == 0 && p.sb1 % 2 == 0 && p.sb2 % 2 == 0 && al(p.A) && al(p.B);
}

// C_z(m, n) = sum_s part[s][z2][m][n], in slice order (the order of a workgroup that runs all slices).
__global__ __launch_bounds__(256) void ordered_reduce(GP p) {
  const int n = blockIdx.x * 256 + threadIdx.x, zl = blockIdx.z;
  if (n >= p.N) return;
  const long mn = (long)p.M * p.N;
  const int z1 = zl / p.nb2, z2 = zl % p.nb2;
  const int zs = p.tab1 ? p.tab1[z1] : z1;
  double* C = p.C + zs * p.sc1 + z2 * p.sc2;
  for (int m = blockIdx.y; m < p.M; m += gridDim.y) {
    const double* x = p.part + zs * p.sp1 + z2 * mn + (long)m * p.N + n;
    double sum = *x;
    for (int sl = 1; sl < p.split; ++sl) sum += x[sl * p.nb2 * mn];
    C[m * p.scm + n * p.scn] = sum;
  }
}

// split > 1: K cut into `split` slices whose partial tiles go to ws, then summed in a fixed order by
// splitk_reduce; ordered: beta is 0 and they are summed in slice order, by ordered_reduce or, without
// ws, by the workgroups themselves.
template <int BM, int BN, int WM, int WN, int S, bool PM = false, bool RED = false>
hipError_t launch_dma(GP p, int nb1, int split, double* ws, bool ordered, hipStream_t s) {
  p.tiles_m = (p.M + BM - 1) / BM;
  p.tiles_n = (p.N + BN - 1) / BN;
  const int nkt = (p.K + kStageK - 1) / kStageK * (RED ? p.nred : 1);
  if (!RED && p.nred != 1) return hipErrorInvalidValue;
  p.it_per_split = (nkt + split - 1) / split;
  p.split = (nkt + p.it_per_split - 1) / p.it_per_split;
  p.part = p.split > 1 ? ws : nullptr;
  p.seq = ordered && p.split > 1 && !ws;
  const int tiles = p.lower ? p.tiles_m * (p.tiles_m + 1) / 2 : p.tiles_m * p.tiles_n;
  if (p.lower && (p.split > 1 || PM || BM != BN || p.tiles_m != p.tiles_n)) return hipErrorInvalidValue;
  if (p.split > 1 && !ws && !ordered) return hipErrorInvalidValue;
  p.per = PM ? 2 * ((tiles + 7) / 8 * 8) : tiles;  // PM: both halves in grid.x, padded to groups of 8
  dim3 grid(p.per * (p.seq ? 1 : p.split), PM ? 1 : p.nb2, nb1);
  hipLaunchKernelGGL((gemm_f64_dma_kernel<BM, BN, WM, WN, S, PM, RED>), grid, dim3(WM * WN * 64), 0, s, p);
  const long outs = (long)p.M * p.N * p.nb2;
  if (p.part && ordered)
    hipLaunchKernelGGL(ordered_reduce, dim3((p.N + 255) / 256, std::min(p.M, 65535), p.nb2 * nb1), dim3(256), 0, s, p);
  else if (p.part)
    hipLaunchKernelGGL(splitk_reduce, splitk_grid(outs, nb1), dim3(256), 0, s, p, outs);
  return hipGetLastError();
}

// Direct-to-LDS launch of a general contraction: the tile and split-K count with the least estimated time,
//   6 us + (stages of a slice + 2) x max(tiles per CU x t, t1) + 5 us and the partial tiles' traffic if split
// with t the time of one stage of one tile on a busy CU and t1 its latency alone (us, measured: sweeps of tile
// and split over 100..3600 squared outputs; the choice stays within 10 % of the best of them).  Where the
// outputs are few, small tiles with K split keep every CU busy: 576 x 576 x 240 75 -> 17 us, 390 x 1521 x 1522 70 -> 55 us
// against 192- to 256-row tiles; in between, the height that fills a round: 1521 x 1521 x 1522 twice takes 254 us in 96 x 96
// tiles (two rounds), 235 in 160 x 128 ones (240 workgroups).
// The choice is made for one operand block, so that a block's sums never depend on the batch.
struct DmaCfg {
  int bm, bn;
  double t, t1;
};
constexpr DmaCfg kDmaCfg[] = {{192, 192, 4.06, 4.06}, {256, 128, 3.68, 3.68}, {224, 128, 3.25, 3.25}, {128, 128, 1.88, 1.88},
                              {96, 96, 1.27, 1.41},   {64, 64, 0.57, 0.69},   {32, 32, 0.185, 0.50},  {192, 128, 2.80, 2.80},
                              {160, 128, 2.36, 2.36}};
struct DmaPlan {
  int cfg, split;
  double us;
};
long dma_tiles(const GP& p, int bm, int bn) {  // of one operand block
  const long tm = (p.M + bm - 1) / bm, tn = (p.N + bn - 1) / bn;
  return p.lower ? tm * (tm + 1) / 2 : tm * tn;
}
inline long dma_stages(const GP& p) { return (long)((p.K + kStageK - 1) / kStageK) * p.nred; }
DmaPlan plan_dma(const GP& p0, bool ws, long ws_elems) {
  const bool red = p0.nred > 1;
  const long outs = (long)p0.M * p0.N * p0.nb2;
  const long nkt = dma_stages(p0);
  DmaPlan best{-1, 1, 0.0};
  for (int c = 0; c < (int)(sizeof kDmaCfg / sizeof kDmaCfg[0]); ++c) {
    const DmaCfg& f = kDmaCfg[c];
    if ((red && f.bm > 64) || (p0.lower && f.bm != f.bn)) continue;
    if (std::max(p0.sam, p0.sbn) * f.bm >= 1L << 28) continue;  // rows past a descriptor's 2 GiB
    const long tiles = dma_tiles(p0, f.bm, f.bn) * p0.nb2;
    for (long sp = 1; sp <= 256; sp += sp < 4 ? 1 : sp / 2) {
      if (sp > 1 && (p0.lower || !ws || tiles * sp > 1536 || nkt < 4 * sp || sp * outs > ws_elems)) break;
      const double per = std::max((double)((tiles * sp + 255) / 256) * f.t, f.t1);
      const double us = 6.0 + (double)((nkt + sp - 1) / sp + 2) * per + (sp > 1 ? 5.0 + (double)((sp + 1) * outs) * 2.7e-6 : 0.0);
      if (best.cfg < 0 || us < best.us) best = {c, (int)sp, us};
    }
  }
  return best;
}

hipError_t launch_dma_auto(const GP& p, int nb1, double* ws, long ws_elems, hipStream_t s) {
  const bool red = p.nred > 1;
  const DmaPlan pl = plan_dma(p, ws != nullptr, ws_elems);
  switch (pl.cfg) {
    case 0: return launch_dma<192, 192, 2, 4, 3>(p, nb1, pl.split, ws, false, s);
    case 1: return launch_dma<256, 128, 4, 2, 3>(p, nb1, pl.split, ws, false, s);
    case 7: return launch_dma<192, 128, 2, 4, 3>(p, nb1, pl.split, ws, false, s);
    case 8: return launch_dma<160, 128, 2, 4, 3>(p, nb1, pl.split, ws, false, s);
    case 2: return launch_dma<224, 128, 2, 4, 3>(p, nb1, pl.split, ws, false, s);
    case 3: return launch_dma<128, 128, 2, 4, 3>(p, nb1, pl.split, ws, false, s);
    case 4: return launch_dma<96, 96, 2, 2, 3>(p, nb1, pl.split, ws, false, s);
    case 5:
      return red ? launch_dma<64, 64, 2, 2, 3, false, true>(p, nb1, pl.split, ws, false, s)
                 : launch_dma<64, 64, 2, 2, 3>(p, nb1, pl.split, ws, false, s);
    default:
      return red ? launch_dma<32, 32, 1, 1, 3, false, true>(p, nb1, pl.split, ws, false, s)
                 : launch_dma<32, 32, 1, 1, 3>(p, nb1, pl.split, ws, false, s);
  }
}

// Ladder tiles: BM x 128, the eight waves side by side (BM / 16 fragment rows each).  Three stages, or
// two where a stage with both rows of each pair leaves no room for a third.
template <int BM, bool PM>
hipError_t launch_ladder(const GP& p, int nb1, int split, double* ws, hipStream_t s) {
  constexpr int S = 3L * (BM + (PM ? 256 : 128)) * kStageK * 8 <= 160 * 1024 ? 3 : 2;
  return launch_dma<BM, 128, 1, 8, S, PM>(p, nb1, split, ws, true, s);
}

// Tile height and split-K count of a ladder of M rows (N columns, both halves).  Time of a launch: whole
// rounds of 256 workgroups x stages of a slice (and about 6 to fill and drain) x (rows + 24 of B staging).
// The split is that of one state's rows Mdec and Ndec columns, so a state's sums do not depend on how many states
// are stacked or which columns are computed together, and takes only counts whose partial tiles fit the scratch; it pays where one state leaves CUs
// idle: its partial tiles cost a pass over the outputs.  Against the best of all heights and splits, us:
// o8 v72 48 / 45, o10 v90 108 / 104, o12 v108 252 / 243, o15 v135 881 / 853, o20 v180 4266 / 4259.
struct LadderPlan {
  int bm, split;
};
LadderPlan ladder_plan(long M, long Mdec, long N, long Ndec, long K, long ws_elems) {
  constexpr int kBM[] = {32, 48, 64, 80, 96, 112, 128, 144, 160, 176, 192, 208, 224, 240, 256};
  const long nkt = (K + kStageK - 1) / kStageK;
  auto cost = [&](int bm, int sp) {
    const double wg = (double)((Mdec + bm - 1) / bm * ((Ndec + 127) / 128) * 2 * sp);
    const double stages = (double)((nkt + sp - 1) / sp + 6) * (bm + 24) * std::ceil(wg / 256);
    return stages + (sp > 1 ? 400.0 + 2.0e-5 * (double)(sp + 1) * (double)Mdec * (double)Ndec * 2 : 0.0);
  };
  LadderPlan best{256, 1};
  double least = -1;
  for (int bm : kBM)
    for (int sp = 1; sp <= 8 && (sp == 1 || (K > kLadderWhole && nkt >= 16 * sp && 2 * sp * Mdec * Ndec <= ws_elems)); ++sp) {
      const double c = cost(bm, sp);
      if (least < 0 || c < least) {
        least = c;
        best = {bm, sp};
      }
    }
  if (M != Mdec || N != Ndec) {
    least = -1;
    for (int bm : kBM) {
      const double c = std::ceil((double)((M + bm - 1) / bm * ((N + 127) / 128) * 2) / 256) * (bm + 24);
      if (least < 0 || c < least) {
        least = c;
        best.bm = bm;
      }
    }
  }
  return best;
}

template <bool PM>
hipError_t launch_ladder_plan(const GP& p, int nb1, LadderPlan pl, double* ws, hipStream_t s) {
  switch (pl.bm) {
    case 32:  // (with pairs, more loads than products in a unit: the next height)
      return launch_ladder<(PM ? 48 : 32), PM>(p, nb1, pl.split, ws, s);
    case 48: return launch_ladder<48, PM>(p, nb1, pl.split, ws, s);
    case 64: return launch_ladder<64, PM>(p, nb1, pl.split, ws, s);
    case 80: return launch_ladder<80, PM>(p, nb1, pl.split, ws, s);
    case 96: return launch_ladder<96, PM>(p, nb1, pl.split, ws, s);
    case 112: return launch_ladder<112, PM>(p, nb1, pl.split, ws, s);
    case 128: return launch_ladder<128, PM>(p, nb1, pl.split, ws, s);
    case 144: return launch_ladder<144, PM>(p, nb1, pl.split, ws, s);
    case 160: return launch_ladder<160, PM>(p, nb1, pl.split, ws, s);
    case 176: return launch_ladder<176, PM>(p, nb1, pl.split, ws, s);
    case 192: return launch_ladder<192, PM>(p, nb1, pl.split, ws, s);
    case 208: return launch_ladder<208, PM>(p, nb1, pl.split, ws, s);
    case 224: return launch_ladder<224, PM>(p, nb1, pl.split, ws, s);
    case 240: return launch_ladder<240, PM>(p, nb1, pl.split, ws, s);
    default: return launch_ladder<256, PM>(p, nb1, pl.split, ws, s);
  }
}

}  // namespace

Gemm gemm_rm(int M, int N, int K, double alpha, const double* A, long lda, bool ta, const double* B, long ldb,
             bool tb, double beta, double* C, long ldc) {
  Gemm g;
  g.M = M;
  g.N = N;
  g.K = K;
  g.alpha = alpha;
  g.beta = beta;
  g.A = A;
  if (!ta) {
    g.sam = lda;
    g.sak = 1;
  } else {
    g.sam = 1;
    g.sak = lda;
  }
  g.B = B;
  if (!tb) {
    g.sbk = ldb;
    g.sbn = 1;
  } else {
    g.sbk = 1;
    g.sbn = ldb;
  }
  g.C = C;
  g.scm = ldc;
  g.scn = 1;
  return g;
}

// Lowest and highest element offset of an affine index expression sum_t i_t * s_t, 0 <= i_t < e_t.
static void affine_range(const long* ext, const long* str, int n, long& lo, long& hi) {
  lo = hi = 0;
  for (int t = 0; t < n; ++t) {
    const long d = (ext[t] - 1) * str[t];
    if (d < 0) lo += d; else hi += d;
  }
}

static bool gemm_in_bounds(const Gemm& g) {
  long lo, hi;
  const long e1 = g.tab1 ? g.tab1_max + 1L : g.nb1;  // batch level 1 spans the table's entries
  const long ea[5] = {g.M, g.K, e1, g.nb2, g.nred}, sa[5] = {g.sam, g.sak, g.sa1, g.sa2, g.sar};
  affine_range(ea, sa, 5, lo, hi);
  if (!range_ok(g.A, lo, hi, sizeof(double), "gemm A")) return false;
  const long eb[5] = {g.K, g.N, e1, g.nb2, g.nred}, sb[5] = {g.sbk, g.sbn, g.sb1, g.sb2, g.sbr};
  affine_range(eb, sb, 5, lo, hi);
  if (!range_ok(g.B, lo, hi, sizeof(double), "gemm B")) return false;
  const long ec[4] = {g.M, g.N, e1, g.nb2}, sc[4] = {g.scm, g.scn, g.sc1, g.sc2};
  affine_range(ec, sc, 4, lo, hi);
  if (!range_ok(g.C, lo, hi, sizeof(double), "gemm C")) return false;
  return !g.ws || range_ok(g.ws, 0, (e1 - 1) * g.ws1 + g.ws_elems - 1, sizeof(double), "gemm split-K scratch");
}

static GP to_gp(const Gemm& g) {
  GP p{};
  p.M = g.M;
  p.N = g.N;
  p.K = g.K;
  p.A = g.A;
  p.sam = g.sam;
  p.sak = g.sak;
  p.sa1 = g.sa1;
  p.sa2 = g.sa2;
  p.sar = g.sar;
  p.B = g.B;
  p.sbk = g.sbk;
  p.sbn = g.sbn;
  p.sb1 = g.sb1;
  p.sb2 = g.sb2;
  p.sbr = g.sbr;
  p.C = g.C;
  p.scm = g.scm;
  p.scn = g.scn;
  p.sc1 = g.sc1;
  p.sc2 = g.sc2;
  p.alpha = g.alpha;
  p.beta = g.beta;
  p.nb2 = g.nb2;
  p.nred = g.nred;
  p.sp1 = g.ws1;
  p.seq = 0;
  p.pm = nullptr;
  p.tab1 = g.tab1;
  p.lower = 0;
  p.lower = g.lower && g.M == g.N && g.beta == 0.0 && g.nred == 1 && dma_eligible(p);
  return p;
}

hipError_t gemm_f64(const Gemm& g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0 || g.nb1 <= 0 || g.nb2 <= 0) return hipSuccess;
  if (bounds_checking() && !gemm_in_bounds(g)) return hipErrorInvalidValue;
  if (dry_run()) return hipSuccess;
  if (g.nb1 > 65535 || g.nb2 > 65535) return hipErrorInvalidValue;
  if (g.K <= 0 || g.nred <= 0) return hipErrorInvalidValue;  // callers never pass an empty contraction
  if (g.ws && g.nb1 > 1 && g.ws1 < g.ws_elems) return hipErrorInvalidValue;  // the blocks' scratches overlap
  GP p = to_gp(g);
  if (dma_eligible(p)) return launch_dma_auto(p, g.nb1, g.fixed ? nullptr : g.ws, g.ws_elems, s);
  // Global-load order: an operand whose m (n) stride is 1 is read m-fast (n-fast).
  const bool amf = (g.sam == 1 && g.sak != 1);
  const bool bnf = (g.sbn == 1) || (g.sbk != 1);
  const long tiles128 = (long)((g.M + 127) / 128) * ((g.N + 127) / 128) * g.nb2;
  if (g.M >= 96 && g.N >= 96 && tiles128 >= 256 && (long)g.K * g.nred > 512) {
    // Large outputs over more than a few stages (a short K is bound by the output's traffic, which two 64 x 64 workgroups per
    // CU keep in flight: -= t1^T W' over 400 outputs of 180 x 180 and K = 20 94 -> 62 us, hole-hole pairs o20 v180 111 -> 102):
    // among 128x128 (4 waves), 256x128 and 192x192 (8 waves) take the least
    // estimated time = whole rounds of 256 tiles x tile area / sustained rate (measured on full
    // rounds: 59.5, 60, 61.5 TFLOP/s), which prices both the padding of M and N and the partly
    // filled last round.
    auto est = [&](int bm, int bn, double rate) {
      const long t = (long)((g.M + bm - 1) / bm) * ((g.N + bn - 1) / bn) * g.nb2;
      return (double)((t + 255) / 256) * bm * bn / rate;
    };
    const double e128 = est(128, 128, 59.5), e256 = est(256, 128, 60.0), e192 = est(192, 192, 61.5);
    if (e192 < e128 && e192 <= e256) return launch_cfg<192, 192, 16, 2, 4, 1>(p, amf, bnf, g.nb1, nullptr, 0, s);
    if (e256 < e128) return launch_cfg<256, 128, 16, 4, 2, 1>(p, amf, bnf, g.nb1, nullptr, 0, s);
    return launch_cfg<128, 128, 16, 2, 2, 2>(p, amf, bnf, g.nb1, g.ws, g.ws_elems, s);
  }
  // a long K lets split-K make up for too few 128 x 128 tiles (down to 16 of them: split into up
  // to 32 slices, a long K still leaves each slice enough iterations to hide its reduction)
  const bool long_k = g.ws && (long)g.K * g.nred >= 2048 && tiles128 >= 16;
  if (g.M >= 96 && g.N >= 96 && long_k) {
    return launch_cfg<128, 128, 16, 2, 2, 2>(p, amf, bnf, g.nb1, g.ws, g.ws_elems, s);
  }
  const long tiles64 = (long)((g.M + 63) / 64) * ((g.N + 63) / 64) * g.nb2;
  if (g.M >= 48 && g.N >= 48 && tiles64 >= 128)
    return launch_cfg<64, 64, 16, 2, 2, 2>(p, amf, bnf, g.nb1, g.ws, g.ws_elems, s);
  // a narrow output over a long K: 64 x 64 tiles of four waves, split along K, keep more of each
  // CU busy (and more loads in flight) than single-wave 32 x 32 tiles
  if (g.ws && g.M >= 16 && g.N >= 16 && (long)g.K * g.nred >= 2048 && tiles64 < 192)
    return launch_cfg<64, 64, 16, 2, 2, 2>(p, amf, bnf, g.nb1, g.ws, g.ws_elems, s);
  return launch_cfg<32, 32, 16, 1, 1, 3>(p, amf, bnf, g.nb1, g.ws, g.ws_elems, s);
}

bool gemm_f64_small(const Gemm& g) {
  const GP p = to_gp(g);
  if (g.M <= 0 || g.N <= 0 || g.K <= 0 || !dma_eligible(p)) return false;
  const DmaPlan pl = plan_dma(p, g.ws && !g.fixed, g.ws_elems);
  return pl.cfg >= 0 && kDmaCfg[pl.cfg].bm <= 64;
}

hipError_t gemm_f64_group(const Gemm* all, int count, hipStream_t s) {
  // Estimated as plan_dma estimates a launch, with one launch overhead and one reduction for all; a unit is one
  // slice of one tile, sliced to about the same number of stages in every problem.  Contractions that take
  // larger tiles go by themselves (those that share an output stay together).
  const int nb1 = count > 0 ? all[0].nb1 : 1;
  Gemm gs[kMaxGroup];
  GP p[kMaxGroup];
  int n = 0;
  auto joins_group = [&](const Gemm& g) {
    return !dry_run() && g.nb1 == nb1 && nb1 <= 65535 && g.ws && g.ws == all[0].ws && g.ws1 == all[0].ws1 && gemm_f64_small(g);
  };
  bool together = true;
  for (int i = 0; i < count; ++i)
    if (all[i].acc >= 0) together = together && joins_group(all[i]);
  double solo = 0.0;
  for (int i = 0; i < count; ++i) {
    const Gemm& g = all[i];
    if (n == kMaxGroup || (g.acc >= 0 ? !together : !joins_group(g))) {
      const hipError_t e = gemm_f64(g, s);
      if (e != hipSuccess) return e;
      continue;
    }
    if (bounds_checking() && !gemm_in_bounds(g)) return hipErrorInvalidValue;
    gs[n] = g;
    p[n++] = to_gp(g);
    if (!g.fixed) solo += plan_dma(p[n - 1], true, g.ws_elems).us;
  }
  const bool group = n > 1;
  struct Choice {
    int bt = 0;
    long unit = 0;
    double us = 0.0;
  } best;
  auto split_of = [&](int i, long unit) {
    const long nkt = dma_stages(p[i]);
    if (gs[i].fixed || p[i].lower) return 1L;
    return std::max(1L, std::min({(nkt + unit - 1) / unit, nkt / 4, 64L}));
  };
  for (int bt : {64, 32}) {
    if (!group) break;
    const double t = bt == 64 ? 0.58 : 0.185, t1 = bt == 64 ? 0.70 : 0.50;
    for (long unit : {8L, 12L, 16L, 24L, 32L, 48L, 64L, 128L, 1L << 40}) {
      double work = 0.0, units = 0.0, parts = 0.0;
      long longest = 0;
      for (int i = 0; i < n; ++i) {
        if (gs[i].fixed) continue;  // the choice does not depend on these
        const long sp = split_of(i, unit), st = (dma_stages(p[i]) + sp - 1) / sp, tl = dma_tiles(p[i], bt, bt) * p[i].nb2;
        work += (double)(tl * sp) * (double)(st + 2);
        units += (double)(tl * sp);
        longest = std::max(longest, st);
        if (sp > 1 || gs[i].acc >= 0) parts += (double)sp * p[i].M * p[i].N * p[i].nb2;
      }
      if (parts > (double)gs[0].ws_elems) continue;
      const double on = std::min(std::ceil(units / 256.0), bt == 64 ? 3.0 : 6.0);  // units sharing a CU
      const double us = 6.0 + std::max(work * t / 256.0, (double)(longest + 2) * std::max(t1, on * t)) +
                        (parts > 0 ? 5.0 + parts * 2.7e-6 : 0.0);
      if (best.bt == 0 || us < best.us) best = {bt, unit, us};
    }
  }
  if (!group || best.bt == 0 || best.us >= solo) {
    for (int i = 0; i < n; ++i) {
      const hipError_t e = gemm_f64(gs[i], s);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  // slices, scratch and launch order (problems that share an output: their slices follow one another)
  if (nb1 > 1 && gs[0].ws1 < gs[0].ws_elems) return hipErrorInvalidValue;  // the blocks' scratches overlap
  GroupP gp{};
  GroupR gr{};
  double* ws = gs[0].ws;
  gp.n = n;
  for (int i = 0; i < n; ++i) {
    GP& q = p[i];
    const long sp = split_of(i, best.unit), nkt = dma_stages(q);
    q.tiles_m = (q.M + best.bt - 1) / best.bt;
    q.tiles_n = (q.N + best.bt - 1) / best.bt;
    q.per = (int)dma_tiles(q, best.bt, best.bt);
    q.it_per_split = (int)((nkt + sp - 1) / sp);
    q.split = (int)((nkt + q.it_per_split - 1) / q.it_per_split);
    const bool joins = gs[i].acc >= 0 && i > 0 && gs[i - 1].acc == gs[i].acc;  // adds to the job before it
    if (q.split > 1 || gs[i].acc >= 0) {
      q.part = ws;
      ws += (long)q.split * q.M * q.N * q.nb2;
      if (joins) {
        gr.slices[gr.n - 1] += q.split;
      } else {
        gr.p[gr.n] = q;
        gr.slices[gr.n] = q.split;
        gr.start[gr.n + 1] = gr.start[gr.n] + (int)(((long)q.M * q.N * q.nb2 + 63) / 64);
        ++gr.n;
      }
    }
    gp.p[i] = q;
    gp.start[i + 1] = gp.start[i] + q.per * q.split * q.nb2;
  }
  const dim3 grid((unsigned)gp.start[n], 1, (unsigned)nb1);
  if (best.bt == 64)
    hipLaunchKernelGGL((gemm_f64_group_kernel<64, 2>), grid, dim3(256), 0, s, gp);
  else
    hipLaunchKernelGGL((gemm_f64_group_kernel<32, 1>), grid, dim3(64), 0, s, gp);
  if (gr.n)
    hipLaunchKernelGGL(group_reduce_kernel, dim3((unsigned)gr.start[gr.n], 1, (unsigned)nb1), dim3(256), 0, s, gr);
  return hipGetLastError();
}

hipError_t gemm_f64_ladder(const Ladder& L, hipStream_t s) {
  if (L.M <= 0 || L.N <= 0) return hipSuccess;
  const bool pmode = L.pm != nullptr;
  const LadderBatch& lb = L.lb;
  if (L.K <= 0 || lb.n > 65535 || L.Mdec <= 0 || L.M % L.Mdec || L.Ndec < L.N) return hipErrorInvalidValue;
  if (bounds_checking()) {
    const long e1 = lb.tab ? lb.tab_max : lb.n - 1;  // last operand block of batch level 1
    const long vlast = pmode ? (L.vrows - 1) * L.ldv + L.K - 1 : L.sv2 + (L.N - 1L) * L.ldv + L.K - 1;
    if (!(range_ok(L.A, 0, e1 * lb.sa + L.sa2 + (L.M - 1L) * L.lda + L.K - 1, sizeof(double), "ladder A") &&
          range_ok(L.C, 0, e1 * lb.sc + L.sc2 + (L.M - 1L) * L.ldc + L.N - 1, sizeof(double), "ladder C") &&
          range_ok(L.V, 0, e1 * lb.sv + vlast, sizeof(double), "ladder V") &&
          (!pmode || range_ok(L.pm, 0, L.N - 1, sizeof(int), "ladder pair rows")) &&
          (!L.ws || range_ok(L.ws, 0, e1 * lb.sw + L.ws_elems - 1, sizeof(double), "ladder split-K scratch"))))
      return hipErrorInvalidValue;
  }
  if (dry_run()) return hipSuccess;
  GP p{};
  p.M = L.M;
  p.N = L.N;
  p.K = L.K;
  p.A = L.A;
  p.sam = L.lda;
  p.sak = 1;
  p.sa2 = L.sa2;
  p.B = L.V;
  p.sbk = 1;
  p.sbn = L.ldv;
  p.sb2 = pmode ? 0 : L.sv2;
  p.C = L.C;
  p.scm = L.ldc;
  p.scn = 1;
  p.sc2 = L.sc2;
  p.alpha = 1.0;
  p.beta = 0.0;
  p.nb2 = 2;
  p.nred = 1;
  p.pm = L.pm;
  p.sa1 = lb.sa;
  p.sb1 = lb.sv;
  p.sc1 = lb.sc;
  p.sp1 = lb.sw;
  p.tab1 = lb.tab;
  if (L.ws && lb.n > 1 && lb.sw < L.ws_elems) return hipErrorInvalidValue;  // the blocks' scratches overlap
  if (!dma_eligible(p) || std::max(p.sam, p.sbn) >= 1L << 20) return hipErrorInvalidValue;  // rows laid out for this kernel
  const LadderPlan pl = ladder_plan(L.M, L.Mdec, L.N, L.Ndec, L.K, L.ws ? L.ws_elems : 0);
  // one slice after another where the partial tiles do not fit the scratch or the blocks fill the chip: the same sums
  double* ws = (long)pl.split * L.M * L.N * 2 * lb.n <= L.ws_elems ? L.ws : nullptr;
  return pmode ? launch_ladder_plan<true>(p, lb.n, pl, ws, s) : launch_ladder_plan<false>(p, lb.n, pl, ws, s);
}

}  // namespace ascc
