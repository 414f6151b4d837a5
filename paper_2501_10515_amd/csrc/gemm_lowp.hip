// Low-precision contractions on the matrix cores, FP64 result:
//
//   C_z(m,n) = alpha * sum_k A_z[m][k] B_z[n][k] + beta * C_z(m,n)
//
// A and B are low-precision shadows of FP64 operands (row-major, K contiguous, zero-padded rows,
// rounded to nearest even by the conversion kernels); C is FP64 with general strides.  Two
// arithmetic policies:
//
//   FP32   : v_mfma_f32_16x16x4_f32 on FP32 shadows.
//   BF16X3 : the shadows are two bf16 planes, x = hi + lo with hi = RNE_bf16(x),
//            lo = RNE_bf16(x - hi); v_mfma_f32_16x16x32_bf16 or 32x32x16 forms
//            lo*hi + hi*lo + hi*hi (the lo*lo term, relative size 2^-16, is dropped).
//
// Both accumulate in FP32 inside a K chunk and add each chunk's partial sum into the FP64 C tile
// (which the workgroup owns for the whole K range), so accumulation across chunks is FP64.
//
// MFMA lane layouts (gfx950, measured): f32 16x16x4 -- lane l supplies A(l%16, l/16) and
// B(l/16, l%16); bf16 16x16x32 -- lane l supplies A(l%16, 8(l/16)+j) and B(8(l/16)+j, l%16),
// j = 0..7; both return register r of lane l as C(4(l/16)+r, l%16); bf16 32x32x16 -- lane l
// supplies A(l%32, 8(l/32)+j) and B(8(l/32)+j, l%32) and returns register q as
// C(8(q/4) + 4(l/32) + q%4, l%32).
#include <algorithm>
#include <cstdint>
#include <type_traits>
#include <utility>

#include "internal.h"
#include "lowp.h"

namespace ascc {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));

// The 32 x 32 split-BF16x3 fragments add a later FP32 chunk's partial sum into the FP64 result with
// a non-returning FP64 atomic add, performed at L2: the old value is never read into registers
// (2.8 % of the o40 v360 split-BF16x3 step; the 16 x 16 output layout, four rows per
// instruction, made the same change twice as slow there, so it keeps the load-add-store).  Each
// element has one writer (the lane that owns it) and its chunks arrive in order, so the sums are
// those of a load-add-store; the stores of a chunk are waited for before any add follows.
__device__ __forceinline__ void add_to(double* p, double v) { unsafeAtomicAdd(p, v); }

// Workgroup to tile, walked in groups of 8 M-tiles (M fastest inside a group): the workgroups resident on one
// XCD at a time cover a compact block of C and share A and B slices in its L2.
__device__ __forceinline__ void tile_of_grouped(int bid, int tiles_m, int tiles_n, int& tm, int& tn) {
  constexpr int GM = 8;
  const int total = tiles_m * tiles_n;
  const int q = total >> 3, rem = total & 7;
  const int x = bid & 7, local = bid >> 3;
  const int t = x * q + min(x, rem) + local;
  const int per = GM * tiles_n;
  const int g = t / per, first = g * GM;
  const int gs = min(tiles_m - first, GM);
  const int r = t - g * per;
  tm = first + r % gs;
  tn = r / gs;
}

// Row-padded conversions: out row r holds in row r (cols values) then zeros up to ldo.
__global__ __launch_bounds__(256) void cvt_f32_2d_kernel(float* __restrict__ out, long ldo, const double* __restrict__ in,
                                                         long ldi, long rows, long cols) {
  const long total = rows * ldo;
  for (long x = blockIdx.x * 256L + threadIdx.x; x < total; x += (long)gridDim.x * 256) {
    const long r = x / ldo, c = x - r * ldo;
    out[x] = (c < cols) ? (float)in[r * ldi + c] : 0.f;
  }
}

// Interleaved split of a row-padded matrix: row r of the output holds, for each K-block kb of 32,
// hi[32] at r * 2ldo + 64kb and lo[32] right after it (ldo a multiple of 32; padding zeroed).
__global__ __launch_bounds__(256) void split_bf16_2d_kernel(unsigned short* __restrict__ out, long ldo,
                                                            const double* __restrict__ in, long ldi, long rows,
                                                            long cols) {
  const long total = rows * ldo;
  for (long x = blockIdx.x * 256L + threadIdx.x; x < total; x += (long)gridDim.x * 256) {
    const long r = x / ldo, c = x - r * ldo;
    unsigned short h = 0, l = 0;
    if (c < cols) {
      const double d = in[r * ldi + c];
      h = bf16_rne((float)d);
      l = bf16_rne((float)(d - (double)bf16_to_f(h)));
    }
    const long o = r * 2 * ldo + (c >> 5) * 64 + (c & 31);
    out[o] = h;
    out[o + 32] = l;
  }
}

// The same two conversions, eight columns per thread (one K-block of 32 never splits a group):
// 16-byte loads of the FP64 source (16-byte aligned rows: `in` aligned, ldi even) and 16-byte
// stores, one index division per eight elements; each element is converted exactly as above.
__global__ __launch_bounds__(256) void cvt_f32_2d_v8_kernel(float* __restrict__ out, long ldo,
                                                            const double* __restrict__ in, long ldi, long rows,
                                                            long cols) {
  const long per = ldo >> 3, total = rows * per;
  for (long x = blockIdx.x * 256L + threadIdx.x; x < total; x += (long)gridDim.x * 256) {
    const long r = x / per, c = (x - r * per) << 3;
    const double* src = in + r * ldi + c;
    double d[8];
    if (c + 8 <= cols) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const double2 v = reinterpret_cast<const double2*>(src)[j];
        d[2 * j] = v.x;
        d[2 * j + 1] = v.y;
      }
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) d[j] = (c + j < cols) ? src[j] : 0.0;
    }
    float4* o = reinterpret_cast<float4*>(out + r * ldo + c);
    o[0] = make_float4((float)d[0], (float)d[1], (float)d[2], (float)d[3]);
    o[1] = make_float4((float)d[4], (float)d[5], (float)d[6], (float)d[7]);
  }
}

__global__ __launch_bounds__(256) void split_bf16_2d_v8_kernel(unsigned short* __restrict__ out, long ldo,
                                                               const double* __restrict__ in, long ldi, long rows,
                                                               long cols) {
  const long per = ldo >> 3, total = rows * per;
  for (long x = blockIdx.x * 256L + threadIdx.x; x < total; x += (long)gridDim.x * 256) {
    const long r = x / per, c = (x - r * per) << 3;
    const double* src = in + r * ldi + c;
    double d[8];
    if (c + 8 <= cols) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const double2 v = reinterpret_cast<const double2*>(src)[j];
        d[2 * j] = v.x;
        d[2 * j + 1] = v.y;
      }
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) d[j] = (c + j < cols) ? src[j] : 0.0;
    }
    uint32_t hw[4], lw[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const unsigned short h0 = bf16_rne((float)d[2 * j]), h1 = bf16_rne((float)d[2 * j + 1]);
      const unsigned short l0 = bf16_rne((float)(d[2 * j] - (double)bf16_to_f(h0)));
      const unsigned short l1 = bf16_rne((float)(d[2 * j + 1] - (double)bf16_to_f(h1)));
      hw[j] = (uint32_t)h0 | ((uint32_t)h1 << 16);
      lw[j] = (uint32_t)l0 | ((uint32_t)l1 << 16);
    }
    unsigned short* o = out + r * 2 * ldo + (c >> 5) * 64 + (c & 31);
    *reinterpret_cast<uint4*>(o) = make_uint4(hw[0], hw[1], hw[2], hw[3]);
    *reinterpret_cast<uint4*>(o + 32) = make_uint4(lw[0], lw[1], lw[2], lw[3]);
  }
}

// Transposing low-precision shadow: out row r (< rows) holds in[c][r] for c < cols, zero padding
// up to ldo (a multiple of 32), laid out as to_lowp_2d lays out its rows.  32 x 32 tiles through
// LDS, so both the reads (along r) and the writes (along c) are coalesced.
template <bool BF>
__global__ __launch_bounds__(256) void lowp_t_kernel(void* __restrict__ outp, long ldo, const double* __restrict__ in,
                                                     long ldi, long rows, long cols) {
  __shared__ double tile[32][33];
  const long r0 = (long)blockIdx.x * 32, c0 = (long)blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int cy = ty + 8 * k;
    const long r = r0 + tx, c = c0 + cy;
    tile[cy][tx] = (r < rows && c < cols) ? in[c * ldi + r] : 0.0;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int ry = ty + 8 * k;
    const long r = r0 + ry, c = c0 + tx;
    if (r >= rows) continue;
    const double d = tile[tx][ry];
    if (BF) {
      unsigned short* out = reinterpret_cast<unsigned short*>(outp);
      const unsigned short h = bf16_rne((float)d);
      const long o = r * 2 * ldo + (c >> 5) * 64 + (c & 31);
      out[o] = h;
      out[o + 32] = bf16_rne((float)(d - (double)bf16_to_f(h)));
    } else {
      reinterpret_cast<float*>(outp)[r * ldo + c] = (float)d;
    }
  }
}

// Low-precision shadow of [(kc|bd) | (kc|ld)]: row m = k*v + b (from kcbd[k][c][b][d]) or ov + k*o + l
// (from kcld[k][c][l][d]), column c*v + d, zero padding up to ldo, laid out as to_lowp_2d lays out its rows.
template <bool BF>
__global__ __launch_bounds__(256) void lowp_gwz_kernel(void* __restrict__ outp, long ldo,
                                                       const double* __restrict__ kcbd,
                                                       const double* __restrict__ kcld, int o, int v) {
  const long ov = (long)o * v, vv = (long)v * v, m = blockIdx.x;
  const double* src = m < ov ? kcbd + m / v * v * vv + m % v * v : kcld + (m - ov) / o * v * ov + (m - ov) % o * v;
  const long sc = m < ov ? vv : ov;
  for (long x = blockIdx.y * 256L + threadIdx.x; x < ldo; x += (long)gridDim.y * 256) {
    const long c = x / v;
    const double d = x < vv ? src[c * sc + (x - c * v)] : 0.0;
    if (BF) {
      unsigned short* out = reinterpret_cast<unsigned short*>(outp);
      const unsigned short h = bf16_rne((float)d);
      const long q = m * 2 * ldo + (x >> 5) * 64 + (x & 31);
      out[q] = h;
      out[q + 32] = bf16_rne((float)(d - (double)bf16_to_f(h)));
    } else {
      reinterpret_cast<float*>(outp)[m * ldo + x] = (float)d;
    }
  }
}

// Low-precision shadow of the vvvv halves formed from the full (ac|bd) matrix in pair order (rows
// at stride ldv): row r = h*Tv + n (h = 0: +, 1: -), column k < Tv, zero padding up to ldo; in FP64
// x = V[n][k] +- V[pm[n]][k], then rounded and laid out as to_lowp_2d does (FP32, or interleaved bf16).
template <bool BF>
__global__ __launch_bounds__(256) void lowp_pm_kernel(unsigned short* __restrict__ bo, float* __restrict__ out,
                                                      long ldo, const double* __restrict__ V, long ldv,
                                                      const int* __restrict__ pm, long Tv) {
  const long total = 2 * Tv * ldo;
  for (long x = blockIdx.x * 256L + threadIdx.x; x < total; x += (long)gridDim.x * 256) {
    const long r = x / ldo, c = x - r * ldo;
    double d = 0.0;
    if (c < Tv) {
      const bool minus = r >= Tv;
      const long n = minus ? r - Tv : r;
      const double u = V[n * ldv + c], w = V[(long)pm[n] * ldv + c];
      d = minus ? u - w : u + w;
    }
    if (BF) {
      const unsigned short h = bf16_rne((float)d);
      const long o = r * 2 * ldo + (c >> 5) * 64 + (c & 31);
      bo[o] = h;
      bo[o + 32] = bf16_rne((float)(d - (double)bf16_to_f(h)));
    } else {
      out[x] = (float)d;
    }
  }
}



// ---------------------------------------------------------------------------------------
// The contraction kernel.  A stage is 32 K-values of every tile row, which both policies keep in one 128-byte line
// (32 FP32 values, or the hi 32 | lo 32 of a split).  The lines go straight from memory to LDS (eight rows per
// 1 KB load; lane l of a load writes LDS bytes 16l .. 16l + 15), S stages deep, with one barrier per stage; rows past M or N
// read as zero through the range of the tile's buffer descriptor, and the K padding of a shadow is zero.  The 16-byte chunk c
// of row r sits at slot c ^ ((r >> 1) & 7): sixteen rows of one chunk cover all 64 LDS banks.
//
// Fragments are read one unit ahead of their MFMAs (a unit is one group of A fragments of one K step), reads and refill
// loads spread between the MFMAs.  Of the three arithmetic orders below every tile shape gives the same bits,
// so the tile is free to follow the sizes and the batch.
//
//   kF32Seq  v_mfma_f32_16x16x4_f32, MFMA t of 16 K-values takes K = 4t .. 4t + 3
//   kF32Str  the same, MFMA t takes K = t, t + 4, t + 8, t + 12 (one 16-byte read per fragment)
//   kBf16    v_mfma_f32_16x16x32_bf16: lo hi, hi lo, hi hi of 32 K-values
//   kBf32    v_mfma_f32_32x32x16_bf16: the same, of 16 K-values
enum { kF32Seq, kF32Str, kBf16, kBf32 };
constexpr int kChunk = 256;  // stages per FP32 accumulation chunk (even: a chunk starts with the first fragment buffers)

struct LP {
  int M, N, K;
  const char* A;  // strides of the operands in bytes
  long lda, sa2;
  const char* B;
  long ldb, sb2;
  double* C;
  long scm, scn, sc2;
  double alpha, beta;
  int tiles_m, tiles_n;
  int ktps;     // stages per split-K slice (blockIdx.z); the whole K when not split
  long cslice;  // C offset between slices (partial tiles of a split launch), 0 otherwise
  // batch: blockIdx.y = z1 * nb + z; z1 selects operand block tab1[z1] (or z1) at strides
  // sa1, sb1, sc1
  int nb;
  const int* tab1;
  long sa1, sb1, sc1;
};

// Buffer descriptor of a wave-uniform range (base, bytes), built from scalar registers: every
// component goes through readfirstlane, so the buffer loads take it straight from SGPRs (left to
// itself the compiler kept parts of it in VGPRs and wrapped each load in a waterfall loop).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t uniform_rsrc(const void* base, uint32_t bytes) {
  const uintptr_t b = reinterpret_cast<uintptr_t>(base);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
  void* ub = reinterpret_cast<void*>(((uintptr_t)hi << 32) | lo);
  return __builtin_amdgcn_make_buffer_rsrc(ub, (short)0, __builtin_amdgcn_readfirstlane((int)bytes), 0x00020000);
}

// Waits until at most N loads of this wave are in flight and its LDS reads have arrived, then for the other waves.
template <int N>
__device__ __forceinline__ void wait_stage() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x070 | (N & 15) | ((N >> 4) << 14));  // vmcnt(N) lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

typedef __attribute__((address_space(3))) void lds_void_t;

// f(0), ..., f(N - 1) with compile-time arguments (the K loop's body is beyond what the unroller takes on).
#define INLINE __attribute__((always_inline))
template <int I>
using Int = std::integral_constant<int, I>;
template <class Fn, int... I>
__device__ __forceinline__ void unrolled_(Fn f, std::integer_sequence<int, I...>) {
  (f(Int<I>()), ...);
}
// of n things spread over the slots 0 .. slots - 1: those before slot x
constexpr int upto(int x, int n, int slots) { return x <= 0 ? 0 : x >= slots ? n : x * n / slots; }
template <int N, class Fn>
__device__ __forceinline__ void unrolled(Fn f) {
  unrolled_(f, std::make_integer_sequence<int, N>());
}

template <int KIND, int BM, int BN, int WM, int WN, int S>
__global__ __launch_bounds__(WM* WN * 64, 1) void gemm_lowp_kernel(LP p) {
  constexpr bool BF = KIND == kBf16 || KIND == kBf32;
  constexpr int F = KIND == kBf32 ? 32 : 16;       // fragment edge
  constexpr int NH = KIND == kBf16 ? 1 : 2;        // K steps of a stage
  constexpr int NP = BF ? 2 : 1, NA = F * F / 64;  // 16-byte parts of a fragment, accumulator values of a lane
  constexpr int NR1 = KIND == kF32Seq ? 4 : NP;    // LDS reads of a fragment
  constexpr int NT1 = BF ? 3 : 4;                  // MFMAs of a fragment pair and K step
  constexpr int NW = WM * WN, TM = BM / WM, TN = BN / WN, RI = TM / F, RJ = TN / F;
  constexpr int IA = BM / 8, NI = (BM + BN) / 8, NPW = (NI + NW - 1) / NW, NPWMIN = NI / NW;  // 1 KB loads of a stage
  constexpr int G = RI * NP >= 8 ? 2 : 1, GI = (RI + G - 1) / G, U = G * NH;  // groups of A fragments, units of a stage
  static_assert(BM % (F * WM) == 0 && BN % (F * WN) == 0 && S >= 2 && NPWMIN >= 1, "tile config");
  typedef float fa_t __attribute__((ext_vector_type(NA)));
  __shared__ __attribute__((aligned(1024))) char T[S][(BM + BN) * 128];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  int tm, tn;
  tile_of_grouped(blockIdx.x, p.tiles_m, p.tiles_n, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;
  const int z = blockIdx.y % p.nb, z1 = blockIdx.y / p.nb;
  const int zs = __builtin_amdgcn_readfirstlane(p.tab1 ? p.tab1[z1] : z1);  // uniform: scalar buffer descriptors
  const char* At = p.A + z * p.sa2 + zs * p.sa1 + (long)m0 * p.lda;
  const char* Bt = p.B + z * p.sb2 + zs * p.sb1 + (long)n0 * p.ldb;
  double* Cb = p.C + z * p.sc2 + zs * p.sc1 + blockIdx.z * p.cslice;
  const uint32_t bytes_a = (uint32_t)(min(BM, p.M - m0) * p.lda), bytes_b = (uint32_t)(min(BN, p.N - n0) * p.ldb);
  uint32_t off[NPW];  // this lane's source in each load its wave issues: byte offset in the tile's rows
#pragma unroll
  for (int j = 0; j < NPW; ++j) {
    const int g = wave + NW * j, r = 8 * g + (lane >> 3);
    const uint32_t ck = 16 * ((lane & 7) ^ ((r >> 1) & 7));
    off[j] = (g < IA ? (uint32_t)(r * p.lda) : (uint32_t)((r - BM) * p.ldb)) + ck;
  }
  // stages [kt0, kt0 + nkt) of this slice; loads past the last one have an empty range (they fetch nothing and write
  // zeros nobody reads), so the K loop runs without branches and counts the same loads in every stage
  const int kt0 = blockIdx.z * p.ktps, nkt = min((p.K + 31) / 32, kt0 + p.ktps) - kt0;
  __amdgpu_buffer_rsrc_t ra, rb;
  auto begin_stage = [&](int kt) INLINE {
    ra = uniform_rsrc(At, kt < nkt ? bytes_a : 0u);
    rb = uniform_rsrc(Bt, kt < nkt ? bytes_b : 0u);
  };
  auto issue1 = [&](int kt, int st, int j) INLINE {  // load j of this wave for stage kt
    const int g = wave + NW * j;
    if (NPW * NW == NI || g < NI) {
      const uint32_t o = off[j];
      __builtin_amdgcn_raw_ptr_buffer_load_lds(g < IA ? ra : rb, (lds_void_t*)&T[st][g * 1024], 16, o, (kt0 + kt) * 128, 0, 0);
    }
  };

  fa_t acc[RI][RJ];
#pragma unroll
  for (int i = 0; i < RI; ++i)
#pragma unroll
    for (int j = 0; j < RJ; ++j)
#pragma unroll
      for (int q = 0; q < NA; ++q) acc[i][j][q] = 0.f;
  auto flush = [&](bool first, bool last) INLINE {
    // addresses formed here, from a lane index the compiler cannot see through: hoisted out of the
    // K loop they would hold registers across it (and spill)
    int ln = lane;
    asm volatile("" : "+v"(ln));
#pragma unroll
    for (int i = 0; i < RI; ++i)
#pragma unroll
      for (int j = 0; j < RJ; ++j)
#pragma unroll
        for (int q = 0; q < NA; ++q) {
          const int fm = F == 32 ? 8 * (q >> 2) + 4 * (ln >> 5) + (q & 3) : 4 * (ln >> 4) + q;
          const int gm = m0 + wm * TM + i * F + fm, gn = n0 + wn * TN + j * F + (ln & (F - 1));
          if (gm < p.M && gn < p.N) {
            double* c = Cb + (long)gm * p.scm + (long)gn * p.scn;
            const double v = p.alpha * (double)acc[i][j][q];
            if (first)
              *c = (p.beta == 0.0) ? v : v + p.beta * *c;
            else if (F == 32)
              add_to(c, v);
            else
              *c += v;
          }
          acc[i][j][q] = 0.f;
        }
    if (!last) __builtin_amdgcn_s_waitcnt(0xF70);  // the stores have reached L2
  };

  // fragments: rows of the lane at l128 within a fragment's rows, chunk c at (c ^ sw) * 16
  const int fr = lane & (F - 1), fg = lane / F, sw = (fr >> 1) & 7;
  f4 fa[2][GI][NP], fb[2][RJ][NP];
  auto read_part = [&](const char* row, int h, int k, f4* x) INLINE {
    if constexpr (KIND == kF32Seq) {
      x[0][k] = *reinterpret_cast<const float*>(row + (((4 * h + k) ^ sw) << 4) + 4 * fg);
    } else {
      const int c = KIND == kF32Str ? 4 * h + fg : KIND == kBf16 ? 4 * k + fg : 4 * k + 2 * h + fg;
      x[k] = *reinterpret_cast<const f4*>(row + ((c ^ sw) << 4));
    }
  };
  // read k of the fragments of unit u (buffers of parity P): the B fragments of a new K step, then the A fragments
  constexpr int RB = RJ * NR1, NR = RB + GI * NR1;
  auto read1 = [&](const char* Ts, auto P, auto u, auto kc) INLINE {
    constexpr int h = u() / G, g = u() % G, k = kc();
    if constexpr (k < RB) {
      if constexpr (g == 0)
        read_part(Ts + (BM + wn * TN + (k / NR1) * F + fr) * 128, h, k % NR1, fb[(P() * NH + h) & 1][k / NR1]);
    } else {
      constexpr int i = (k - RB) / NR1;
      if constexpr (g * GI + i < RI)
        read_part(Ts + (wm * TM + (g * GI + i) * F + fr) * 128, h, k % NR1, fa[(P() * U + u()) & 1][i]);
    }
  };
  auto product = [&](const f4* a, const f4* b, int t, fa_t& c) INLINE {
    if constexpr (BF) {
      const bf8 x = __builtin_bit_cast(bf8, a[t == 0 ? 1 : 0]), y = __builtin_bit_cast(bf8, b[t == 1 ? 1 : 0]);
      if constexpr (F == 32)
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, y, c, 0, 0, 0);
      else
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, y, c, 0, 0, 0);
    } else {
      c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[0][t], b[0][t], c, 0, 0, 0);
    }
  };

  unrolled<S>([&](auto st) INLINE {
    begin_stage(st());
    unrolled<NPW>([&](auto j) INLINE { issue1(st(), st(), j()); });
  });
  wait_stage<(S - 1) * NPWMIN>();
  unrolled<NR>([&](auto k) INLINE { read1(T[0], Int<0>(), Int<0>(), k); });
  // one stage, in slot st; P: parity of the fragment buffers its first unit uses (those of the next stage's follow)
  auto stage = [&](int kt, int st, int st1, auto P) INLINE {
    unrolled<U>([&](auto uc) INLINE {
      constexpr int u = uc(), h = u / G, g = u % G, NM = NT1 * GI * RJ;
      constexpr int MR = BF ? NM : (NM + 1) / 2, ML = BF ? 0 : MR;  // reads go in slots 0 .. MR - 1, loads from ML on
      constexpr bool last = u + 1 == U;
      const char* Tn = T[last ? st1 : st];
      if constexpr (last) {
        // stage kt + 1 has landed once no more than the later stages' loads of this wave are in flight; past the
        // barrier it has for every wave, and every wave holds the last fragments of stage kt in registers,
        // so its slot is refilled from here on
        wait_stage<(S - 2) * NPWMIN>();
        begin_stage(kt + S);
      }
      unrolled<NM>([&](auto mc) INLINE {
        constexpr int m = mc(), t = m / (GI * RJ), i = m / RJ % GI, j = m % RJ;
        if constexpr (g * GI + i < RI)
          product(fa[(P() * U + u) & 1][i], fb[(P() * NH + h) & 1][j], t, acc[g * GI + i][j]);
        constexpr int k0 = upto(m, NR, MR), k1 = upto(m + 1, NR, MR);
        constexpr int l0 = upto(m - ML, NPW, NM - ML), l1 = upto(m + 1 - ML, NPW, NM - ML);
        unrolled<k1 - k0>([&](auto k) INLINE {
          read1(Tn, Int<last ? P() ^ 1 : P()>(), Int<last ? 0 : u + 1>(), Int<k0 + k()>());
        });
        if constexpr (last) unrolled<l1 - l0>([&](auto k) INLINE { issue1(kt + S, st, l0 + k()); });
        __builtin_amdgcn_sched_barrier(0);
      });
    });
  };
  for (int kc = 0, st = 0; kc < nkt; kc += kChunk) {
    const int kend = min(nkt, kc + kChunk);
    auto next = [](int x) { return x + 1 == S ? 0 : x + 1; };
    int kt = kc;
    for (; kt < kend; ++kt) {
      int st1 = next(st);
      stage(kt, st, st1, Int<0>());
      st = st1;
      if (++kt == kend) break;
      st1 = next(st);
      stage(kt, st, st1, Int<1>());
      st = st1;
    }
    flush(kc == 0, kend == nkt);
  }
  if (nkt <= 0) flush(true, true);
  __builtin_amdgcn_s_waitcnt(0xF70);  // no load may reach LDS after the workgroup has left
}

// C_z(m,n) = beta * C_z(m,n) + sum_s part[s][z][m][n] for outer block blockIdx.y (partial tiles ws1 apart), summed in slice order.
__global__ __launch_bounds__(256) void lowp_splitk_reduce(double* C, long scm, long scn, long sc2, long sc1, int nb,
                                                          const int* tab1, double beta, const double* part, long ws1,
                                                          int M, int N, int split) {
  const long mn = (long)M * N, outs = mn * nb;
  const int zs = tab1 ? tab1[blockIdx.y] : blockIdx.y;
  for (long x = blockIdx.x * 256L + threadIdx.x; x < outs; x += (long)gridDim.x * 256) {
    double acc = 0.0;
    for (int sl = 0; sl < split; ++sl) acc += part[zs * ws1 + sl * outs + x];
    const long r = x % mn;
    const int z = (int)(x / mn), m = (int)(r / N), n = (int)(r % N);
    double* c = C + z * sc2 + zs * sc1 + m * scm + n * scn;
    *c = (beta == 0.0) ? acc : acc + beta * *c;
  }
}

// Stages of a split-K slice for a launch of `tiles` workgroups (one per CU) over nkt stages of 32: slices of at least
// 16 stages (the last one of what is left), enough of them for one round of 256 workgroups, of which the scratch holds
// fit sets of partial tiles.
int stages_per_slice(long tiles, int nkt, long fit) {
  if (tiles >= 192 || nkt < 32) return nkt;
  const long n = std::min<long>({(256 + tiles - 1) / tiles, (long)nkt / 16, fit});
  return n < 2 ? nkt : (int)((nkt + n - 1) / n);
}

// Tile shapes.  A launch of c = ceil(workgroups / 256) tiles per CU and k stages is taken as f + k max(t1, c ts) + c e:
// t1 is the stage of a workgroup with a CU to itself (load and LDS latency), ts that of one among many
// (MFMA and load rate), e the store of a tile; us, fitted (1 to 13 % rms by shape) to 194 contractions of o4 v36 to o40 v130
// and o36 v260 systems, over which the choice comes within 0.5 to 1.3 % of the best shape in the mean (14 % at most).  Where
// the fit put t1 below ts it has no effect, and ts stands for it.  All shapes of an order give the same bits.
// Measured there against register-staged 256 x 128 / 128 x 128 tiles (kBf16, kF32Seq) and 256 x 256 direct-to-LDS
// ones: 2.2 and 2.05 times as fast, 1.2 (kBf32) and 1.4 (kF32Str).  Split-BF16x3, o8 v72: ladder 36 x 2628 x 2628 108 -> 22 us,
// rings 576^3 30 -> 8.8 us; o20 v180: ladder 210 x 16290 x 16290 910 -> 643 us, rings 3600^3 460 -> 423 us.  FP32,
// o17 v131: ladder 153 x 8646 x 8646 1.42 -> 0.62 ms, rings 2227^3 535 -> 360 us.
struct Shape {
  int kind, bm, bn, threads;
  double t1, ts, f, e;
  void (*kernel)(LP);
};
#define SHAPE(KIND, BM, BN, WM, WN, S, T1, TS, F, E) \
  { KIND, BM, BN, WM * WN * 64, T1, TS, F, E, gemm_lowp_kernel<KIND, BM, BN, WM, WN, S> }
const Shape kShapes[] = {
    SHAPE(kBf16, 64, 64, 2, 2, 3, 0.238, 0.238, 4.0, 0.0),    SHAPE(kBf16, 64, 64, 2, 2, 4, 0.236, 0.236, 3.6, 0.54),
    SHAPE(kBf16, 96, 96, 2, 2, 3, 0.415, 0.374, 3.9, 1.28),   SHAPE(kBf16, 128, 64, 2, 2, 3, 0.373, 0.365, 4.4, 0.63),
    SHAPE(kBf16, 128, 128, 2, 2, 4, 0.565, 0.565, 1.6, 5.44), SHAPE(kBf16, 256, 128, 4, 2, 3, 0.910, 0.867, 6.9, 0.0),
    SHAPE(kBf32, 64, 128, 2, 2, 3, 1.0, 0.386, 0.0, 1.57),    SHAPE(kBf32, 128, 256, 2, 4, 3, 1.240, 1.042, 0.0, 8.87),
    SHAPE(kBf32, 192, 192, 2, 2, 3, 1.239, 1.156, 0.0, 11.8), SHAPE(kBf32, 256, 128, 4, 2, 3, 1.231, 1.025, 0.0, 8.55),
    SHAPE(kBf32, 192, 256, 2, 4, 2, 1.563, 1.563, 0.0, 9.75), SHAPE(kBf32, 256, 256, 2, 4, 2, 1.849, 1.849, 0.0, 15.0),
    SHAPE(kF32Seq, 64, 64, 2, 2, 3, 0.706, 0.561, 3.1, 1.17), SHAPE(kF32Seq, 64, 64, 2, 2, 4, 0.691, 0.583, 2.7, 1.72),
    SHAPE(kF32Seq, 96, 96, 2, 2, 3, 1.526, 1.243, 1.1, 4.38), SHAPE(kF32Seq, 128, 64, 2, 2, 3, 1.204, 1.031, 2.3, 2.89),
    SHAPE(kF32Str, 64, 64, 2, 2, 3, 0.706, 0.499, 6.3, 0.78), SHAPE(kF32Str, 128, 256, 2, 4, 3, 3.731, 3.665, 1.0, 8.94),
    SHAPE(kF32Str, 224, 192, 2, 4, 3, 4.938, 4.938, 1.0, 10.2), SHAPE(kF32Str, 256, 256, 2, 4, 2, 7.135, 7.135, 5.9, 10.4),
};
#undef SHAPE

}  // namespace



hipError_t to_lowp_2d(int prec, float* out, long ldo, const double* in, long ldi, long rows, long cols,
                      hipStream_t s) {
  const long total = rows * ldo;
  if (total <= 0) return hipSuccess;
  if (bounds_checking() && !(range_ok(out, 0, total - 1, 4, "lowp shadow") &&
                             range_ok(in, 0, (rows - 1) * ldi + cols - 1, 8, "lowp source")))
    return hipErrorInvalidValue;
  if (dry_run()) return hipSuccess;
  // eight columns per thread where the rows allow 16-byte accesses (ldo is a multiple of 32)
  const bool v8 = (reinterpret_cast<uintptr_t>(in) & 15) == 0 && (reinterpret_cast<uintptr_t>(out) & 15) == 0 &&
                  (ldi & 1) == 0 && (ldo & 31) == 0;
  long g = ((v8 ? total / 8 : total) + 255) / 256;
  if (g > 8192) g = 8192;
  if (prec == kPrecBF16x3) {
    if (v8)
      hipLaunchKernelGGL(split_bf16_2d_v8_kernel, dim3((unsigned)g), dim3(256), 0, s,
                         reinterpret_cast<unsigned short*>(out), ldo, in, ldi, rows, cols);
    else
      hipLaunchKernelGGL(split_bf16_2d_kernel, dim3((unsigned)g), dim3(256), 0, s,
                         reinterpret_cast<unsigned short*>(out), ldo, in, ldi, rows, cols);
  } else {
    if (v8)
      hipLaunchKernelGGL(cvt_f32_2d_v8_kernel, dim3((unsigned)g), dim3(256), 0, s, out, ldo, in, ldi, rows, cols);
    else
      hipLaunchKernelGGL(cvt_f32_2d_kernel, dim3((unsigned)g), dim3(256), 0, s, out, ldo, in, ldi, rows, cols);
  }
  return hipGetLastError();
}

hipError_t gemm_lowp(const GemmLP& g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0 || g.nb <= 0 || g.nb1 <= 0) return hipSuccess;
  if (g.K <= 0 || (long)g.nb * g.nb1 > 65535 || (g.prec != kPrecFP32 && g.prec != kPrecBF16x3))
    return hipErrorInvalidValue;
  const bool bf = (g.prec == kPrecBF16x3);
  // whole stages: rows of K padded to 32 values (128 bytes), 16-byte aligned (bf16: interleaved K-blocks)
  const int nkt = (g.K + 31) / 32;
  const long unit = bf ? 64 : 32, el = bf ? 2 : 4, row = unit * nkt;
  auto al16 = [](const void* x) { return (reinterpret_cast<uintptr_t>(x) & 15) == 0; };
  if (((g.lda | g.ldb | g.sa2 | g.sb2 | g.sa1 | g.sb1) & (unit - 1)) || g.lda < row || g.ldb < row || !al16(g.A) || !al16(g.B))
    return hipErrorInvalidValue;
  const long nz1 = g.tab1 ? g.tab1_max + 1 : g.nb1;  // operand blocks of the outer batch level
  if (bounds_checking()) {
    const long la = (long)(g.M - 1) * g.lda + row - 1 + (long)(g.nb - 1) * g.sa2 + (nz1 - 1) * g.sa1;
    const long lb = (long)(g.N - 1) * g.ldb + row - 1 + (long)(g.nb - 1) * g.sb2 + (nz1 - 1) * g.sb1;
    long lo = 0, hi = 0;
    const long dc[4] = {(long)(g.M - 1) * g.scm, (long)(g.N - 1) * g.scn, (long)(g.nb - 1) * g.sc2, (nz1 - 1) * g.sc1};
    for (long d : dc) {
      if (d < 0) lo += d; else hi += d;
    }
    if (!(range_ok(g.A, 0, la, el, "lowp A") && range_ok(g.B, 0, lb, el, "lowp B") && range_ok(g.C, lo, hi, 8, "lowp C") &&
          (!g.ws || range_ok(g.ws, 0, (nz1 - 1) * g.ws1 + g.ws_elems - 1, 8, "lowp split-K scratch"))))
      return hipErrorInvalidValue;
  }
  if (dry_run()) return hipSuccess;
  if (g.ws && g.nb1 > 1 && g.ws1 < g.ws_elems) return hipErrorInvalidValue;  // the blocks' scratches overlap
  const int nbz = g.nb * g.nb1;  // grid.y
  const int mdec = g.m_dec > 0 ? g.m_dec : g.M;
  // The order and the slices, which the bits of a result depend on, follow from the shape of one state alone: the wide
  // orders (32 x 32 products, one read per FP32 fragment) from half a round of 256 x 256 tiles on, or a quarter with
  // scratch, K cut so that all slices fill one round; the others in slices of at least 512.
  const long t2 = (long)((mdec + 255) / 256) * ((g.N + 255) / 256) * g.nb;
  const long fit = g.ws ? g.ws_elems / ((long)g.M * g.N * g.nb) : 0;  // slices that the scratch of a block holds
  int kind = bf ? kBf16 : kF32Seq, ktps = nkt;
  if (t2 >= 128) {
    kind = bf ? kBf32 : kF32Str;
  } else {
    const long n = t2 >= 64 ? std::min<long>({256 / t2, (long)nkt / 16, fit}) : 0;
    if (n >= 2) {
      kind = bf ? kBf32 : kF32Str;
      ktps = (int)((nkt + n - 1) / n);
    } else {
      const long bm = bf ? 256 : 128;
      ktps = stages_per_slice(((g.M + bm - 1) / bm) * ((g.N + 127) / 128) * g.nb, nkt, fit);
    }
  }
  const int split = (nkt + ktps - 1) / ktps;
  const Shape* best = nullptr;
  double best_us = 0.0;
  for (const Shape& f : kShapes) {
    // a tile's rows lie within the 4 GiB range of a buffer descriptor
    if (f.kind != kind || std::min(f.bm, g.M) * g.lda * el >= (1L << 32) || std::min(f.bn, g.N) * g.ldb * el >= (1L << 32)) continue;
    const long tiles = (long)((g.M + f.bm - 1) / f.bm) * ((g.N + f.bn - 1) / f.bn);
    const double c = (double)((tiles * nbz * split + 255) / 256);
    const double us = f.f + ktps * std::max(f.t1, c * f.ts) + c * f.e;
    if (!best || us < best_us) {
      best = &f;
      best_us = us;
    }
  }
  if (!best) return hipErrorInvalidValue;
  LP p;
  p.M = g.M;
  p.N = g.N;
  p.K = g.K;
  p.A = reinterpret_cast<const char*>(g.A);
  p.lda = g.lda * el;
  p.sa2 = g.sa2 * el;
  p.B = reinterpret_cast<const char*>(g.B);
  p.ldb = g.ldb * el;
  p.sb2 = g.sb2 * el;
  p.C = g.C;
  p.scm = g.scm;
  p.scn = g.scn;
  p.sc2 = g.sc2;
  p.alpha = g.alpha;
  p.beta = g.beta;
  p.tiles_m = (g.M + best->bm - 1) / best->bm;
  p.tiles_n = (g.N + best->bn - 1) / best->bn;
  p.ktps = ktps;
  p.cslice = 0;
  p.nb = g.nb;
  p.tab1 = g.tab1;
  p.sa1 = g.sa1 * el;
  p.sb1 = g.sb1 * el;
  p.sc1 = g.sc1;
  if (split > 1) {  // partial tiles [split][nb][M][N] in the scratch of each block
    p.C = g.ws;
    p.scm = g.N;
    p.scn = 1;
    p.sc2 = (long)g.M * g.N;
    p.sc1 = g.ws1;
    p.cslice = (long)g.M * g.N * g.nb;
    p.beta = 0.0;
  }
  hipLaunchKernelGGL(best->kernel, dim3(p.tiles_m * p.tiles_n, nbz, split), dim3(best->threads), 0, s, p);
  if (split > 1) {
    const dim3 grid((unsigned)std::min<long>((p.cslice + 255) / 256, 4096), (unsigned)g.nb1);
    hipLaunchKernelGGL(lowp_splitk_reduce, grid, dim3(256), 0, s, g.C, g.scm, g.scn, g.sc2, g.sc1, g.nb, g.tab1, g.beta, g.ws,
                       g.ws1, g.M, g.N, split);
  }
  return hipGetLastError();
}

hipError_t to_lowp_gwz(int prec, float* out, long ldo, const double* kcbd, const double* kcld, int o, int v,
                       hipStream_t s) {
  const long ov = (long)o * v, vv = (long)v * v, rows = ov + (long)o * o;
  if (ldo < vv || ldo % 32) return hipErrorInvalidValue;
  if (bounds_checking() && !(range_ok(kcbd, 0, ov * vv - 1, 8, "Gwz shadow (kc|bd)") &&
                             range_ok(kcld, 0, ov * ov - 1, 8, "Gwz shadow (kc|ld)") &&
                             range_ok(out, 0, rows * ldo - 1, 4, "Gwz shadow")))
    return hipErrorInvalidValue;
  if (dry_run()) return hipSuccess;
  const dim3 grid((unsigned)rows, (unsigned)std::min<long>((ldo + 255) / 256, 64));
  if (prec == kPrecBF16x3)
    hipLaunchKernelGGL(lowp_gwz_kernel<true>, grid, dim3(256), 0, s, out, ldo, kcbd, kcld, o, v);
  else
    hipLaunchKernelGGL(lowp_gwz_kernel<false>, grid, dim3(256), 0, s, out, ldo, kcbd, kcld, o, v);
  return hipGetLastError();
}

hipError_t to_lowp_pm(int prec, float* out, long ldo, const double* V, long ldv, long vrows, const int* pm, long Tv,
                      hipStream_t s) {
  const long total = 2 * Tv * ldo;
  if (total <= 0) return hipSuccess;
  if (ldo < Tv || ldv < Tv || vrows < Tv) return hipErrorInvalidValue;
  if (bounds_checking() && !(range_ok(out, 0, total - 1, 4, "vvvv shadow") &&
                             range_ok(V, 0, (vrows - 1) * ldv + Tv - 1, 8, "full vvvv") &&
                             range_ok(pm, 0, Tv - 1, 4, "pair rows")))
    return hipErrorInvalidValue;
  if (dry_run()) return hipSuccess;
  long g = (total + 255) / 256;
  if (g > 8192) g = 8192;
  if (prec == kPrecBF16x3)
    hipLaunchKernelGGL(lowp_pm_kernel<true>, dim3((unsigned)g), dim3(256), 0, s,
                       reinterpret_cast<unsigned short*>(out), nullptr, ldo, V, ldv, pm, Tv);
  else
    hipLaunchKernelGGL(lowp_pm_kernel<false>, dim3((unsigned)g), dim3(256), 0, s, nullptr, out, ldo, V, ldv, pm, Tv);
  return hipGetLastError();
}

hipError_t to_lowp_t(int prec, float* out, long ldo, const double* in, long ldi, long rows, long cols, hipStream_t s) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  if ((ldo & 31) || ldo < cols || ldi < rows || (rows + 31) / 32 > 0x7fffffffL || ldo / 32 > 65535)
    return hipErrorInvalidValue;
  if (bounds_checking() && !(range_ok(out, 0, rows * ldo - 1, 4, "transposed shadow") &&
                             range_ok(in, 0, (cols - 1) * ldi + rows - 1, 8, "transposed shadow source")))
    return hipErrorInvalidValue;
  if (dry_run()) return hipSuccess;
  const dim3 grid((unsigned)((rows + 31) / 32), (unsigned)(ldo / 32));
  if (prec == kPrecBF16x3)
    hipLaunchKernelGGL(lowp_t_kernel<true>, grid, dim3(256), 0, s, (void*)out, ldo, in, ldi, rows, cols);
  else
    hipLaunchKernelGGL(lowp_t_kernel<false>, grid, dim3(256), 0, s, (void*)out, ldo, in, ldi, rows, cols);
  return hipGetLastError();
}

}  // namespace ascc
