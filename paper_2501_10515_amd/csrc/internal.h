// Internal declarations shared by the libascc translation units (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <string>

struct ascc_ints;
struct ascc_diis;
struct ascc_opts;
struct ascc_result;

namespace ascc {

// Status used inside the library; converted to the ASCC_E_* codes at the ABI boundary.
struct Error {
  int code;
  std::string msg;
};

void set_error(const std::string& msg);

// Optional host-side bounds checking of every strided launch (environment variable
// ASCC_CHECK_BOUNDS=1): device buffers are registered with their sizes, and each GEMM /
// permute launch first verifies that the lowest and highest element it can touch lie in one
// registered buffer.  A violation is reported as an error instead of being launched.
bool bounds_checking();
// Dry run (environment variable ASCC_DRY_RUN=1, implies bounds checking): device
// allocations return unbacked addresses and no kernel, copy or synchronisation is issued,
// so the complete host-side launch sequence -- every stride and extent -- can be validated
// on a machine without a GPU.
bool dry_run();
void register_buffer(const void* p, size_t bytes);
void unregister_buffer(const void* p);
// true if [base + lo, base + hi] (in elements of `elem` bytes) lies inside a registered buffer
bool range_ok(const void* base, long lo, long hi, size_t elem, const char* what);

// ---------------------------------------------------------------------------------------
// Strided batched FP64 GEMM on the matrix cores:
//   C_z(m,n) = alpha * sum_{r < nred} sum_k A_{z,r}(m,k) B_{z,r}(k,n) + beta * C_z(m,n)
// Every operand is a general strided 2-D view, e.g. A(m,k) = A[m*sam + k*sak].  The batch
// index z runs over nb1 x nb2 (z1 outer, z2 inner) with one stride per level; the reduction
// index r (nred >= 1) adds products of further (A, B) pairs into the same C.
// beta == 0 never reads C.
struct Gemm {
  int M = 0, N = 0, K = 0;
  const double* A = nullptr;
  long sam = 0, sak = 0, sa1 = 0, sa2 = 0, sar = 0;
  const double* B = nullptr;
  long sbk = 0, sbn = 0, sb1 = 0, sb2 = 0, sbr = 0;
  double* C = nullptr;
  long scm = 0, scn = 0, sc1 = 0, sc2 = 0;
  double alpha = 1.0, beta = 0.0;
  int nb1 = 1, nb2 = 1, nred = 1;
  // Optional scratch for split-K: when the output has too few tiles to fill the chip, the
  // (reduction x K) iteration space is cut into slices whose partial tiles land here and
  // are then summed in a fixed order (deterministic).  nullptr disables splitting.  Every block of batch level 1
  // has ws_elems of its own, ws1 apart, and takes the tiles and slices that it takes alone, so that its
  // sums do not depend on nb1.
  double* ws = nullptr;
  long ws_elems = 0, ws1 = 0;
  // Optional table of batch level 1: grid index z1 takes operand block tab1[z1] (device array of
  // nb1 entries, each at most tab1_max); nullptr: block z1.
  const int* tab1 = nullptr;
  int tab1_max = 0;
  // C = A B with B(k, n) = A(n, k) is symmetric: when M == N, beta == 0 and the rows qualify for
  // the direct-to-LDS kernel, only the tiles on and below the diagonal are computed, each stored
  // at its transposed place too (otherwise the full product)
  bool lower = false;
  // In a group (gemm_f64_group): consecutive contractions with the same acc >= 0 add to one output (the same
  // C, M x N elements in the same order, beta = 1); fixed: K is summed whole by any launch.
  int acc = -1;
  bool fixed = false;
};

// Batch level of the particle-particle ladder: n operand blocks (A, V, C and the scratch offset by sa, sv, sc, sw
// elements per block; the pair-row table, which depends on v only, is shared), block z taken from
// tab[z] when tab is given (entries at most tab_max).
struct LadderBatch {
  int n = 1;
  const int* tab = nullptr;
  int tab_max = 0;
  long sa = 0, sv = 0, sc = 0, sw = 0;
};

// Convenience constructors for row-major matrices:
//   A is M x K with leading dimension lda (ta = false) or stored K x M (ta = true), etc.
Gemm gemm_rm(int M, int N, int K, double alpha, const double* A, long lda, bool ta, const double* B, long ldb,
             bool tb, double beta, double* C, long ldc);

hipError_t gemm_f64(const Gemm& g, hipStream_t s);
// Independent contractions in order (each output read and written by one of them, or added to by several with
// the same acc): small ones as one launch where that is estimated to take less time than their own launches, a
// choice made from the shapes of one operand block (not from those marked fixed).
hipError_t gemm_f64_group(const Gemm* gs, int n, hipStream_t s);
// Whether a contraction would take small direct-to-LDS tiles (64 x 64 or 32 x 32) by itself.
bool gemm_f64_small(const Gemm& g);

// Particle-particle ladder over pair indices, both halves h = 0 (+), 1 (-) in one launch:
//   C_h[m][n] = sum_k A_h[m][k] * V_h(n, k),   m < M, n < N, k < K
// A_h and C_h are rows at strides lda, ldc, the halves sa2, sc2 apart.  pm == nullptr: V_h is stored,
// N rows at stride ldv, the halves sv2 apart.  Otherwise V is the full (ac|bd) matrix in pair order
// (see pack_full), vrows rows at stride ldv, and V_h(n, k) = V[n][k] +- V[pm[n]][k] = (ac|bd) +- (ad|bc)
// for n = (a <= b), k = (c <= d) (its diagonal columns hold (ac|bc) / 2, so V_+ is (ac|bc) there).
// Rows are 16-byte aligned, K even (zero past T(v)).  A row's sums do not depend on M or N: K is cut into
// slices as for Mdec rows (those of one state; M a multiple of it) and Ndec columns, summed in slice order.
struct Ladder {
  int M = 0, Mdec = 0, N = 0, Ndec = 0, K = 0;
  const double* A = nullptr;
  long lda = 0, sa2 = 0;
  const double* V = nullptr;
  long ldv = 0, sv2 = 0, vrows = 0;
  const int* pm = nullptr;
  double* C = nullptr;
  long ldc = 0, sc2 = 0;
  double* ws = nullptr;  // optional scratch for the slices' partial tiles
  long ws_elems = 0;
  LadderBatch lb;
};
constexpr int kLadderWhole = 31 * 16;  // K up to this is never cut
hipError_t gemm_f64_ladder(const Ladder& L, hipStream_t s);

// Low-precision contraction with FP64 result (gemm_lowp.hip):
//   C_z(m,n) = alpha * sum_k A_z[m*lda + k] * B_z[n*ldb + k] + beta * C_z(m,n)
// A, B are FP32 (K contiguous); prec selects FP32 MFMA or split-BF16x3 MFMA; FP32 accumulation
// inside chunks of 8192 K-values, FP64 accumulation across chunks.
constexpr int kPrecFP64 = 0, kPrecFP32 = 1, kPrecBF16x3 = 2;
struct GemmLP {
  int M = 0, N = 0, K = 0, nb = 1;
  const float* A = nullptr;
  long lda = 0, sa2 = 0;
  const float* B = nullptr;
  long ldb = 0, sb2 = 0;
  double* C = nullptr;
  long scm = 0, scn = 1, sc2 = 0;
  double alpha = 1.0, beta = 0.0;
  int prec = kPrecFP32;
  // rows zero-padded to whole K-blocks of 32; BF16X3: interleaved splits (see to_lowp_2d), lda, ldb,
  // sa2, sb2 count bf16 elements
  // Optional split-K scratch: an output with too few tiles to fill the chip has its K range cut
  // into slices (all but the last at least 512 of K, each FP32 chunk starting at its slice's start)
  // whose FP64 partial tiles land here and are then summed in slice order (deterministic).  Every outer block has
  // ws_elems of its own, ws1 apart, and takes the order and the slices that it takes alone (see Gemm).
  double* ws = nullptr;
  long ws_elems = 0, ws1 = 0;
  // Optional outer batch level over operand blocks: nb1 blocks at strides sa1, sb1 (in the units of
  // lda) and sc1 (FP64 elements); block z1 taken from tab1[z1] when tab1 is given (entries at most
  // tab1_max).
  int nb1 = 1;
  long sa1 = 0, sb1 = 0, sc1 = 0;
  const int* tab1 = nullptr;
  int tab1_max = 0;
  // rows that decide the kernel (0: M): operands stacking the rows of several states pass one
  // state's rows, so that every state's rows are summed exactly as when it is alone
  int m_dec = 0;
};
hipError_t gemm_lowp(const GemmLP& g, hipStream_t s);
// Low-precision shadow of a row-major FP64 matrix with the leading dimension padded to ldo
// (a multiple of 32; padding zeroed).  FP32: one float per element, row stride ldo.  BF16X3: the
// same bytes as bf16, row stride 2 ldo, each K-block of 32 stored as hi[32] then lo[32] with
// hi = RNE_bf16(x), lo = RNE_bf16(x - hi).
hipError_t to_lowp_2d(int prec, float* out, long ldo, const double* in, long ldi, long rows, long cols, hipStream_t s);
// Transposed shadow: out row r (r < rows) = column r of in ([cols][ldi] FP64), padded to ldo.
hipError_t to_lowp_t(int prec, float* out, long ldo, const double* in, long ldi, long rows, long cols, hipStream_t s);
// Rows m = k*v + b: (kc|bd) = kcbd[k][c][b][d] and m = ov + k*o + l: (kc|ld) = kcld[k][c][l][d] over the
// columns c*v + d (zero padded to ldo) in low precision.
hipError_t to_lowp_gwz(int prec, float* out, long ldo, const double* kcbd, const double* kcld, int o, int v,
                       hipStream_t s);
// Packed vvvv halves [2][Tv][ldo] (zero padded) in low precision, formed from the full (ac|bd)
// matrix in pair order [vrows][ldv] as gemm_f64_ladder forms them (V[n][k] +- V[pm[n]][k]).
hipError_t to_lowp_pm(int prec, float* out, long ldo, const double* V, long ldv, long vrows, const int* pm, long Tv,
                      hipStream_t s);
inline long lowp_ld(long k) { return (k + 31) / 32 * 32; }

// Hand-over test of a low-precision bulk phase: the residual norm has reached the rounding floor
// of the contractions when it has not set a new minimum (by 1%) for kPatience iterations.  Eight,
// not fewer: the excited-state (ASCC) iteration has plateaus of several iterations well above the
// floor, and a low-precision iteration costs less than half an FP64 one, so waiting longer is
// cheap while an early hand-over leaves most of the work to FP64.
struct LowpStall {
  static constexpr int kPatience = 8;
  double best = 0.0;
  int since = 0;
  bool stalled(double rnorm) {
    if (since == 0 && best == 0.0) best = rnorm;
    if (rnorm < 0.99 * best) {
      best = rnorm;
      since = 0;
    } else {
      ++since;
    }
    return since >= kPatience;
  }
};

// ---------------------------------------------------------------------------------------
// Element-wise kernels (elementwise.hip).

// out[i0,i1,i2,i3] = c0*out + sum_t coef[t] * in_t[i0*s_t0 + i1*s_t1 + i2*s_t2 + i3*s_t3]
// for up to four strided inputs (an input with coef 0 is not read; c0 == 0 never reads out).
struct Perm4In {
  const double* p = nullptr;
  long s[4] = {0, 0, 0, 0};
  double coef = 0.0;
};
hipError_t permute4(double* out, const int dims[4], double c0, const Perm4In* in, int nin, hipStream_t s);
// Same with an explicitly strided output view.
hipError_t permute4_strided(double* out, const long ostr[4], const int dims[4], double c0, const Perm4In* in,
                            int nin, hipStream_t s);

// Assembly of the doubles residual from the ring, ladder and E-term pieces (formula at the kernel).
// rminus: the ladders are pair rows rl = R+ and rminus = R- at stride ldr (unpack_rpm) instead of RL.
hipError_t assemble_r2(double* r2, const double* g1, const double* rl, const double* em, const double* p1,
                       const double* p2, int no, int nv, hipStream_t s, const double* rminus = nullptr, long ldr = 0);

// Pair packing of the particle-particle ladder (p(i,j) = row-major index of i <= j).
// Full (ac|bd) storage in pair order R(a,b) (a <= b: p(a,b); a > b: T(v) + strict index of (b,a)), rows at
// stride ldv: pm[n] = R(b,a) for pair n = (a <= b); pack_full scatters W[a - a0][c][b][d] = (ac|bd),
// a0 <= a < a1, to V[R(a,b)][R(c,d)], the diagonal columns c = d halved.
hipError_t pair_minus_rows(int* pm, int v, hipStream_t s);
hipError_t pack_full(double* V, long ldv, const double* W, int a0, int a1, int v, hipStream_t s);
// Pair rows (+ and - halves over the pairs c <= d, rows at stride ldo >= T(v), zero past T(v)):
// t+-[T(o)], t+ = (t^cd + t^dc)/2, and V+-[T(v)] and G+-[ov + o^2], sums and differences of (ac|bd) and
// (ad|bc), of (kc|bd) and (kd|bc) and of (kc|ld) and (kd|lc) (diagonal: the element itself, and 0).
hipError_t pack_tpm(double* tplus, double* tminus, long ldo, const double* t2, int o, int v, hipStream_t s);
// rows a0 <= a < a1 from W[a - a0][c][b - a0][d] = (ac|bd)
hipError_t pack_vvvv(double* vplus, double* vminus, long ldo, const double* W, int a0, int a1, int v, hipStream_t s);
// (kc|bd) as kcbd[k][c][b][d], (kc|ld) as kcld[k][c][l][d]
hipError_t pack_gwz(double* gplus, double* gminus, long ldo, const double* kcbd, const double* kcld, int o, int v,
                    hipStream_t s);
// Tx, U (rows at stride ld, zero past o v) and, with tplus given, t+- from t2; Xc and Zd of the rings
// (formulas at the kernels)
hipError_t amp_views(double* Tx, double* U, long ld, double* tplus, double* tminus, long ldo, const double* t2, int o,
                     int v, hipStream_t s);
hipError_t ring_xz_lowp(int prec, float* xz, long ld, const double* g2, const double* g3, const double* y1, const double* y2,
                        int o, int v, hipStream_t s);  // as the shadow [2][ov][ld] alone
hipError_t ring_xz(double* xc, double* zd, long ld, const double* g2, const double* g3, const double* y1,
                   const double* y2, int o, int v, hipStream_t s);
// W' and chi+- from the W/Z columns of the ladder's pair rows (formulas at the kernel)
hipError_t wz_chi(double* wp, long ldw, double* chip, double* chim, const double* rp, const double* rm, long ldr,
                  const double* g4, const double* foo, const double* t1, int o, int v, hipStream_t s);
// RL[i][j][a][b] from the pair rows R+- (stride ldr)
hipError_t unpack_rpm(double* RL, const double* Rplus, const double* Rminus, long ldr, int o, int v, hipStream_t s);

// T1 dressing and the dressed Fock matrix (formulas at the kernels).  B is [p][q] rows of ldq fitting values
// (zero past naux), likewise D [o][n], bvv [v][v], bvo [o][v] (B^_ai at [i][a]) and boo [o][o]:
//   dress_right  D[k][p] = (B Y^T)_pk
//   dress_left   bvv, bvo, boo and f = h + 2 sum_Q J_Q B, J_Q = sum_k D[k][k]
//   coulomb      f = f0 + alpha sum_Q J_Q B, J_Q = sum_k B[k][k]
//   fock_finish  F^ = X f Y^T: fvv [v][v], foo [o][o], r1 = F^_ai at [i][a], fov [o][v] (zero to ldf elements)
hipError_t dress_right(double* D, const double* B, const double* t1, int o, int v, long ldq, hipStream_t s);
// (with svv given also their low-precision shadows, rows at stride lowp_ld(ldq))
hipError_t dress_left(double* bvv, double* bvo, double* boo, double* f, const double* B, const double* D,
                      const double* t1, const double* h, int o, int v, long ldq, int prec, float* svv, float* svo, float* soo,
                      hipStream_t s);
hipError_t coulomb(double* f, const double* f0, const double* B, double alpha, int o, int n, long ldq, hipStream_t s);
hipError_t fock_finish(double* fvv, double* foo, double* r1, double* fov, long ldf, const double* f, const double* t1,
                       int o, int v, hipStream_t s);

// x -> (1 + c E_hp) x (1 - c E_hp) in place on an n x n matrix of rows of len values at stride ld (E_hp: one at
// row h, column p).
hipError_t onebody_transform(double* X, int n, long ld, long len, int h, int p, double c, hipStream_t s);
// A cross index set: over the n = no * nv indices r = i * nv + a, the members with i == h or
// a == pa (m = no + nv - 1 of them), listed compactly as (h, 0 .. nv-1), then (i, pa) for i != h
// ascending.  With (no, nv, h, pa) = (o, v, hole, particle) it is the set of (i, a) rows of an
// ov x ov matrix that touch a primary orbital; (o, o, h, h) and (v, v, pa, pa) are the pair
// indices ij and ab that do.
struct Cross {
  int no = 1, nv = 1, h = 0, pa = 0;
  __host__ __device__ long n() const { return (long)no * nv; }
  __host__ __device__ long m() const { return (long)no + nv - 1; }
};
//   cross_gather_rows: dst[k][c] = src[row k of X][c], c < ncols (zero_diag: the corner entry
//                      at row and column h*nv + pa written as 0).
//   cross_gather_cols: dst[r][k] = src[r][col k of X] for k < m, 0 for m <= k < ldd; zero_rows:
//                      rows r that are members of *zero_rows written as 0.
//   cross_scatter_add_rows / _cols / _block: the inverse placements, dst += alpha * src.
//   cross_rows_without_corner: dst[k][c] = Y[row k][c] - [row k == hp] T[hp][hp] K[hp][c] for
//                      X.n() x X.n() operands, T and K rows at stride ldk (the cross rows of T' K,
//                      T' = T minus its corner entry, from Y = T K).
//   em_cross_column:   EM[ij][a][b] += tc[ij][v + a - [a > pa]] * A[b][pa] for a != pa.
// mixed_doubles: dst = src on the mixed doubles (index set holds h or pa, not all primary), else 0.
hipError_t cross_gather_rows(double* dst, long ldd, const double* src, long lds, long src_rows, long ncols,
                             const Cross& X, bool zero_diag, hipStream_t s);
hipError_t cross_gather_cols(double* dst, long ldd, const double* src, long lds, long nrows, const Cross& X,
                             const Cross* zero_rows, hipStream_t s);
hipError_t cross_scatter_add_rows(double* dst, long ldd, long dst_rows, const double* src, long lds, long ncols,
                                  double alpha, const Cross& X, hipStream_t s);
hipError_t cross_scatter_add_cols(double* dst, long ldd, long nrows, const double* src, long lds, double alpha,
                                  const Cross& X, hipStream_t s);
hipError_t cross_scatter_add_block(double* dst, long ldd, const double* src, long lds, double alpha, const Cross& X,
                                   hipStream_t s);
hipError_t cross_rows_without_corner(double* dst, long ldd, const double* Y, const double* T, const double* K,
                                     long ldk, const Cross& X, hipStream_t s);
hipError_t em_cross_column(double* em, const double* tc, long ldt, const double* A, int o, int v, int pa,
                           hipStream_t s);
hipError_t mixed_doubles(double* dst, const double* src, int o, int v, int h, int pa, hipStream_t s);
// e0[0] = sum_{i<o} (h[i * hs] + f[i * fs]) (hlen, flen: elements of h and f, for the bounds check).
hipError_t reference_energy(double* e0, const double* h, long hs, long hlen, const double* f, long fs, long flen,
                            int o, hipStream_t s);
// t1 = 0, t2 = 0 except t1[h][a] = s1 and t2[h][h][a][a] = s2.
hipError_t initial_guess(double* t1, double* t2, int no, int nv, int h, int a, double s1, double s2, hipStream_t s);

// Deterministic two-stage energy reduction:
//   e = sum_{ijab} (t2 + t1_ia t1_jb) L[ijab] + 2 sum_ia f_ia t1_ia
hipError_t energy(double* e, double* partial, const double* t1, const double* t2, const double* Lijab,
                  const double* fov, int no, int nv, hipStream_t s);

// DIIS device state (one per amplitude set), kept in device memory.
constexpr int kMaxDiis = 16;
struct DiisState {
  int nvec;     // stored pairs
  int head;     // slot that receives the next pair
  int calls;    // update calls so far
  int flags;    // last call's flags
  double e_prev;
  int has_prev;
  int pad_;
  double Bm[kMaxDiis * kMaxDiis];  // error-vector overlaps, indexed by slot
  double coef[kMaxDiis];           // extrapolation coefficients by slot (0 for unused)
  int slot_age[kMaxDiis];          // insertion counter of each slot (-1 empty)
  int counter;
  int pad2_;
};

struct UpdateArgs {
  double* t1;  // written; read as the step's start too unless t1i, t2i are given
  double* t2;
  const double* t1i = nullptr;
  const double* t2i = nullptr;
  const double* r1;
  const double* r2;
  const double* e;
  const double* eps;  // diagonal of the Fock matrix [n]
  double* hist_t;     // [m][len]
  double* hist_e;     // [m][len]
  double* partial;    // [nblk][2 + m] reduction scratch
  DiisState* st;
  double* stats;
  int no, nv, m;
  int start;  // calls before this (device-side count) store no pair in the history
  long len;   // no*nv + no*no*nv*nv
  double shift;
  // Batched update of nslot amplitude sets: every pointer above except stats names slot 0 of a
  // layout repeated at a byte stride ss (slot k at + k ss, k = tab[z] for grid row z when tab is
  // given, entries at most tab_max); stats is [slot][8].
  int nslot = 1;
  long ss = 0;
  const int* tab = nullptr;
  int tab_max = 0;
};
hipError_t diis_update(const UpdateArgs& u, hipStream_t s);
int update_partial_blocks();

// The solve loop of ascc_solve with its DIIS state and work arrays carved from [ws, ws + ws_bytes)
// (ws == nullptr: allocated, as ascc_solve does), and the bytes that carving needs.
size_t solve_workspace_bytes(long o, long v, int diis_size);
int solve_impl(ascc_ints* I, const ascc_opts* opts, double* t1, double* t2, ascc_result* res, void* stream, char* ws,
               size_t ws_bytes);
// An unbacked, never dereferenced device address range for a dry run.
uintptr_t dry_run_address(size_t bytes);
// One iteration (residual, then the Jacobi/DIIS update) of n slots that repeat one layout at a
// byte stride: I, D and the amplitude / residual / energy pointers are those of the base slot,
// whose layout spans [region, region + stride); slot z of the batch is the base slot + htab[z]
// (dtab: the same table in device memory, read by the batched contractions and the update).
// stats receives one row of 8 statistics per slot, row htab[z] for slot z (see ascc_update).
int iterate_slots(ascc_ints* I, ::ascc_diis* D, int n, const int* dtab, const int* htab, const char* region,
                  long stride, double* t1, double* t2, double* r1, double* r2, double* e, double* stats,
                  hipStream_t s);

}  // namespace ascc
