// Projector refresh on the device (Sec. 3.3, Eq. 7 and the "if t mod T = 0" branch of Algorithm 1: every
// T steps P is replaced by the leading r singular vectors of the current gradient, on the short side).
// The paper calls an SVD; only the subspace spanned by the leading vectors enters the step (the step is
// invariant to a rotation of P inside that subspace up to the Adam state's coordinates, which the paper
// resets to nothing: M and V carry over), so the basis is computed by subspace iteration:
//
//     Q <- orth( G G^T Q )   (m <= n),        Q <- orth( G^T G Q )   (m > n),
//
// a fixed number of times from a seeded random start.  The two big products are the projection
// kernel itself: T = (G applied along the short side) is exactly R for the projector Q, and the way
// back is the same kernel run on the other orientation of G with T as its K-blocked operand, which the way there writes
// from its accumulators (store_projection).
// The small dense algebra of the orthonormalisation (CholeskyQR: C = Y^T Y, C = L L^T, Q = Y L^-T by forward substitution) is
// done in fp64, on the matrix pipe, so that it survives gradients with a steep spectrum: r^2 S flops per matrix, every listed
// matrix in one grouped launch.  Whether a second orthonormalisation is needed is asked of bf16 plane products first.
#pragma once
#include "fira_device.h"
#include "fira_elementwise.h"
#include "fira_gemm.h"


// splitmix64 finaliser: one independent 64-bit value per counter
__device__ __forceinline__ unsigned long long refresh_mix64(unsigned long long z) {
  z += 0x9e3779b97f4a7c15ull;
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  return z ^ (z >> 31);
}

// The first round's basis as the projection's operand PT: uniform(-1, 1) entries, a function of (seed, matrix, element)
// only, which nothing else reads.  Also clears the flags of the second orthonormalisation pass.
// (168 bases of the 1B shapes at r = 512: 181 us; 335 + 329 as an fp32 basis and a pass that made both operand copies of it.)
__global__ __launch_bounds__(256) void fira_refresh_start_kernel(const FiraMat* __restrict__ mats, const FiraRefreshEnt* __restrict__ ents,
                                                                 unsigned long long seed, int* __restrict__ done) {
  const FiraRefreshEnt e = ents[blockIdx.y];
  if (blockIdx.x == 0 && threadIdx.x == 0) as_global(done)[blockIdx.y] = 0;
  const unsigned long long key = refresh_mix64(seed ^ ((unsigned long long)(unsigned)e.mat << 32));
  prep_projector_tiles<false>(mats[e.mat], [&](long long idx) {
    const unsigned long long h = refresh_mix64(key + (unsigned long long)idx);
    return (float)((double)(h >> 11) * (2.0 / 9007199254740992.0) - 1.0);
  });
}

// 64 x 64 tile of a product accumulated in fp64 on the matrix pipe (v_mfma_f64_16x16x4_f64): 256 threads, wave w
// owns the 32 x 32 block at rows 32 (w >> 1), columns 32 (w & 1), as 2 x 2 blocks of 16 x 16.  Operand layout of
// the instruction: lane l supplies A[m = l % 16][k = l / 16] and B[k = l / 16][n = l % 16]; of its four result
// values, number v is D[m = l / 16 + 4 v][n = l % 16] (checked on the device against a plain product).  The products are fp64 multiply-adds like the vector
// unit's; the matrix pipe has the same peak on this chip but takes one instruction for 2048 of them, which
// frees the issue slots that the vector form spends on conversions and LDS reads.
typedef double f64x4_t __attribute__((ext_vector_type(4)));
struct RefreshAcc { f64x4_t v[2][2]; };
__device__ __forceinline__ void refresh_acc_zero(RefreshAcc& acc) {
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc.v[i][j] = f64x4_t{0.0, 0.0, 0.0, 0.0};
}
__device__ __forceinline__ void refresh_acc_step(RefreshAcc& acc, double a0, double a1, double b0, double b1) {
  acc.v[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b0, acc.v[0][0], 0, 0, 0);
  acc.v[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b1, acc.v[0][1], 0, 0, 0);
  acc.v[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b0, acc.v[1][0], 0, 0, 0);
  acc.v[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b1, acc.v[1][1], 0, 0, 0);
}
// K steps [0, KN) of a staged pair of operands: A(k, m) = sa[k * ak + m * am], B(k, n) = sb[k * bk + n * bn],
// m and n counted inside the workgroup's 64 x 64 tile.
template <int KN, typename TA, typename TB>
__device__ __forceinline__ void refresh_acc_steps(RefreshAcc& acc, const TA* sa, int ak, int am, const TB* sb, int bk, int bn) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int m0 = 32 * (wave >> 1) + (lane & 15), n0 = 32 * (wave & 1) + (lane & 15), kq = lane >> 4;
#pragma unroll
  for (int k4 = 0; k4 < KN; k4 += 4) {
    const int k = k4 + kq;
    const double a0 = (double)sa[k * ak + m0 * am], a1 = (double)sa[k * ak + (m0 + 16) * am];
    const double b0 = (double)sb[k * bk + n0 * bn], b1 = (double)sb[k * bk + (n0 + 16) * bn];
    refresh_acc_step(acc, a0, a1, b0, b1);
  }
}
// Calls f(row, col, value) for every element of the workgroup's tile that this lane holds.
template <typename F>
__device__ __forceinline__ void refresh_acc_foreach(const RefreshAcc& acc, F f) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        f(32 * (wave >> 1) + 16 * i + (lane >> 4) + 4 * v, 32 * (wave & 1) + 16 * j + (lane & 15), acc.v[i][j][v]);
}
#define FIRA_STAGE_LD 80   // floats per staged K row of 64: the four K rows that one load instruction touches fall on distinct banks

// Four consecutive floats of a row-major fp32 array (row `row`, columns col .. col + 3, leading dimension ld,
// `rows` x `cols` valid): one 16-byte load when ld is a multiple of 4 (col is), else element by element.
__device__ __forceinline__ f32x4 refresh_load4(gptr<const float> A, int row, int col, int rows, int cols, int ld) {
  if (row >= rows || col >= cols) return f32x4{0.f, 0.f, 0.f, 0.f};
  gptr<const float> p = A + (long long)row * ld + col;
  if ((ld & 3) == 0) return *reinterpret_cast<gptr<const f32x4>>(p);
  return f32x4{p[0], col + 1 < cols ? p[1] : 0.f, col + 2 < cols ? p[2] : 0.f, col + 3 < cols ? p[3] : 0.f};
}

// The second orthonormalisation pass asks of the basis it is given whether max |Y^T Y - I| is within done_tol, and for
// bf16 matrices (1e-4) three bf16 plane products h h + h m + m h answer that: a matrix whose products come out within
// refresh_check_tolerance, done_tol less all that they can be off by, is within done_tol, so it needs no fp64 Gram matrix; any
// other (FIRA_PASS_UNSURE, and every fp32 matrix, whose 1e-6 lies below that margin) is decided by it.
//
// What they can be off by, in units of ||y_a|| ||y_b|| (a matrix that is let through has squared norms within 1e-4 of 1):
//   2^-15 = 3.052e-5 for what the products leave out: bf16 has eight significant bits, so |m| <= 2^-8 |y| and |l| <= 2^-17 |y|,
//     and a product loses |m_a m_b + l_a y_b + y_a l_b - l_a l_b| <= (2^-16 + 2 * 2^-17) |y_a y_b|;
//   4.2e-6 for the sums of 32 rows, which start from zero, the small products first.  However a multiply adds its sixteen products up, each of
//     them and the result cost at most a unit in the last place, 2^-23, of the largest number there is at that point, and none
//     is larger than 1.016 (2^-7 while only h m and m h are there) of the 32 rows' share of ||y_a|| ||y_b||: 17 (2 * 1.016 + 4 * 2^-7) 2^-23
//     of that share, and the shares add up to ||y_a|| ||y_b|| at most (Cauchy and Schwarz);
//   2^-24 for each of the S / 32 additions of those sums, 1.863e-9 per row.
// Tiles of 128 x 128, a wavefront 64 x 64 of it; K stages of 32 rows, split in registers on the way into LDS, as the fp32
// projection's.  168 matrices of 2048 rows at r = 512: 592 us; the fp64 Gram matrices 1820.
#define FIRA_PASS_NEEDED 1
#define FIRA_PASS_UNSURE 2
__host__ __device__ __forceinline__ float refresh_check_tolerance(float done_tol, int S) {
  return done_tol - 3.06e-5f - 4.3e-6f - 1.87e-9f * (float)((S + 31) & ~31);
}
__global__ __launch_bounds__(256, 2) void fira_refresh_check_kernel(const FiraRefreshEnt* __restrict__ ents) {
  __shared__ __attribute__((aligned(16))) char lds[4 * FIRA_SPLIT_PLANE];
  const FiraRefreshEnt e = ents[blockIdx.y];
  const int nt = (e.r + 127) / 128;
  int ta = 0, rem = blockIdx.x;                     // linear index -> (ta >= tb)
  while (ta < nt && rem > ta) { rem -= ta + 1; ++ta; }
  if (ta >= nt) return;
  const int tb = rem;
  const float tol = refresh_check_tolerance(e.done_tol, e.S);
  if (!(tol > 0.0f)) {
    if (threadIdx.x == 0) *as_global(e.done) = FIRA_PASS_UNSURE;
    return;
  }
  gptr<const float> Y = as_global<const float>(e.Y);
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int a0 = 64 * (wave >> 1), b0 = 64 * (wave & 1), b = split_b(t), kq = split_kq(t), store_at = split_store_at(t);
  const bool diag = ta == tb, upper = diag && wave == 1;      // (nobody asks for the wave above the diagonal)
  char* lb = diag ? lds : lds + 2 * FIRA_SPLIT_PLANE;
  f32x16_t sum[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) sum[i][j][v] = 0.0f;
  f32x4 va[4], vb[4];
  auto fetch = [&](int s0) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      va[j] = refresh_load4(Y, s0 + 4 * kq + j, ta * 128 + 4 * b, e.S, e.r, e.r);
      if (!diag) vb[j] = refresh_load4(Y, s0 + 4 * kq + j, tb * 128 + 4 * b, e.S, e.r, e.r);
    }
  };
  auto store = [&](char* dst, const f32x4 (&v)[4]) {
    float x[4][4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i][j] = v[j][i];
    split_store_plane<0>(dst + store_at, x);
    split_store_plane<1>(dst + store_at + FIRA_SPLIT_PLANE, x);
  };
  fetch(0);
  for (int s0 = 0; s0 < e.S; s0 += 32) {
    store(lds, va);
    if (!diag) store(lb, vb);
    __syncthreads();
    if (s0 + 32 < e.S) fetch(s0 + 32);
    if (!upper) {
      bf16x8_t fa[2][2][2], fb[2][2][2];     // [slice][plane][block]
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const int off = p * FIRA_SPLIT_PLANE + (32 * i + (lane & 31)) * FIRA_SPLIT_PITCH + (2 * kk + (lane >> 5)) * 16;
            fa[kk][p][i] = *reinterpret_cast<const bf16x8_t*>(lds + a0 * FIRA_SPLIT_PITCH + off);
            fb[kk][p][i] = *reinterpret_cast<const bf16x8_t*>(lb + b0 * FIRA_SPLIT_PITCH + off);
          }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          f32x16_t part;
#pragma unroll
          for (int v = 0; v < 16; ++v) part[v] = 0.0f;
#pragma unroll
          for (int kk = 0; kk < 2; ++kk) {
            part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[kk][0][i], fb[kk][1][j], part, 0, 0, 0);
            part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[kk][1][i], fb[kk][0][j], part, 0, 0, 0);
          }
#pragma unroll
          for (int kk = 0; kk < 2; ++kk) part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[kk][0][i], fb[kk][0][j], part, 0, 0, 0);
          sum[i][j] += part;
        }
    }
    __syncthreads();
  }
  bool off = false;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row = ta * 128 + a0 + 32 * i + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3), col = tb * 128 + b0 + 32 * j + (lane & 31);
        const float d = sum[i][j][v] - (row == col ? 1.0f : 0.0f);
        off = off || (!upper && row < e.r && col <= row && !(fabsf(d) <= tol));      // (true for a NaN)
      }
  if (off) *as_global(e.done) = FIRA_PASS_UNSURE;
}

// C = Y^T Y (lower triangle tiles only), fp64.  K stages of 32 rows; the next stage's rows are requested into
// registers before the current one is multiplied.  What is not a multiply on the matrix pipe costs here: with the
// register count left to the compiler it kept the sums in the other half of the register file between stages and moved all
// of them there and back per stage (168 matrices of 2048 rows at r = 512: 1.82 ms, 2.04 before; five workgroups per CU).
#define FIRA_GRAM_KS 32
__global__ __launch_bounds__(256, 5) void fira_refresh_gram_kernel(const FiraRefreshEnt* __restrict__ ents) {
  __shared__ __attribute__((aligned(16))) float sa[FIRA_GRAM_KS * FIRA_STAGE_LD], sb[FIRA_GRAM_KS * FIRA_STAGE_LD];
  const FiraRefreshEnt e = ents[blockIdx.y];
  if (e.done && !(*as_global<const int>(e.done) & FIRA_PASS_UNSURE)) return;
  const int nt = (e.r + 63) / 64;
  // linear index -> (ta >= tb)
  int ta = 0, rem = blockIdx.x;
  while (ta < nt && rem > ta) { rem -= ta + 1; ++ta; }
  if (ta >= nt) return;
  const int tb = rem;
  gptr<const float> Y = as_global<const float>(e.Y);
  const int t = threadIdx.x;
  RefreshAcc acc;
  refresh_acc_zero(acc);
  const bool upper = ta == tb && (t >> 6) == 1;      // the wave above the diagonal: nobody stores its block
  f32x4 ra[2], rb[2];
  auto fetch = [&](int s0) {
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const int x = t + 256 * p, sl = x >> 4, c4 = (x & 15) * 4;
      ra[p] = refresh_load4(Y, s0 + sl, ta * 64 + c4, e.S, e.r, e.r);
      rb[p] = refresh_load4(Y, s0 + sl, tb * 64 + c4, e.S, e.r, e.r);
    }
  };
  fetch(0);
  for (int s0 = 0; s0 < e.S; s0 += FIRA_GRAM_KS) {
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const int x = t + 256 * p, sl = x >> 4, c4 = (x & 15) * 4;
      *reinterpret_cast<f32x4*>(&sa[sl * FIRA_STAGE_LD + c4]) = ra[p];
      *reinterpret_cast<f32x4*>(&sb[sl * FIRA_STAGE_LD + c4]) = rb[p];
    }
    __syncthreads();
    if (s0 + FIRA_GRAM_KS < e.S) fetch(s0 + FIRA_GRAM_KS);
    if (!upper) refresh_acc_steps<FIRA_GRAM_KS>(acc, sa, FIRA_STAGE_LD, 1, sb, FIRA_STAGE_LD, 1);
    __syncthreads();
  }
  gptr<double> C = as_global(e.C);
  bool off = false;
  refresh_acc_foreach(acc, [&](int row, int col, double v) {
    const int ra_ = ta * 64 + row, cb = tb * 64 + col;
    if (ra_ < e.r && cb < e.r && cb <= ra_) {
      C[(long long)ra_ * e.r + cb] = v;
      off = off || !(fabs(v - (ra_ == cb ? 1.0 : 0.0)) <= (double)e.done_tol);   // (true for a NaN)
    }
  });
  // Second pass only: is the basis that the pass was given orthonormal already, max |C - I| within the entry's tolerance?
  // (Every tile that finds it is not stores the same value.)
  if (e.done && off) *as_global(e.done) = FIRA_PASS_UNSURE | FIRA_PASS_NEEDED;
}

// (FIRA_PASS_NEEDED counts against the pass: unset until a tile of the Gram matrix shows that the basis is not orthonormal yet)
__device__ __forceinline__ bool refresh_pass_done(const FiraRefreshEnt& e) { return e.done && !(*as_global<const int>(e.done) & FIRA_PASS_NEEDED); }

// In-place Cholesky factorisation of the lower triangle of C (fp64), one workgroup per matrix, blocked by 32
// columns: factor the diagonal block, solve the panel below it one row per thread, update the trailing triangle from
// the panel.  A pivot that is not safely positive is replaced by a small multiple of the largest diagonal entry.  That
// carries a Y that is deficient by rounding, not one whose gradient has a numerical rank below r: the rounding left of
// the missing directions, divided by such pivots, grows from panel to panel and can end in a basis of NaNs.
//
// What bounds it is the chain of dependent steps of one panel, not its arithmetic, so both triangular parts work in
// registers: the diagonal block with one row per lane and the column's entries handed round by lane reads, the panel
// with one row per thread and independent multiply-adds per column; the triangle's old values are requested before
// the products that are taken off them.  168 matrices of r = 512: 870 us; 56 of r = 128: 88 us (1890 and 255 us
// while both parts went through LDS element by element and the largest diagonal entry was looked for by one thread).
#define FIRA_CHOL_THREADS 512
#define FIRA_CHOL_NB 32
#define FIRA_CHOL_PAN_ROWS 544   // panel rows kept in LDS: 544 x 33 doubles = 140 KB (every panel of a matrix with r <= 576)

// sqrt(x) and 1 / sqrt(x) for a normal x > 0: two rounds of Goldschmidt's coupled iteration from the hardware's estimate
// and a last Newton correction of each (within one ulp), a third of the instructions of a square root and a division.
__device__ __forceinline__ void sqrt_and_inverse(double x, double& root, double& inv) {
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y, h = 0.5 * y;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const double e = fma(-h, g, 0.5);
    g = fma(g, e, g);
    h = fma(h, e, h);
  }
  root = fma(fma(-g, g, x), h, g);
  inv = 2.0 * h;
  inv = fma(inv, fma(-inv, root, 1.0), inv);
}

// Factor of a 32 x 32 diagonal block by one wavefront, lane i its row i (d[k], k <= i; lanes 32 .. 63 repeat them): pivot(j, 1 / L_jj) is
// called by lane j.
template <typename Pivot>
__device__ __forceinline__ void chol_diagonal(double (&d)[FIRA_CHOL_NB], double floor_piv, Pivot pivot) {
  const int lane = threadIdx.x & 63, row = lane & (FIRA_CHOL_NB - 1);
#pragma unroll
  for (int j = 0; j < FIRA_CHOL_NB; ++j) {
    double piv, inv;
    sqrt_and_inverse(fmax(lane_value(d[j], j), floor_piv), piv, inv);
    const double lj = d[j] * inv;          // (rows above j hold what nobody reads)
    d[j] = row == j ? piv : lj;
    if (lane == j) pivot(j, inv);
#pragma unroll
    for (int k = j + 1; k < FIRA_CHOL_NB; ++k) d[k] = fma(-lj, lane_value(lj, k), d[k]);
    __builtin_amdgcn_sched_barrier(0);     // (else the lane reads of many columns are gathered, and spill)
  }
}
// One row of the panel below it, x D^T = x: DT holds the factor by columns, rinv the reciprocals of its diagonal.
__device__ __forceinline__ void chol_panel_row(double (&x)[FIRA_CHOL_NB], const double* DT, const double* rinv) {
#pragma unroll
  for (int k = 0; k < FIRA_CHOL_NB; ++k) {
    int col = k * (FIRA_CHOL_NB + 2);      // known only when x[k] is: the factor is read column by column (gathered at the top, it spills)
    asm volatile("" : "+s"(col) : "v"(x[k]));
    x[k] *= rinv[k];
#pragma unroll
    for (int j = k + 1; j < FIRA_CHOL_NB; ++j) x[j] = fma(-x[k], DT[col + j], x[j]);
  }
}

__global__ __launch_bounds__(FIRA_CHOL_THREADS) void fira_refresh_chol_kernel(const FiraRefreshEnt* __restrict__ ents, int pan_rows) {
  constexpr int NB = FIRA_CHOL_NB, PP = NB + 1, DP = NB + 2;
  __shared__ __attribute__((aligned(16))) double DT[NB * DP];   // the diagonal block's factor, by columns: L[i][k] at k * DP + i
  __shared__ double rinv_s[NB];
  __shared__ double dmax_s[FIRA_CHOL_THREADS / 64];
  // the panel below the diagonal block, [rows][PP], while it fits (pan_rows rows of dynamic LDS):
  // the panel solve and the trailing update then read it from LDS instead of walking through memory
  extern __shared__ __attribute__((aligned(16))) double chol_pan[];
  const FiraRefreshEnt e = ents[blockIdx.x];
  if (refresh_pass_done(e)) return;
  const int r = e.r, t = threadIdx.x, lane = t & 63, wave = t >> 6;
  gptr<double> C = as_global(e.C);
  {
    double mx = 0.0;
    for (int i = t; i < r; i += FIRA_CHOL_THREADS) mx = fmax(mx, C[(long long)i * r + i]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o, 64));
    if (lane == 0) dmax_s[wave] = mx;
  }
  __syncthreads();
  double dmax = 0.0;
#pragma unroll
  for (int w = 0; w < FIRA_CHOL_THREADS / 64; ++w) dmax = fmax(dmax, dmax_s[w]);
  const double floor_piv = dmax * 1e-24 + 1e-300;
  for (int jb = 0; jb < r; jb += NB) {
    const int nb = min(NB, r - jb);
    // (1) diagonal block -> LDS -> registers of the first wavefront (lane i: row i; identity past the end)
    for (int x = t; x < NB * NB; x += FIRA_CHOL_THREADS) {
      const int i = x / NB, k = x % NB;
      DT[k * DP + i] = (i < nb && k <= i) ? C[(long long)(jb + i) * r + jb + k] : (i == k ? 1.0 : 0.0);
    }
    __syncthreads();
    if (wave == 0) {
      const int row = lane & (NB - 1);
      double d[NB];
#pragma unroll
      for (int k = 0; k < NB; ++k) d[k] = DT[k * DP + row];
      chol_diagonal(d, floor_piv, [&](int j, double inv) { rinv_s[j] = inv; });
      if (lane < NB) {
#pragma unroll
        for (int k = 0; k < NB; ++k) DT[k * DP + row] = k <= row ? d[k] : 0.0;
      }
    }
    __syncthreads();
    for (int x = t; x < NB * NB; x += FIRA_CHOL_THREADS) {
      const int i = x / NB, k = x % NB;
      if (i < nb && k <= i) C[(long long)(jb + i) * r + jb + k] = DT[k * DP + i];
    }
    // (2) panel: rows below the block (which is then a whole one), X D^T = C_panel, forward substitution along its columns
    const int below = r - (jb + nb);
    const bool in_lds = below <= pan_rows;
    if (in_lds) {
      for (int x = t; x < below * NB; x += FIRA_CHOL_THREADS) {
        const int i = x / NB, k = x % NB;
        chol_pan[i * PP + k] = C[(long long)(jb + NB + i) * r + jb + k];
      }
      __syncthreads();
    }
    for (int i = t; i < below; i += FIRA_CHOL_THREADS) {
      gptr<double> grow = C + (long long)(jb + NB + i) * r + jb;
      double x[NB];
#pragma unroll
      for (int k = 0; k < NB; ++k) x[k] = in_lds ? chol_pan[i * PP + k] : grow[k];
      chol_panel_row(x, DT, rinv_s);
#pragma unroll
      for (int k = 0; k < NB; ++k) {
        if (in_lds) chol_pan[i * PP + k] = x[k];
        else grow[k] = x[k];
      }
    }
    __syncthreads();   // (HIP's barrier also waits for this wave's global stores)
    if (in_lds) {
      for (int x = t; x < below * NB; x += FIRA_CHOL_THREADS) {
        const int i = x / NB, k = x % NB;
        C[(long long)(jb + NB + i) * r + jb + k] = chol_pan[i * PP + k];
      }
      // (3) trailing triangle: C[i][k] -= sum_p P[i][p] P[k][p],  jb+NB <= k <= i < r,  P = the panel, on the matrix
      // pipe: 32 x 32 blocks of the triangle dealt out to the wavefronts, operands from the panel in
      // LDS (rows past the end are clamped to the last row; what they produce is not stored)
      const int nb32 = (below + 31) / 32;
      int cnt = 0;
      for (int bi = 0; bi < nb32; ++bi)
        for (int bk = 0; bk <= bi; ++bk, ++cnt) {
          if (cnt % (FIRA_CHOL_THREADS / 64) != wave) continue;
          double old[2][2][4];
          gptr<double> Cb = C + (long long)(jb + NB + 32 * bi) * r + jb + NB + 32 * bk;
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
              for (int v = 0; v < 4; ++v) {
                const int ri = 16 * i + (lane >> 4) + 4 * v, ck = 16 * j + (lane & 15);
                const bool in = 32 * bi + ri < below && 32 * bk + ck <= 32 * bi + ri;
                old[i][j][v] = in ? Cb[(long long)ri * r + ck] : 0.0;
              }
          const int m0 = min(32 * bi + (lane & 15), below - 1), m1 = min(32 * bi + 16 + (lane & 15), below - 1);
          const int n0 = min(32 * bk + (lane & 15), below - 1), n1 = min(32 * bk + 16 + (lane & 15), below - 1);
          RefreshAcc acc;
          refresh_acc_zero(acc);
#pragma unroll
          for (int k4 = 0; k4 < NB; k4 += 4) {
            const int k = k4 + (lane >> 4);
            const double a0 = chol_pan[m0 * PP + k], a1 = chol_pan[m1 * PP + k];
            const double b0 = chol_pan[n0 * PP + k], b1 = chol_pan[n1 * PP + k];
            refresh_acc_step(acc, a0, a1, b0, b1);
          }
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
              for (int v = 0; v < 4; ++v) {
                const int ri = 16 * i + (lane >> 4) + 4 * v, ck = 16 * j + (lane & 15);
                if (32 * bi + ri < below && 32 * bk + ck <= 32 * bi + ri) Cb[(long long)ri * r + ck] = old[i][j][v] - acc.v[i][j][v];
              }
        }
    } else {
    const int nt4 = (below + 3) / 4;
    for (int x = t; x < nt4 * nt4; x += FIRA_CHOL_THREADS) {
      const int bi = x / nt4, bk = x % nt4;
      if (bk > bi) continue;
      const int i0 = jb + nb + 4 * bi, k0 = jb + nb + 4 * bk;
      double acc[4][4];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[i][k] = 0.0;
      for (int p = 0; p < nb; ++p) {
        double a[4], b[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          a[i] = (i0 + i < r) ? C[(long long)(i0 + i) * r + jb + p] : 0.0;
          b[i] = (k0 + i < r) ? C[(long long)(k0 + i) * r + jb + p] : 0.0;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int k = 0; k < 4; ++k) acc[i][k] += a[i] * b[k];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (i0 + i < r && k0 + k <= i0 + i) C[(long long)(i0 + i) * r + k0 + k] -= acc[i][k];
    }
    }
    __syncthreads();
  }
}

// Factorisation and the inverses of its diagonal blocks in one launch for ranks up to 128 (lists of nothing larger), whose whole matrix fits
// in LDS: the kernels above and below go through memory between their steps.  The same operations in the same order, and the chain
// of those is what is left: 56 matrices of r = 128 98 us, 88 and 16 in two launches (a refresh of 8 blocks of 512 x 1376 729 -> 693 us, where
// the estimate's last kernel, whose loads run side by side now, has 11 of it; 24 of 1024 x 2736 at r = 128 2672 -> 2600).
// LDS: the factor in rows of FIRA_CHOL_SMALL_PITCH (an odd number of doubles), identity past r.  Of the half above the diagonal, rows 0 .. 63
// of columns 64 .. 127 take the inverses of the 32 x 32 triangles; when the factor has left, the quarter below takes the products.
#define FIRA_CHOL_SMALL_R 128
#define FIRA_CHOL_SMALL_PITCH (FIRA_CHOL_SMALL_R + 1)
#define FIRA_CHOL_SMALL_LDS (FIRA_CHOL_SMALL_R * FIRA_CHOL_SMALL_PITCH * 8)
__global__ __launch_bounds__(FIRA_CHOL_THREADS) void fira_refresh_chol_small_kernel(const FiraRefreshEnt* __restrict__ ents) {
  constexpr int NB = FIRA_CHOL_NB, DP = NB + 2, P = FIRA_CHOL_SMALL_PITCH, N = FIRA_CHOL_SMALL_R, WAVES = FIRA_CHOL_THREADS / 64;
  __shared__ __attribute__((aligned(16))) double DT[NB * DP];   // the diagonal block's factor, by columns: L[i][k] at k * DP + i
  __shared__ double rinv_s[N];
  __shared__ double dmax_s[WAVES];
  extern __shared__ __attribute__((aligned(16))) double chol_a[];
  const FiraRefreshEnt e = ents[blockIdx.x];
  if (refresh_pass_done(e)) return;
  const int r = e.r, r32 = (r + NB - 1) / NB * NB, t = threadIdx.x, lane = t & 63, wave = t >> 6;
  gptr<double> C = as_global(e.C);
  {
    constexpr int PASSES = N * N / FIRA_CHOL_THREADS;
    double mx = 0.0;
#pragma unroll
    for (int g = 0; g < PASSES; g += 8) {
      double v[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int x = t + FIRA_CHOL_THREADS * (g + q), i = x / N, k = x % N;
        v[q] = k <= i && i < r ? C[(unsigned)(i * r + k)] : (i == k ? 1.0 : 0.0);
      }
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int x = t + FIRA_CHOL_THREADS * (g + q), i = x / N, k = x % N;
        chol_a[i * P + k] = v[q];
        if (i == k && i < r) mx = fmax(mx, v[q]);
      }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o, 64));
    if (lane == 0) dmax_s[wave] = mx;
  }
  __syncthreads();
  double dmax = 0.0;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) dmax = fmax(dmax, dmax_s[w]);
  const double floor_piv = dmax * 1e-24 + 1e-300;
  for (int jb = 0; jb < r; jb += NB) {
    double* D = chol_a + jb * P + jb;
    if (wave == 0) {
      const int row = lane & (NB - 1);
      double d[NB];
#pragma unroll
      for (int k = 0; k < NB; ++k) d[k] = k <= row ? D[row * P + k] : 0.0;
      chol_diagonal(d, floor_piv, [&](int j, double inv) { rinv_s[j] = inv; });
      if (lane < NB) {
#pragma unroll
        for (int k = 0; k < NB; ++k) {
          const double v = k <= row ? d[k] : 0.0;
          DT[k * DP + row] = v;
          if (k <= row) D[row * P + k] = v;
        }
      }
    }
    __syncthreads();
    const int below = r32 - jb - NB;
    double* pan = chol_a + (jb + NB) * P + jb;
    if (t < below) {
      double x[NB];
#pragma unroll
      for (int k = 0; k < NB; ++k) x[k] = pan[t * P + k];
      chol_panel_row(x, DT, rinv_s);
#pragma unroll
      for (int k = 0; k < NB; ++k) pan[t * P + k] = x[k];
    }
    __syncthreads();
    // trailing triangle: blocks of 32 x 32 (what lies above the diagonal in the diagonal ones is never read)
    int cnt = 0;
    for (int bi = 0; bi < below; bi += NB)
      for (int bk = 0; bk <= bi; bk += NB, ++cnt) {
        if (cnt % WAVES != wave) continue;
        const int m0 = bi + (lane & 15), n0 = bk + (lane & 15);
        RefreshAcc acc;
        refresh_acc_zero(acc);
#pragma unroll
        for (int k4 = 0; k4 < NB; k4 += 4) {
          const int k = k4 + (lane >> 4);
          refresh_acc_step(acc, pan[m0 * P + k], pan[(m0 + 16) * P + k], pan[n0 * P + k], pan[(n0 + 16) * P + k]);
        }
        double* T = chol_a + (jb + NB + bi) * P + jb + NB + bk;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              const int ri = 16 * i + (lane >> 4) + 4 * v, ck = 16 * j + (lane & 15);
              if (bk < bi || ck <= ri) T[ri * P + ck] -= acc.v[i][j][v];
            }
      }
    __syncthreads();
  }
  for (int x = t; x < r * N; x += FIRA_CHOL_THREADS) {
    const int i = x / N, k = x % N;
    if (k <= i) C[(unsigned)(i * r + k)] = chol_a[i * P + k];
  }
  if (t < N) rinv_s[t] = 1.0 / chol_a[t * P + t];
  __syncthreads();
  // fira_refresh_diaginv_kernel's steps, wave w < 4 the triangle at 32 w
  const int blocks = (r + 63) / 64;
  double* X = chol_a + 64;                            // triangle w: X[(32 (w >> 1) + i) P + 32 (w & 1) + c]
  if (wave < 2 * blocks && lane < NB) {
    const double* L = chol_a + NB * wave * (P + 1);
    double x[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) x[i] = i == lane ? 1.0 : 0.0;
#pragma unroll
    for (int p = 0; p < NB; ++p) {
      x[p] *= rinv_s[NB * wave + p];
#pragma unroll
      for (int i = p + 1; i < NB; ++i) x[i] = fma(-L[i * P + p], x[p], x[i]);
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) X[(NB * (wave >> 1) + i) * P + NB * (wave & 1) + lane] = x[i];
  }
  __syncthreads();
  const int J = t >> 8, row = (t & 255) >> 3, c4 = (t & 7) * 4;      // 256 threads to a block, four of a row's values each
  const double* XA = X + NB * J * P;
  const double* XB = XA + NB;
  double* W = chol_a + 64 * P + NB * J * P;           // (the factor's lower left quarter has left)
  double q[4] = {0.0, 0.0, 0.0, 0.0};
  if (J < blocks) {
    const double* Cq = chol_a + (64 * J + NB) * P + 64 * J;
    for (int k = 0; k < NB; ++k)
#pragma unroll
      for (int c = 0; c < 4; ++c) q[c] = fma(Cq[row * P + k], XA[k * P + c4 + c], q[c]);
#pragma unroll
    for (int c = 0; c < 4; ++c) W[row * P + c4 + c] = q[c];
  }
  __syncthreads();
  if (J >= blocks) return;
#pragma unroll
  for (int c = 0; c < 4; ++c) q[c] = 0.0;
  for (int k = 0; k < NB; ++k)
#pragma unroll
    for (int c = 0; c < 4; ++c) q[c] = fma(XB[row * P + k], W[k * P + c4 + c], q[c]);
  gptr<double> inv = reinterpret_cast<gptr<double>>(as_global(e.inst)) + (size_t)J * 64 * 64;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    inv[row * 64 + c4 + c] = XA[row * P + c4 + c];
    inv[row * 64 + NB + c4 + c] = 0.0;
    inv[(NB + row) * 64 + c4 + c] = -q[c];
    inv[(NB + row) * 64 + NB + c4 + c] = XB[row * P + c4 + c];
  }
}

// Q = Y L^-T, i.e. every row solves  q L^T = y  by forward substitution, done in column blocks of 64:
//     Q_J = (Y_J - Q_{<J} L_{J,<J}^T) inv(L_JJ)^T.
// Rows do not depend on each other, so a workgroup takes 64 of them through all column blocks, reading back the blocks of Q
// that it wrote before (fp32, as the result is stored).  Everything but the 64 x 64 inverses of the diagonal blocks is a dense
// product, tiled like the Gram kernel (64 x 64 output tile, fp64 on the matrix pipe, operands staged through LDS
// with the next stage's values requested into registers meanwhile).  The inverses of the diagonal blocks come from a small
// kernel of their own (one thread per column of an inverse) and live in the scratch of the installation,
// which is idle until the solves are done.  (Forms that kept a workgroup's rows in LDS and walked along
// the columns, one row per lane with L read from memory or staged in LDS, ran at a tenth of the fp64
// rate: bound by the latency, or the LDS bandwidth, of the operand every lane shares.)
// The staged operands and, after them, Y_J - update share the LDS (33 KB, four workgroups per CU: the stages of 16 k
// are short, and what hides their barriers is other workgroups); the first half of the inverse is requested before
// the barrier in front of the products it meets.  168 matrices of 2048 rows at r = 512: 1.95 ms; 2.45 ms with a
// launch per column block, whose staged operands met in LDS four to a bank.
#define FIRA_SOLVE_LD 66   // doubles per row of Y_J - update: the fragment reads of 16 rows x 2 columns fall on distinct banks
#define FIRA_SOLVE_LDS (64 * FIRA_SOLVE_LD * 8)   // [64][FIRA_SOLVE_LD] Y_J - update; before that the staged Q and L
// Column swizzle of a staged K row: four rows that one store instruction touches fall on distinct banks.
__device__ __forceinline__ int solve_swz_q(int k) { return 16 * ((k >> 2) & 3); }
__device__ __forceinline__ int solve_swz_l(int k) { return 8 * ((k >> 2) & 3); }

// inv(L_JJ) for every diagonal block J of a matrix: inv[J][k][c], k >= c (zero above the diagonal).
// Rows and columns beyond r act as an identity.  By halves: the inverses of the two 32 x 32 triangles A and B, one
// column per lane in registers (independent multiply-adds per row of the substitution), then the lower left quarter
// -inv(B) C inv(A).  (48 us for 168 matrices of r = 512; 390 us as one chain of 64 dependent rows per lane.)
__global__ __launch_bounds__(256) void fira_refresh_diaginv_kernel(const FiraRefreshEnt* __restrict__ ents) {
  constexpr int H = 32, DP = H + 2;
  __shared__ __attribute__((aligned(16))) double LT[2][H * DP];   // the triangles by columns: L[i][k] at k * DP + i
  __shared__ double Cq[H][H + 1], W[H][H + 1], rinv[2][H];
  __shared__ double X[2][H][H + 1];
  const FiraRefreshEnt e = ents[blockIdx.y];
  const int r = e.r, j0 = blockIdx.x * FIRA_SOLVE_JB, t = threadIdx.x;
  if (j0 >= r || refresh_pass_done(e)) return;
  gptr<const double> Lm = as_global<const double>(e.C);
#pragma unroll
  for (int p = 0; p < 16; ++p) {
    const int x = t + 256 * p, i = x >> 6, k = x & 63;
    const bool in = j0 + i < r && k <= i;
    const double v = in ? Lm[(long long)(j0 + i) * r + j0 + k] : (i == k ? 1.0 : 0.0);
    if (i >= H && k < H) Cq[i - H][k] = v;
    else if (i < H && k < H) LT[0][k * DP + i] = v;
    else if (i >= H) LT[1][(k - H) * DP + i - H] = v;
    if (i == k) rinv[i / H][i % H] = 1.0 / v;
  }
  __syncthreads();
  if (t < 2 * H) {
    const int half = t / H, c = t % H;      // column c of the inverse of a triangle: L x = e_c
    double x[H];
#pragma unroll
    for (int i = 0; i < H; ++i) x[i] = i == c ? 1.0 : 0.0;
#pragma unroll
    for (int p = 0; p < H; ++p) {
      x[p] *= rinv[half][p];
#pragma unroll
      for (int i = p + 1; i < H; ++i) x[i] = fma(-LT[half][p * DP + i], x[p], x[i]);
    }
#pragma unroll
    for (int i = 0; i < H; ++i) X[half][i][c] = x[i];
  }
  __syncthreads();
  const int row = t >> 3, c4 = (t & 7) * 4;
  double q[4] = {0.0, 0.0, 0.0, 0.0};
  for (int k = 0; k < H; ++k)
#pragma unroll
    for (int c = 0; c < 4; ++c) q[c] = fma(Cq[row][k], X[0][k][c4 + c], q[c]);
#pragma unroll
  for (int c = 0; c < 4; ++c) W[row][c4 + c] = q[c];
  __syncthreads();
#pragma unroll
  for (int c = 0; c < 4; ++c) q[c] = 0.0;
  for (int k = 0; k < H; ++k)
#pragma unroll
    for (int c = 0; c < 4; ++c) q[c] = fma(X[1][row][k], W[k][c4 + c], q[c]);
  gptr<double> inv = reinterpret_cast<gptr<double>>(as_global(e.inst)) + (size_t)blockIdx.x * 64 * 64;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    inv[row * 64 + c4 + c] = X[0][row][c4 + c];
    inv[row * 64 + H + c4 + c] = 0.0;
    inv[(H + row) * 64 + c4 + c] = -q[c];
    inv[(H + row) * 64 + H + c4 + c] = X[1][row][c4 + c];
  }
}

// All of Q for 64 rows.
__global__ __launch_bounds__(256, 4) void fira_refresh_solve_kernel(const FiraRefreshEnt* __restrict__ ents) {
  __shared__ __attribute__((aligned(16))) char solve_lds[FIRA_SOLVE_LDS];
  float* sa = reinterpret_cast<float*>(solve_lds);                                   // [16][FIRA_STAGE_LD]  Q[s0 + i][k0 + kk]
  double* sb = reinterpret_cast<double*>(solve_lds + 16 * FIRA_STAGE_LD * 4);        // [16][FIRA_STAGE_LD]  L[j0 + j][k0 + kk]
  double (*st)[FIRA_SOLVE_LD] = reinterpret_cast<double (*)[FIRA_SOLVE_LD]>(solve_lds);   // Y_J - update
  const FiraRefreshEnt e = ents[blockIdx.y];
  const int r = e.r, s0 = blockIdx.x * 64;
  if (s0 >= e.S || refresh_pass_done(e)) return;
  gptr<const float> Y = as_global<const float>(e.Y);
  gptr<const double> Lm = as_global<const double>(e.C);
  gptr<float> Q = as_global(e.Q);
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int m0 = 32 * (wave >> 1) + (lane & 15), n0 = 32 * (wave & 1) + (lane & 15), kq = lane >> 4;
  const int lr = t >> 2, lk = (t & 3) * 4;      // staging: row (or column of the block) lr, four k from lk
  for (int j0 = 0; j0 < r; j0 += FIRA_SOLVE_JB) {
    RefreshAcc acc;
    refresh_acc_zero(acc);
    // (j0 is a multiple of 64: whole tiles along k, all inside the matrix.)  The next stage's values are requested
    // into registers before the current one is multiplied.
    f32x4 rq;
    double rl[4];
    auto fetch = [&](int k0) {
      rq = refresh_load4(Q + (long long)s0 * r + k0, lr, lk, e.S - s0, r, r);
      if (j0 + lr < r) {
        gptr<const double> pl = Lm + (long long)j0 * r + k0 + (unsigned)(lr * r + lk);
        if ((r & 1) == 0) {
          typedef double f64x2_t __attribute__((ext_vector_type(2)));
          const f64x2_t u = *reinterpret_cast<gptr<const f64x2_t>>(pl), w = *reinterpret_cast<gptr<const f64x2_t>>(pl + 2);
          rl[0] = u.x; rl[1] = u.y; rl[2] = w.x; rl[3] = w.y;
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q) rl[q] = pl[q];
        }
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) rl[q] = 0.0;
      }
    };
    if (j0 > 0) fetch(0);
    for (int k0 = 0; k0 < j0; k0 += 16) {
      const float qv[4] = {rq.x, rq.y, rq.z, rq.w};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        sa[(lk + q) * FIRA_STAGE_LD + (lr ^ solve_swz_q(lk))] = qv[q];
        sb[(lk + q) * FIRA_STAGE_LD + (lr ^ solve_swz_l(lk))] = rl[q];
      }
      __syncthreads();
      if (k0 + 16 < j0) fetch(k0 + 16);
#pragma unroll
      for (int k4 = 0; k4 < 16; k4 += 4) {       // sum_k Q[row][k] L[j0 + col][k]
        const int k = k4 + kq;
        const float* pa = sa + k * FIRA_STAGE_LD;
        const double* pb = sb + k * FIRA_STAGE_LD;
        refresh_acc_step(acc, (double)pa[m0 ^ solve_swz_q(k4)], (double)pa[(m0 + 16) ^ solve_swz_q(k4)],
                         pb[n0 ^ solve_swz_l(k4)], pb[(n0 + 16) ^ solve_swz_l(k4)]);
      }
      __syncthreads();
    }
    // T = Y_J - update  (the last stage's barrier has freed the staged operands)
    gptr<const double> inv = reinterpret_cast<gptr<const double>>(as_global(e.inst)) + (size_t)j0 * 64;
    double b0[8], b1[8];
    auto fetch_inv = [&](int k0) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        b0[i] = inv[n0 * 64 + k0 + 4 * i + kq];
        b1[i] = inv[(n0 + 16) * 64 + k0 + 4 * i + kq];
      }
    };
    gptr<const float> Yb = Y + (long long)s0 * r + j0;
    gptr<float> Qb = Q + (long long)s0 * r + j0;
    refresh_acc_foreach(acc, [&](int row, int col, double v) {
      const double yv = (s0 + row < e.S && j0 + col < r) ? (double)Yb[row * r + col] : 0.0;
      st[row][col] = yv - v;
    });
    fetch_inv(0);
    __syncthreads();
    // Q_J = T inv^T:  q[row][k] = sum_{c <= k} T[row][c] inv[k][c]   (inv is zero above its diagonal: the left columns take half the c)
    refresh_acc_zero(acc);
    auto half = [&](int k0) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int k = k0 + 4 * i + kq;
        refresh_acc_step(acc, st[m0][k], st[m0 + 16][k], b0[i], b1[i]);
      }
    };
    half(0);
    if (wave & 1) {
      fetch_inv(32);
      half(32);
    }
    refresh_acc_foreach(acc, [&](int row, int k, double v) {
      if (s0 + row < e.S && j0 + k < r) Qb[row * r + k] = (float)v;
    });
    __syncthreads();   // this block of Q is there for the whole workgroup, and T has been read
  }
}

// ------------------------------------------------------------------------------------------------
// Installation of the listed matrices' projectors from their Q buffers, one launch per phase for all
// of them (blockIdx.y = list entry) instead of four launches per matrix: the operand copies Pn / PT
// (fira_prep_projector_kernel) and the estimate of ||P^T P - I|| behind the Gram gate (the three
// fira_ortho_* kernels), each with its own scratch.
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void fira_refresh_prep_kernel(const FiraMat* __restrict__ mats, const FiraRefreshEnt* __restrict__ ents) {
  const FiraRefreshEnt e = ents[blockIdx.y];
  if (e.q_dtype == 1) prep_projector_body<true>(mats[e.mat], reinterpret_cast<const bf16_raw*>(e.Q));
  else prep_projector_body<true>(mats[e.mat], (const float*)(refresh_pass_done(e) ? e.Y : e.Q));   // (a second pass that had nothing to do left its input as the result)
}
// Between two rounds: the basis as PT only (271 us there, 329 with both copies).
__global__ __launch_bounds__(256) void fira_refresh_round_kernel(const FiraMat* __restrict__ mats, const FiraRefreshEnt* __restrict__ ents) {
  const FiraRefreshEnt e = ents[blockIdx.y];
  prep_projector_body<false>(mats[e.mat], (const float*)e.Q);
}
__global__ __launch_bounds__(256) void fira_refresh_ortho_y_kernel(const FiraMat* __restrict__ mats, const FiraRefreshEnt* __restrict__ ents) {
  const FiraRefreshEnt e = ents[blockIdx.y];
  if ((int)blockIdx.x * 4 >= e.S) return;
  ortho_y_body(mats[e.mat], e.inst);
}
__global__ __launch_bounds__(256) void fira_refresh_ortho_z_kernel(const FiraMat* __restrict__ mats, const FiraRefreshEnt* __restrict__ ents) {
  const FiraRefreshEnt e = ents[blockIdx.y];
  ortho_z_body(mats[e.mat], e.inst, e.inst + (size_t)e.S * 4);
}
__global__ __launch_bounds__(256) void fira_refresh_ortho_final_kernel(const FiraMat* __restrict__ mats, const FiraRefreshEnt* __restrict__ ents,
                                                                       FiraScal* __restrict__ scal, FiraGate* __restrict__ gate) {
  __shared__ float red[4][4];
  const FiraRefreshEnt e = ents[blockIdx.x];
  ortho_final_body(mats[e.mat], e.inst + (size_t)e.S * 4, scal, gate, e.mat, red);
}
