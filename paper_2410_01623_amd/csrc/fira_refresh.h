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
// unit's.  Both have the same peak, of which the matrix pipe sustains 77 TFLOP/s, on one sum in turn as on eight, and the vector unit 55 to 60; together they give
// 72 (fira_microbench).  One instruction does 1024 of them, which frees the issue slots that the vector form spends on conversions and LDS reads.
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

// Place of element (row, col), col <= row, of the Gram matrix and its factor.  Above the ranks of fira_refresh_chol_small_kernel they are kept as 32 x 32
// tiles, block row after block row of the lower triangle (r^2 / 2 + 16 r doubles of the r^2 there are).  A quarter of a tile, 16 x 16, holds its
// columns two by two, those with (column % 4) / 2 = 0 first: the 16 rows x 8 columns that one instruction reads as an operand of the factorisation are
// 1 KB of contiguous memory in lane order (fira_refresh_chol_kernel over 168 matrices of r = 512, as it was then: 667 us; 920 with a tile's rows one after the
// other, of which sixteen bytes each make an operand's instruction, and the same with rows of r).
#define FIRA_CHOL_SMALL_R 128
__device__ __forceinline__ bool chol_tiled(int r) { return r > FIRA_CHOL_SMALL_R; }
__device__ __forceinline__ unsigned chol_row(int r, int row) {      // element (row, 0)
  const unsigned i = (unsigned)row, b = i >> 5;
  return chol_tiled(r) ? (b * (b + 1) / 2) * 1024u + ((i >> 4) & 1u) * 512u + (i & 15u) * 2u : i * (unsigned)r;
}
__device__ __forceinline__ unsigned chol_col(int r, int col) {      // ... from there to (row, col)
  const unsigned k = (unsigned)col;
  return chol_tiled(r) ? (k >> 5) * 1024u + ((k >> 4) & 1u) * 256u + ((k >> 1) & 1u) * 128u + ((k >> 2) & 3u) * 32u + (k & 1u) : k;
}
__device__ __forceinline__ unsigned chol_at(int r, int row, int col) { return chol_row(r, row) + chol_col(r, col); }

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
// SMALL: the matrices with r <= FIRA_CHOL_SMALL_R, whose rows are summed in four parts, one after the other or, in lists of few tiles (parts = 4), by a workgroup
// each: a wavefront that has its SIMD to itself waits for its LDS reads, conversions and barriers between multiplies (512 rows are 512 multiplies of 64 cycles, 14 us, and took 32), and
// tiles which leave the chip idle have nothing beside them.  The parts lie in C, in Q, which the solve has yet to write, and in Top, which the way back has read; the factorisation adds
// them up in the same order.  (56 matrices of 512 rows at r = 128: 32 us for a workgroup per
// tile, 23 for four.  A refresh step in one part and in four: 28 matrices of 256 x 688 at r = 64 233 and 220 us; r = 128, 14 of 512 x 1376 362 and 333, 56
// 495 and 485, 84 of 1024 x 2736 1361 and 1344, 168 of 512 x 1376 1005 and 1021.)
#define FIRA_GRAM_KS 32
#define FIRA_GRAM_PARTS 4
// Whether a matrix's Gram matrix lies in parts (where there is room for them), and where part 1 .. 3 does.
__device__ __forceinline__ bool gram_in_parts(const FiraRefreshEnt& e, int parts) {
  return parts == FIRA_GRAM_PARTS && !e.done && e.r <= FIRA_CHOL_SMALL_R && e.S >= 2 * e.r && (long long)e.Lp * e.rq >= 8 * e.r * e.r;
}
__device__ __forceinline__ gptr<double> gram_part(const FiraRefreshEnt& e, int part) {
  return part == 1 ? reinterpret_cast<gptr<double>>(as_global(e.Q)) : reinterpret_cast<gptr<double>>(as_global(e.Top)) + (part - 2) * e.r * e.r;
}
template <bool SMALL>
__global__ __launch_bounds__(256, SMALL ? 4 : 5) void fira_refresh_gram_kernel(const FiraRefreshEnt* __restrict__ ents, int parts) {
  __shared__ __attribute__((aligned(16))) float sa[FIRA_GRAM_KS * FIRA_STAGE_LD], sb[FIRA_GRAM_KS * FIRA_STAGE_LD];
  const FiraRefreshEnt e = ents[blockIdx.y];
  if ((e.r <= FIRA_CHOL_SMALL_R) != SMALL) return;
  if (e.done && !(*as_global<const int>(e.done) & FIRA_PASS_UNSURE)) return;
  const int nt = (e.r + 63) / 64;
  // linear index -> (ta >= tb)
  int ta = 0, rem = blockIdx.x;
  while (ta < nt && rem > ta) { rem -= ta + 1; ++ta; }
  if (ta >= nt) return;
  const int tb = rem;
  const bool own = SMALL && gram_in_parts(e, parts);        // this workgroup has a part of its own
  const int part = own ? (int)blockIdx.z : 0;
  if (SMALL && !own && blockIdx.z > 0) return;
  gptr<const float> Y = as_global<const float>(e.Y);
  const int t = threadIdx.x;
  RefreshAcc acc, sum;
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
  // rows of a part: a quarter of them in whole stages
  const int rows = ((e.S + FIRA_GRAM_PARTS - 1) / FIRA_GRAM_PARTS + FIRA_GRAM_KS - 1) / FIRA_GRAM_KS * FIRA_GRAM_KS;
  const int begin = own ? part * rows : 0, end = own ? min(begin + rows, e.S) : e.S;
  if (SMALL) refresh_acc_zero(sum);
  fetch(begin);
  int until = begin + rows;
  for (int s0 = begin; s0 < end; s0 += FIRA_GRAM_KS) {
    if (SMALL && s0 == until) {                      // one part after the other: the parts' sums are added up as the factorisation adds them
      until += rows;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) sum.v[i][j] += acc.v[i][j];
      refresh_acc_zero(acc);
    }
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const int x = t + 256 * p, sl = x >> 4, c4 = (x & 15) * 4;
      *reinterpret_cast<f32x4*>(&sa[sl * FIRA_STAGE_LD + c4]) = ra[p];
      *reinterpret_cast<f32x4*>(&sb[sl * FIRA_STAGE_LD + c4]) = rb[p];
    }
    __syncthreads();
    if (s0 + FIRA_GRAM_KS < end) fetch(s0 + FIRA_GRAM_KS);
    if (!upper) refresh_acc_steps<FIRA_GRAM_KS>(acc, sa, FIRA_STAGE_LD, 1, sb, FIRA_STAGE_LD, 1);
    __syncthreads();
  }
  if (SMALL) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc.v[i][j] = sum.v[i][j] + acc.v[i][j];
  }
  gptr<double> C = part == 0 ? as_global(e.C) : gram_part(e, part);
  bool off = false;
  refresh_acc_foreach(acc, [&](int row, int col, double v) {
    const int ra_ = ta * 64 + row, cb = tb * 64 + col;
    if (ra_ < e.r && cb < e.r && cb <= ra_) {
      C[chol_at(e.r, ra_, cb)] = v;
      off = off || !(fabs(v - (ra_ == cb ? 1.0 : 0.0)) <= (double)e.done_tol);   // (true for a NaN)
    }
  });
  // Second pass only: is the basis that the pass was given orthonormal already, max |C - I| within the entry's tolerance?
  // (Every tile that finds it is not stores the same value.)
  if (e.done && off) *as_global(e.done) = FIRA_PASS_UNSURE | FIRA_PASS_NEEDED;
}

// (FIRA_PASS_NEEDED counts against the pass: unset until a tile of the Gram matrix shows that the basis is not orthonormal yet)
__device__ __forceinline__ bool refresh_pass_done(const FiraRefreshEnt& e) { return e.done && !(*as_global<const int>(e.done) & FIRA_PASS_NEEDED); }

// In-place Cholesky factorisation of the lower triangle of C (fp64), one workgroup per matrix, 32 columns (a panel) at a time, each panel brought
// up to date with all the columns before it when its turn comes (left-looking: the triangle is read, never rewritten).  A pivot that is not
// safely positive is replaced by a small multiple of the largest diagonal entry.  That
// carries a Y that is deficient by rounding, not one whose gradient has a numerical rank below r: the rounding left of
// the missing directions, divided by such pivots, grows from panel to panel and can end in a basis of NaNs.
//
// What bounds it is the chain of dependent steps of one panel, not its arithmetic.  chol_eliminate therefore does the diagonal block and the rows
// below it in one pass: every wavefront repeats the block's elimination in its lanes 0 .. 31 and carries 32 rows of the panel along in the
// others, whose multiply-adds are the same instructions (and 64 more in a second set of registers where there are many rows; the lane
// reads, two for each multiply-add, are shared).  Rows of the identity carried along become the block's inverse, which the solve needs.
// A column is scaled by 1 / pivot as it is eliminated, and by the square roots when all are known, side by side.
// 168 matrices of r = 512, the inverses of the diagonal blocks included: 560 us (680 while offsets, masks and rows of one panel after the other were held
// across them and 132 registers went to memory); 930 with the panel solved after its block by one row per thread and a trailing triangle rewritten for every panel.
#define FIRA_CHOL_THREADS 512
#define FIRA_CHOL_NB 32
#define FIRA_CHOL_ROWS 512        // rows of a panel that are in LDS at a time, the diagonal block's among them
#define FIRA_CHOL_PITCH (FIRA_CHOL_NB + 1)

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

// Lane i < 32: row i of a 32 x 32 diagonal block (d[k], k <= i; what stands above is never handed on), lanes 32 .. 63 and x, where EXTRA,
// a row each of what lies below it.  Afterwards the block's factor D, and X D^T = what was there.
// (Lane reads in groups of eight: one right before the multiply-add that takes it costs twice as much, 22 cycles against 14.  The next pivot's
// reciprocal is formed beside a column's later groups.)
template <bool EXTRA>
__device__ __forceinline__ void chol_eliminate(double (&d)[FIRA_CHOL_NB], double (&x)[EXTRA ? FIRA_CHOL_NB : 1], int lane, double floor_piv) {
  constexpr int NB = FIRA_CHOL_NB, GROUP = 8;
  double own = 1.0;                        // lane j: pivot j
  double piv, inv;
  auto pivot = [&](int j) {
    piv = fmax(lane_value(d[j], j), floor_piv);
    inv = __builtin_amdgcn_rcp(piv);
    inv = fma(inv, fma(-piv, inv, 1.0), inv);
    inv = fma(inv, fma(-piv, inv, 1.0), inv);
  };
  pivot(0);
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const double t = -d[j] * inv;          // (rows above j hold what nobody reads)
    double tx = 0.0;
    if (EXTRA) tx = -x[j] * inv;
    const double p = piv;
#pragma unroll
    for (int k0 = j + 1; k0 < NB; k0 += GROUP) {
      double b[GROUP];
#pragma unroll
      for (int k = k0; k < NB && k < k0 + GROUP; ++k) b[k - k0] = lane_value(d[j], k);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int k = k0; k < NB && k < k0 + GROUP; ++k) {
        d[k] = fma(t, b[k - k0], d[k]);
        if (EXTRA) x[k] = fma(tx, b[k - k0], x[k]);
      }
      if (k0 == j + 1) pivot(j + 1);
    }
    d[j] = lane == j ? p : d[j];
    own = lane == j ? p : own;
    __builtin_amdgcn_sched_barrier(0);     // (else the lane reads of many columns are gathered, and spill)
  }
  double root, scale;
  sqrt_and_inverse(own, root, scale);
#pragma unroll
  for (int j0 = 0; j0 < NB; j0 += GROUP) {
    double b[GROUP];
#pragma unroll
    for (int j = 0; j < GROUP; ++j) b[j] = lane_value(scale, j0 + j);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < GROUP; ++j) {
      d[j0 + j] *= b[j];
      if (EXTRA) x[j0 + j] *= b[j];
    }
  }
}

// Floor of the pivots: from the largest diagonal entry that a thread has seen.  red: a value per wavefront.
__device__ __forceinline__ double chol_floor(double mx, double* red) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o, 64));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
  __syncthreads();
  double dmax = 0.0;
#pragma unroll
  for (int w = 0; w < FIRA_CHOL_THREADS / 64; ++w) dmax = fmax(dmax, red[w]);
  return dmax * 1e-24 + 1e-300;
}

// acc[i][j] += the products of four k of 16 rows and 16 columns.
template <int RB, int CB>
__device__ __forceinline__ void chol_products(f64x4_t (&acc)[RB][CB], const double (&a)[RB], const double (&b)[CB]) {
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int j = 0; j < CB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
}
// Puts f(row, col, value) in the place of each value that this lane holds.
template <int RB, int CB, typename F>
__device__ __forceinline__ void chol_foreach(f64x4_t (&acc)[RB][CB], int lane, F f) {
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int j = 0; j < CB; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[i][j][v] = f(16 * i + (lane >> 4) + 4 * v, 16 * j + (lane & 15), acc[i][j][v]);
}

// Rows row0 .. row0 + 16 RB - 1 of the panel of columns jb .. jb + 31, C - L[rows][<jb] L[jb ..][<jb]^T, into LDS; row x of pan is the
// matrix's row at(x).  The sums start from -C, which is on its way meanwhile; operands are requested four stages of 16 k ahead.  Of these, lane l
// takes four from 4 (l / 16), and an instruction those with the same place among the four.
template <int RB, typename At>
__device__ __forceinline__ void chol_update(double* pan, gptr<const double> C, int r, int jb, int row0, int lane, At at) {
  typedef double __attribute__((ext_vector_type(2), aligned(8))) f64x2_a8;
  f64x4_t acc[RB][2];
  chol_foreach(acc, lane, [&](int row, int col, double) {
    const int g = at(row0 + row), c = jb + col;
    return g < r && c <= g ? -C[chol_at(r, g, c)] : 0.0;
  });
  gptr<const double> pa[RB], pb[2];
#pragma unroll
  for (int i = 0; i < RB; ++i) pa[i] = C + (chol_row(r, min(at(row0 + 16 * i + (lane & 15)), r - 1)) + chol_col(r, 4 * (lane >> 4)));
#pragma unroll
  for (int i = 0; i < 2; ++i) pb[i] = C + (chol_row(r, min(jb + 16 * i + (lane & 15), r - 1)) + chol_col(r, 4 * (lane >> 4)));
  struct Operands { double a[4][RB], b[4][2]; };
  const int pair = (int)chol_col(r, 2);
  auto load = [&](Operands& o, int k) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int i = 0; i < RB; ++i) {
        const f64x2_a8 u = *reinterpret_cast<gptr<const f64x2_a8>>(pa[i] + (k + h * pair));
        o.a[2 * h][i] = u.x;
        o.a[2 * h + 1][i] = u.y;
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const f64x2_a8 u = *reinterpret_cast<gptr<const f64x2_a8>>(pb[i] + (k + h * pair));
        o.b[2 * h][i] = u.x;
        o.b[2 * h + 1][i] = u.y;
      }
    }
  };
  auto multiply = [&](const Operands& o) {
#pragma unroll
    for (int s = 0; s < 4; ++s) chol_products(acc, o.a[s], o.b[s]);
  };
  if (jb > 0) {                            // (a multiple of 32: an even number of stages; what is requested past the end is not used)
    Operands o[4];
    auto stage = [&](int s) { return (int)chol_col(r, 16 * min(s, jb / 16 - 1)); };
#pragma unroll
    for (int s = 0; s < 4; ++s) load(o[s], stage(s));
    int s0 = 0;
    for (; s0 + 4 <= jb / 16; s0 += 4) {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        multiply(o[s]);
        load(o[s], stage(s0 + s + 4));
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (s0 < jb / 16) {
      multiply(o[0]);
      multiply(o[1]);
    }
  }
  chol_foreach(acc, lane, [&](int row, int col, double v) {
    const int x = row0 + row;
    return pan[x * FIRA_CHOL_PITCH + col] = at(x) < r ? -v : (x == col ? 1.0 : 0.0);      // (identity past the end)
  });
}

// Lower left quarter -B C A of a 64 x 64 inverse, from the inverses A and B of the 32 x 32 triangles and what lies below the first, C, by four wavefronts:
// a wavefront's 16 x 16 of C A goes to W, and then, when all are there, of -B W to store(row, col, value).  Arrays in LDS, P doubles a row.
template <int P>
__device__ __forceinline__ void chol_quarter(f64x4_t& acc, const double* left, const double* right) {
  const int lane = threadIdx.x & 63, wave = (threadIdx.x >> 6) & 3;
  const double *pa = left + (16 * (wave >> 1) + (lane & 15)) * P + (lane >> 4), *pb = right + (lane >> 4) * P + 16 * (wave & 1) + (lane & 15);
  acc = f64x4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int k = 0; k < FIRA_CHOL_NB; k += 4) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(pa[k], pb[k * P], acc, 0, 0, 0);
}
template <typename F>
__device__ __forceinline__ void chol_quarter_foreach(const f64x4_t& acc, F f) {
  const int lane = threadIdx.x & 63, wave = (threadIdx.x >> 6) & 3;
#pragma unroll
  for (int v = 0; v < 4; ++v) f(16 * (wave >> 1) + (lane >> 4) + 4 * v, 16 * (wave & 1) + (lane & 15), acc[v]);
}

__global__ __launch_bounds__(FIRA_CHOL_THREADS) void fira_refresh_chol_kernel(const FiraRefreshEnt* __restrict__ ents) {
  constexpr int NB = FIRA_CHOL_NB, PP = FIRA_CHOL_PITCH, WAVES = FIRA_CHOL_THREADS / 64, PANEL = FIRA_CHOL_ROWS - NB;
  static_assert(FIRA_CHOL_ROWS <= 3 * NB * (WAVES - 1) + NB, "the wavefronts hold a panel's rows and the identity's");
  __shared__ double red[WAVES];
  // the diagonal block's 32 rows and, below them, up to PANEL of the others: [rows][PP]
  extern __shared__ __attribute__((aligned(16))) double chol_pan[];
  const FiraRefreshEnt e = ents[blockIdx.x];
  if (refresh_pass_done(e)) return;
  const int r = e.r, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int t = threadIdx.x;
  gptr<double> C = as_global(e.C);
  double mx = 0.0;
  for (int i = t; i < r; i += FIRA_CHOL_THREADS) mx = fmax(mx, C[chol_at(r, i, i)]);
  const double floor_piv = chol_floor(mx, red);
  for (int jb = 0; jb < r; jb += NB) {
    // (each part of the rows repeats the diagonal block, which is stored with the last)
    for (int base = jb + NB;; base += PANEL) {
      asm volatile("" : "+v"(t));          // (else the offsets, and 32 masks, of all that follows are formed out here, and spill)
      const int lane = t & 63;
      const int rows = max(min(PANEL, r - base), 0), blocks = 1 + (rows + NB - 1) / NB;
      const bool last = base + PANEL >= r;
      auto at = [&](int x) { return x < NB ? jb + x : base + x - NB; };
      // 32 rows to a wavefront at a time, or 16 where that keeps more of them busy
      if (blocks > WAVES)
        for (int b = wave; b < blocks; b += WAVES) chol_update<2>(chol_pan, C, r, jb, NB * b, lane, at);
      else
        for (int b = wave; b < 2 * blocks; b += WAVES) chol_update<1>(chol_pan, C, r, jb, NB / 2 * b, lane, at);
      __syncthreads();
      // the panel's rows, 96 to a wavefront, and the identity's 32 to the last one
      const bool identity = wave == WAVES - 1;
      const int end = NB * blocks, row0 = 3 * NB * wave + lane;
      const bool works = identity ? base == jb + NB : wave == 0 || NB * (3 * wave + 1) < end;
      // (Registers, which this kernel is short of: rows that are set wherever they are used do not live from panel to panel, and x stays one register a
      // value only if its elimination cannot move into the store below. 132 spilled without these two and with lanes formed per function.)
      double d[NB], x[NB];
#pragma unroll
      for (int k = 0; k < NB; ++k) d[k] = x[k] = 0.0;
      if (works) {
        const double* from = chol_pan + (lane < NB ? lane : min(row0, end - 1)) * PP;
#pragma unroll
        for (int k = 0; k < NB; ++k) d[k] = identity && lane >= NB ? (k == lane - NB ? 1.0 : 0.0) : from[k];
        from = chol_pan + min(row0 + 2 * NB, end - 1) * PP;
#pragma unroll
        for (int k = 0; k < NB; ++k) x[k] = from[k];
      }
      __syncthreads();                     // (the block's rows have been read by everybody)
      if (works) {
        chol_eliminate<true>(d, x, lane, floor_piv);
#pragma unroll
        for (int k = 0; k < NB; ++k) asm volatile("" : "+v"(x[k]));
        if (identity) {                    // D^-T, a row per lane
          if (lane >= NB) {
            gptr<double> inv = reinterpret_cast<gptr<double>>(as_global(e.inst)) + (size_t)(jb / 64) * 64 * 64 + (jb & 32) * 65 + lane - NB;
#pragma unroll
            for (int k = 0; k < NB; ++k) inv[k * 64] = k >= lane - NB ? d[k] : 0.0;
          }
        } else {
          if (lane < NB ? wave == 0 : row0 < end) {
            double* to = chol_pan + (lane < NB ? lane : row0) * PP;
#pragma unroll
            for (int k = 0; k < NB; ++k) to[k] = d[k];
          }
          if (row0 + 2 * NB < end) {
            double* to = chol_pan + (row0 + 2 * NB) * PP;
#pragma unroll
            for (int k = 0; k < NB; ++k) to[k] = x[k];
          }
        }
      }
      __syncthreads();
      if (chol_tiled(r)) {                 // a tile is 16 bytes a thread (what stands above the diagonal and past the end is nobody's)
        typedef double f64x2_t __attribute__((ext_vector_type(2)));
        const int i = 16 * (t >> 8) + (t & 15), k = 16 * ((t >> 7) & 1) + 4 * ((t >> 4) & 3) + 2 * ((t >> 6) & 1);
#pragma unroll 4
        for (int b = last ? 0 : 1; b < blocks; ++b) {
          const double* from = chol_pan + (NB * b + i) * PP + k;
          *reinterpret_cast<gptr<f64x2_t>>(C + (chol_at(r, b ? base + NB * (b - 1) : jb, jb) + 2 * t)) = f64x2_t{from[0], from[1]};
        }
      } else {
        for (int y = t + (last ? 0 : NB * NB); y < (NB + rows) * NB; y += FIRA_CHOL_THREADS) {
          const int i = y / NB, k = y % NB, g = at(i);
          if (g < r && jb + k <= g) C[chol_at(r, g, jb + k)] = chol_pan[i * PP + k];
        }
      }
      __syncthreads();                     // (HIP's barrier also waits for this wave's global stores)
      if (last) break;
    }
  }
}

// Factorisation and the inverses of its diagonal blocks in one launch for ranks up to 128 (lists of nothing larger), whose whole matrix fits
// in LDS: the kernels above and below go through memory between their steps.  The same operations in the same order.  56 matrices of r = 128: 38 us, 42
// with the parts of the Gram matrices to add up; 98 with one row per thread below a block and the inverses formed afterwards, a step each for every column (a refresh of 8 blocks of 512 x 1376
// 683 -> 559 us).
// LDS: the factor in rows of FIRA_CHOL_SMALL_PITCH (an odd number of doubles), identity past r.  Of the half above the diagonal, rows 0 .. 63
// of columns 64 .. 127 take the inverses of the 32 x 32 triangles; when the factor has left, the quarter below takes the products.
#define FIRA_CHOL_SMALL_PITCH (FIRA_CHOL_SMALL_R + 1)
#define FIRA_CHOL_SMALL_LDS (FIRA_CHOL_SMALL_R * FIRA_CHOL_SMALL_PITCH * 8)
__global__ __launch_bounds__(FIRA_CHOL_THREADS) void fira_refresh_chol_small_kernel(const FiraRefreshEnt* __restrict__ ents, int parts) {
  constexpr int NB = FIRA_CHOL_NB, P = FIRA_CHOL_SMALL_PITCH, N = FIRA_CHOL_SMALL_R, WAVES = FIRA_CHOL_THREADS / 64;
  __shared__ double red[WAVES];
  extern __shared__ __attribute__((aligned(16))) double chol_a[];
  const FiraRefreshEnt e = ents[blockIdx.x];
  if (refresh_pass_done(e)) return;
  const int r = e.r, t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int blocks = (r + 63) / 64, r32 = (r + NB - 1) / NB * NB;
  gptr<double> C = as_global(e.C);
  double* X = chol_a + 64;                            // the inverse of triangle w: X[(32 (w >> 1) + i) P + 32 (w & 1) + c]
  double mx = 0.0;
  {
    constexpr int PASSES = N * N / FIRA_CHOL_THREADS;
    auto load = [&](auto at_once, auto in_parts) {       // AT values of a thread at a time, and the other parts', in flight
      constexpr int AT = decltype(at_once)::value, MORE = decltype(in_parts)::value ? FIRA_GRAM_PARTS - 1 : 0;
#pragma unroll
      for (int g = 0; g < PASSES; g += AT) {
        double v[MORE + 1][AT];
#pragma unroll
        for (int p = 0; p <= MORE; ++p) {
          gptr<const double> from = p == 0 ? (gptr<const double>)C : (gptr<const double>)gram_part(e, p);
#pragma unroll
          for (int q = 0; q < AT; ++q) {
            const int x = t + FIRA_CHOL_THREADS * (g + q), i = x / N, k = x % N;
            v[p][q] = k <= i && i < r ? from[(unsigned)(i * r + k)] : (i == k && p == 0 ? 1.0 : 0.0);
          }
        }
#pragma unroll
        for (int q = 0; q < AT; ++q) {
          const int x = t + FIRA_CHOL_THREADS * (g + q), i = x / N, k = x % N;
#pragma unroll
          for (int p = 1; p <= MORE; ++p) v[0][q] += v[p][q];
          chol_a[i * P + k] = v[0][q];
          if (i == k && i < r) mx = fmax(mx, v[0][q]);
        }
      }
    };
    if (gram_in_parts(e, parts)) load(std::integral_constant<int, 8>{}, std::true_type{});
    else load(std::integral_constant<int, 16>{}, std::false_type{});
  }
  const double floor_piv = chol_floor(mx, red);
  if (r32 < 64 * blocks)                              // the last 64 columns' second triangle is past the end
    for (int x = t; x < NB * NB; x += FIRA_CHOL_THREADS) X[(r32 / 64 * NB + x / NB) * P + NB + x % NB] = x / NB == x % NB ? 1.0 : 0.0;
  for (int jb = 0; jb < r; jb += NB) {
    const int below = r32 - jb - NB;
    if (jb > 0) {                                     // (rows past r take zeros off an identity)
      for (int u = wave; u < 4 * (below / NB + 1); u += WAVES) {      // 16 x 16 at a time
        const int row0 = jb + 16 * (u >> 1), col0 = jb + 16 * (u & 1);
        f64x4_t acc[1][1];
        chol_foreach(acc, lane, [&](int row, int col, double) { return -chol_a[(row0 + row) * P + col0 + col]; });
        const double *pa = chol_a + (row0 + (lane & 15)) * P + 4 * (lane >> 4), *pb = chol_a + (col0 + (lane & 15)) * P + 4 * (lane >> 4);
        for (int k = 0; k < jb; k += NB) {
          double a[8], b[8];
#pragma unroll
          for (int s = 0; s < 8; ++s) {
            a[s] = pa[k + 16 * (s >> 2) + (s & 3)];
            b[s] = pb[k + 16 * (s >> 2) + (s & 3)];
          }
#pragma unroll
          for (int s = 0; s < 8; ++s) acc[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], b[s], acc[0][0], 0, 0, 0);
        }
        chol_foreach(acc, lane, [&](int row, int col, double v) { return chol_a[(row0 + row) * P + col0 + col] = -v; });
      }
      __syncthreads();
    }
    // wavefront w carries the panel's rows 32 w ..; the one after them, the identity's
    const bool identity = NB * wave == below;
    double d[NB], none[1];
    double* at = chol_a + (jb + (lane < NB ? 0 : NB * wave) + lane) * P + jb;
    if (NB * wave <= below) {
#pragma unroll
      for (int k = 0; k < NB; ++k) d[k] = identity && lane >= NB ? (k == lane - NB ? 1.0 : 0.0) : at[k];
    }
    __syncthreads();
    if (NB * wave <= below) {
      chol_eliminate<false>(d, none, lane, floor_piv);
      if (lane >= NB && identity) {
#pragma unroll
        for (int k = 0; k < NB; ++k) X[(jb / 64 * NB + k) * P + (jb & 32) + lane - NB] = k >= lane - NB ? d[k] : 0.0;
      } else if (lane >= NB || wave == 0) {
#pragma unroll
        for (int k = 0; k < NB; ++k) at[k] = d[k];     // (nobody reads what stands above the diagonal)
      }
    }
    __syncthreads();
  }
  for (int x = t; x < r * N; x += FIRA_CHOL_THREADS) {
    const int i = x / N, k = x % N;
    if (k <= i) C[(unsigned)(i * r + k)] = chol_a[i * P + k];
  }
  // fira_refresh_diaginv_kernel's steps, four wavefronts to a block
  const int J = t >> 8;
  const double* XA = X + NB * J * P;
  const double* XB = XA + NB;
  double* W = chol_a + 64 * P + NB * J * P;           // (the factor's lower left quarter)
  f64x4_t q;
  chol_quarter<P>(q, chol_a + (64 * J + NB) * P + 64 * J, XA);
  __syncthreads();                                    // (which has left)
  chol_quarter_foreach(q, [&](int row, int col, double v) { W[row * P + col] = v; });
  __syncthreads();
  if (J >= blocks) return;
  chol_quarter<P>(q, XB, W);
  gptr<double> inv = reinterpret_cast<gptr<double>>(as_global(e.inst)) + (size_t)J * 64 * 64;
  chol_quarter_foreach(q, [&](int row, int col, double v) {
    inv[row * 64 + col] = XA[row * P + col];
    inv[row * 64 + NB + col] = 0.0;
    inv[(NB + row) * 64 + col] = -v;
    inv[(NB + row) * 64 + NB + col] = XB[row * P + col];
  });
}

// Q = Y L^-T, i.e. every row solves  q L^T = y  by forward substitution, done in column blocks of 64:
//     Q_J = (Y_J - Q_{<J} L_{J,<J}^T) inv(L_JJ)^T.
// Rows do not depend on each other, so a workgroup takes 64 of them through all column blocks, reading back the blocks of Q
// that it wrote before (fp32, as the result is stored).  Everything but the 64 x 64 inverses of the diagonal blocks is a dense
// product, tiled like the Gram kernel (64 x 64 output tile, fp64 on the matrix pipe, operands staged through LDS
// with the next stage's values requested into registers meanwhile).  The inverses of the diagonal blocks are there
// already (their 32 x 32 triangles from the factorisation, which carries rows of an identity along, the quarters below from fira_refresh_diaginv_kernel)
// and live in the scratch of the installation, which is idle until the solves are done.  (Forms that kept a workgroup's rows in LDS and walked along
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
// Rows and columns beyond r act as an identity.  The inverses A and B of the two 32 x 32 triangles are there already (fira_refresh_chol_kernel);
// this adds the lower left quarter -B C A and the zeros.
__global__ __launch_bounds__(256) void fira_refresh_diaginv_kernel(const FiraRefreshEnt* __restrict__ ents) {
  constexpr int H = 32;
  __shared__ double Cq[H][H + 1], W[H][H + 1], X[2][H][H + 1];
  const FiraRefreshEnt e = ents[blockIdx.y];
  const int r = e.r, j0 = blockIdx.x * FIRA_SOLVE_JB, t = threadIdx.x;
  if (j0 >= r || refresh_pass_done(e)) return;
  gptr<const double> Lm = as_global<const double>(e.C);
  gptr<double> inv = reinterpret_cast<gptr<double>>(as_global(e.inst)) + (size_t)blockIdx.x * 64 * 64;
  const bool second = j0 + H < r;          // (the second triangle is past the end otherwise)
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const int x = t + 256 * p, i = x >> 5, k = x & 31;
    X[0][i][k] = inv[i * 64 + k];
    X[1][i][k] = second ? inv[(H + i) * 64 + H + k] : (i == k ? 1.0 : 0.0);
    Cq[i][k] = j0 + H + i < r ? Lm[chol_at(r, j0 + H + i, j0 + k)] : 0.0;
  }
  __syncthreads();
  f64x4_t q;
  chol_quarter<H + 1>(q, &Cq[0][0], &X[0][0][0]);
  chol_quarter_foreach(q, [&](int row, int col, double v) { W[row][col] = v; });
  __syncthreads();
  chol_quarter<H + 1>(q, &X[1][0][0], &W[0][0]);
  chol_quarter_foreach(q, [&](int row, int col, double v) {
    inv[row * 64 + H + col] = 0.0;
    inv[(H + row) * 64 + col] = -v;
    if (!second) inv[(H + row) * 64 + H + col] = X[1][row][col];
  });
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
    const unsigned lrow = chol_row(r, j0 + lr);
    auto fetch = [&](int k0) {
      rq = refresh_load4(Q + (long long)s0 * r + k0, lr, lk, e.S - s0, r, r);
      if (j0 + lr < r) {
        gptr<const double> pl = Lm + (lrow + chol_col(r, k0 + lk));
        if (chol_tiled(r) || (r & 1) == 0) {
          typedef double f64x2_t __attribute__((ext_vector_type(2)));
          const f64x2_t u = *reinterpret_cast<gptr<const f64x2_t>>(pl), w = *reinterpret_cast<gptr<const f64x2_t>>(pl + chol_col(r, 2));
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
