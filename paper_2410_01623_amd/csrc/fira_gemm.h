// Grouped bf16 MFMA contractions of the Fira step for gfx950 (v_mfma_f32_32x32x16_bf16).
//
// Every contraction has the form  D[a][b] = sum_k A[a][k] * B[b][k]  ("A" is the MFMA A operand,
// "B" the MFMA B operand) and runs in 256-thread workgroups, two per CU, each wavefront owning a
// 128 (A) x 64 (B) block of accumulators.  Two independent workgroups per CU matter more than a
// bigger tile: the phases of one (operand requests, LDS traffic, the HBM-bound epilogue) overlap the
// multiplies of the other, which a single workgroup in lockstep on its barriers cannot do.
//
// Operands that the library stores itself (P in both orientations, Z, R) are K-blocked
// ([K/32][rows][32], see kblk_index) and go from global memory straight into an LDS ring with
// LDS-direct loads.  The gradient is the caller's: its rows start at any 2-byte boundary and, when P
// multiplies from the left, it is K-slow (element (a, k) at base[k*ld + a]); it passes through
// registers (K-slow: 4(k) x 8(a) blocks, row-contiguous 16-byte loads, transposed in registers
// before the LDS write).
//
// Accumulator layout of one 32 x 32 block (per lane, 16 floats v = 0..15):
//     b (B row) = lane % 32,   a (A row) = 8*(v/4) + 4*(lane/32) + v%4
// so a lane owns 4 consecutive A rows per group of 4 registers.
#pragma once
#include <type_traits>
#include "fira_device.h"

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16_t;


// [row][64 k] bf16 tile, 128 B per row, 16-byte chunks XOR-swizzled by row so that fragment reads
// and tile writes spread over all banks.
__device__ __forceinline__ int lds_tile_off(int row, int chunk) {
  return row * 128 + (((chunk ^ row ^ (row >> 3) ^ (row >> 6)) & 7) << 4);
}

// 8 consecutive bf16 of a row that has `limit` valid elements, starting at element idx; elements
// outside [0, limit) read as zero and are never touched in memory.  No alignment assumed.
// Branch-free for limit >= 8: the 16-byte load is moved back so that it ends inside the row and the
// value is shifted down again, which also shifts zeros into the out-of-range positions.  (A ragged
// chunk handled with per-element loads costs a serialized memory round trip per element.)
__device__ __forceinline__ u32x4 load8_bf16(gptr<const bf16_raw> row, long long idx, long long limit) {
  if (limit >= 8) {
    long long start = idx < limit - 8 ? idx : limit - 8;
    if (start < 0) start = 0;
    const u32x4 v = *reinterpret_cast<gptr<const u32x4_a2>>(row + start);
    const long long d = idx - start;          // elements to shift out at the low end
    const unsigned sh = d < 8 ? (unsigned)d : 8u;
    // 128-bit logical shift right by 16*sh bits
    const unsigned long long lo = ((unsigned long long)v.y << 32) | v.x, hi = ((unsigned long long)v.w << 32) | v.z;
    const unsigned bits = 16u * sh;
    unsigned long long rlo, rhi;
    if (bits == 0) { rlo = lo; rhi = hi; }
    else if (bits < 64) { rlo = (lo >> bits) | (hi << (64 - bits)); rhi = hi >> bits; }
    else if (bits < 128) { rlo = hi >> (bits - 64); rhi = 0; }
    else { rlo = 0; rhi = 0; }
    return u32x4{(unsigned)rlo, (unsigned)(rlo >> 32), (unsigned)rhi, (unsigned)(rhi >> 32)};
  }
  unsigned w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int e = 0; e < 8; ++e)
    if (idx + e >= 0 && idx + e < limit) w[e >> 1] |= ((unsigned)row[idx + e]) << ((e & 1) * 16);
  return u32x4{w[0], w[1], w[2], w[3]};
}

// 8 bf16 moved down by d (>= 0) elements, zeros from above.
__device__ __forceinline__ u32x4 shift8_bf16(u32x4 v, int d) {
  v = d & 4 ? u32x4{v.z, v.w, 0u, 0u} : v;
  v = d & 2 ? u32x4{v.y, v.z, v.w, 0u} : v;
  v = d & 1 ? u32x4{__builtin_amdgcn_alignbit(v.y, v.x, 16), __builtin_amdgcn_alignbit(v.z, v.y, 16), __builtin_amdgcn_alignbit(v.w, v.z, 16), v.w >> 16} : v;
  return d < 8 ? v : u32x4{0u, 0u, 0u, 0u};
}

struct GemmOperands {
  gptr<const bf16_raw> A;  // A side
  long long lda;      // gradient operand: elements between consecutive A rows (K-contiguous) or K steps
                      // (K-slow); K-blocked operand: its padded row count
  int a_row0, a_rows; // first A row of this tile, number of valid A rows
  int KA;             // valid contraction length on the A side (elements beyond read as zero)
  gptr<const bf16_raw> B;  // B side: always K-blocked, zero padded to a multiple of 64 in K
  long long ldb;      // padded row count of B
  int b_row0, b_rows;
  int KB;             // stored contraction length of B (>= KA, a multiple of 64; ring core: of 32)
  int wrapA = 0, wrapB = 0;   // ring core only: K blocks of 32 after which the operand repeats (Z in two planes meets P twice); 0 = never
};

// Fragments of one k-slice (16) of a wave's 32 TM (A) x 32 TN (B) block and its TM TN MFMAs.
template <int TM, int TN>
struct Frags { bf16x8_t a[TM], b[TN]; };
template <int TM, int TN>
__device__ __forceinline__ void gemm_mfma_slice(f32x16_t (&acc)[TM][TN], const Frags<TM, TN>& f) {
#pragma unroll
  for (int tm = 0; tm < TM; ++tm)
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
      acc[tm][tn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[tm], f.b[tn], acc[tm][tn], 0, 0, 0);
}
// Sum of squares of the A fragments (v_dot2c_f32_bf16: two bf16 products per instruction): with the
// gradient on the A side this accumulates ||G_i||^2 for the wave's A rows at no extra memory traffic.
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float frag_sumsq(const bf16x8_t& f, float sq) {
  const u32x4 w = __builtin_bit_cast(u32x4, f);
  const unsigned d[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const bf16x2_t v = __builtin_bit_cast(bf16x2_t, d[e]);
    sq = __builtin_amdgcn_fdot2_f32_bf16(v, v, sq, false);
  }
  return sq;
}
// ------------------------------------------------------------------------------------------------
// Ring core for the rank-axis contractions (K = r is short, the epilogue is long): 256 threads,
// 256 (A) x 128 (B) tile, two workgroups per CU, so one runs its HBM-bound epilogue while the other
// multiplies.  Both operands are K-blocked, so they go from global memory straight into LDS
// (global_load_lds_dwordx4: lane l of a wave writes 16 bytes at M0 + 16*l) without passing through
// registers, and one load instruction (16 rows x 32 k) reads 1 KB of contiguous memory: row
// segments of 64 B spread over 16 separate rows reach only two thirds of that L2 bandwidth.
// LDS holds a ring of three K stages of 32
// ([row][32 k] bf16, 64 B per row, 24 KB per stage): while stage s is multiplied, stages s+1 and
// s+2 are in flight, and there is one barrier per stage.
//
// The loads are written as inline assembly because the compiler, which cannot tell the ring's
// buffers apart, would wait for every outstanding LDS-direct load before each fragment read.  The
// waits are explicit instead: loads retire in order, so vmcnt(6) (one stage = 6 loads per thread)
// means "everything but the newest stage has landed".  Other vector memory operations the compiler
// may have in flight only make that wait stricter.
//
// Slot layout of a stage: the 16-byte chunk c (8 k) of row r sits at  r*64 + 16*((c ^ f(r)) & 3),
// f(r) = bit2(r) | (bit3(r) ^ bit1(r)) << 1, which makes the fragment reads (32 consecutive rows,
// one chunk) hit distinct 16-byte bank groups within every aligned group of 8 and of 16 lanes.
// Since a lane may fetch any global address, the loader realises the permutation on the global
// side: lane l of a load covers row l/4 of a 16-row group and fetches chunk (l%4) ^ f(l/4).
// Operand rows are padded to whole tiles (zeros), so no row index needs clamping; what the padding
// rows produce lands in accumulators that are never stored.
// ------------------------------------------------------------------------------------------------
#define FIRA_BACK_THREADS 256
#define FIRA_RK 32
#define FIRA_RING_STAGES 3

typedef __attribute__((address_space(3))) char* lds_ptr;

__device__ __forceinline__ int ring_swz(int row) { return ((row >> 2) & 1) | ((((row >> 3) ^ (row >> 1)) & 1) << 1); }
__device__ __forceinline__ int ring_tile_off(int row, int chunk) {
  return row * 64 + (((chunk ^ ring_swz(row)) & 3) << 4);
}

// 16 bytes per lane from base + voff (base wave-uniform) to LDS byte address lds_addr + 16*lane.
// M0 is not preserved; on this target the compiler loads M0 right before each of its own uses.
__device__ __forceinline__ void lds_dma16(const void* base, unsigned voff, unsigned lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :: "v"(voff), "s"(base), "s"(lds_addr) : "memory");
}

// Two wavefronts along either side, each with 32 TM (A) x 32 TN (B): (4, 2) is the tile above, (2, 1) a quarter of it for
// launches that leave the chip idle otherwise.
template <int TM, int TN>
struct RingShape {
  static constexpr int A = 64 * TM * 64, B = 64 * TN * 64, STAGE = A + B;   // bytes of a stage
};
template <int TM, int TN>
__device__ __forceinline__ void ring_compute(f32x16_t (&acc)[TM][TN], const char* stage) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave & 1, wn = wave >> 1;
  const char* la = stage;
  const char* lb = stage + RingShape<TM, TN>::A;
  Frags<TM, TN> f[2];
  auto read = [&](int kk, int q) {           // fragment q (of TM + TN) of slice kk
    const int chunk = 2 * kk + (lane >> 5);
    if (q < TM) f[kk].a[q] = *reinterpret_cast<const bf16x8_t*>(la + ring_tile_off(wm * 32 * TM + 32 * q + (lane & 31), chunk));
    else f[kk].b[q - TM] = *reinterpret_cast<const bf16x8_t*>(lb + ring_tile_off(wn * 32 * TN + 32 * (q - TM) + (lane & 31), chunk));
  };
  // The second slice's fragments are read between the first one's multiplies (see proj_compute): the update over the 7B
  // shapes at r = 1024 16155 -> 15700 us, over the 1B shapes at r = 512 2057 -> 2041.
#pragma unroll
  for (int q = 0; q < TM + TN; ++q) read(0, q);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int x = 0; x < TM * TN; ++x) {
    acc[x / TN][x % TN] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[0].a[x / TN], f[0].b[x % TN], acc[x / TN][x % TN], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < TM + TN; ++q)
      if (q * TM * TN / (TM + TN) == x) read(1, q);
    __builtin_amdgcn_sched_barrier(0);
  }
  gemm_mfma_slice(acc, f[1]);
}

// Both operands K-blocked with lda / ldb padded rows (multiples of 256); KB of the stored k (a multiple of 32).
template <int TM, int TN>
__device__ __forceinline__ void ring_mainloop(f32x16_t (&acc)[TM][TN], char* lds, const GemmOperands& g) {
  typedef RingShape<TM, TN> Shape;
#pragma unroll
  for (int tm = 0; tm < TM; ++tm)
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[tm][tn][v] = 0.0f;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const unsigned lds0 = (unsigned)(size_t)(lds_ptr)lds;
  const int KT = g.KB / FIRA_RK;
  const int lrow = lane >> 2;
  const int chunk = (lane & 3) ^ ring_swz(lrow);
  const unsigned off = (unsigned)(lrow * 64 + chunk * 16);   // inside a 16-row group (1 KB, contiguous)
  // this wave's first group of each operand in K block 0; a K block is rows * 64 bytes further
  const char* pa = reinterpret_cast<const char*>((const bf16_raw*)g.A) + ((long long)g.a_row0 + 16 * TM * wave) * 64;
  const char* pb = reinterpret_cast<const char*>((const bf16_raw*)g.B) + ((long long)g.b_row0 + 16 * TN * wave) * 64;
  auto issue = [&](int s) {
    const unsigned dst = lds0 + (unsigned)((s % FIRA_RING_STAGES) * Shape::STAGE);
    const int sa = (g.wrapA && s >= g.wrapA) ? s - g.wrapA : s, sb = (g.wrapB && s >= g.wrapB) ? s - g.wrapB : s;
    const char* ka = pa + (long long)sa * g.lda * 64;
    const char* kb = pb + (long long)sb * g.ldb * 64;
#pragma unroll
    for (int q = 0; q < TM; ++q) lds_dma16(ka + q * 1024, off, dst + (unsigned)((TM * wave + q) * 1024));
#pragma unroll
    for (int q = 0; q < TN; ++q) lds_dma16(kb + q * 1024, off, dst + (unsigned)(Shape::A + (TN * wave + q) * 1024));
  };
  issue(0);
  if (KT > 1) issue(1);
  for (int s = 0; s < KT; ++s) {
    // stage s has landed (this wave's share; the TM + TN requests of stage s + 1 may be in flight), then everybody's;
    // everybody is also done with stage s-1
    if (s + 1 < KT) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" :: "n"(TM + TN) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
    if (s + 2 < KT) issue(s + 2);            // into the buffer of stage s-1
    ring_compute(acc, lds + (s % FIRA_RING_STAGES) * Shape::STAGE);
  }
}

// ------------------------------------------------------------------------------------------------
// Kernel 1 (pipelined form): low-rank gradient, long-side major:  Rt[i][a] = sum_s G(s, i) P[s][a]
//   LEFT  (m <= n): i = column of G, s = row of G      -> A side is G read K-slow
//   RIGHT (m >  n): i = row of G,    s = column of G   -> A side is G read K-contiguous
//   B side is PT (rank rows, short side along K, K-blocked).
// 256 threads, 128 (A: gradient side) x 256 (B: rank) tile, two independent workgroups per CU so
// that the load/store phases of one overlap the multiplies of the other.  Wave w owns all 128 A rows
// and B rows 64 w .. 64 w + 63.
//   B goes straight from global memory into a three-stage LDS ring (K stages of 32, as in the ring
//   core above).
//   A cannot: a gradient row starts at any 2-byte boundary and the left orientation needs a
//   transpose.  It passes through registers, one K stage of 64 per two ring stages, into a single
//   128-B-per-row LDS tile.
// Per K stage of 64 ("E" half, then "O" half; D(s) = ring stage s of B, A(S) = register stage):
//   E: wait A(S), D(2S); barrier; registers -> LDS A; request D(2S+2), A(S+1); barrier; multiply
//      k = 0..31 of the stage
//   O: wait D(2S+1); barrier; request D(2S+3); multiply k = 32..63
// All requests of the interior path are inline assembly, so the waits can be exact: loads retire in
// order, each request group is 4 instructions per thread, and the queue order is
// A(0) D(0) D(1) | D(2) A(1) | D(3) | D(4) A(2) | D(5) ...; E waits with vmcnt(4) (only the newest
// D may be in flight), O with vmcnt(8).  Matrices with a side of less than eight load A with ordinary guarded loads at the same
// points of the sequence; the compiler's own waits for those only wait longer.
// ------------------------------------------------------------------------------------------------
#define FIRA_PROJ_THREADS 256
#define FIRA_PROJ_LDS_A (FIRA_PA * 128)
#define FIRA_PROJ_RING_STAGE (FIRA_PB * 64)
#define FIRA_PROJ_LDS (FIRA_PROJ_LDS_A + FIRA_RING_STAGES * FIRA_PROJ_RING_STAGE)

// 16 bytes per lane from base + voff into registers; the result may only be read after a wait that
// names the registers (wait_loads below; the names also go into a comment on the instruction, which
// is what the static check of the compiled code keys on).
__device__ __forceinline__ void gload16_async(u32x4& dst, const void* base, unsigned voff) {
  asm volatile("global_load_dwordx4 %0, %1, %2" : "=v"(dst) : "v"(voff), "s"(base) : "memory");
}
template <int N>
__device__ __forceinline__ void wait_loads(u32x4 (&r)[4]) {
  asm volatile("s_waitcnt vmcnt(%4) ; %0 %1 %2 %3" : "+v"(r[0]), "+v"(r[1]), "+v"(r[2]), "+v"(r[3]) : "n"(N) : "memory");
}

// Thread -> element mapping of the A loaders (256 threads, 64 k x 128 rows per stage):
//   K-contiguous: chunk cc = t & 7, rows rr + 32*q, rr = t >> 3, q = 0..3.
//   K-slow:       one 4(k) x 8(a) block per thread: a-block ib (16), k-quad kq (16).  Thread bits
//                 [0:3) -> ib low, bit 3 -> kq low, bit 4 -> ib high, bits [5:8) -> kq high: 8 lanes
//                 read 128 contiguous bytes of one gradient row, and any 16 consecutive lanes write
//                 16 distinct 8-byte LDS slots of a 128-byte bank window (8 chunk positions from the
//                 row swizzle x the two halves of a chunk from kq's low bit).
__device__ __forceinline__ int proj_kslow_ib(int t) { return (t & 7) | ((t >> 1) & 8); }
__device__ __forceinline__ int proj_kslow_kq(int t) { return ((t >> 3) & 1) | ((t >> 4) & ~1); }

// How a tile's gradient is read: all of it there; up to the matrix's edge or the end of the contraction (EDGE): pieces that would leave it are moved back,
// stay in flight like any other, and are moved into place in registers when they are stored; or, for matrices with a side of less than
// eight, value by value (GUARDED).  A launch of few tiles waits for its edge tiles: 56 matrices of 512 x 512 and 512 x 1376, fused
// kernel at r = 128, multiply phase of an edge tile 29 us where pieces were realigned as they were loaded, of any other 12.
enum ProjLoads { PROJ_FAST, PROJ_EDGE, PROJ_GUARDED };
template <bool LEFT, ProjLoads MODE>
struct ProjALoader {
  const GemmOperands& g;
  const char* base;       // wave-uniform, advances along K
  unsigned off[4];        // byte offsets of this thread's four 16-byte loads
  long long step;         // bytes per K stage of 64
  int k0;
  int down;               // EDGE: elements by which a loaded piece is moved down (LEFT: in every stage, RIGHT: in the last)
  __device__ __forceinline__ ProjALoader(const GemmOperands& g_) : g(g_), k0(0), down(0) {
    const int t = threadIdx.x;
    if (LEFT) {
      const int ib = proj_kslow_ib(t), kq = proj_kslow_kq(t);
      int a0 = g.a_row0, a = 8 * ib;
      if (MODE == PROJ_EDGE) {
        a0 = min(a0, g.a_rows - 8);
        const int at = min(g.a_row0 + 8 * ib, g.a_rows - 8);
        down = min(g.a_row0 + 8 * ib - at, 8);
        a = at - a0;
      }
      base = reinterpret_cast<const char*>((const bf16_raw*)g.A + a0);
#pragma unroll
      for (int j = 0; j < 4; ++j) off[j] = (unsigned)(((4 * kq + j) * g.lda + a) * 2);
      step = 64 * g.lda * 2;
    } else {
      const int cc = t & 7, rr = t >> 3;
      base = reinterpret_cast<const char*>((const bf16_raw*)g.A + (long long)g.a_row0 * g.lda);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        int row = rr + 32 * q;
        if (MODE == PROJ_EDGE) row = min(row, g.a_rows - 1 - g.a_row0);     // (rows past the end are nobody's)
        off[q] = (unsigned)((row * g.lda + 8 * cc) * 2);
      }
      step = 64 * 2;
    }
    if (MODE == PROJ_EDGE && g.KB == 64) last();
  }
  // All but GUARDED: request j of the four of a stage (the caller issues all four, in order, then advance())
  __device__ __forceinline__ void load_one(u32x4 (&ra)[4], int j) { gload16_async(ra[j], base, off[j]); }
  __device__ __forceinline__ void advance() { base += step; }
  // EDGE, before the requests of the last stage: those past the end of the contraction go to where it ends
  __device__ __forceinline__ void last() {
    const int t = threadIdx.x, left = g.KA - (g.KB - 64);      // k of the stage that there are
    if (left >= 64) return;
    if (LEFT) {
      const int kq = proj_kslow_kq(t);
#pragma unroll
      for (int j = 0; j < 4; ++j) off[j] -= (unsigned)(max(4 * kq + j - (left - 1), 0) * g.lda * 2);
    } else {
      const int k = 8 * (t & 7), back = min(left - 8, 0);      // (the stage may hold less than a piece)
      down = min(max(k - (left - 8), 0), 8);
      base += 2 * back;
#pragma unroll
      for (int q = 0; q < 4; ++q) off[q] = (unsigned)((int)off[q] + 2 * (min(k, left - 8) - k - back));
    }
  }
  // EDGE, after the wait for a stage: everything in its place, zeros past the ends
  template <bool LAST>
  __device__ __forceinline__ void settle(u32x4 (&ra)[4]) {
    const int left = g.KA - (g.KB - 64);
    if (LEFT) {
      if (g.a_row0 + FIRA_PA > g.a_rows) {
#pragma unroll
        for (int j = 0; j < 4; ++j) ra[j] = shift8_bf16(ra[j], down);
      }
      if (LAST && left < 64) {
        const int kq = proj_kslow_kq(threadIdx.x);
#pragma unroll
        for (int j = 0; j < 4; ++j) ra[j] = 4 * kq + j < left ? ra[j] : u32x4{0u, 0u, 0u, 0u};
      }
    } else if (LAST && left < 64) {
#pragma unroll
      for (int q = 0; q < 4; ++q) ra[q] = shift8_bf16(ra[q], down);
    }
  }
  __device__ __forceinline__ void load(u32x4 (&ra)[4]) {
    if (MODE != PROJ_GUARDED) {
#pragma unroll
      for (int j = 0; j < 4; ++j) gload16_async(ra[j], base, off[j]);
      base += step;
    } else {
      const int t = threadIdx.x;
      const u32x4 zero = u32x4{0u, 0u, 0u, 0u};
      if (LEFT) {
        const int ib = proj_kslow_ib(t), kq = proj_kslow_kq(t);
        const long long a = (long long)g.a_row0 + 8 * ib;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int k = k0 + 4 * kq + j;
          const int kc = k < g.KA ? k : g.KA - 1;
          const u32x4 v = load8_bf16(g.A + (long long)kc * g.lda, a, g.a_rows);
          ra[j] = k < g.KA ? v : zero;
        }
      } else {
        const int cc = t & 7, rr = t >> 3;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int row = g.a_row0 + rr + 32 * q;
          const int rc = row < g.a_rows ? row : g.a_rows - 1;
          ra[q] = load8_bf16(g.A + (long long)rc * g.lda, k0 + 8 * cc, g.KA);
        }
      }
      k0 += 64;
    }
  }
};
// The loads that a tile takes.
__device__ __forceinline__ bool proj_interior(const GemmOperands& g) { return g.a_row0 + FIRA_PA <= g.a_rows && g.KA == g.KB; }
__device__ __forceinline__ bool proj_guarded(bool left, const GemmOperands& g) { return (left ? g.a_rows : g.KA) < 8; }

// Registers -> LDS tile of one K stage (128 rows x 64 k, lds_tile_off layout), written as eight parts.  t = the thread's place among the 256 loaders.
//   K-slow (LEFT): ra[j] holds row k = 4*kq + j of a 4(k) x 8(a) block, dword d of it the elements
//   a = 2d, 2d+1.  Part p emits output row a = p: its four k values, two byte permutes and one 8-byte
//   write.  The row's chunk position is (chunk ^ row ^ row>>3 ^ row>>6) & 7 with row = 8*ib + p, i.e.
//   a per-thread constant XOR p.
//   K-contiguous: part p is half p & 1 of the 16-byte piece q = p >> 1 (row rr + 32 q); the chunk
//   position is a per-thread constant XOR a constant of q.
template <bool LEFT>
__device__ __forceinline__ void proj_store_a_part(char* la, const u32x4 (&ra)[4], int p, int t) {
  if (LEFT) {
    const int ib = proj_kslow_ib(t), kq = proj_kslow_kq(t);
    const int bx = ((kq >> 1) ^ ib ^ (ib >> 3)) & 7;
    char* row0 = la + ib * 1024 + 8 * (kq & 1);
    const unsigned in[16] = {ra[0].x, ra[0].y, ra[0].z, ra[0].w, ra[1].x, ra[1].y, ra[1].z, ra[1].w,
                             ra[2].x, ra[2].y, ra[2].z, ra[2].w, ra[3].x, ra[3].y, ra[3].z, ra[3].w};  // in[4*j + d]
    const unsigned sel = (p & 1) ? 0x07060302u : 0x05040100u;   // the high or the low halves of (x, y)
    const unsigned w0 = __builtin_amdgcn_perm(in[4 + (p >> 1)], in[0 + (p >> 1)], sel);    // k = 0, 1
    const unsigned w1 = __builtin_amdgcn_perm(in[12 + (p >> 1)], in[8 + (p >> 1)], sel);   // k = 2, 3
    *reinterpret_cast<u32x2*>(row0 + p * 128 + ((bx ^ p) << 4)) = u32x2{w0, w1};
  } else {
    const int cc = t & 7, rr = t >> 3, q = p >> 1;
    const int bx = (cc ^ rr ^ (rr >> 3)) & 7;
    const int cq = (4 * (q & 1)) ^ (q >> 1);
    const u32x2 half = (p & 1) ? u32x2{ra[q].z, ra[q].w} : u32x2{ra[q].x, ra[q].y};
    *reinterpret_cast<u32x2*>(la + rr * 128 + q * 4096 + ((bx ^ cq) << 4) + 8 * (p & 1)) = half;
  }
}

template <bool LEFT>
__device__ __forceinline__ void proj_store_a(char* la, const u32x4 (&ra)[4], int t = threadIdx.x) {
#pragma unroll
  for (int p = 0; p < 8; ++p) proj_store_a_part<LEFT>(la, ra, p, t);
}

// 32 k of the wave's 128 x 64 sub-tile: A fragments from the 128-B-per-row tile (k-slices kk4, kk4+1
// of its 4), B fragments from a ring stage.
// A wavefront issues in order, and a multiply holds the matrix pipe for 32 cycles: sixteen multiplies
// in a row leave the wavefront unable to issue anything else for as long as they queue, and whatever
// else the half stage has to do (the second slice's fragment reads, the requests of the next ring stage
// and gradient tile) then runs with the matrix pipe idle.  So that work is dealt out between the
// multiplies of the first slice: `piece(j)`, j = 0..7, is called after the j-th of them, and scheduling
// barriers keep the compiler from gathering the multiplies again.
// TM: row blocks of 32 that the wave owns, from row a0; its 64 B rows start at b0.
template <int TM, bool SUMSQ, typename Piece>
__device__ __forceinline__ void proj_compute(f32x16_t (&acc)[TM][2], const char* la, const char* lb, int a0, int b0, int kk4,
                                             float (&sq)[TM], Piece piece) {
  const int lane = threadIdx.x & 63;
  bf16x8_t fa[2][TM], fb[2][2];
  auto read_a = [&](int kk, int t) {
    fa[kk][t] = *reinterpret_cast<const bf16x8_t*>(la + lds_tile_off(a0 + 32 * t + (lane & 31), 2 * (kk4 + kk) + (lane >> 5)));
  };
  auto read_b = [&](int kk, int t) {
    fb[kk][t] = *reinterpret_cast<const bf16x8_t*>(lb + ring_tile_off(b0 + 32 * t + (lane & 31), 2 * kk + (lane >> 5)));
  };
  auto sumsq = [&](int kk) {
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) sq[tm] = frag_sumsq(fa[kk][tm], sq[tm]);
  };
#pragma unroll
  for (int t = 0; t < TM; ++t) read_a(0, t);
#pragma unroll
  for (int t = 0; t < 2; ++t) read_b(0, t);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int j = 0; j < 2 * TM; ++j) {
    const int tm = j >> 1, tn = j & 1;
    acc[tm][tn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[0][tm], fb[0][tn], acc[tm][tn], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    if (j < TM) read_a(1, j);
    else if (j < TM + 2) read_b(1, j - TM);
#pragma unroll
    for (int c = 0; c < 4 / TM; ++c) piece(j * (4 / TM) + c);
    __builtin_amdgcn_sched_barrier(0);
  }
  if (SUMSQ) sumsq(0);
#pragma unroll
  for (int tm = 0; tm < TM; ++tm)
#pragma unroll
    for (int tn = 0; tn < 2; ++tn)
      acc[tm][tn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[1][tm], fb[1][tn], acc[tm][tn], 0, 0, 0);
  if (SUMSQ) sumsq(1);
}

// RT = rank tiles of 256 that one workgroup covers (256*RT threads, wave w owns rank rows 64 w ..).
// With RT = 2 both tiles share the A tile, which only the first four wavefronts load and store
// (LOADER); the other four have no A requests in their queue, so their O-half wait is vmcnt(4) where a
// loading wavefront's is vmcnt(8).
// (LOADER is a template parameter rather than a test inside, so that each kind of wavefront runs
// straight-line code in which every request is followed by its own wait.)
// TM = 2: half a rank tile (r <= 128), two wavefronts along the factors (64 each) and two along the rank; a ring
// stage is 128 rows, two requests per wave, and the queue depths are TM where four requests make them 4 above.
// prologue(): called when the first operands have been requested, for work that would otherwise stand before or after the contraction.
template <bool LEFT, ProjLoads MODE, bool SUMSQ, int RT = 1, bool LOADER = true, int TM = 4, typename Prologue>
__device__ __forceinline__ void proj_pipeline(f32x16_t (&acc)[TM][2], char* lds, const GemmOperands& g, float (&sq)[TM], Prologue prologue) {
  static_assert(LOADER || RT == 2, "only the second rank tile's wavefronts go without the gradient");
  static_assert(TM == 4 || RT == 1, "half a rank tile, or whole ones");
  constexpr int STAGE = RT * TM * 4096;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  constexpr bool loader = LOADER;
  char* la = lds;
  char* ring = lds + FIRA_PROJ_LDS_A;
  const unsigned ring0 = (unsigned)(size_t)(lds_ptr)ring;
  const int SS = g.KB / 64;                    // K stages of 64; the ring runs 2*SS stages of 32
  const int lrow = lane >> 2;
  const int chunk = (lane & 3) ^ ring_swz(lrow);
  const unsigned offb = (unsigned)(lrow * 64 + chunk * 16);
  const int a0 = TM == 2 ? 64 * (wave >> 1) : 0, b0 = TM == 2 ? 64 * (wave & 1) : 64 * wave;
  const char* pb = reinterpret_cast<const char*>((const bf16_raw*)g.B) + ((long long)g.b_row0 + 16 * TM * wave) * 64;
  // request q (of TM) of ring stage s
  auto request_b1 = [&](int s, int q) {
    const unsigned dst = ring0 + (unsigned)((s % FIRA_RING_STAGES) * STAGE);
    const char* kb = pb + (long long)s * g.ldb * 64;
    lds_dma16(kb + q * 1024, offb, dst + (unsigned)((TM * wave + q) * 1024));
  };
  auto request_b = [&](int s) {
#pragma unroll
    for (int q = 0; q < TM; ++q) request_b1(s, q);
  };
  ProjALoader<LEFT, MODE> al(g);
  u32x4 ra[4];
  if (loader) al.load(ra);                     // A(0)
  request_b(0);
  request_b(1);
  prologue();
  // LAST: the final K stage requests nothing more.  It is written out separately rather than
  // guarded inside the loop, so that on every path a request is followed by the wait that covers it.
  auto stage = [&](auto last, int S) {
    constexpr bool LAST = decltype(last)::value;
    // E half
    if (loader) wait_loads<TM>(ra);            // A(S) and D(2S) have landed; D(2S+1) may be in flight
    else asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
    asm volatile("s_barrier" ::: "memory");    // everybody is done with the previous stage's A tile and ring slot
    if (loader) {
      if (MODE == PROJ_EDGE) al.template settle<LAST>(ra);
      proj_store_a<LEFT>(la, ra);
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    // the requests of D(2S+2) (into the slot of D(2S-1), free since the first barrier) and of A(S+1)
    // (whose registers proj_store_a has just released) go out between the multiplies
    proj_compute<TM, SUMSQ>(acc, la, ring + ((2 * S) % FIRA_RING_STAGES) * STAGE, a0, b0, 0, sq, [&](int j) {
      if (LAST) return;
      if (j < TM) request_b1(2 * S + 2, j);
      else if (j >= 4 && loader) {
        if (MODE != PROJ_GUARDED) {
          if (MODE == PROJ_EDGE && j == 4 && S + 2 == SS) al.last();
          al.load_one(ra, j - 4);
          if (j == 7) al.advance();
        } else if (j == 4) {
          al.load(ra);
        }
      }
    });
    // O half
    // D(2S+1) has landed.  Guarded A loads are the compiler's and may be fewer than 4 instructions,
    // so that path only lets D(2S+2)'s stay in flight.
    if (LAST) asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
    else if (MODE != PROJ_GUARDED && loader) {
      if (TM == 4) asm volatile("s_waitcnt vmcnt(8)\n\ts_barrier" ::: "memory");
      else asm volatile("s_waitcnt vmcnt(6)\n\ts_barrier" ::: "memory");
    } else {
      if (TM == 4) asm volatile("s_waitcnt vmcnt(4)\n\ts_barrier" ::: "memory");
      else asm volatile("s_waitcnt vmcnt(2)\n\ts_barrier" ::: "memory");
    }
    proj_compute<TM, SUMSQ>(acc, la, ring + ((2 * S + 1) % FIRA_RING_STAGES) * STAGE, a0, b0, 2, sq, [&](int j) {
      if (!LAST && j < TM) request_b1(2 * S + 3, j);
    });
  };
  for (int S = 0; S + 1 < SS; ++S) stage(std::false_type{}, S);
  stage(std::true_type{}, SS - 1);
}

// ------------------------------------------------------------------------------------------------
// Kernel 1 for fp32 matrices.  The gradient is read in fp32: a thread holds a 4 x 4 block of it in
// registers, splits the values into bf16 planes (x = h + m + l, split3) and writes the plane in turn to an
// LDS tile.  The six plane products run one after the other over the whole contraction, the largest first (sequences A
// and B): what the small ones add meets a sum that is already whole, and is rounded at the size of the result, where
// all six taken together per block of k round six times as often at the size of the running sum (twice the error of R
// where it cancels).  So G is read six times (10 GB through the fabric where G is 1.2, measured at the size below), which with
// the requests of two stages in flight is what bounds the kernel: 1491 us over the 168 matrices of 1024 x 1024 and
// 1024 x 2736 at r = 256, 1807 with one stage's; the way through memory took 1361 + 1123 + 918 (six planes written, read
// back, and a pass of its own for ||G_i||^2, which falls out of the first product here).
// (Sums of all six products per block of 32 k, apart from the running sum: 930 us and a quarter
// of the error of R, but single weights then differ from the former results by more than rounding explains locally:
// an element whose R is tiny in every step hands its relative error on to N.)
//
// Tile: 128 factors x 64 TM rank components; wave w holds 32 TM factors x 64 rank components, TM = 4, 2
// or 1 (the smallest that covers r, so that no wavefront multiplies padding only).  A stage is one product over 32 k:
//   registers -> LDS tile [128][32 k], 80 bytes per row (conflict-free for the 8-byte writes of
//   four rows and the 16-byte fragment reads of sixteen), doubled, the projector's plane beside it in a ring of three; one
//   barrier per stage; the operands of the stage after next are requested between the multiplies.
// Loads never leave the matrix: a group of four that would is moved back and shifted in registers, rows
// past the end read the last row; values past the contraction length are set to zero.
// ------------------------------------------------------------------------------------------------
#define FIRA_PANEL_MAX_S 416
#define FIRA_PANEL_MAX_R 256
// fp32 matrices that the panel kernel below takes
__host__ __device__ __forceinline__ bool panel_projection(const FiraMat& mt) { return mt.kx != 1 && mt.S <= FIRA_PANEL_MAX_S && mt.r <= FIRA_PANEL_MAX_R; }
#define FIRA_SPLIT_PITCH 80
#define FIRA_SPLIT_PLANE (FIRA_PA * FIRA_SPLIT_PITCH)
#define FIRA_SPLIT_LDS (2 * FIRA_SPLIT_PLANE + FIRA_RING_STAGES * FIRA_PROJ_RING_STAGE)

// Thread t holds rows 4 b .. 4 b + 3 and k = 4 kq .. 4 kq + 3 of the tile; 32 consecutive threads write
// four rows' whole 64 bytes.
__device__ __forceinline__ int split_b(int t) { return (t & 3) | ((t >> 5) << 2); }
__device__ __forceinline__ int split_kq(int t) { return (t >> 2) & 7; }

// The lane number, formed anew at each call, so that no address made from it is kept from one block to the next: one
// reloaded from scratch waits for every load in flight.  Kept, the fp32 update spills 41 registers instead of 15 and the fp32
// norm pass 23 instead of 7.
__device__ __forceinline__ int fresh_lane() {
  unsigned zero = 0;
  asm volatile("" : "+s"(zero));
  return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, zero));
}

// ASYNC: 16-byte inline-assembly loads (at least four elements along the contiguous axis); otherwise
// element by element (matrices with fewer).  What does not change from block to block is formed once: 300 vector instructions a
// stage, most of them addresses, were what bounded the kernel once its loads ran ahead.
template <bool LEFT, bool ASYNC>
struct SplitALoader {
  gptr<const float> G;
  long long ld;
  int row0, L, S, b, kq;    // b, kq: this thread's place in the tile (split_b, split_kq)
  unsigned off[LEFT ? 1 : 4];
  __device__ __forceinline__ SplitALoader(gptr<const float> G_, long long ld_, int row0_, int L_, int S_)
      : G(G_), ld(ld_), row0(row0_), L(L_), S(S_), b(split_b(threadIdx.x)), kq(split_kq(threadIdx.x)) {
    if (LEFT) off[0] = (unsigned)(min(row0 + 4 * b, L - 4) - min(row0, L - 4)) * 4u;
    else
#pragma unroll
      for (int q = 0; q < 4; ++q) off[LEFT ? 0 : q] = (unsigned)(min(row0 + 4 * b + q, L - 1) - row0) * (unsigned)(ld * 4);
    if (!LEFT)
#pragma unroll
      for (int q = 0; q < 4; ++q) off[LEFT ? 0 : q] += 16u * (unsigned)kq;
    else off[0] += 4u * (unsigned)kq * (unsigned)(ld * 4);
  }
  // request q (of 4) of the block of 32 k that starts at k0
  __device__ __forceinline__ void load_one(u32x4 (&ra)[4], int k0, int q) {
    if (ASYNC) {
      // (a block that ends past S takes its last rows or columns again instead)
      if (LEFT) {
        unsigned o = off[0];
        const char* base = reinterpret_cast<const char*>((const float*)G + (long long)(k0 + q) * ld + min(row0, L - 4));
        if (k0 + 32 > S) {
          base -= (long long)q * ld * 4;
          o = (unsigned)(min(row0 + 4 * b, L - 4) - min(row0, L - 4)) * 4u + (unsigned)min(4 * kq + q, S - 1 - k0) * (unsigned)(ld * 4);
        }
        gload16_async(ra[q], base, o);
      } else {
        unsigned o = off[LEFT ? 0 : q];
        const char* base = reinterpret_cast<const char*>((const float*)G + (long long)row0 * ld + k0);
        if (k0 + 32 > S) {
          base -= (long long)k0 * 4;
          o += (unsigned)(min(k0 + 4 * kq, S - 4) - 4 * kq) * 4u;
        }
        gload16_async(ra[q], base, o);
      }
    } else {
      unsigned w[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int k = k0 + 4 * kq + (LEFT ? q : e), row = row0 + 4 * b + (LEFT ? e : q);
        w[e] = (k < S && row < L) ? __float_as_uint(LEFT ? G[(long long)k * ld + row] : G[(long long)row * ld + k]) : 0u;
      }
      ra[q] = u32x4{w[0], w[1], w[2], w[3]};
    }
  }
  static __device__ __forceinline__ u32x4 shifted(u32x4 v, int d) {
    if (d & 1) v = u32x4{v.y, v.z, v.w, 0u};
    if (d & 2) v = u32x4{v.z, v.w, 0u, 0u};
    return d < 4 ? v : u32x4{0u, 0u, 0u, 0u};
  }
  // after the wait: the loaded groups as x[e][j] = element (row 4 b + e, k = k0 + 4 kq + j), zeros past S
  __device__ __forceinline__ void unpack(u32x4 (&ra)[4], int k0, float (&x)[4][4]) {
    if (ASYNC) {
      if (LEFT) {
        if (row0 + FIRA_PA > L) {            // a group of four columns that was moved back
          const int c = row0 + 4 * b, shift = c - min(c, L - 4);
#pragma unroll
          for (int q = 0; q < 4; ++q) ra[q] = shifted(ra[q], shift);
        }
        if (k0 + 32 > S) {
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (k0 + 4 * kq + q >= S) ra[q] = u32x4{0u, 0u, 0u, 0u};
        }
      } else if (k0 + 32 > S) {
        const int k = k0 + 4 * kq, d = k - min(k, S - 4);
#pragma unroll
        for (int q = 0; q < 4; ++q) ra[q] = shifted(ra[q], d);
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const unsigned w[4] = {ra[q].x, ra[q].y, ra[q].z, ra[q].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) (LEFT ? x[e][q] : x[q][e]) = __uint_as_float(w[e]);
    }
  }
};

// Plane PL (0, 1, 2: h, m, l) of the block -> its tile.  dst: the thread's first row there (split_store_at).
__device__ __forceinline__ int split_store_at(int t) { return 4 * split_b(t) * FIRA_SPLIT_PITCH + 8 * split_kq(t); }
template <int PL>
__device__ __forceinline__ void split_store_plane(char* dst, const float (&x)[4][4]) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float d[4] = {x[e][0], x[e][1], x[e][2], x[e][3]};
    u32x2 v = u32x2{pack_bf16x2(d[0], d[1]), pack_bf16x2(d[2], d[3])};
#pragma unroll
    for (int p = 0; p < PL; ++p) {
      d[0] -= __uint_as_float(v.x << 16); d[1] -= __uint_as_float(v.x & 0xffff0000u);
      d[2] -= __uint_as_float(v.y << 16); d[3] -= __uint_as_float(v.y & 0xffff0000u);
      v = u32x2{pack_bf16x2(d[0], d[1]), pack_bf16x2(d[2], d[3])};
    }
    *reinterpret_cast<u32x2*>(dst + e * FIRA_SPLIT_PITCH) = v;
  }
}

// All three planes of four values.
__device__ __forceinline__ void split3_planes(const float (&x)[4], u32x2 (&pl)[3]) {
  float d[4] = {x[0], x[1], x[2], x[3]};
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    pl[p] = u32x2{pack_bf16x2(d[0], d[1]), pack_bf16x2(d[2], d[3])};
    d[0] -= __uint_as_float(pl[p].x << 16); d[1] -= __uint_as_float(pl[p].x & 0xffff0000u);
    d[2] -= __uint_as_float(pl[p].y << 16); d[3] -= __uint_as_float(pl[p].y & 0xffff0000u);
  }
}
// ||G_i||^2 over the four k that a thread holds of a block.  Spelled out, and added up block after block in both projection kernels:
// which of the two serves a matrix depends on what else is listed, its norms must not.
__device__ __forceinline__ float split_sumsq(const float (&x)[4]) {
  return __builtin_fmaf(x[0], x[0], x[1] * x[1]) + __builtin_fmaf(x[2], x[2], x[3] * x[3]);
}
// One stage: 32 k of a plane product, `piece(j)`, j = 0..7, between its first multiplies (see proj_compute).
template <int TM, typename Piece>
__device__ __forceinline__ void split_compute(f32x16_t (&acc)[TM][2], const char* la, const char* lb, int a0, int b0, Piece piece) {
  const int lane = threadIdx.x & 63;
  bf16x8_t fa[2][TM], fb[2][2];
  auto read_a = [&](int kk, int t) {
    fa[kk][t] = *reinterpret_cast<const bf16x8_t*>(la + (a0 + 32 * t + (lane & 31)) * FIRA_SPLIT_PITCH + (2 * kk + (lane >> 5)) * 16);
  };
  auto read_b = [&](int kk, int t) {
    fb[kk][t] = *reinterpret_cast<const bf16x8_t*>(lb + ring_tile_off(b0 + 32 * t + (lane & 31), 2 * kk + (lane >> 5)));
  };
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
    for (int t = 0; t < TM; ++t) read_a(kk, t);
    read_b(kk, 0);
    read_b(kk, 1);
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int kk = 0; kk < 2; ++kk)
#pragma unroll
    for (int j = 0; j < 2 * TM; ++j) {
      acc[j >> 1][j & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[kk][j >> 1], fb[kk][j & 1], acc[j >> 1][j & 1], 0, 0, 0);
      if (kk == 0) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < 4 / TM; ++c) piece(j * (4 / TM) + c);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
}

// acc and sq (rows 4 b + e, this thread's k) must be zero on entry.  B: the projector's planes (sequence B).
template <bool LEFT, int TM, bool ASYNC>
__device__ __forceinline__ void split_pipeline(f32x16_t (&acc)[TM][2], char* lds, const FiraMat& mt, const float* G, int a_row0, int b_row0,
                                               int a0, int b0, float (&sq)[4]) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  constexpr int SLOT = TM * 4096;
  char* lb = lds + 2 * FIRA_SPLIT_PLANE;
  const unsigned lb0 = (unsigned)(size_t)(lds_ptr)lb;
  const int nblocks = (mt.S + 31) / 32, planes = mt.Sp / 32;
  const char* pb = reinterpret_cast<const char*>(mt.PT) + ((long long)b_row0 + 16 * TM * wave) * 64;
  const int lane = threadIdx.x & 63, lrow = lane >> 2, store_at = split_store_at(threadIdx.x);
  const unsigned offb = (unsigned)(lrow * 64 + ((lane & 3) ^ ring_swz(lrow)) * 16);
  // request q (of TM) of this wave's share of the projector's plane `pos` of sequence B, block kb
  auto request_b = [&](int pos, int kb, int slot, int q) {
    lds_dma16(pb + ((long long)(pos * planes + kb) * mt.rq) * 64 + q * 1024, offb, lb0 + (unsigned)(slot * SLOT + (TM * wave + q) * 1024));
  };
  SplitALoader<LEFT, ASYNC> al(as_global(G), mt.ld, a_row0, mt.L, mt.S);
  // Block of 32 k of a plane product: requests of two stages are in flight while one is multiplied, each stage's the
  // projector's plane (TM instructions per wavefront), then the gradient's block (4, into the set of registers that is free).
  // The last two stages request the first two blocks again, which nobody reads: every stage is the same code, with no
  // copy of a register that a load is on its way to.  (Neighbouring blocks may share lines of the gradient, and a last block asks
  // for its last row or column several times: these are loads into registers, which return in order whatever they ask for.)
  struct Block { int pos, kb; };
  auto next = [&](Block b) { return b.kb + 1 < nblocks ? Block{b.pos, b.kb + 1} : Block{b.pos == 5 ? 0 : b.pos + 1, 0}; };
  u32x4 ra[2][4];
  auto request = [&](u32x4 (&r)[4], Block b, int bslot) {
#pragma unroll
    for (int q = 0; q < TM; ++q) request_b(b.pos, b.kb, bslot, q);
#pragma unroll
    for (int q = 0; q < 4; ++q) al.load_one(r, 32 * b.kb, q);
  };
  auto stage = [&](u32x4 (&r)[4], int aslot, int bslot, Block b) {
    if (nblocks == 1) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (the next stage's block of G is this one again)
    wait_loads<ASYNC ? TM + 4 : 0>(r);           // this stage's operands have landed (guarded loads are the compiler's, of whatever number)
    float x[4][4];
    al.unpack(r, 32 * b.kb, x);
    if (b.pos == 0) {
#pragma unroll
      for (int e = 0; e < 4; ++e) sq[e] += split_sumsq(x[e]);
    }
    char* dst = lds + aslot * FIRA_SPLIT_PLANE + store_at;       // sequence A: planes 0 0 1 0 2 1
    if (b.pos == 4) split_store_plane<2>(dst, x);
    else if (b.pos == 2 || b.pos == 5) split_store_plane<1>(dst, x);
    else split_store_plane<0>(dst, x);
    // everybody's share is there, and everybody is done with the stage before
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    const Block b2 = next(next(b));
    const int bslot2 = bslot == 0 ? 2 : bslot - 1;   // (bslot + 2) % 3: the slot of the stage before
    split_compute<TM>(acc, lds + aslot * FIRA_SPLIT_PLANE, lb + bslot * SLOT, a0, b0, [&](int j) {
      if (j < TM) request_b(b2.pos, b2.kb, bslot2, j);
      else if (j >= 4) al.load_one(r, 32 * b2.kb, j - 4);
    });
  };
  Block b{0, 0};
  int bslot = 0, left = 3 * nblocks;             // 6 nblocks stages, two at a time
  auto step = [&]() { b = next(b); bslot = bslot == 2 ? 0 : bslot + 1; };
  request(ra[0], b, 0);
  request(ra[1], next(b), 1);
  do {
    stage(ra[0], 0, bslot, b);
    step();
    stage(ra[1], 1, bslot, b);
    step();
  } while (--left > 0);
  wait_loads<0>(ra[0]);
  wait_loads<0>(ra[1]);
}

// A wave's 32 TM x 32 TN block of R, from row row0 and column col0: into Rt, or (the projector refresh) rounded to bf16 into the
// K-blocked operand of the way back, `top` (rows = rank, K = factors).  A lane holds four consecutive factors of a
// rank row, and a 32 x 32 block of the operand is 2 KB of contiguous memory.  Factors past the end are the
// contraction's padding and are written as zeros; rank rows past r only feed columns that nobody stores.
// (168 matrices of the 1B shapes at r = 512, twice a refresh: with T in fp32, a pass that packed it and one that cleared
// the padding the way there took 1375 + 464 us, and 83 once; with the operand written here 1360.)
template <int TM, int TN = 2>
__device__ __forceinline__ void store_projection(const f32x16_t (&acc)[TM][TN], const FiraMat& mt, bf16_raw* top, int row0, int col0) {
  const int lane = threadIdx.x & 63, hi4 = 4 * (lane >> 5);
  if (top) {
    gptr<bf16_raw> Top = as_global(top);
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
      for (int tn = 0; tn < TN; ++tn) {
        const int col = col0 + 32 * tn + (lane & 31), rb = row0 + 32 * tm;
        if (rb >= ((mt.L + 63) & ~63)) continue;
#pragma unroll
        for (int vg = 0; vg < 4; ++vg) {
          const f32x16_t& a = acc[tm][tn];
          const int row = rb + 8 * vg + hi4, live = mt.L - row;
          *reinterpret_cast<gptr<u32x2>>(Top + kblk_index(mt.rq, col, row)) =
              u32x2{pack_bf16x2(live > 0 ? a[4 * vg] : 0.0f, live > 1 ? a[4 * vg + 1] : 0.0f),
                    pack_bf16x2(live > 2 ? a[4 * vg + 2] : 0.0f, live > 3 ? a[4 * vg + 3] : 0.0f)};
        }
      }
    return;
  }
  gptr<float> Rt = as_global(mt.Rt);
#pragma unroll
  for (int tm = 0; tm < TM; ++tm)
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) {
      const int col = col0 + 32 * tn + (lane & 31);
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row = row0 + 32 * tm + 8 * (v >> 2) + hi4 + (v & 3);
        if (row < mt.L && col < mt.r) Rt[(long long)row * mt.r + col] = acc[tm][tn][v];
      }
    }
}

template <bool LEFT, int TM>
__device__ __forceinline__ void project_split_tile(char* lds, const FiraMat& mt, const FiraEnt& ent, const FiraTile& tile, int norm_mode, int pack) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int a_row0 = tile.ta * FIRA_PA, b_row0 = tile.tb * FIRA_PB;
  const int a0 = 32 * TM * (wave % (4 / TM)), b0 = 64 * (wave / (4 / TM));
  const float* G = reinterpret_cast<const float*>(ent.G);
  f32x16_t acc[TM][2];
  float sq[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int tm = 0; tm < TM; ++tm)
#pragma unroll
    for (int tn = 0; tn < 2; ++tn)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[tm][tn][v] = 0.0f;
  if ((LEFT ? mt.L : mt.S) >= 4) split_pipeline<LEFT, TM, true>(acc, lds, mt, G, a_row0, b_row0, a0, b0, sq);
  else split_pipeline<LEFT, TM, false>(acc, lds, mt, G, a_row0, b_row0, a0, b0, sq);
  if (norm_mode == 1 && tile.tb == 0) {
    gptr<float> g2 = as_global(mt.g2);
#pragma unroll
    for (int e = 0; e < 4; ++e) {          // the eight threads that share a row
      float s = sq[e];
      s += __shfl_xor(s, 4, 64);
      s += __shfl_xor(s, 8, 64);
      s += __shfl_xor(s, 16, 64);
      const int row = a_row0 + 4 * split_b(threadIdx.x) + e;
      if (split_kq(threadIdx.x) == 0 && row < mt.L) g2[row] = s;
    }
  }
  store_projection<TM>(acc, mt, pack ? reinterpret_cast<bf16_raw*>(ent.W) : nullptr, a_row0 + a0, b_row0 + b0);
}

// bf16 matrices: TM = 2 where the rank fits half a rank tile (64 < r <= 128 in a step; a refresh also brings smaller
// ones), else 4.  (Both orientations of 56 matrices of 512 x 512 and 512 x 1376 at r = 128: 31 us; 38 us with TM = 4; 22 since edge tiles keep
// their loads in flight.)
template <bool LEFT, int TM>
__device__ __forceinline__ void project_tile_as(char* lds, const FiraMat& mt, const FiraEnt& ent, const FiraTile& tile, int norm_mode, int pack) {
  GemmOperands g;
  g.a_row0 = tile.ta * FIRA_PA;
  g.a_rows = mt.L;
  g.b_row0 = tile.tb * FIRA_PB;
  g.b_rows = mt.r;
  g.B = as_global<const bf16_raw>(mt.PT);
  g.ldb = mt.rq;
  g.KB = mt.Sp;
  g.A = as_global(reinterpret_cast<const bf16_raw*>(ent.G));
  g.lda = mt.ld;
  g.KA = mt.S;
  f32x16_t acc[TM][2];
  float sq[TM];
#pragma unroll
  for (int tm = 0; tm < TM; ++tm) {
    sq[tm] = 0.0f;
#pragma unroll
    for (int tn = 0; tn < 2; ++tn)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[tm][tn][v] = 0.0f;
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int a0 = TM == 2 ? 64 * (wave >> 1) : 0, b0 = TM == 2 ? 64 * (wave & 1) : 64 * wave;   // this wave's part of the tile
  // Gram route: ||G_i||^2 of the tile's 128 factors falls out of the A fragments of the waves with the
  // first 64 columns of each panel's first rank tile.
  const bool sumsq = norm_mode == 1 && tile.tb == 0 && b0 == 0;
  // LEFT: the k rows of G are whole rows of the matrix (any ld); RIGHT: a row of G holds KA values
  auto run = [&](auto mode) {
    if (sumsq) proj_pipeline<LEFT, decltype(mode)::value, true, 1, true, TM>(acc, lds, g, sq, [] {});
    else proj_pipeline<LEFT, decltype(mode)::value, false, 1, true, TM>(acc, lds, g, sq, [] {});
  };
  if (proj_interior(g)) run(std::integral_constant<ProjLoads, PROJ_FAST>{});
  else if (TM == 4 || !proj_guarded(LEFT, g)) run(std::integral_constant<ProjLoads, PROJ_EDGE>{});
  else if constexpr (TM == 2) run(std::integral_constant<ProjLoads, PROJ_GUARDED>{});      // (r <= min(m, n) < 8)
  if (sumsq) {
    gptr<float> g2 = as_global(mt.g2);
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
      const float tot = sq[tm] + __shfl_xor(sq[tm], 32, 64);
      const int row = g.a_row0 + a0 + 32 * tm + (lane & 31);
      if (lane < 32 && row < mt.L) g2[row] = tot;
    }
  }
  store_projection<TM>(acc, mt, pack ? reinterpret_cast<bf16_raw*>(ent.W) : nullptr, g.a_row0 + a0, g.b_row0 + b0);
}

template <bool LEFT>
__device__ __forceinline__ void project_tile(char* lds, const FiraMat* __restrict__ mats, const FiraEnt* __restrict__ ents,
                                             const FiraTile& tile, int norm_mode, int pack, const FiraScal* __restrict__ scal, const FiraHp& hp) {
  const FiraEnt ent = ents[tile.ent];
  if (hp.mixed && use_gram(hp, scal[ent.mat])) return;   // the fused kernel serves this matrix
  const FiraMat mt = mats[ent.mat];

  if (mt.kx != 1) return;                                // fira_fp32_project_kernel's
  if (mt.r <= 128) project_tile_as<LEFT, 2>(lds, mt, ent, tile, norm_mode, pack);
  else project_tile_as<LEFT, 4>(lds, mt, ent, tile, norm_mode, pack);
}

// One grid for both orientations: workgroups [0, blocks_left) take the tiles of the matrices with
// m <= n (gradient K-slow), the rest those with m > n, so that only one partly filled round of
// workgroups ends the launch.  blocks_left is a multiple of 8, which keeps the XCD-aware mapping of
// each part.  scal is read only when hp.mixed is set (a step in which the fused kernel serves the
// matrices on the Gram route and this kernel the others).  pack (the projector refresh's way there): the product leaves
// rounded to bf16 as the operand of the way back, at the address in the entry's W, instead of in fp32.
__global__ __launch_bounds__(FIRA_PROJ_THREADS, 2) void fira_project_kernel(const FiraMat* __restrict__ mats,
                                                                            const FiraEnt* __restrict__ ents,
                                                                            const FiraTile* __restrict__ tiles_left, int ntiles_left,
                                                                            int blocks_left,
                                                                            const FiraTile* __restrict__ tiles_right, int ntiles_right,
                                                                            int norm_mode, int pack, const FiraScal* __restrict__ scal, FiraHp hp) {
  extern __shared__ __attribute__((aligned(16))) char lds[];   // FIRA_PROJ_LDS bytes
  if ((int)blockIdx.x < blocks_left) {
    const int ti = xcd_chunked_index(blockIdx.x, ntiles_left);
    if (ti < 0) return;
    project_tile<true>(lds, mats, ents, tiles_left[ti], norm_mode, pack, scal, hp);
  } else {
    const int ti = xcd_chunked_index((int)blockIdx.x - blocks_left, ntiles_right);
    if (ti < 0) return;
    project_tile<false>(lds, mats, ents, tiles_right[ti], norm_mode, pack, scal, hp);
  }
}

// panels: fira_panel_project_kernel serves the matrices that it can take.
// The fp32 matrices of the same tile lists (the tiles of bf16 matrices leave at once, as those of fp32 ones do above; in
// one kernel for both the two forms together took more registers than either).
template <bool LEFT>
__device__ __forceinline__ void project_fp32_tile(char* lds, const FiraMat* __restrict__ mats, const FiraEnt* __restrict__ ents,
                                                  const FiraTile& tile, int norm_mode, int pack, int panels) {
  const FiraEnt ent = ents[tile.ent];
  const FiraMat mt = mats[ent.mat];
  if (mt.kx == 1 || (panels && panel_projection(mt))) return;
  if (mt.r <= 64) project_split_tile<LEFT, 1>(lds, mt, ent, tile, norm_mode, pack);
  else if (mt.r <= 128) project_split_tile<LEFT, 2>(lds, mt, ent, tile, norm_mode, pack);
  else project_split_tile<LEFT, 4>(lds, mt, ent, tile, norm_mode, pack);
}
__global__ __launch_bounds__(FIRA_PROJ_THREADS, 2) void fira_fp32_project_kernel(const FiraMat* __restrict__ mats,
                                                                                 const FiraEnt* __restrict__ ents,
                                                                                 const FiraTile* __restrict__ tiles_left, int ntiles_left,
                                                                                 int blocks_left,
                                                                                 const FiraTile* __restrict__ tiles_right, int ntiles_right,
                                                                                 int norm_mode, int pack, int panels) {
  extern __shared__ __attribute__((aligned(16))) char lds[];   // FIRA_SPLIT_LDS bytes
  if ((int)blockIdx.x < blocks_left) {
    const int ti = xcd_chunked_index(blockIdx.x, ntiles_left);
    if (ti < 0) return;
    project_fp32_tile<true>(lds, mats, ents, tiles_left[ti], norm_mode, pack, panels);
  } else {
    const int ti = xcd_chunked_index((int)blockIdx.x - blocks_left, ntiles_right);
    if (ti < 0) return;
    project_fp32_tile<false>(lds, mats, ents, tiles_right[ti], norm_mode, pack, panels);
  }
}

// ------------------------------------------------------------------------------------------------
// Kernel 1 for fp32 matrices whose short side is at most FIRA_PANEL_MAX_S (the three planes of 64 whole factors fit in LDS) and
// whose rank is at most FIRA_PANEL_MAX_R.
// A workgroup reads its panel of the gradient once and splits it once; the six plane products then run from LDS over all
// rank columns, wave w with 32 factors x 32 TN rank components, the projector's fragments straight from memory into
// registers (a 32 x 32 block of a plane is 2 KB of contiguous memory), U blocks of 32 k ahead.  No barrier after the
// split, and a tenth of the instructions per multiply of the kernel above, whose 6 S / 32 stages in turn are what a small
// matrix waits for.  Same products and sums in the same order: R and ||G_i||^2 are the same bit for bit.
// It holds a CU's LDS, or half its registers, so it is for lists whose workgroups all run at once (host: acquire_list); with more of them the
// smaller tiles above keep the chip busier.  What counts is the workgroups that are launched, with those that have no panel: they take
// their turns on the XCDs.  A step of 256 x 256 and 256 x 688 matrices at r = 64, with tiles and with panels:
// 67 and 48 us for 49 panels, 78 and 60 for 196, 89 and 86 for 392, 130 and 143 for 784; of 400 x 400 and 400 x 800 at
// r = 128: 103 and 75 us for 67 panels, 126 and 127 for 268, 197 and 220 for 536.  256 x 688 alone: 35 and 13 us of projection.
// The projection alone, with tiles and with panels: 400 x 800 at r = 256 73 and 56 us for 252 workgroups, 75 and 105 for 266; at two to
// a CU 64 x 30000 at r = 16 14.4 and 12.6 us (470 workgroups), 16 x 40000 13.0 and 15.9 (626), 128 x 40000 at r = 128 31 and 35 (626).
// Above r = 256 a panel takes a third and fourth pass over rank columns, where tiles take more workgroups: 400 x 800 at r = 260 71 and 61 us for one
// matrix, 72 and 71 (73 and 80 with cold operands) at r = 384, 73 and 176 for eighteen at r = 400.
// Row pitch of a plane: an odd number of 16-byte chunks, so that the fragment reads of sixteen rows are conflict-free.
// ------------------------------------------------------------------------------------------------
#define FIRA_PANEL_F 64
#define FIRA_PANEL_WG_PER_CU 2
__host__ __device__ __forceinline__ int panel_pitch(int S) { return ((S + 31) & ~31) * 2 + 16; }
__host__ __device__ __forceinline__ int panel_lds(int S) { return FIRA_SPLIT_PLANES * FIRA_PANEL_F * panel_pitch(S); }

template <int TN>
__device__ __forceinline__ void panel_products(const char* lds, const FiraMat& mt, const FiraEnt& ent, int a_row0, int col0, int pack) {
  constexpr int U = 6 / TN;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), hi = lane >> 5;
  const int nblocks = (mt.S + 31) / 32, planes = mt.Sp / 32, pitch = panel_pitch(mt.S);
  const int a0 = 32 * (wave & 1), b0 = col0 + 32 * TN * (wave >> 1);
  const char* la = lds + (a0 + (lane & 31)) * pitch + hi * 16;
  gptr<const char> pb = reinterpret_cast<gptr<const char>>(as_global<const bf16_raw>(mt.PT)) + (b0 + (lane & 31)) * 64 + hi * 16;
  f32x16_t acc[1][TN];
#pragma unroll
  for (int tn = 0; tn < TN; ++tn)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[0][tn][v] = 0.0f;
  // the projector's plane pos of sequence B (as stored), block kb
  struct Block { int pos, kb; };
  auto next = [&](Block b) { return b.kb + 1 < nblocks ? Block{b.pos, b.kb + 1} : Block{b.pos == 5 ? 0 : b.pos + 1, 0}; };
  u32x4 fb[2][U][2][TN];
  Block ahead{0, 0}, b{0, 0};
  auto request = [&](u32x4 (&f)[U][2][TN]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      gptr<const char> p = pb + (long long)(ahead.pos * planes + ahead.kb) * mt.rq * 64;
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) f[u][kk][tn] = *reinterpret_cast<gptr<const u32x4>>(p + tn * 2048 + kk * 32);
      ahead = next(ahead);
    }
  };
  auto multiply = [&](const u32x4 (&f)[U][2][TN]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const char* pa = la + ((0x610 >> (2 * b.pos)) & 3) * (FIRA_PANEL_F * pitch) + b.kb * 64;   // sequence A: planes 0 0 1 0 2 1
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        const bf16x8_t fa = *reinterpret_cast<const bf16x8_t*>(pa + kk * 32);
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
          acc[0][tn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, __builtin_bit_cast(bf16x8_t, f[u][kk][tn]), acc[0][tn], 0, 0, 0);
      }
      b = next(b);
    }
  };
  // 6 nblocks blocks in groups of U, two groups at a time; an odd last group is multiplied by itself
  const int groups = 6 * nblocks / U;
  request(fb[0]);
  for (int g = 0; g < groups; g += 2) {
    if (g + 1 < groups) request(fb[1]);
    multiply(fb[0]);
    if (g + 1 < groups) {
      if (g + 2 < groups) request(fb[0]);
      multiply(fb[1]);
    }
  }
  store_projection<1, TN>(acc, mt, pack ? reinterpret_cast<bf16_raw*>(ent.W) : nullptr, a_row0 + a0, b0);
}

template <bool LEFT>
__device__ __forceinline__ void project_panel(char* lds, const FiraMat& mt, const FiraEnt& ent, int a_row0, int norm_mode, int pack) {
  // Thread t: rows 4 b .. 4 b + 3 and k = 4 kq .. 4 kq + 3 of every second block of 32 k (b, kq as in the tiles above)
  const int t = threadIdx.x & 127, half = threadIdx.x >> 7, b = split_b(t), kq = split_kq(t), pitch = panel_pitch(mt.S);
  const int nblocks = (mt.S + 31) / 32, L = mt.L, S = mt.S;
  gptr<const float> G = as_global(reinterpret_cast<const float*>(ent.G));
  const bool wide = (LEFT ? L : S) >= 4;
  constexpr int U = 4, GROUPS = 2;           // blocks in flight; groups of them
  static_assert(64 * U * GROUPS >= FIRA_PANEL_MAX_S, "every block of this half belongs to a group");
  f32x4 sq[GROUPS][U];                       // this thread's share of ||G_i||^2 by block
  char* dst = lds + 4 * b * pitch + 8 * kq;
#pragma unroll
  for (int g = 0; g < GROUPS; ++g) {
    const int kb0 = half + 2 * U * g;
    if (kb0 >= nblocks) break;
    f32x4 v[U][4];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int k0 = 32 * (kb0 + 2 * u);
        v[u][q] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (k0 >= S) continue;
        if (wide) {                          // a group of four that would leave the matrix is moved back (and shifted below)
          const int row = LEFT ? min(a_row0 + 4 * b, L - 4) : min(a_row0 + 4 * b + q, L - 1);
          const int k = LEFT ? min(k0 + 4 * kq + q, S - 1) : min(k0 + 4 * kq, S - 4);
          v[u][q] = *reinterpret_cast<gptr<const f32x4_a4>>(G + (LEFT ? (long long)k * mt.ld + row : (long long)row * mt.ld + k));
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int k = k0 + 4 * kq + (LEFT ? q : e), row = a_row0 + 4 * b + (LEFT ? e : q);
            if (k < S && row < L) v[u][q][e] = LEFT ? G[(long long)k * mt.ld + row] : G[(long long)row * mt.ld + k];
          }
        }
      }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k0 = 32 * (kb0 + 2 * u);
      if (k0 >= S) break;
      float x[4][4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        u32x4 w = __builtin_bit_cast(u32x4, v[u][q]);
        if (wide) {
          const int at = LEFT ? a_row0 + 4 * b : k0 + 4 * kq;
          w = SplitALoader<LEFT, true>::shifted(w, at - min(at, (LEFT ? L : S) - 4));
          if (LEFT && k0 + 4 * kq + q >= S) w = u32x4{0u, 0u, 0u, 0u};
        }
        const unsigned ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) (LEFT ? x[e][q] : x[q][e]) = __uint_as_float(ww[e]);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) sq[g][u][e] = split_sumsq(x[e]);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        u32x2 pl[3];
        split3_planes(x[e], pl);
#pragma unroll
        for (int p = 0; p < 3; ++p) *reinterpret_cast<u32x2*>(dst + p * (FIRA_PANEL_F * pitch) + e * pitch + 2 * k0) = pl[p];
      }
    }
  }
  __syncthreads();
  for (int col0 = 0; col0 < mt.r; ) {
    if (mt.r - col0 <= 64) {
      panel_products<1>(lds, mt, ent, a_row0, col0, pack);
      col0 += 64;
    } else {
      panel_products<2>(lds, mt, ent, a_row0, col0, pack);
      col0 += 128;
    }
  }
  if (norm_mode == 1) {
    f32x4* odd = reinterpret_cast<f32x4*>(lds);       // [odd block][128]
    __syncthreads();                                  // the products are done with the panel
    if (half) {
#pragma unroll
      for (int i = 0; i < GROUPS * U; ++i)
        if (2 * i + 1 < nblocks) odd[128 * i + t] = sq[i / U][i % U];
    }
    __syncthreads();
    if (half) return;
    f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < GROUPS * U; ++i) {            // block after block, as the tiles above add them
      if (2 * i < nblocks) s += sq[i / U][i % U];
      if (2 * i + 1 < nblocks) s += odd[128 * i + t];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {                     // the eight threads that share a row
      float x = s[e];
      x += __shfl_xor(x, 4, 64);
      x += __shfl_xor(x, 8, 64);
      x += __shfl_xor(x, 16, 64);
      if (kq == 0 && a_row0 + 4 * b + e < L) as_global(mt.g2)[a_row0 + 4 * b + e] = x;
    }
  }
}

// Two workgroups per tile of the projection's lists (which also hold other matrices and their further rank tiles).
__global__ __launch_bounds__(256, FIRA_PANEL_WG_PER_CU) void fira_panel_project_kernel(const FiraMat* __restrict__ mats,
                                                                    const FiraEnt* __restrict__ ents,
                                                                    const FiraTile* __restrict__ tiles_left, int ntiles_left,
                                                                    const FiraTile* __restrict__ tiles_right, int norm_mode, int pack) {
  extern __shared__ __attribute__((aligned(16))) char lds[];   // panel_lds(S) of the widest listed matrix
  const int ti = blockIdx.x >> 1;
  const bool left = ti < ntiles_left;
  const FiraTile tile = left ? tiles_left[ti] : tiles_right[ti - ntiles_left];
  if (tile.tb != 0) return;
  const FiraEnt ent = ents[tile.ent];
  const FiraMat mt = mats[ent.mat];
  const int a_row0 = tile.ta * FIRA_PA + FIRA_PANEL_F * (blockIdx.x & 1);
  if (!panel_projection(mt) || a_row0 >= mt.L) return;
  if (left) project_panel<true>(lds, mt, ent, a_row0, norm_mode, pack);
  else project_panel<false>(lds, mt, ent, a_row0, norm_mode, pack);
}

// ------------------------------------------------------------------------------------------------
// The rank-axis contraction of fp32 matrices: every block of 32 k holds the planes h, m, l of both operands in LDS
// (72 KB, single-buffered, two workgroups per CU) and runs the six plane products from there, so that a plane is
// brought in once instead of two or three times, summed per block apart from the running sum, which is then rounded to
// nearest once per three products.  First B's
// plane h against A's l, m, h, while B's m and l arrive; then those against A's h and m, while the next
// block's A l and B h arrive in the places that are free by then.  350M shapes at r = 256, update: 1240 us, against
// 1293 us with the six products one after the other through the ring.
// ------------------------------------------------------------------------------------------------
template <bool FIRST, int TM, int TN>
__device__ __forceinline__ void back_split_compute(f32x16_t (&acc)[TM][TN], const char* la, const char* lb) {
  const int lane = fresh_lane(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int a0 = 32 * TM * (wave & 1), b0 = 32 * TN * (wave >> 1);
  constexpr int BLOCKS = TM * TN;
  // product i: A fragment FA(i) = 2 * plane (of la) + slice, B fragment FB(i) = 2 * plane (of lb) + slice
  constexpr int NA = FIRST ? 6 : 4, NB = FIRST ? 2 : 4;
  constexpr int FA[6] = {FIRST ? 4 : 2, FIRST ? 5 : 3, FIRST ? 2 : 0, FIRST ? 3 : 1, 0, 1};
  constexpr int FB[6] = {0, 1, FIRST ? 0 : 2, FIRST ? 1 : 3, 0, 1};
  bf16x8_t fa[NA], fb[TN][NB];
  auto read_a = [&](int f, int t) {
    fa[f] = *reinterpret_cast<const bf16x8_t*>(la + (f >> 1) * RingShape<TM, TN>::A + ring_tile_off(a0 + 32 * t + (lane & 31), 2 * (f & 1) + (lane >> 5)));
  };
#pragma unroll
  for (int f = 0; f < NA; ++f) read_a(f, 0);
#pragma unroll
  for (int t = 0; t < TN; ++t)
#pragma unroll
    for (int f = 0; f < NB; ++f)
      fb[t][f] = *reinterpret_cast<const bf16x8_t*>(lb + (f >> 1) * RingShape<TM, TN>::B + ring_tile_off(b0 + 32 * t + (lane & 31), 2 * (f & 1) + (lane >> 5)));
  __builtin_amdgcn_sched_barrier(0);
  f32x16_t part[2];
#pragma unroll
  for (int blk = 0; blk < BLOCKS; ++blk) {
    const int tm = blk / TN, tn = blk % TN;
    f32x16_t& p = part[blk & 1];
#pragma unroll
    for (int v = 0; v < 16; ++v) p[v] = 0.0f;
#pragma unroll
    for (int i = 0; i < 6; ++i) {
      p = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[FA[i]], fb[tn][FB[i]], p, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if (tn == TN - 1 && tm < TM - 1 && (FIRST || i < 2 || i > 3)) read_a(FA[i], tm + 1);   // after this fragment's last use
      if (blk > 0 && i >= 2) {
        f32x16_t& d = acc[(blk - 1) / TN][(blk - 1) % TN];
#pragma unroll
        for (int v = 4 * (i - 2); v < 4 * (i - 1); ++v) d[v] += part[(blk - 1) & 1][v];
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  acc[TM - 1][TN - 1] += part[(BLOCKS - 1) & 1];
}

// nblocks: blocks of 32 k in use; kplane: blocks per stored plane.  The low-rank operand (A if left) stores the planes
// h, m, l one after the other, the projector in sequence B (h m . l).
template <int TM, int TN>
__device__ __forceinline__ void split_mainloop(f32x16_t (&acc)[TM][TN], char* lds, const GemmOperands& g, int nblocks, int kplane, bool left) {
#pragma unroll
  for (int tm = 0; tm < TM; ++tm)
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[tm][tn][v] = 0.0f;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const unsigned lds0 = (unsigned)(size_t)(lds_ptr)lds;
  const char* pa = reinterpret_cast<const char*>((const bf16_raw*)g.A) + ((long long)g.a_row0 + 16 * TM * wave) * 64;
  const char* pb = reinterpret_cast<const char*>((const bf16_raw*)g.B) + ((long long)g.b_row0 + 16 * TN * wave) * 64;
  constexpr int RA = RingShape<TM, TN>::A, RB = RingShape<TM, TN>::B;
  // this wave's share of a plane of block kb: TM requests of A's, TN of B's
  auto request = [&](const char* base, long long ld, bool lowrank, int pl, int kb, int dst, int n) {
    const int lane = fresh_lane(), lrow = lane >> 2;
    const unsigned off = (unsigned)(lrow * 64 + ((lane & 3) ^ ring_swz(lrow)) * 16);
    const char* src = base + (long long)((pl == 2 && !lowrank ? 3 : pl) * kplane + kb) * ld * 64;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (q < n) lds_dma16(src + q * 1024, off, (unsigned)__builtin_amdgcn_readfirstlane((int)(lds0 + (unsigned)(dst + (n * wave + q) * 1024))));
  };
  auto request_a = [&](int pl, int kb) { request(pa, g.lda, left, pl, kb, pl * RA, TM); };
  auto request_b = [&](int pl, int kb) { request(pb, g.ldb, !left, pl, kb, 3 * RA + pl * RB, TN); };
  request_a(2, 0);
  request_b(0, 0);
  auto block = [&](auto last, int kb) {
    asm volatile("s_barrier" ::: "memory");              // everybody is done with the previous block
    request_a(0, kb);
    request_a(1, kb);
    request_b(1, kb);
    request_b(2, kb);
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" :: "n"(2 * TN) : "memory");   // all but B's m and l have landed
    back_split_compute<true>(acc, lds, lds + 3 * RA);
    asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
    if (!decltype(last)::value) {
      request_a(2, kb + 1);
      request_b(0, kb + 1);
    }
    back_split_compute<false>(acc, lds, lds + 3 * RA + RB);
  };
  for (int kb = 0; kb + 1 < nblocks; ++kb) block(std::false_type{}, kb);
  block(std::true_type{}, nblocks - 1);
}

// ------------------------------------------------------------------------------------------------
// Kernels 2 and 3 share the contraction  U[i][j] = sum_a X[i][a] Y[j][a]  over the rank axis, with
// X = P (m x r) and Y = Z or R long-side major (n x r) when left, X = Z or R (m x r) and Y = Q (n x r)
// when right.  The A side is Y (so a lane owns 4 consecutive columns j), the B side is X.
// The accumulators are re-laid out through LDS, one 32(i) x 64(j) slab per wave at a time, so that
// G and W are touched with 16-byte, row-contiguous accesses.
//   MODE 0: partial[tile] = sum_ij (k (G - U))^2            with Y/X built from R      (Eq. 12's norm)
//   MODE 1: W -= lr*alpha*(U + c k G)                       with Y/X built from Z = N - c k R
// ------------------------------------------------------------------------------------------------
template <typename T>
struct Elem8;  // 8 consecutive elements of W or G: raw registers, conversion to floats, store
template <>
struct Elem8<bf16_raw> {
  typedef u32x4 Raw;
  // W and G are touched once per step: non-temporal accesses keep them from evicting the operand
  // panels that the 32 CUs of an XCD share through its L2.
  template <bool INTERIOR>
  static __device__ __forceinline__ Raw load_raw(gptr<const bf16_raw> row, long long idx, long long limit) {
    if (INTERIOR) return __builtin_nontemporal_load(reinterpret_cast<gptr<const u32x4_a2>>(row + idx));
    return load8_bf16(row, idx, limit);
  }
  static __device__ __forceinline__ Raw load_edge(gptr<const bf16_raw> row, long long idx) { return *reinterpret_cast<gptr<const u32x4_a2>>(row + idx); }
  static __device__ __forceinline__ Raw zero() { return u32x4{0u, 0u, 0u, 0u}; }
  static __device__ __forceinline__ Raw shift(const Raw& v, int d) { return shift8_bf16(v, d); }
  static __device__ __forceinline__ void unpack(const Raw& v, float (&x)[8]) {
    const unsigned w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      x[2 * d] = __uint_as_float(w[d] << 16);
      x[2 * d + 1] = __uint_as_float(w[d] & 0xffff0000u);
    }
  }
  template <bool INTERIOR>
  static __device__ __forceinline__ void store(const float (&x)[8], gptr<bf16_raw> row, long long idx, long long limit) {
    if (INTERIOR || idx + 8 <= limit) {
      const u32x4 v = u32x4{pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]), pack_bf16x2(x[4], x[5]),
                            pack_bf16x2(x[6], x[7])};
      __builtin_nontemporal_store(v, reinterpret_cast<gptr<u32x4_a2>>(row + idx));
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (idx + e < limit) row[idx + e] = f32_to_bf16(x[e]);
    }
  }
};
template <>
struct Elem8<float> {
  struct Raw { f32x4 a, b; };
  template <bool INTERIOR>
  static __device__ __forceinline__ Raw load_raw(gptr<const float> row, long long idx, long long limit) {
    Raw r;
    if (INTERIOR || idx + 8 <= limit) {
      r.a = *reinterpret_cast<gptr<const f32x4_a4>>(row + idx);
      r.b = *reinterpret_cast<gptr<const f32x4_a4>>(row + idx + 4);
    } else {
      float x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = (idx + e < limit) ? row[idx + e] : 0.0f;
      r.a = f32x4{x[0], x[1], x[2], x[3]};
      r.b = f32x4{x[4], x[5], x[6], x[7]};
    }
    return r;
  }
  static __device__ __forceinline__ Raw load_edge(gptr<const float> row, long long idx) { return load_raw<true>(row, idx, 0); }
  static __device__ __forceinline__ Raw zero() { Raw r; r.a = f32x4{0.f, 0.f, 0.f, 0.f}; r.b = r.a; return r; }
  static __device__ __forceinline__ Raw shift(Raw r, int d) {
    const f32x4 z = f32x4{0.f, 0.f, 0.f, 0.f};
    if (d & 4) { r.a = r.b; r.b = z; }
    if (d & 2) { r.a = f32x4{r.a.z, r.a.w, r.b.x, r.b.y}; r.b = f32x4{r.b.z, r.b.w, 0.f, 0.f}; }
    if (d & 1) { r.a = f32x4{r.a.y, r.a.z, r.a.w, r.b.x}; r.b = f32x4{r.b.y, r.b.z, r.b.w, 0.f}; }
    if (d >= 8) { r.a = z; r.b = z; }
    return r;
  }
  static __device__ __forceinline__ void unpack(const Raw& r, float (&x)[8]) {
    x[0] = r.a.x; x[1] = r.a.y; x[2] = r.a.z; x[3] = r.a.w; x[4] = r.b.x; x[5] = r.b.y; x[6] = r.b.z; x[7] = r.b.w;
  }
  template <bool INTERIOR>
  static __device__ __forceinline__ void store(const float (&x)[8], gptr<float> row, long long idx, long long limit) {
    if (INTERIOR || idx + 8 <= limit) {
      *reinterpret_cast<gptr<f32x4_a4>>(row + idx) = f32x4{x[0], x[1], x[2], x[3]};
      *reinterpret_cast<gptr<f32x4_a4>>(row + idx + 4) = f32x4{x[4], x[5], x[6], x[7]};
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (idx + e < limit) row[idx + e] = x[e];
    }
  }
};

// Epilogue of the rank-axis contractions.  Two waves that share 64 tile rows (i) own 256 adjacent
// columns (j) between them; their accumulators are re-laid out through one LDS slab of 32 rows x 256
// columns per step, so that every global instruction covers two full 256-column row segments
// (512 B of bf16, 1 KB of fp32, contiguous) instead of 64-column pieces.  That matters most when
// ld is odd and no 16-byte access is aligned: the number of partially covered 128-byte lines per
// instruction drops four-fold.  DEPTH passes of G (and W) values are in flight: a pass is requested that
// many passes before it is consumed, across the change of slab.
// Edge tiles keep their loads in flight as well: they load whole pieces that stay inside the matrix, and move the values into
// place where they are used, if the row's end is not a whole piece (realigned as they were loaded, every pass waited for its own).  The
// element-by-element loads of matrices with fewer than eight columns are a form of their own: a copy of them beside every pass made
// launches with many edge tiles wait for instructions.  Edge pieces are loaded through the caches, since a tile covers their lines in
// part: past them, repeated steps of lists that fit the memory-side cache took 2 to 7 % longer (60M shapes 117 and 107 us, 21 matrices
// of 704 x 704 and 704 x 1736 at r = 144 106 and 100), ones whose arrays just exceed it up to 2 % less (112 of 335 x 335 and 335 x 482 at r = 66
// 130 and 133), large ones and first passes neither.  8 blocks of 1003 x 1003 and 1003 x 3001 at r = 64, update and norm pass: 146 and 73 us; 190 and 88 with one form for both and non-temporal loads, 210
// and 99 realigned while loading; 31 matrices of 384 x 1168 at r = 4 22.8 and 14.5, 23.8 and 17.3, 24.7 and 14.4; the update over the 1B shapes
// 2019, 2033 and 2071 us.
// (The norm pass, MODE 0, over 168 matrices of 1024 x 1024 and 1024 x 2736 at r = 256: 271 us = 0.57 PFLOP/s; 628 us
// while it had no loads in flight and spilled 72 registers.)
template <int TM, int TN>
struct EpiShape {
  static constexpr int COLS = 64 * TM, ROWS = 64 * TN;         // of the tile (n side, m side)
  static constexpr int STRIDE = COLS + 4;                      // floats per staged row (keeps 16-byte alignment, shifts banks)
  static constexpr int SLAB = 2 * 32 * STRIDE * 4;
  static constexpr int LDS = SLAB + ROWS * 4;                  // the slabs, then one factor per tile row (matrices with m > n)
  static constexpr int RING = FIRA_RING_STAGES * RingShape<TM, TN>::STAGE, ALL = LDS > RING ? LDS : RING;
};
#define FIRA_BACK_LDS (EpiShape<4, 2>::ALL)
enum EpiForm { kInside, kEdge, kNarrow };   // tiles inside the matrix, at its edge, of matrices with fewer than eight columns
template <int MODE, typename T, EpiForm FORM, int TM, int TN>
__device__ __forceinline__ float backproject_epilogue(f32x16_t (&acc)[TM][TN], char* lds, const FiraMat& mt,
                                                      const FiraEnt& ent, int i0, int j0, float c, float lr_alpha, bool unitk) {
  typedef typename Elem8<T>::Raw Raw;
  constexpr bool INTERIOR = FORM == kInside;
  // passes in flight: 64 registers of G and W values beside the accumulators
  typedef EpiShape<TM, TN> Shape;
  constexpr int LANES = 8 * TM, PROWS = 64 / LANES, PASSES = 16 / PROWS;   // lanes of a row, rows of a pass, passes of a wave's share of a slab
  constexpr int DEPTH = PASSES * TN < 8 ? PASSES * TN : sizeof(T) == 2 ? 8 : 4;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave & 1, wn = wave >> 1;
  float* buf = reinterpret_cast<float*>(lds) + wn * (32 * Shape::STRIDE);
  float* rowphi = reinterpret_cast<float*>(lds + Shape::SLAB);
  gptr<const T> G = as_global(reinterpret_cast<const T*>(ent.G));
  gptr<T> W = as_global(reinterpret_cast<T*>(ent.W));
  gptr<const float> phi = as_global<const float>(mt.phi);
  const int jl = 8 * (lane % LANES);          // this lane's 8 columns inside the staged 64 TM
  const int ih = lane / LANES;                // which of the rows of a pass
  const long long j = (long long)j0 + jl;
  // slab tn holds tile rows 32 TN wn + 32 tn .. +31; this wave consumes 16 of them.
  // Interior tiles address a pass as a wave-uniform row pointer plus one 32-bit lane offset.
  const long long wave_row0 = (long long)i0 + wn * 32 * TN + 16 * wm;
  const long long lane_off = (unsigned)(ih * (int)mt.ld + jl);
  auto slab_row = [&](int p) { return 16 * wm + PROWS * p + ih; };
  // Edge tiles: the first column loaded, this lane's behind it, and what its values have to be moved down by.
  const int jc0 = min(j0, mt.n - 8), jc = min((int)j, mt.n - 8) - jc0, jshift = (int)j - min((int)j, mt.n - 8);
  const bool moved = FORM == kEdge && (mt.n & 7) != 0 && j0 + Shape::COLS > mt.n;
  auto fetch = [&](int q, Raw& gr, Raw& wr) {   // pass q = PASSES * slab + pass of the slab
    const int tn = q / PASSES, p = q % PASSES;
    if constexpr (FORM == kInside) {
      const long long base = (wave_row0 + 32 * tn + PROWS * p) * mt.ld + j0;
      gr = Elem8<T>::template load_raw<true>(G + base, lane_off, 0);
      if (MODE == 1) wr = Elem8<T>::template load_raw<true>(W + base, lane_off, 0);
    } else if constexpr (FORM == kEdge) {
      // rows and columns past the end repeat the last ones
      const int first = min((int)wave_row0 + 32 * tn + PROWS * p, mt.m - 1);
      const long long base = (long long)first * mt.ld + jc0;
      const long long off = (unsigned)((min(first + ih, mt.m - 1) - first) * (int)mt.ld + jc);
      gr = Elem8<T>::load_edge(G + base, off);
      if (MODE == 1) wr = Elem8<T>::load_edge(W + base, off);
    } else {
      const long long i = (long long)i0 + wn * 32 * TN + 32 * tn + slab_row(p);
      const bool ok = i < mt.m && j < mt.n;
      gr = ok ? Elem8<T>::template load_raw<false>(G + i * mt.ld, j, mt.n) : Elem8<T>::zero();
      if (MODE == 1) wr = ok ? Elem8<T>::template load_raw<false>(W + i * mt.ld, j, mt.n) : Elem8<T>::zero();
    }
  };
  Raw gbuf[DEPTH], wbuf[MODE == 1 ? DEPTH : 1];
#pragma unroll
  for (int q = 0; q < DEPTH; ++q) fetch(q, gbuf[q], wbuf[MODE == 1 ? q : 0]);
  float cphi[8];
  if (mt.left) {
#pragma unroll
    for (int e = 0; e < 8; ++e) cphi[e] = (INTERIOR || j + e < mt.n) ? (unitk ? c : c * phi[j + e]) : 0.0f;
  }
  float sum = 0.0f;
#pragma unroll
  for (int tn = 0; tn < TN; ++tn) {
    __syncthreads();  // previous slab fully consumed (first time: the main loop's LDS reads are done)
    // One factor per row (m > n): the tile's go through LDS.  Loaded from global memory inside a pass
    // they would have to be waited for there, and the memory counter being in order, that wait would
    // cover every request in flight for the later passes.
    if (tn == 0 && !mt.left && threadIdx.x < Shape::ROWS) {
      const long long i = (long long)i0 + threadIdx.x;
      rowphi[threadIdx.x] = (INTERIOR || i < mt.m) ? (unitk ? c : c * phi[i]) : 0.0f;
    }
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
      for (int vg = 0; vg < 4; ++vg) {
        const f32x16_t& a = acc[tm][tn];
        const f32x4 val = f32x4{a[4 * vg], a[4 * vg + 1], a[4 * vg + 2], a[4 * vg + 3]};
        *reinterpret_cast<f32x4*>(buf + (lane & 31) * Shape::STRIDE + 32 * TM * wm + 32 * tm + 8 * vg + 4 * (lane >> 5)) = val;
      }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
      const int il = slab_row(p);
      const long long i = (long long)i0 + wn * 32 * TN + 32 * tn + il;
      const int q = PASSES * tn + p;
      Raw& gr = gbuf[q % DEPTH];
      Raw& wr = wbuf[MODE == 1 ? q % DEPTH : 0];
      if (INTERIOR || (i < mt.m && j < mt.n)) {
        const f32x4 u0 = *reinterpret_cast<const f32x4*>(buf + il * Shape::STRIDE + jl);
        const f32x4 u1 = *reinterpret_cast<const f32x4*>(buf + il * Shape::STRIDE + jl + 4);
        const float u[8] = {u0.x, u0.y, u0.z, u0.w, u1.x, u1.y, u1.z, u1.w};
        if (moved) {
          gr = Elem8<T>::shift(gr, jshift);
          if (MODE == 1) wr = Elem8<T>::shift(wr, jshift);
        }
        float g[8];
        Elem8<T>::unpack(gr, g);
        if (!mt.left) {
          const float f = rowphi[wn * 32 * TN + 32 * tn + il];
#pragma unroll
          for (int e = 0; e < 8; ++e) cphi[e] = f;
        }
        if (MODE == 0) {
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float sv = cphi[e] * (g[e] - u[e]);   // c = 1 here: k_i (G - P R)
            sum += (INTERIOR || j + e < mt.n) ? sv * sv : 0.0f;
          }
        } else {
          float w[8];
          Elem8<T>::unpack(wr, w);
#pragma unroll
          for (int e = 0; e < 8; ++e) w[e] = w[e] - lr_alpha * (u[e] + cphi[e] * g[e]);
          if (INTERIOR) Elem8<T>::template store<true>(w, W + ((wave_row0 + 32 * tn + PROWS * p) * mt.ld + j0), lane_off, 0);
          else Elem8<T>::template store<false>(w, W + i * mt.ld, j, mt.n);
        }
      }
      if (q + DEPTH < PASSES * TN) fetch(q + DEPTH, gr, wr);
      // Nothing is stored in the norm pass, so nothing but this keeps the compiler from gathering every pass's loads at
      // the top and the whole chain of additions at the end, with all values spilled in between.
      if (MODE == 0) asm volatile("" : "+v"(sum) :: "memory");
    }
  }
  return sum;
}

// T: storage type of W and G of every matrix in the tile list (the host keeps one list per type).
// (TM, TN) = (2, 1): four workgroups of 128 x 64 per listed tile, which fill the chip for lists of few tiles (host: launch_update);
// the norm pass, whose partial sums are laid out by tile, has the one form.  A step with whole and with quarter tiles, by
// the whole tiles of its list: 256 x 688 in fp32 (6) 42 and 31 us; bf16, 512 x 512 and 512 x 1376 at r = 128: 59 and 51 (102),
// 95 and 90 (816); 1024 x 1024 and 1024 x 2736: r = 192 172 and 166 (1568), 320 and 323 (3136); r = 256 137 and 130 (784), 192 and
// 187 (1568), 255 and 261 (2352), 1156 and 1207 (12544); r = 512 222 and 230 (1176); 1024 x 1024 at r = 512 98 and 102 (448);
// 2048 x 5461 at r = 512 196 and 183 (352), with 2048 x 2048 510 and 534 (3120); fp32, 1024 x 2736: r = 512 523 and 510 (784),
// r = 400 698 and 700 (1176), r = 256 3143 and 3212 (9408).  With operands that are in no cache: 512 x 512 and 512 x 1376 at r = 128
// 75 and 66 (102), 124 and 119 (816), 161 and 152 (1224); 1024 x 1024 and 1024 x 2736 at r = 256 143 and 138 (784), 281 and 286 (2352);
// 2048 x 5461 at r = 512 208 and 203 (352), 1024 x 1024 112 and 115 (384); fp32, 1024 x 2736 at r = 256 276 and 257 (392).
template <int MODE, typename T, int TM = 4, int TN = 2>
__global__ __launch_bounds__(FIRA_BACK_THREADS, TM == 4 ? 2 : sizeof(T) == 4 ? 3 : 4) void fira_backproject_kernel(const FiraMat* __restrict__ mats,
                                                                           const FiraScal* __restrict__ scal,
                                                                           const FiraEnt* __restrict__ ents,
                                                                           const FiraTile* __restrict__ tiles,
                                                                           int ntiles, int backwards, float* __restrict__ partial,
                                                                           FiraHp hp) {
  extern __shared__ __attribute__((aligned(16))) char lds[];   // FIRA_BACK_LDS bytes
  __shared__ float red[4];
  static_assert(TM == 4 || MODE == 1, "partial sums are laid out by tile");
  constexpr int PARTS = 8 / (TM * TN);           // workgroups of a listed tile
  const int wi = xcd_chunked_index(blockIdx.x, ntiles * PARTS);
  if (wi < 0) return;
  const int sub = wi % PARTS;
  // backwards: what the kernels before it read last, G of the last matrices, is still in the memory-side cache.  Update over the
  // 350M shapes at r = 256 435 -> 423 us, 1B 2098 -> 2078, residual route 420 -> 412.  That holds after Adam on the Gram route as well, which
  // has then come back to the first matrices (forwards / backwards, 350M shapes: two planes 544 / 534, r = 96 380 / 370, 8 blocks at r = 768
  // 242 / 236; with Adam forwards as well 545, 381 and 245).  At ranks up to 64 the update is a plain stream and the direction is worth 1 % on one
  // shape and nothing on another: steps 607 / 602 us over the 350M shapes at r = 16, 657 / 647 at r = 64, 2290 / 2287 over the 1B
  // shapes at r = 64, 6819 / 6856 over the fine-tuning shapes at r = 16, 7199 / 7183 at r = 64 (runs differ by 60): those go forwards.
  const FiraTile tile = tiles[backwards ? ntiles - 1 - wi / PARTS : wi / PARTS];
  const FiraEnt ent = ents[tile.ent];
  if (MODE == 0 && use_gram(hp, scal[ent.mat])) return;   // this matrix takes the Gram route to ||S||
  const FiraMat mt = mats[ent.mat];
  if (PARTS > 1 && (tile.ta * FIRA_BA + 64 * TM * (sub & 1) >= mt.n || tile.tb * FIRA_BB + 64 * TN * (sub >> 1) >= mt.m)) return;
  const float lr_alpha = MODE == 1 ? *hp.lr_alpha : 0.0f;

  // Y (n side) is the A operand, X (m side) the B operand.
  gptr<const bf16_raw> lowrank = as_global<const bf16_raw>((MODE == 0) ? mt.Rb : mt.Nb);
  gptr<const bf16_raw> proj = as_global<const bf16_raw>(mt.Pn);
  GemmOperands g;
  g.a_row0 = tile.ta * FIRA_BA + 64 * TM * (sub & 1);
  g.a_rows = mt.n;
  g.b_row0 = tile.tb * FIRA_BB + 64 * TN * (sub >> 1);
  g.b_rows = mt.m;
  // Z in two planes (hi + lo): the contraction runs over 2 rp, and the projector's K blocks are used twice
  const bool split = MODE == 1 && two_planes(hp, mt);
  g.KA = g.KB = split ? 2 * mt.rp : (mt.r + 31) / 32 * 32;   // (fp32 matrices: split_mainloop counts for itself)
  g.wrapA = (split && !mt.left) ? mt.rp / FIRA_RK : 0;
  g.wrapB = (split && mt.left) ? mt.rp / FIRA_RK : 0;
  g.A = mt.left ? lowrank : proj;
  g.B = mt.left ? proj : lowrank;
  g.lda = mt.left ? mt.Lq : mt.Sq;
  g.ldb = mt.left ? mt.Sq : mt.Lq;
  f32x16_t acc[TM][TN];
  if (sizeof(T) == 4) split_mainloop(acc, lds, g, (mt.r + 31) / 32, mt.rp / 32, mt.left != 0);
  else ring_mainloop(acc, lds, g);

  const float c = (MODE == 0) ? 1.0f : scal[ent.mat].c;
  const int i0 = g.b_row0, j0 = g.a_row0;
  const bool interior = i0 + 64 * TN <= mt.m && j0 + 64 * TM <= mt.n;
  float sum;
  // matrix-level factor: the residual norm is taken with unit factors and scaled by the limiter kernel
  const bool unitk = MODE == 0 && hp.scaling == 1;
  if (mt.n < 8) sum = backproject_epilogue<MODE, T, kNarrow, TM, TN>(acc, lds, mt, ent, i0, j0, c, lr_alpha, unitk);
  else if (interior) sum = backproject_epilogue<MODE, T, kInside, TM, TN>(acc, lds, mt, ent, i0, j0, c, lr_alpha, unitk);
  else sum = backproject_epilogue<MODE, T, kEdge, TM, TN>(acc, lds, mt, ent, i0, j0, c, lr_alpha, unitk);

  if (MODE == 0) {
    // deterministic workgroup reduction: xor-butterfly inside each wave, then waves in order
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) sum += __shfl_xor(sum, off, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0)
      as_global(partial)[tile.part] = (red[0] + red[1]) + (red[2] + red[3]);
  }
}
