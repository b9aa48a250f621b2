// Projection and Adam in one kernel (Algorithm 1: R = P^T G, the moment updates of Eqs. 2-4, the factor
// k_i of Eq. 11, and the back-projection operand Z_i = N_i - k_i R_i).
//
// When the rank fits one workgroup (r <= 512) the whole row R_i of a factor sits in the accumulators of
// the workgroup that projected it, so Adam can run on it there: R never goes to memory, and neither
// does a second launch read it back.  Per factor and rank component that leaves M and V read and
// written once (16 B) and Z written once (2 B), against 26 B for the two-kernel sequence.
//
// Tile: 128 factors x 256 RT rank components, 256 RT threads; wave w holds all 128 factors x rank
// components 64 w .. 64 w + 63 (RT = 1: r <= 256; two workgroups per CU, r = 128 in a form of its own; RT = 2: r <= 512, one per CU,
// the two rank tiles share one copy of the gradient tile, which is then read from memory once).
// The multiply phase is proj_pipeline.  The epilogue cannot keep many loads of M and V in flight from
// registers (the accumulators fill them), so M and V travel through LDS, which the multiply phase
// has left free: the tile is worked through in eight chunks of 16 factors, and while chunk c is
// processed the rows of M and V of chunk c + 1 arrive by LDS-direct loads (1 KB per instruction) in the
// other of two landing buffers.  Per chunk:
//   1. every lane updates M and V in place in the landing buffer for its 16 elements, forms N (kept in
//      registers) and sums N^2 and R^2 per factor; the sums are reduced over the 32 lanes that share a
//      factor (a reduce-scatter, fixed order) and left in LDS per wave;
//   2. one thread per factor adds the waves' sums in order, forms k_i, writes phi and q;
//   3. Z = N - k R is rounded to bf16 into an LDS image of the K-blocked operand;
//   4. the new M and V and Z leave LDS in 16-byte pieces, whole rows contiguous.
// Waits on the LDS-direct loads are explicit (see fira_gemm.h).  The wait for chunk c + 1 stands between
// steps 3 and 4 of chunk c, before the chunk's stores are issued, and waits for everything in flight: that
// is the loads of chunk c + 1 and the stores of chunk c - 1, which are a whole chunk old.  The stores of
// chunk c then stay in flight while chunk c + 1 is processed.  No count of instructions, and no
// assumption about the order in which loads and stores retire relative to each other, is involved.
//
// A step takes this kernel only if every listed matrix is bf16 with r % 4 == 0, 64 < r <= 512, column
// factors, Algorithm 1 proper.  On the Gram route to ||S|| R is written below FIRA_FUSE_DROP_R only.  On the residual route (with the operand
// copy of R that it contracts) and with Z in two planes a form of its own leaves R in memory whatever the rank, as two kernels do (fira_fused_leave_r_kernel, for lists that fill
// its rounds of workgroups).
// The limiter runs after it; for a matrix whose factor c came out below 1, fira_makez_kernel turns the Z
// written here (for c = 1) into c Z + (1 - c) N, with N formed again from the updated M and V.
#pragma once
#include "fira_device.h"
#include "fira_elementwise.h"
#include "fira_gemm.h"

#define FIRA_FUSE_F 16   // factors per chunk of the epilogue
#define FIRA_FUSE_LDS_MAIN(RT) (FIRA_PROJ_LDS_A + FIRA_RING_STAGES * (RT) * FIRA_PROJ_RING_STAGE)
// two landing buffers (M and V of a chunk, fp32), the Z image (bf16), per-wave sums, ||G_i||^2 of the tile, k_i
#define FIRA_FUSE_LDS_EPI(RT) (2 * FIRA_FUSE_F * 256 * (RT) * 8 + FIRA_FUSE_F * 256 * (RT) * 2 + 4 * (RT) * FIRA_FUSE_F * 8 + 128 * 4 + 2 * FIRA_FUSE_F * 4)
#define FIRA_FUSE_LDS(RT) (FIRA_FUSE_LDS_MAIN(RT) > FIRA_FUSE_LDS_EPI(RT) ? FIRA_FUSE_LDS_MAIN(RT) : FIRA_FUSE_LDS_EPI(RT))

// Sum of x[v] over the 32 lanes of a half wave, for 8 values at once.  Afterwards every lane holds the
// total of value  v = 4*bit4(l) + 2*bit3(l) + bit2(l).
__device__ __forceinline__ float half_wave_reduce8(const float (&x)[8]) {
  const int lane = threadIdx.x & 63;
  float a[4], b[2];
#pragma unroll
  for (int j = 0; j < 4; ++j) {          // x[j] stays in the even rows of 16 lanes, x[4 + j] in the odd ones
    const u32x2_s s = __builtin_amdgcn_permlane16_swap(__float_as_uint(x[j]), __float_as_uint(x[4 + j]), false, false);
    a[j] = __uint_as_float(s[0]) + __uint_as_float(s[1]);
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const float keep = (lane & 8) ? a[2 + j] : a[j], send = (lane & 8) ? a[j] : a[2 + j];
    b[j] = keep + lane_xor<8>(send);
  }
  const float keep = (lane & 4) ? b[1] : b[0], send = (lane & 4) ? b[0] : b[1];
  return add_xor<1>(add_xor<2>(keep + lane_xor<4>(send)));
}

// A wave-uniform pointer, in scalar registers whatever the compiler holds it in.
__device__ __forceinline__ const char* scalar_pointer(const char* p) {
  const unsigned long long a = (unsigned long long)p;
  const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)a), hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(a >> 32));
  return (const char*)(((unsigned long long)hi << 32) | lo);
}

// TM = 4: a wave's factors of a chunk are the chunk's 16.  TM = 2 (r <= 128): a chunk is 16 factors of either half of
// the tile, 32 rows of 128 in the same LDS, and half as many chunks.
// KEEP: R is left in memory, and as an operand too where operand_r is set (its image has Z's place in LDS before Z has); Z has a second plane where
// the step asks for one, whose image has it afterwards.
template <int RT, int TM, bool INTERIOR, bool KEEP>
__device__ __forceinline__ void project_adam_epilogue(f32x16_t (&acc)[TM][2], char* lds, const FiraMat& mt, const FiraHp& hp,
                                                      float bias, int a_row0, const float (&sq)[TM], bool operand_r) {
  constexpr int HALVES = 4 / TM, NW = 4 * RT / HALVES, THREADS = 256 * RT, C = 64 * NW, F = FIRA_FUSE_F * HALVES, NCHUNK = 128 / F;
  constexpr int ARR = F * C * 4;                                   // bytes of one array (M or V) of a chunk
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l32 = lane & 31, hi = lane >> 5;
  const int half = TM == 2 ? wave >> 1 : 0, wcol = TM == 2 ? wave & 1 : wave;   // this wave's half of the factors, its 64 rank columns
  bf16_raw* zl = reinterpret_cast<bf16_raw*>(lds + 4 * ARR);       // [C / 32 K blocks][F factors][32]
  float* part = reinterpret_cast<float*>(lds + 4 * ARR + F * C * 2);   // [NW][F factors][2]
  float* g2s = part + NW * F * 2;                                  // [128]
  float* ks = g2s + 128;                                           // [F]
  const unsigned lds0 = (unsigned)(size_t)(lds_ptr)lds;
  const int r = mt.r, L = mt.L;
  const int kblocks = mt.rp >> 5;
  const char* Mg = reinterpret_cast<const char*>(mt.M);
  const char* Vg = reinterpret_cast<const char*>(mt.V);

  // row `row` (0 .. F - 1) of chunk c, as a factor of the matrix
  auto factor = [&](int c, int row) { return a_row0 + (TM == 2 ? 64 * (row >> 4) + 16 * c + (row & 15) : F * c + row); };
  // Requests of chunk c, 8 instructions of 1 KB per wave for M and V: a row of C floats is RT pieces of 256 floats,
  // or half an instruction.
  auto request = [&](int c) {
    const unsigned dst0 = lds0 + (unsigned)((c & 1) * 2 * ARR);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int q = wave * 8 + i;                                  // 0 .. 32 RT - 1
      if (TM == 4) {
        const int arr = q / (F * RT), row = (q % (F * RT)) / RT, piece = q % RT;
        const long long grow = (long long)a_row0 + F * c + row;
        const char* src = scalar_pointer((arr ? Vg : Mg) + (grow * r + piece * 256) * 4);
        const unsigned dst = dst0 + (unsigned)(arr * ARR + (row * C + piece * 256) * 4);
        if (INTERIOR) {
          lds_dma16(src, (unsigned)lane * 16u, dst);
        } else if (grow < L) {
          if (piece * 256 + lane * 4 < r) lds_dma16(src, (unsigned)lane * 16u, dst);
        }
      } else {                                                     // rows 2 q', 2 q' + 1 of the chunk, one per half wave
        const int arr = q / (F / 2), row = 2 * (q % (F / 2)), grow = factor(c, row);
        const char* src = scalar_pointer((arr ? Vg : Mg) + (long long)grow * r * 4);
        const unsigned dst = dst0 + (unsigned)(arr * ARR + row * C * 4);
        const unsigned voff = (unsigned)(hi * r * 4 + l32 * 16);
        if (INTERIOR) {
          lds_dma16(src, voff, dst);
        } else if (grow + hi < L) {
          if (l32 * 4 < r) lds_dma16(src, voff, dst);
        }
      }
    }
  };

  __syncthreads();                                                 // the multiply phase is done with LDS
  request(0);
  if (wcol == 0) {
    gptr<float> g2 = as_global(mt.g2);
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
      const float tot = sq[tm] + __shfl_xor(sq[tm], 32, 64);
      const int rl = 64 * half + 32 * tm + l32;
      if (lane < 32) {
        g2s[rl] = tot;
        if (a_row0 + rl < L) g2[a_row0 + rl] = tot;
      }
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();

  // the factor (of a chunk of 16) whose sums this lane holds after half_wave_reduce8
  const int vown = (lane >> 2) & 7;
  const int rl_own = 16 * half + 8 * (vown >> 2) + 4 * hi + (vown & 3);
  // this lane's element (v', tn) of a chunk sits at float index (16*half + 8*(v'>>2) + 4*hi + (v'&3)) * C + 64*wcol + 32*tn + l32
  const int row_lane = 16 * half + 4 * hi, lane_idx = row_lane * C + 64 * wcol + l32;

  // an operand's pieces of a chunk from their image: C/32 K blocks x F rows of 64 bytes, 2 pieces of 16 per thread
  // (KEEP: offsets formed anew for every chunk; held over all of them, some would not fit the registers)
  auto thread = [&] {
    int t = threadIdx.x;
    if (KEEP) asm volatile("" : "+v"(t));
    return t;
  };
  auto store_operand_rows = [&](bf16_raw* to, int c, int kb0) {
    const int t = thread();
    gptr<char> out = reinterpret_cast<gptr<char>>(as_global(to));
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int p = t + THREADS * i;                               // K block, quarter p % 4 of a row
      const int kb = p / (4 * F);
      if (INTERIOR || kb < kblocks)
        *reinterpret_cast<gptr<u32x4>>(out + ((long long)(kb0 + kb) * mt.Lq + factor(c, (p % (4 * F)) >> 2)) * 64 + (p & 3) * 16) =
            *reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(zl) + p * 16);
    }
  };
  const bool planes = KEEP && two_planes(hp, mt);

  // One body for all chunks, with the chunk's sixteen accumulators moved to a place of their own first (they can only be indexed
  // statically): written out per chunk the epilogue was 6 KB of code eight times over, which a workgroup of a launch of one round
  // fetched as it went; the kernels are half as long now (427 -> 422 us over the 350M shapes, 2104 -> 2094 over the 1B shapes).
#pragma unroll 1
  for (int c = 0; c < NCHUNK; ++c) {
    float cur[2][8];
#pragma unroll
    for (int k = 0; k < NCHUNK; ++k)
      if (c == k) {
#pragma unroll
        for (int tn = 0; tn < 2; ++tn)
#pragma unroll
          for (int v = 0; v < 8; ++v) {
            cur[tn][v] = acc[k >> 1][tn][8 * (k & 1) + v];
            asm volatile("" : "+v"(cur[tn][v]));      // (a branch, not a chain of selects)
          }
      }
    const int row_w = factor(c, 16 * half);                        // first of the wave's sixteen factors
    float* landM = reinterpret_cast<float*>(lds + (c & 1) * 2 * ARR);
    float* landV = landM + F * C;
    if (c + 1 < NCHUNK) request(c + 1);
    float nv[2][8], nn[8], rr[8];
#pragma unroll
    for (int tn = 0; tn < 2; ++tn) {
      const int col = 64 * wcol + 32 * tn + l32;
#pragma unroll
      for (int v = 0; v < 8; ++v) {
        const int dr = 8 * (v >> 2) + (v & 3);
        const int idx = lane_idx + dr * C + 32 * tn;
        const bool ok = INTERIOR || (col < r && row_w + 4 * hi + dr < L);
        const float x = cur[tn][v];
        if (KEEP && operand_r) zl[((2 * wcol + tn) * F + row_lane + dr) * 32 + l32] = f32_to_bf16(ok ? x : 0.0f);
        const float m0 = ok ? landM[idx] : 0.0f, v0 = ok ? landV[idx] : 0.0f;
        const float m1 = hp.b1 * m0 + hp.omb1 * x;
        const float v1 = hp.b2 * v0 + hp.omb2 * (x * x);
        float n = adam_direction(m1, v1, bias, hp.epsf);
        if (!ok) n = 0.0f;
        landM[idx] = m1;
        landV[idx] = v1;
        nv[tn][v] = n;
        // (spelled out, for square_sum_as_fused to take the same sums)
        nn[v] = tn == 0 ? n : __builtin_fmaf(nn[v], nn[v], n * n);
        rr[v] = tn == 0 ? x : __builtin_fmaf(rr[v], rr[v], x * x);
      }
    }
    {
      const float tn_ = half_wave_reduce8(nn), tr_ = half_wave_reduce8(rr);
      if ((lane & 3) == 0) *reinterpret_cast<float2*>(part + (wcol * F + rl_own) * 2) = float2{tn_, tr_};
    }
    __syncthreads();
    if (KEEP && operand_r) store_operand_rows(mt.Rb, c, 0);
    if (threadIdx.x < F) {
      float snn = 0.0f, srr = 0.0f;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const float2 p = *reinterpret_cast<const float2*>(part + (w * F + threadIdx.x) * 2);
        snn += p.x;
        srr += p.y;
      }
      const int row = factor(c, threadIdx.x);
      float k = sqrtf(snn) / (sqrtf(srr) + hp.epsf);
      if (row < L) {
        as_global(mt.phi)[row] = k;
        as_global(mt.q)[row] = k * k * residual_sq(hp, g2s[row - a_row0], srr);
      } else {
        k = 0.0f;
      }
      ks[threadIdx.x] = k;
    }
    __syncthreads();
    auto z_image = [&](auto plane) {                               // Z, or what its rounding leaves
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        const f32x4 kq = *reinterpret_cast<const f32x4*>(ks + 8 * g + row_lane);
#pragma unroll
        for (int tn = 0; tn < 2; ++tn) {
          const int kb = 2 * wcol + tn;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int v = 4 * g + e;
            const bool ok = INTERIOR || (64 * wcol + 32 * tn + l32 < r && row_w + 8 * g + 4 * hi + e < L);
            float z = ok ? nv[tn][v] - kq[e] * cur[tn][v] : 0.0f;
            if (decltype(plane)::value == 1) z -= bf16_to_f32(f32_to_bf16(z));
            zl[(kb * F + 8 * g + row_lane + e) * 32 + l32] = f32_to_bf16(z);
          }
        }
      }
    };
    z_image(std::integral_constant<int, 0>{});
    __syncthreads();
    // The next chunk has landed (this wave's share of it).  The wait stands before this chunk's stores are
    // issued, so that it can be "everything": the only other operations in flight are the previous chunk's
    // stores, which have had this whole chunk to complete.  (Placed after the stores, the wait would have
    // to let exactly their number stay in flight, which is right only if stores never retire before older
    // loads and the compiler emits exactly the instructions counted.)
    if (c + 1 < NCHUNK) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    // M and V: 2 x F rows x C/4 pieces of 16 bytes, 8 per thread
    const int tx = thread();
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int arr = i >> 2, rem = tx + THREADS * (i & 3);
      const int row = rem / (C / 4), c4 = rem % (C / 4);
      const long long grow = factor(c, row);
      if (INTERIOR || (grow < L && 4 * c4 < r)) {
        const u32x4 val = *reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(landM) + arr * ARR + (row * C + 4 * c4) * 4);
        gptr<char> dst = reinterpret_cast<gptr<char>>(as_global(arr ? mt.V : mt.M)) + (grow * r + 4 * c4) * 4;
        *reinterpret_cast<gptr<u32x4>>(dst) = val;
      }
    }
    store_operand_rows(mt.Nb, c, 0);
    if (KEEP || (TM == 2 && r < FIRA_FUSE_DROP_R)) {
#pragma unroll
      for (int tn = 0; tn < 2; ++tn) {                             // (128 bytes of a factor's row per half wave)
        const int col = 64 * wcol + 32 * tn + l32;
#pragma unroll
        for (int v = 0; v < 8; ++v) {
          const int row = row_w + 4 * hi + 8 * (v >> 2) + (v & 3);
          if (INTERIOR || (col < r && row < L)) as_global(mt.Rt)[(unsigned)(row * r + col)] = cur[tn][v];
        }
      }
      if (planes) {
        __syncthreads();
        z_image(std::integral_constant<int, 1>{});
        __syncthreads();
        store_operand_rows(mt.Nb, c, kblocks);
      }
    }
    // everybody's share of the next chunk has landed, and all are done reading this chunk's LDS (the stores
    // above have read it into registers: the compiler waits for those LDS reads before the barrier)
    if (c + 1 < NCHUNK) __syncthreads();
  }
}

template <bool LEFT, int RT, int TM, bool KEEP>
__device__ __forceinline__ void project_adam_tile_as(char* lds, const FiraMat& mt, const FiraScal* __restrict__ scal,
                                                     const FiraEnt& ent, const FiraTile& tile, const FiraHp& hp, bool gram) {
  GemmOperands g;
  g.a_row0 = tile.ta * FIRA_PA;
  g.a_rows = mt.L;
  g.b_row0 = 0;
  g.b_rows = mt.r;
  g.B = as_global<const bf16_raw>(mt.PT);
  g.ldb = mt.rq;
  g.KB = mt.Sp;
  g.A = as_global(reinterpret_cast<const bf16_raw*>(ent.G));
  g.lda = mt.ld;
  g.KA = mt.S;
  const int t = scal[ent.mat].t + 1;             // 1-based
  // RT = 2 has no register to spare while loads are in flight (one value went to memory and back there)
  float bias = RT == 2 ? bias_correction(hp, t) : 0.0f;
  auto prologue = [&] {
    if (RT == 2) return;
    bias = bias_correction(hp, t);
    asm volatile("" : "+v"(bias));                 // (here, not where it is used)
  };
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
  const int wave = threadIdx.x >> 6;
  const bool sumsq = TM == 2 ? (wave & 1) == 0 : wave == 0;      // the waves of the first 64 rank columns
  auto run = [&](auto mode) {
    constexpr ProjLoads MODE = decltype(mode)::value;
    if (sumsq) proj_pipeline<LEFT, MODE, true, RT, true, TM>(acc, lds, g, sq, prologue);
    else if (RT == 1 || wave < 4) proj_pipeline<LEFT, MODE, false, RT, true, TM>(acc, lds, g, sq, prologue);
    else if constexpr (RT == 2) proj_pipeline<LEFT, MODE, false, 2, false, TM>(acc, lds, g, sq, prologue);
  };
  if (proj_interior(g)) run(std::integral_constant<ProjLoads, PROJ_FAST>{});
  else run(std::integral_constant<ProjLoads, PROJ_EDGE>{});        // (both sides are at least r >= FIRA_FUSE_MIN_R)
  if (g.a_row0 + FIRA_PA <= mt.L && mt.r == 64 * TM * RT) project_adam_epilogue<RT, TM, true, KEEP>(acc, lds, mt, hp, bias, g.a_row0, sq, !gram);
  else project_adam_epilogue<RT, TM, false, KEEP>(acc, lds, mt, hp, bias, g.a_row0, sq, !gram);
}

// Ranks up to 128 fill half a rank tile; their tiles multiply 64 x 64 per wave and go through
// Adam in four chunks instead of eight (56 matrices of 512 x 512 and 512 x 1376 at r = 128: 48 us instead of 65; 40 since edge tiles keep their loads
// in flight).
template <bool LEFT, int RT, bool KEEP>
__device__ __forceinline__ void project_adam_tile(char* lds, const FiraMat* __restrict__ mats, const FiraScal* __restrict__ scal, FiraScal* __restrict__ scal_out,
                                                  const FiraEnt* __restrict__ ents, const FiraTile& tile, const FiraHp& hp) {
  const FiraEnt ent = ents[tile.ent];
  const bool gram = use_gram(hp, scal[ent.mat]);
  if (!gram && !KEEP) return;    // this matrix takes the residual route: the two-kernel path serves it
  if (tile.ta == 0 && threadIdx.x == 0) set_limiter_inputs(scal_out + ent.mat, scal[ent.mat]);
  const FiraMat mt = mats[ent.mat];
  if (RT == 1 && mt.r <= 128) project_adam_tile_as<LEFT, 1, 2, KEEP>(lds, mt, scal, ent, tile, hp, gram);
  else project_adam_tile_as<LEFT, RT, 4, KEEP>(lds, mt, scal, ent, tile, hp, gram);
}

// One grid for both orientations: workgroups [0, blocks_left) take the tiles of the matrices with
// m <= n, the rest those with m > n.  With one workgroup per CU (RT = 2) a launch ends in a round that is
// only partly filled; one launch instead of two has one such round.  blocks_left is a multiple of 8,
// which keeps the XCD-aware mapping of each part.
template <int RT, bool KEEP>
__device__ __forceinline__ void project_adam_block(char* lds, const FiraMat* __restrict__ mats, const FiraScal* __restrict__ scal, FiraScal* __restrict__ scal_out,
                                                   const FiraEnt* __restrict__ ents, const FiraTile* __restrict__ tiles_left, int ntiles_left, int blocks_left,
                                                   const FiraTile* __restrict__ tiles_right, int ntiles_right, const FiraHp& hp) {
  if ((int)blockIdx.x < blocks_left) {
    const int ti = xcd_chunked_index(blockIdx.x, ntiles_left);
    if (ti < 0) return;
    project_adam_tile<true, RT, KEEP>(lds, mats, scal, scal_out, ents, tiles_left[ti], hp);
  } else {
    const int ti = xcd_chunked_index((int)blockIdx.x - blocks_left, ntiles_right);
    if (ti < 0) return;
    project_adam_tile<false, RT, KEEP>(lds, mats, scal, scal_out, ents, tiles_right[ti], hp);
  }
}
template <int RT>
__global__ __launch_bounds__(256 * RT, RT == 1 ? 2 : 1) void fira_project_adam_kernel(const FiraMat* __restrict__ mats,
                                                                                      const FiraScal* __restrict__ scal, FiraScal* __restrict__ scal_out,
                                                                                      const FiraEnt* __restrict__ ents,
                                                                                      const FiraTile* __restrict__ tiles_left, int ntiles_left,
                                                                                      int blocks_left,
                                                                                      const FiraTile* __restrict__ tiles_right, int ntiles_right,
                                                                                      FiraHp hp) {
  extern __shared__ __attribute__((aligned(16))) char lds[];   // FIRA_FUSE_LDS(RT) bytes
  project_adam_block<RT, false>(lds, mats, scal, scal_out, ents, tiles_left, ntiles_left, blocks_left, tiles_right, ntiles_right, hp);
}
// The same with R left behind (KEEP), on every route, for lists whose matrices all do that (and which leave_r_fill finds long enough).
template <int RT>
__global__ __launch_bounds__(256 * RT, RT == 1 ? 2 : 1) void fira_fused_leave_r_kernel(const FiraMat* __restrict__ mats,
                                                                                       const FiraScal* __restrict__ scal, FiraScal* __restrict__ scal_out,
                                                                                       const FiraEnt* __restrict__ ents,
                                                                                       const FiraTile* __restrict__ tiles_left, int ntiles_left,
                                                                                       int blocks_left,
                                                                                       const FiraTile* __restrict__ tiles_right, int ntiles_right,
                                                                                       FiraHp hp) {
  extern __shared__ __attribute__((aligned(16))) char lds[];   // FIRA_FUSE_LDS(RT) bytes
  project_adam_block<RT, true>(lds, mats, scal, scal_out, ents, tiles_left, ntiles_left, blocks_left, tiles_right, ntiles_right, hp);
}

// ------------------------------------------------------------------------------------------------
// Projection and Adam for small ranks (r <= 64, the fine-tuning setting's r = 32), bf16 matrices on every route and with any
// rank.  The tile is 128 (gradient side) x 64 (rank): with a 256-wide rank tile three quarters or more of the multiplies
// would work on padding.  Wave w owns gradient rows 32 w .. 32 w + 31 and all 64 rank columns (two accumulator
// blocks), so the kernel needs few registers and 34 KB of LDS (Adam's rows; the multiplies take 28), four workgroups share a CU, and the
// gradient stream is what bounds it.  Same pipeline as proj_pipeline (single gradient tile, E and O halves);
// a ring stage is 64 rows x 32 k = 4 KB, one request instruction per wavefront, so the E-half wait is
// vmcnt(1) and the O-half wait vmcnt(5) (one ring request and the four of A(S+1) are younger).
//
// A wave holds the whole rows R_i of its factors, so Adam runs on them there, without a barrier: the rows pass through LDS, so that
// a factor's row is 8 or 16 lanes' four values each, and M, V, R and Z come and go in 16- and 8-byte pieces of whole rows.  R is
// written, since fira_get_lowrank and the limited steps read it, but no pass of its own reads it back.
// A step with the projection and Adam in two launches and in this one: 160 matrices of 4096 x 4096 and 4096 x 11008 at r = 32 6830 and 6700 us
// (the projection alone 1745, Adam 334, this kernel 1958); 350M shapes at r = 16, 32 and 64 602, 612, 644 and 525, 540, 590, on the residual
// route at r = 32 790 and 701; 8 blocks of 512 x 512 and 512 x 1376 at r = 64 87 and 74; one block of 256 x 256 and 256 x 688
// 26.8 and 24.4 at r = 16, 26.0 and 26.1 at r = 64.  Ranks that are no multiple of four, whose N and R went out as operands
// for a pass of their own to form Z from: 350M shapes at r = 50 791 and 577, the 1B shapes 2595 and 2165.  (The four workgroups' 128
// registers leave five values of an edge tile in memory during its multiplies, outside the loop over K.)
// ------------------------------------------------------------------------------------------------
#define FIRA_PROJ_SMALL_STAGE (FIRA_PS * 64)
#define FIRA_PROJ_SMALL_PITCH 68   // floats of a factor's row in LDS: 16-byte alignment, banks shifted from row to row
#define FIRA_PROJ_SMALL_LDS (FIRA_PA * FIRA_PROJ_SMALL_PITCH * 4)   // more than the gradient tile and the ring take
static_assert(FIRA_PROJ_SMALL_LDS >= FIRA_PROJ_LDS_A + FIRA_RING_STAGES * FIRA_PROJ_SMALL_STAGE, "the multiply phase fits");

template <bool SUMSQ>
__device__ __forceinline__ void proj_compute_small(f32x16_t (&acc)[2], const char* la, const char* lb, int kk4, float& sq) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  bf16x8_t fa[2], fb[2][2];
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) {
    fa[kk] = *reinterpret_cast<const bf16x8_t*>(la + lds_tile_off(32 * wave + (lane & 31), 2 * (kk4 + kk) + (lane >> 5)));
#pragma unroll
    for (int t = 0; t < 2; ++t)
      fb[kk][t] = *reinterpret_cast<const bf16x8_t*>(lb + ring_tile_off(32 * t + (lane & 31), 2 * kk + (lane >> 5)));
  }
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
    for (int t = 0; t < 2; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[kk], fb[kk][t], acc[t], 0, 0, 0);
    if (SUMSQ) sq = frag_sumsq(fa[kk], sq);
  }
}

template <bool LEFT, ProjLoads MODE, bool SUMSQ, typename Prologue>
__device__ __forceinline__ void proj_pipeline_small(f32x16_t (&acc)[2], char* lds, const GemmOperands& g, float& sq, Prologue prologue) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  char* la = lds;
  char* ring = lds + FIRA_PROJ_LDS_A;
  const unsigned ring0 = (unsigned)(size_t)(lds_ptr)ring;
  const int SS = g.KB / 64;
  const int lrow = lane >> 2;
  const int chunk = (lane & 3) ^ ring_swz(lrow);
  const unsigned offb = (unsigned)(lrow * 64 + chunk * 16);
  const char* pb = reinterpret_cast<const char*>((const bf16_raw*)g.B) + ((long long)g.b_row0 + 16 * wave) * 64;
  auto request_b = [&](int s) {   // this wave's 16 of the stage's 64 rows
    lds_dma16(pb + (long long)s * g.ldb * 64, offb, ring0 + (unsigned)((s % FIRA_RING_STAGES) * FIRA_PROJ_SMALL_STAGE + wave * 1024));
  };
  ProjALoader<LEFT, MODE> al(g);
  u32x4 ra[4];
  al.load(ra);                                 // A(0)
  request_b(0);
  request_b(1);
  prologue();
  auto stage = [&](auto last, int S) {
    constexpr bool LAST = decltype(last)::value;
    wait_loads<1>(ra);                         // A(S) and D(2S) have landed; D(2S+1) may be in flight
    asm volatile("s_barrier" ::: "memory");
    if (MODE == PROJ_EDGE) al.template settle<LAST>(ra);
    proj_store_a<LEFT>(la, ra);
    if (!LAST) {
      request_b(2 * S + 2);
      if (MODE == PROJ_EDGE && S + 2 == SS) al.last();
      al.load(ra);                             // A(S+1)
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    proj_compute_small<SUMSQ>(acc, la, ring + ((2 * S) % FIRA_RING_STAGES) * FIRA_PROJ_SMALL_STAGE, 0, sq);
    // D(2S+1) has landed (guarded A loads may be fewer than 4 instructions: that path lets one stay)
    if (LAST) asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
    else if (MODE != PROJ_GUARDED) asm volatile("s_waitcnt vmcnt(5)\n\ts_barrier" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(1)\n\ts_barrier" ::: "memory");
    if (!LAST) request_b(2 * S + 3);
    proj_compute_small<SUMSQ>(acc, la, ring + ((2 * S + 1) % FIRA_RING_STAGES) * FIRA_PROJ_SMALL_STAGE, 2, sq);
  };
  for (int S = 0; S + 1 < SS; ++S) stage(std::false_type{}, S);
  stage(std::true_type{}, SS - 1);
}

// Adam on the wave's 32 factors, row0 the first one: LPR lanes to a row of r <= 4 LPR, two passes of 64 / LPR rows at a time, the next two's M
// and V requested before.  What a launch of few tiles waits for here is instructions, so what can be is formed once: offsets are
// 32 bits (L r <= 2^28), the factors k_i are stored in one piece at the end, and ||N_i|| and ||R_i|| share a square root.
// rows: [32][FIRA_PROJ_SMALL_PITCH], for R's way through LDS, k_i and ||R_i||^2 behind it.  g2: ||G_i||^2 of factor row0 + lane % 32.
template <int LPR>
__device__ __forceinline__ void small_adam_rows(const f32x16_t (&acc)[2], float* rows, const FiraMat& mt, const FiraScal& sc, const FiraHp& hp,
                                                float bias, int row0, float g2) {
  const int lane = threadIdx.x & 63, a = 4 * (lane % LPR), lrow = lane / LPR, r = mt.r;
  constexpr int ROWS = 64 / LPR, PASSES = 32 / ROWS;
  const bool matrix = hp.scaling == 1;              // one factor per matrix: the limiter kernel forms it from the rows' sums
  const bool leave = matrix || leaves_n_and_r(mt, sc.c), operand_r = leave || !use_gram(hp, sc);
  const bool planes = two_planes(hp, mt), rounded = rounds_n_and_r(mt);
  const int mine = min(max(r - a, 0), 4);           // this lane's values of a row
  const f32x4 zero = f32x4{0.f, 0.f, 0.f, 0.f};
  auto load4 = [&](gptr<char> base, unsigned off) { return load_row4(reinterpret_cast<gptr<const float>>(base + off), mine); };
  auto store4 = [&](gptr<char> base, unsigned off, const f32x4& v) { store_row4(reinterpret_cast<gptr<float>>(base + off), v, mine); };
  gptr<char> M = reinterpret_cast<gptr<char>>(as_global(mt.M)), V = reinterpret_cast<gptr<char>>(as_global(mt.V));
  gptr<char> Rt = reinterpret_cast<gptr<char>>(as_global(mt.Rt)), Nb = reinterpret_cast<gptr<char>>(as_global(mt.Nb)), Rb = reinterpret_cast<gptr<char>>(as_global(mt.Rb));
#pragma unroll
  for (int tn = 0; tn < 2; ++tn)
#pragma unroll
    for (int v = 0; v < 16; ++v)
      rows[(8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)) * FIRA_PROJ_SMALL_PITCH + 32 * tn + (lane & 31)] = acc[tn][v];
  // of this lane's next pass: its place in M, V and Rt, in the operands (whose second plane lies mt.rp / 32 K blocks on), and how many
  // factors there are from its own
  unsigned off = (unsigned)((row0 + lrow) * r + a) * 4u, op = (unsigned)(((a >> 5) * mt.Lq + row0 + lrow) * 32 + (a & 31)) * 2u;
  const unsigned step = (unsigned)(ROWS * r) * 4u, plane = (unsigned)((mt.rp >> 5) * mt.Lq) * 64u;
  int left = mt.L - row0 - lrow;
  const u32x2 keep = row4_mask(mine);
  f32x4 mnext[2], wnext[2];
  auto request = [&](unsigned o, int n) {
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      mnext[p] = wnext[p] = zero;
      if (n > ROWS * p && mine > 0) {
        mnext[p] = load4(M, o + p * step);
        wnext[p] = load4(V, o + p * step);
      }
    }
  };
  request(off, left);
  float* here = rows + lrow * FIRA_PROJ_SMALL_PITCH;
  // (the wave's lanes meet in LDS: its own accesses are in order, so a wait before the reads is all they need)
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll 1
  for (int p0 = 0; p0 < PASSES; p0 += 2) {
    f32x4 m[2], x[2];
    float nn[2], rr[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const bool live = left > ROWS * p && mine > 0;
      x[p] = *reinterpret_cast<const f32x4*>(here + p * ROWS * FIRA_PROJ_SMALL_PITCH + a);
      f32x4 w;
      nn[p] = rr[p] = 0.0f;
#pragma unroll
      for (int e = 0; e < 4; ++e) {                 // (the operand's padding multiplies a non-finite gradient to NaN)
        x[p][e] = live && e < mine ? x[p][e] : 0.0f;
        m[p][e] = hp.b1 * mnext[p][e] + hp.omb1 * x[p][e];
        w[e] = hp.b2 * wnext[p][e] + hp.omb2 * (x[p][e] * x[p][e]);
      }
      if (live) {
        store4(M, off + p * step, m[p]);
        store4(V, off + p * step, w);
        store4(Rt, off + p * step, x[p]);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {                 // (zero where m is)
        m[p][e] = adam_direction(m[p][e], w[e], bias, hp.epsf);
        nn[p] += m[p][e] * m[p][e];
        rr[p] += x[p][e] * x[p][e];
      }
    }
    if (p0 + 2 < PASSES) request(off + 2 * step, left - 2 * ROWS);
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const float snn = row_sum<LPR>(nn[p]), srr = row_sum<LPR>(rr[p]);
      const float root = sqrtf((lane & 1) ? srr : snn), other = lane_xor<1>(root);
      const float k = hp.scaling == 2 ? 1.0f : ((lane & 1) ? other : root) / (((lane & 1) ? root : other) + hp.epsf);
      if (a == 0) *reinterpret_cast<float2*>(here + p * ROWS * FIRA_PROJ_SMALL_PITCH + 64) = float2{matrix ? snn : k, srr};
      f32x4 z = m[p];
      if (!leave) z = rounded ? bf16_rounded(m[p]) - k * bf16_rounded(x[p]) : m[p] - k * x[p];
      const bool live = left > ROWS * p;
      // rows past L are zero; the rows of a K block follow each other, 64 bytes each (a second block that is all padding holds the zeros
      // it was initialised with)
      const u32x2 h = pack_bf16x4(z), mask = live ? keep : u32x2{0u, 0u};
      *reinterpret_cast<gptr<u32x2>>(Nb + (op + p * ROWS * 64)) = h & mask;
      if (planes) *reinterpret_cast<gptr<u32x2>>(Nb + (op + p * ROWS * 64 + plane)) = split_remainder(z, h) & mask;
      if (operand_r) *reinterpret_cast<gptr<u32x2>>(Rb + (op + p * ROWS * 64)) = pack_bf16x4(x[p]);
    }
    off += 2 * step;
    op += 2 * ROWS * 64;
    left -= 2 * ROWS;
    here += 2 * ROWS * FIRA_PROJ_SMALL_PITCH;
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  if (lane < 32 && row0 + lane < mt.L) {
    const float2 kr = *reinterpret_cast<const float2*>(rows + lane * FIRA_PROJ_SMALL_PITCH + 64);
    as_global(mt.phi)[row0 + lane] = kr.x;
    if (matrix) as_global(mt.q)[row0 + lane] = kr.y;
    else if (have_g2(hp)) as_global(mt.q)[row0 + lane] = kr.x * kr.x * residual_sq(hp, g2, kr.y);
  }
}

template <bool LEFT, typename Prologue>
__device__ __forceinline__ void project_small_tile(f32x16_t (&acc)[2], char* lds, const FiraMat& mt, const FiraEnt& ent, const FiraTile& tile,
                                                   bool sumsq, float& sq, Prologue prologue) {
  GemmOperands g;
  g.a_row0 = tile.ta * FIRA_PA;
  g.a_rows = mt.L;
  g.b_row0 = 0;
  g.b_rows = mt.r;
  g.B = as_global<const bf16_raw>(mt.PT);
  g.ldb = mt.rq;
  g.KB = mt.Sp;
  g.A = as_global(reinterpret_cast<const bf16_raw*>(ent.G));
  g.lda = mt.ld;
  g.KA = mt.S;
  auto run = [&](auto mode) {
    if (sumsq) proj_pipeline_small<LEFT, decltype(mode)::value, true>(acc, lds, g, sq, prologue);
    else proj_pipeline_small<LEFT, decltype(mode)::value, false>(acc, lds, g, sq, prologue);
  };
  if (proj_interior(g)) run(std::integral_constant<ProjLoads, PROJ_FAST>{});
  else if (!proj_guarded(LEFT, g)) run(std::integral_constant<ProjLoads, PROJ_EDGE>{});
  else run(std::integral_constant<ProjLoads, PROJ_GUARDED>{});
}

// Both orientations in one grid, as in fira_project_kernel.
__global__ __launch_bounds__(FIRA_PROJ_THREADS, 4) void fira_project_small_kernel(const FiraMat* __restrict__ mats,
                                                                                  const FiraEnt* __restrict__ ents,
                                                                                  const FiraTile* __restrict__ tiles_left, int ntiles_left,
                                                                                  int blocks_left,
                                                                                  const FiraTile* __restrict__ tiles_right, int ntiles_right,
                                                                                  int norm_mode, const FiraScal* __restrict__ scal, FiraScal* __restrict__ scal_out, FiraHp hp) {
  extern __shared__ __attribute__((aligned(16))) char lds[];   // FIRA_PROJ_SMALL_LDS bytes
  const bool left = (int)blockIdx.x < blocks_left;
  const int ti = left ? xcd_chunked_index(blockIdx.x, ntiles_left) : xcd_chunked_index((int)blockIdx.x - blocks_left, ntiles_right);
  if (ti < 0) return;
  const FiraTile tile = left ? tiles_left[ti] : tiles_right[ti];
  const FiraEnt ent = ents[tile.ent];
  const FiraMat mt = mats[ent.mat];
  f32x16_t acc[2];
  float sq = 0.0f;
#pragma unroll
  for (int tn = 0; tn < 2; ++tn)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[tn][v] = 0.0f;
  const bool sumsq = norm_mode == 1;           // every wave owns its own 32 factors
  if (tile.ta == 0 && threadIdx.x == 0) set_limiter_inputs(scal_out + ent.mat, scal[ent.mat]);
  const int t = scal[ent.mat].t + 1;           // 1-based
  float bias;
  auto prologue = [&] {
    bias = bias_correction(hp, t);
    asm volatile("" : "+v"(bias));               // (here, not where it is used)
  };
  if (left) project_small_tile<true>(acc, lds, mt, ent, tile, sumsq, sq, prologue);
  else project_small_tile<false>(acc, lds, mt, ent, tile, sumsq, sq, prologue);
  const int lane = threadIdx.x & 63, row0 = tile.ta * FIRA_PA + 32 * (threadIdx.x >> 6);
  const float g2 = sq + __shfl_xor(sq, 32, 64);
  if (sumsq && lane < 32 && row0 + lane < mt.L) as_global(mt.g2)[row0 + lane] = g2;
  __syncthreads();                             // the multiplies are done with LDS
  float* rows = reinterpret_cast<float*>(lds) + 32 * __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * FIRA_PROJ_SMALL_PITCH;
  if (mt.r <= 32) small_adam_rows<8>(acc, rows, mt, scal[ent.mat], hp, bias, row0, g2);
  else small_adam_rows<16>(acc, rows, mt, scal[ent.mat], hp, bias, row0, g2);
}
