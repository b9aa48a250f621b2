// Fused element-wise / reduction passes of the Fira step (HBM-bound): Adam on the low-rank gradient
// with the per-factor norms, the limiter scalar, the construction of the back-projection operand,
// and the operand conversions done when a projector is installed.
#pragma once
#include <type_traits>
#include "fira_device.h"


// Work-list lookup for the row-blocked kernels: entry e covers row-blocks [ents[e].row0, ents[e+1].row0).
__device__ __forceinline__ int find_entry(const FiraEnt* __restrict__ ents, int count, int rowblock) {
  int lo = 0, hi = count - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (ents[mid].row0 <= rowblock) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// ||G_i - P R_i||^2 from ||G_i||^2 and ||R_i||^2 (Gram route), or ||G_i||^2 itself for the variant that
// scales the full gradient.
__device__ __forceinline__ float residual_sq(const FiraHp& hp, float g2, float rr) {
  return hp.variant == 1 ? g2 : fmaxf(g2 - rr, 0.0f);
}

// Adam's direction for one element (Eqs. 2-4), N = bias * m / (sqrt(v) + eps), bias = sqrt(1 - beta2^t) /
// (1 - beta1^t), from the hardware's square root and reciprocal (1 ulp each) rather than the correctly
// rounded library forms, which cost about five times the instructions: in the fused kernel that
// arithmetic is not hidden behind memory traffic.  The square-root instruction takes no subnormal
// input, so v is raised to the smallest normal number first: sqrt(v) then reads 1.1e-19 where it is
// smaller, which only an eps of that order could tell apart.  Otherwise the result is within a few
// ulp of the exact quotient.
__device__ __forceinline__ float adam_direction(float m1, float v1, float bias, float eps) {
  const float s = __builtin_amdgcn_sqrtf(fmaxf(v1, 0x1p-126f));
  return bias * m1 * __builtin_amdgcn_rcpf(s + eps);
}

// A lane's double, in every lane.
__device__ __forceinline__ double lane_value(double x, int lane) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)u, lane);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u >> 32), lane);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
// Adam's bias correction after t steps (Eq. 4), in double: 1 - beta2^t loses all accuracy in fp32 at small t.  Called by whole
// wavefronts, whose halves take one power each: a power is a chain of some three hundred instructions, which a launch of few tiles waits for.
__device__ __forceinline__ float bias_correction(const FiraHp& hp, int t) {
  const double p = 1.0 - pow((threadIdx.x & 32) ? hp.beta1 : hp.beta2, (double)t);
  return (float)(sqrt(lane_value(p, 0)) / lane_value(p, 32));
}

// x of lane l ^ OFF, and x plus that, between registers (a shuffle goes through LDS, ten times as far): sums over the lanes of a factor
// are chains of them.  Called by whole wavefronts.
typedef unsigned u32x2_s __attribute__((__vector_size__(2 * sizeof(unsigned))));
template <int CTRL>
__device__ __forceinline__ float dpp_move(float x) { return __uint_as_float((unsigned)__builtin_amdgcn_mov_dpp((int)__float_as_uint(x), CTRL, 0xf, 0xf, true)); }
template <int OFF>
__device__ __forceinline__ float lane_xor(float x) {
  static_assert(OFF == 1 || OFF == 2 || OFF == 4 || OFF == 8, "inside a row of 16 lanes");
  if (OFF == 1) return dpp_move<0xb1>(x);                       // quad_perm 1 0 3 2
  if (OFF == 2) return dpp_move<0x4e>(x);                       // quad_perm 2 3 0 1
  if (OFF == 4) return dpp_move<0x1b>(dpp_move<0x141>(x));      // l ^ 7 (row_half_mirror), then ^ 3 (quad_perm 3 2 1 0)
  return dpp_move<0x128>(x);                                    // row_ror 8
}
template <int OFF>
__device__ __forceinline__ float add_xor(float x) {
  if constexpr (OFF < 16) {
    return x + lane_xor<OFF>(x);
  } else {      // the swap leaves both lanes' values in every lane
    const unsigned u = __float_as_uint(x);
    const u32x2_s s = OFF == 16 ? __builtin_amdgcn_permlane16_swap(u, u, false, false) : __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __uint_as_float(s[0]) + __uint_as_float(s[1]);
  }
}
// Sum over the LPR lanes that share a factor's row.
template <int LPR>
__device__ __forceinline__ float row_sum(float x) {
  static_assert(LPR == 8 || LPR == 16 || LPR == 64, "");
  if (LPR == 64) x = add_xor<16>(add_xor<32>(x));
  if (LPR >= 16) x = add_xor<8>(x);
  return add_xor<1>(add_xor<2>(add_xor<4>(x)));
}
__device__ __forceinline__ float wave_sum(float x) { return row_sum<64>(x); }

// store one low-rank value as an MFMA operand element (plain bf16, or the three planes of the split)
// (`op` is a K-blocked array with `rows` padded rows; plane p of the split occupies k = p*rp + a.)
template <int KX>
__device__ __forceinline__ void store_operand(gptr<bf16_raw> op, int rows, long long row, int rp, int a, float x) {
  if (KX == 1) {
    op[kblk_index(rows, row, a)] = f32_to_bf16(x);
  } else {
    bf16_raw h, m, l;
    split3(x, h, m, l);
    op[kblk_index(rows, row, a)] = h;
    op[kblk_index(rows, row, rp + a)] = m;
    op[kblk_index(rows, row, 2 * rp + a)] = l;
  }
}
// Such an element of a fp32 matrix.
__device__ __forceinline__ float load_split_operand(gptr<const bf16_raw> op, int rows, long long row, int rp, int a) {
  return (bf16_to_f32(op[kblk_index(rows, row, a)]) + bf16_to_f32(op[kblk_index(rows, row, rp + a)])) +
         bf16_to_f32(op[kblk_index(rows, row, 2 * rp + a)]);
}

// ------------------------------------------------------------------------------------------------
// Adam on R (Eqs. 2-4 applied to R, Algorithm 1's Adam block) fused with the two norms of every
// factor (Algorithm 1, "Norm-Based Scaling").  One wavefront per long-side row:
//   M <- b1 M + (1-b1) R;  V <- b2 V + (1-b2) R^2;  N = bias * M / (sqrt(V) + eps)
//   k_i = ||N_i|| / (||R_i|| + eps);  N and R are also written as bf16 MFMA operands.
// ------------------------------------------------------------------------------------------------
template <int KX, int VEC>
__device__ __forceinline__ void adam_row(const FiraMat& mt, const FiraHp& hp, float bias, long long row, bool gram) {
  const int lane = threadIdx.x & 63;
  const int r = mt.r;
  gptr<const float> R = as_global<const float>(mt.Rt) + row * r;
  gptr<float> M = as_global(mt.M) + row * r;
  gptr<float> V = as_global(mt.V) + row * r;
  gptr<bf16_raw> Nb = as_global(mt.Nb);
  gptr<bf16_raw> Rb = as_global(mt.Rb);
  float nn = 0.0f, rr = 0.0f;
  for (int a = lane * VEC; a < r; a += 64 * VEC) {
    float rv[VEC], mv[VEC], vv[VEC], nv[VEC];
    if (VEC == 4) {
      *reinterpret_cast<f32x4*>(rv) = *reinterpret_cast<gptr<const f32x4>>(R + a);
      *reinterpret_cast<f32x4*>(mv) = *reinterpret_cast<gptr<const f32x4>>(M + a);
      *reinterpret_cast<f32x4*>(vv) = *reinterpret_cast<gptr<const f32x4>>(V + a);
    } else {
      rv[0] = R[a]; mv[0] = M[a]; vv[0] = V[a];
    }
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      mv[e] = hp.b1 * mv[e] + hp.omb1 * rv[e];
      vv[e] = hp.b2 * vv[e] + hp.omb2 * (rv[e] * rv[e]);
      nv[e] = adam_direction(mv[e], vv[e], bias, hp.epsf);
      nn += nv[e] * nv[e];
      rr += rv[e] * rv[e];
    }
    if (VEC == 4) {
      *reinterpret_cast<gptr<f32x4>>(M + a) = *reinterpret_cast<const f32x4*>(mv);
      *reinterpret_cast<gptr<f32x4>>(V + a) = *reinterpret_cast<const f32x4*>(vv);
    } else {
      M[a] = mv[0]; V[a] = vv[0];
    }
    if (KX == 1 && VEC == 4) {
      const long long o = kblk_index(mt.Lq, row, a);
      *reinterpret_cast<gptr<u32x2>>(Nb + o) = u32x2{pack_bf16x2(nv[0], nv[1]), pack_bf16x2(nv[2], nv[3])};
      *reinterpret_cast<gptr<u32x2>>(Rb + o) = u32x2{pack_bf16x2(rv[0], rv[1]), pack_bf16x2(rv[2], rv[3])};
    } else {
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        store_operand<KX>(Nb, mt.Lq, row, mt.rp, a + e, nv[e]);
        store_operand<KX>(Rb, mt.Lq, row, mt.rp, a + e, rv[e]);
      }
    }
  }
  nn = wave_sum(nn);
  rr = wave_sum(rr);
  if (lane == 0) {
    if (hp.scaling == 1) {
      // one factor per matrix: leave the row's ||N_i||^2 and ||R_i||^2 for the limiter kernel, which
      // sums them, forms the factor and writes it over phi
      as_global(mt.phi)[row] = nn;
      as_global(mt.q)[row] = rr;
    } else {
      const float k = (hp.scaling == 2) ? 1.0f : sqrtf(nn) / (sqrtf(rr) + hp.epsf);
      as_global(mt.phi)[row] = k;
      // Gram route: ||G_i - P R_i||^2 = ||G_i||^2 - ||R_i||^2 when P^T P = I (G_i^T P = R_i^T always)
      if (have_g2(hp)) as_global(mt.q)[row] = k * k * residual_sq(hp, as_global<const float>(mt.g2)[row], rr);
    }
  }
}

// What is left of four values when their nearest-even bf16 `hi` is taken off (exact).
__device__ __forceinline__ f32x4 bf16_remainder(const f32x4& z, const u32x2& hi) {
  return f32x4{z[0] - __uint_as_float(hi.x << 16), z[1] - __uint_as_float(hi.x & 0xffff0000u),
               z[2] - __uint_as_float(hi.y << 16), z[3] - __uint_as_float(hi.y & 0xffff0000u)};
}
__device__ __forceinline__ u32x2 pack_bf16x4(const f32x4& z) { return u32x2{pack_bf16x2(z[0], z[1]), pack_bf16x2(z[2], z[3])}; }
// Second bf16 plane of four values whose first plane (nearest-even bf16) is `hi`: bf16(z - hi), so that
// hi + lo carries 16 mantissa bits of z.
__device__ __forceinline__ u32x2 split_remainder(const f32x4& z, const u32x2& hi) { return pack_bf16x4(bf16_remainder(z, hi)); }

// The values a .. a + 3 of a low-rank row of r, `mine` of which exist (a row starts at any element if r is no multiple of four), and back.
__device__ __forceinline__ f32x4 load_row4(gptr<const float> p, int mine) {
  if (mine >= 4) return *reinterpret_cast<gptr<const f32x4_a4>>(p);
  f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int e = 0; e < 3; ++e)
    if (e < mine) v[e] = p[e];
  return v;
}
__device__ __forceinline__ void store_row4(gptr<float> p, const f32x4& v, int mine) {
  if (mine >= 4) *reinterpret_cast<gptr<f32x4_a4>>(p) = v;
  else
#pragma unroll
    for (int e = 0; e < 3; ++e)
      if (e < mine) p[e] = v[e];
}
// The same without a branch for rows of at least four values: the last four instead of a group that ends past r, moved down.
__device__ __forceinline__ f32x4 load_row4_inside(gptr<const float> row, int a, int r) {
  const int at = min(a, r - 4), d = a - at;
  f32x4 v = *reinterpret_cast<gptr<const f32x4_a4>>(row + at);
  if (d & 1) v = f32x4{v.y, v.z, v.w, 0.f};
  if (d & 2) v = f32x4{v.z, v.w, 0.f, 0.f};
  return v;
}
// Mask of their bf16 pairs: an operand's columns past r stay zero, even for a non-finite factor.
__device__ __forceinline__ u32x2 row4_mask(int mine) {
  return u32x2{mine <= 0 ? 0u : mine == 1 ? 0xffffu : ~0u, mine < 3 ? 0u : mine == 3 ? 0xffffu : ~0u};
}

// Planes of an operand row element: 1, 2 (Z of a bf16 matrix with hp.zsplit) or 3 (fp32 matrices).
template <int KX>
__device__ __forceinline__ int z_planes(const FiraHp& hp, const FiraMat& mt) { return KX == 1 ? (two_planes(hp, mt) ? 2 : 1) : 3; }
// Four consecutive values as that many planes (each the rounding of what the ones before leave).
template <int KX>
__device__ __forceinline__ void bf16_planes(const f32x4& z, int planes, u32x2 (&pl)[3]) {
  pl[0] = pack_bf16x4(z);
  if (KX != 1 || planes == 2) {
    const f32x4 d = bf16_remainder(z, pl[0]);
    pl[1] = pack_bf16x4(d);
    if (KX != 1) pl[2] = pack_bf16x4(bf16_remainder(d, pl[1]));
  }
}

// Sums of the squares of 64 consecutive values of a row, four to a lane of a row of 16 lanes and zeros past the end, in the order in which the fused
// projection/Adam kernel takes them: columns 32 apart (lanes 8 apart) in one lane, then by 16, 8 and 4 (lanes), 2 and 1 (a lane's four). At every
// step across lanes but the last ones each lane goes on with half of its values.
__device__ __forceinline__ float square_sum_of_64(const f32x4& x) {
  const bool upper = (threadIdx.x & 8) != 0, odd = (threadIdx.x & 4) != 0;
  float s[2];                                   // of values e, or 2 + e in the upper lanes
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const float keep = upper ? x[2 + e] : x[e], got = lane_xor<8>(upper ? x[e] : x[2 + e]);
    const float lo = upper ? got : keep, hi = upper ? keep : got;
    s[e] = __builtin_fmaf(lo, lo, hi * hi);
  }
  const float t = add_xor<1>(add_xor<2>((odd ? s[1] : s[0]) + lane_xor<4>(odd ? s[0] : s[1])));
  return add_xor<4>(add_xor<8>(t));
}
// Such sums of a row of up to 128 values in a half wave, and of up to 256 NIT in a wavefront (one after the other, as that kernel adds its waves' up).
__device__ __forceinline__ float square_sum_as_fused(const f32x4& x) { return add_xor<16>(square_sum_of_64(x)); }
template <int NIT>
__device__ __forceinline__ float square_sum_as_fused(const f32x4 (&x)[NIT]) {
  float sum = 0.0f;
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int part = (int)__float_as_uint(square_sum_of_64(x[it]));
#pragma unroll
    for (int w = 0; w < 4; ++w) sum += __uint_as_float((unsigned)__builtin_amdgcn_readlane(part, 16 * w));
  }
  return sum;
}

// Same update for matrices with r <= FIRA_ZREADY_MAX_R (fp32: FIRA_ZREADY_MAX_R_F32): the factor's N
// and R stay in registers until k_i is known, and the row is written once as the back-projection operand for
// an inactive limiter, Z_i = N_i - k_i R_i, rounded from fp32 a single time.  R is written as an
// operand only when the residual contraction will need it.  Z is K-blocked, 64 B per row and K
// block, so the workgroup's 16 rows are collected in LDS ([K block][16 rows][32]) and leave as
// 1 KB contiguous pieces (fira_adam_kernel).  fp32 matrices move 26 bytes per element here; with N and R written
// as planes and turned into Z by a pass of their own it was 92 (350M shapes at r = 256: 916 + 602 -> 364 us).
// rl: the same image of R for bf16 matrices on the residual route (null: R goes out from here, in 64-byte pieces).
// AS_FUSED: ranks whose lists take the fused projection/Adam kernel or this one by their length and by what else they hold.  What a matrix gets
// must not depend on that, so the two norms are summed as that kernel sums them.
template <int KX, int NIT, bool ODD>   // 256 * NIT >= r; ODD: r is no multiple of four
__device__ __forceinline__ void adam_row_zready(const FiraMat& mt, const FiraHp& hp, float bias, long long row, bool gram,
                                                bf16_raw* zl, bf16_raw* rl, int rowlocal, bool leave) {
  const int lane = threadIdx.x & 63;
  const int r = mt.r;
  gptr<const float> R = as_global<const float>(mt.Rt) + row * r;
  gptr<float> M = as_global(mt.M) + row * r;
  gptr<float> V = as_global(mt.V) + row * r;
  gptr<bf16_raw> Rb = as_global(mt.Rb);
  constexpr bool AS_FUSED = KX == 1 && !ODD && 256 * NIT <= FIRA_FUSE_MAX_R;
  float nn = 0.0f, rr = 0.0f;
  f32x4 nv[NIT], rv[NIT];
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int a = lane * 4 + 256 * it;
    if (AS_FUSED) nv[it] = rv[it] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (a < r) {
      auto load = [&](gptr<const float> p) { return ODD ? load_row4_inside(p, a, r) : (f32x4)*reinterpret_cast<gptr<const f32x4>>(p + a); };
      rv[it] = load(R);
      f32x4 mv = load(M), vv = load(V);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        mv[e] = hp.b1 * mv[e] + hp.omb1 * rv[it][e];
        vv[e] = hp.b2 * vv[e] + hp.omb2 * (rv[it][e] * rv[it][e]);
        nv[it][e] = adam_direction(mv[e], vv[e], bias, hp.epsf);
        if (!AS_FUSED) {
          nn += nv[it][e] * nv[it][e];
          rr += rv[it][e] * rv[it][e];
        }
      }
      store_row4(M + a, mv, ODD ? r - a : 4);
      store_row4(V + a, vv, ODD ? r - a : 4);
    }
  }
  if constexpr (AS_FUSED) {
    nn = square_sum_as_fused(nv);
    rr = square_sum_as_fused(rv);
  } else {
    nn = wave_sum(nn);
    rr = wave_sum(rr);
  }
  const float k = (hp.scaling == 2) ? 1.0f : sqrtf(nn) / (sqrtf(rr) + hp.epsf);
  const int planes = z_planes<KX>(hp, mt), plane_off = (mt.rp >> 5) * (FIRA_ROWS_PER_WG * 32);   // planes of the LDS image
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int a = lane * 4 + 256 * it;
    if (a < mt.rp) {
      u32x2 zp[3];
      zp[0] = zp[1] = zp[2] = u32x2{0u, 0u};
      if (a < r) {
        if (ODD && KX == 1) bf16_planes<KX>(leave ? nv[it] : bf16_rounded(nv[it]) - k * bf16_rounded(rv[it]), planes, zp);
        else bf16_planes<KX>(nv[it] - k * rv[it], planes, zp);
        if (ODD) {
          const u32x2 mask = row4_mask(r - a);
#pragma unroll
          for (int p = 0; p < 3; ++p) zp[p] &= mask;
        }
        if ((!gram || (ODD && leave)) && !rl) {
          u32x2 rb[3];
          bf16_planes<KX>(rv[it], KX == 1 ? 1 : 3, rb);
#pragma unroll
          for (int p = 0; p < (KX == 1 ? 1 : 3); ++p)
            *reinterpret_cast<gptr<u32x2>>(Rb + kblk_index(mt.Lq, row, p * mt.rp + a)) = rb[p];
        }
      }
      const int at = (a >> 5) * (FIRA_ROWS_PER_WG * 32) + rowlocal * 32 + (a & 31);
#pragma unroll
      for (int p = 0; p < (KX == 1 ? 2 : 3); ++p)
        if (p < planes) *reinterpret_cast<u32x2*>(zl + at + p * plane_off) = zp[p];
      if (KX == 1 && rl) *reinterpret_cast<u32x2*>(rl + at) = a < r ? pack_bf16x4(rv[it]) : u32x2{0u, 0u};
    }
  }
  if (lane == 0) {
    as_global(mt.phi)[row] = k;
    if (have_g2(hp)) as_global(mt.q)[row] = k * k * residual_sq(hp, as_global<const float>(mt.g2)[row], rr);
  }
}

// Rows of few values: LPR lanes to a row, so that a wavefront takes 64 / LPR rows at once.  16 for fp32 matrices with r <= 64; 32 for bf16 ones with
// 64 < r <= 128, r a multiple of four (whose norms are summed as the fused kernel sums them, see AS_FUSED above).
// Bound by instructions in short lists and by memory in long ones.  A row at a time, half the lanes idle, and two at a time, a step at r = 96 of one block of
// 256 x 688 28.9 and 26.4 us, two of 512 x 1376 53.3 and 49.7, 24 of 1024 x 2736 on the residual route 903 and 854 and in two planes 802 and 743.
template <int KX, int LPR>   // 4 LPR >= r
__device__ __forceinline__ void adam_rows_short(const FiraMat& mt, const FiraHp& hp, float bias, long long row_base,
                                                bool gram, bf16_raw* zl, bf16_raw* rl, int wave, int i) {
  const int lane = threadIdx.x & 63;
  const int g = lane / LPR, a = (lane % LPR) * 4;
  const int r = mt.r;
  const long long row = row_base + g;
  const bool live = row < mt.L && a < r;
  const int mine = KX == 1 ? 4 : r - a;
  gptr<const float> R = as_global<const float>(mt.Rt) + row * r;
  gptr<float> M = as_global(mt.M) + row * r;
  gptr<float> V = as_global(mt.V) + row * r;
  f32x4 nv = f32x4{0.f, 0.f, 0.f, 0.f}, rv = nv;
  float nn = 0.0f, rr = 0.0f;
  if (live) {
    rv = load_row4(R + a, mine);
    f32x4 mv = load_row4(M + a, mine);
    f32x4 vv = load_row4(V + a, mine);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      mv[e] = hp.b1 * mv[e] + hp.omb1 * rv[e];
      vv[e] = hp.b2 * vv[e] + hp.omb2 * (rv[e] * rv[e]);
      nv[e] = adam_direction(mv[e], vv[e], bias, hp.epsf);
      nn += nv[e] * nv[e];
      rr += rv[e] * rv[e];
    }
    store_row4(M + a, mv, mine);
    store_row4(V + a, vv, mine);
  }
  if constexpr (KX == 1) {
    nn = square_sum_as_fused(nv);
    rr = square_sum_as_fused(rv);
  } else {
    nn = row_sum<16>(nn);
    rr = row_sum<16>(rr);
  }
  const float k = (hp.scaling == 2) ? 1.0f : sqrtf(nn) / (sqrtf(rr) + hp.epsf);
  if (a < mt.rp) {
    const int planes = z_planes<KX>(hp, mt);
    u32x2 zp[3];
    zp[0] = zp[1] = zp[2] = u32x2{0u, 0u};   // rows beyond L and columns beyond r: the operand's zero padding
    if (live) {
      bf16_planes<KX>(nv - k * rv, planes, zp);
      const u32x2 mask = row4_mask(mine);
#pragma unroll
      for (int p = 0; p < 3; ++p) zp[p] &= mask;
      if (!gram && !rl) {
        u32x2 rb[3];
        bf16_planes<KX>(rv, KX == 1 ? 1 : 3, rb);
#pragma unroll
        for (int p = 0; p < (KX == 1 ? 1 : 3); ++p)
          *reinterpret_cast<gptr<u32x2>>(as_global(mt.Rb) + kblk_index(mt.Lq, row, p * mt.rp + a)) = rb[p];
      }
    }
    const int at = (a >> 5) * (FIRA_ROWS_PER_WG * 32) + (wave * 4 + i + g) * 32 + (a & 31);
#pragma unroll
    for (int p = 0; p < (KX == 1 ? 2 : 3); ++p)
      if (p < planes) *reinterpret_cast<u32x2*>(zl + at + p * (mt.rp >> 5) * (FIRA_ROWS_PER_WG * 32)) = zp[p];
    if (KX == 1 && rl) *reinterpret_cast<u32x2*>(rl + at) = live ? pack_bf16x4(rv) : u32x2{0u, 0u};
  }
  if (a == 0 && row < mt.L) {
    as_global(mt.phi)[row] = k;
    if (have_g2(hp)) as_global(mt.q)[row] = k * k * residual_sq(hp, as_global<const float>(mt.g2)[row], rr);
  }
}

// Rows that are no multiple of four values (ODD) have forms of their own, so that the others do not pay for their tails: N and R
// used to leave as operands there, for a pass of their own to form Z from.  A step over 24 blocks of 1024 x 2736 at r = 97 904 us then, 781
// now, on the residual route 1056 and 954; 8 blocks of 2048 x 5461 at r = 255, 511 and 770 1277, 1938, 2967 and 1096, 1646, 2447; four
// blocks of 800 x 2000 in fp32 at r = 130 394 and 334.
// STAGE_R: the launch's LDS has room for R beside Z (bf16 matrices with 64 < r <= FIRA_RSTAGE_MAX_R on the residual route): R, too, then
// leaves in pieces of 1 KB.  Above that rank the image would halve the wavefronts in flight.  Adam on the residual route over
// 168 matrices of the 1B shapes at r = 512: 1420 us, 1725 with R in 64-byte pieces; 350M shapes at r = 256: 346, 397.
// KX: the matrices that this launch serves, bf16 (1) or fp32 (FIRA_KX_SPLIT); the row-blocks of the others leave.
// (One kernel for both took ten registers too many for four wavefronts per SIMD, and 2 % of the bf16 time.)
template <int KX, bool STAGE_R>
__global__ __launch_bounds__(256, 4) void fira_adam_kernel(const FiraMat* __restrict__ mats,
                                                        const FiraScal* __restrict__ scal, FiraScal* __restrict__ scal_out,
                                                        const FiraEnt* __restrict__ ents, int count,
                                                        int total_rowblocks, int backwards, FiraHp hp) {
  extern __shared__ __attribute__((aligned(16))) char adam_lds[];   // zready matrices: 16 rows x planes x rp bf16 (and R's)
  // backwards: R of the last matrices is still in the memory-side cache
  const int rb = backwards ? total_rowblocks - 1 - (int)blockIdx.x : (int)blockIdx.x;
  if (rb < 0 || rb >= total_rowblocks) return;
  const int e = find_entry(ents, count, rb);
  const FiraEnt ent = ents[e];
  const FiraMat mt = mats[ent.mat];
  if ((mt.kx == 1) != (KX == 1) || (KX == 1 && mt.r <= FIRA_PS)) return;   // (small ranks: fira_project_small_kernel)
  bf16_raw* zl = reinterpret_cast<bf16_raw*>(adam_lds);
  const bool zready = mt.zready && hp.scaling != 1;   // the matrix-level factor is not known in this kernel
  const FiraScal sc = scal[ent.mat];
  const bool gram = use_gram(hp, sc);
  if (hp.mixed && gram) return;                // the fused kernel has served this matrix
  if (rb == ent.row0 && threadIdx.x == 0) set_limiter_inputs(scal_out + ent.mat, sc);
  const float bias = bias_correction(hp, sc.t + 1);   // (the step count is 1-based)
  const int wave = threadIdx.x >> 6;
  const long long row_base = (long long)(rb - ent.row0) * FIRA_ROWS_PER_WG + wave * 4;
  const int planes = z_planes<KX>(hp, mt);
  const bool leave = leaves_n_and_r(mt, sc.c);
  const bool staged = STAGE_R && zready && !gram && mt.r <= FIRA_RSTAGE_MAX_R;
  bf16_raw* rl = staged ? zl + planes * (mt.rp >> 5) * (FIRA_ROWS_PER_WG * 32) : nullptr;
  constexpr int LPR = KX == 1 ? 32 : 16;
  if (zready && mt.r <= 4 * LPR && (KX != 1 || (mt.r & 3) == 0)) {
    for (int i = 0; i < 4; i += 64 / LPR) adam_rows_short<KX, LPR>(mt, hp, bias, row_base + i, gram, zl, rl, wave, i);
  } else if (zready) {
    auto rows = [&](auto nit, auto odd) __attribute__((always_inline)) {
      for (int i = 0; i < 4; ++i) {
        const long long row = row_base + i;
        if (row < mt.L) {
          adam_row_zready<KX, decltype(nit)::value, decltype(odd)::value>(mt, hp, bias, row, gram, zl, rl, wave * 4 + i, leave);
        } else {   // rows of the padding: zeros
          for (int a = (threadIdx.x & 63) * 4; a < (planes + (staged ? 1 : 0)) * mt.rp; a += 256)
            *reinterpret_cast<u32x2*>(zl + (a >> 5) * (FIRA_ROWS_PER_WG * 32) + (wave * 4 + i) * 32 + (a & 31)) = u32x2{0u, 0u};
        }
      }
    };
    auto by_rank = [&](auto odd) __attribute__((always_inline)) {
      if (mt.r <= 256) rows(std::integral_constant<int, 1>{}, odd);
      else if (mt.r <= 512) rows(std::integral_constant<int, 2>{}, odd);
      else if constexpr (KX == 1) rows(std::integral_constant<int, FIRA_ZREADY_MAX_R / 256>{}, odd);
    };
    if ((mt.r & 3) == 0) by_rank(std::false_type{});
    else by_rank(std::true_type{});
  } else {
    for (int i = 0; i < 4; ++i) {
      const long long row = row_base + i;
      if (row >= mt.L) break;
      if (KX == 1 && (mt.r & 3) == 0) adam_row<1, 4>(mt, hp, bias, row, gram);
      else adam_row<KX, 1>(mt, hp, bias, row, gram);
    }
  }
  if (zready) {
    __syncthreads();
    // the 16 rows of one K block are 1 KB of contiguous memory
    const long long row0 = (long long)(rb - ent.row0) * FIRA_ROWS_PER_WG;
    auto flush = [&](bf16_raw* op, const char* image, int nplanes) {      // plane p: K blocks from p rp/32
      gptr<char> out = reinterpret_cast<gptr<char>>(as_global(op));
      const int nbytes = nplanes * (mt.rp >> 5) * (FIRA_ROWS_PER_WG * 64);
      for (int o = threadIdx.x * 16; o < nbytes; o += 256 * 16) {
        const int kb = o / (FIRA_ROWS_PER_WG * 64), w = o % (FIRA_ROWS_PER_WG * 64);
        *reinterpret_cast<gptr<u32x4>>(out + ((long long)kb * mt.Lq + row0) * 64 + w) = *reinterpret_cast<const u32x4*>(image + o);
      }
    };
    flush(mt.Nb, adam_lds, planes);
    if (staged) flush(mt.Rb, reinterpret_cast<const char*>(rl), 1);
  }
}

// ------------------------------------------------------------------------------------------------
// Norm-growth limiter (Eq. 12 in Algorithm 1's form): one workgroup per listed matrix sums the
// tile partials of ||S||^2 in a fixed order (fp64), derives the factor c, and advances the state.
// ------------------------------------------------------------------------------------------------
#define FIRA_LIMITER_THREADS 256
// Workgroup sum in a fixed order: butterfly inside each wavefront, then the four wavefronts in order.
__device__ __forceinline__ double limiter_block_sum(double x, double* red) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) x += __shfl_xor(x, off, 64);
  __syncthreads();                       // red may still be read from the previous call
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}

// This thread's share of a sum of n values, in a fixed order; eight loads in flight.
__device__ __forceinline__ double limiter_thread_sum(gptr<const float> x, int n) {
  double a = 0.0;
  for (int i = threadIdx.x; i < n; i += 8 * FIRA_LIMITER_THREADS) {
    float v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = x[min(i + k * FIRA_LIMITER_THREADS, n - 1)];
#pragma unroll
    for (int k = 0; k < 8; ++k) a += i + k * FIRA_LIMITER_THREADS < n ? (double)v[k] : 0.0;
  }
  return a;
}
// ||S||^2 (acc) of a matrix with a factor per row or none, and where both routes' data are at hand the Gram route's value of it (accg).
__device__ __forceinline__ void limiter_sums(const FiraMat& mt, const FiraEnt& ent, const float* __restrict__ partial, bool gram, bool calibrate,
                                             double* red, double& acc, double& accg) {
  const double a = gram || calibrate ? limiter_thread_sum(as_global<const float>(mt.q), mt.L) : 0.0;
  acc = limiter_block_sum(gram ? a : limiter_thread_sum(as_global<const float>(partial) + ent.part0, ent.npart), red);
  accg = calibrate ? limiter_block_sum(a, red) : 0.0;     // (uniform over the workgroup)
}
// The limiter's factor for ||S|| = sn (Eq. 12).
__device__ __forceinline__ double limiter_factor(const FiraHp& hp, double sn, int has_prev, double s_prev) {
  if (!has_prev || isinf(hp.gamma) || sn == 0.0) return 1.0;
  const double den = s_prev + hp.eps;
  const double ratio = den > 0.0 ? sn / den : INFINITY;
  return hp.gamma / fmax(ratio, hp.gamma);
}
// The state after the step (one thread).
__device__ __forceinline__ void limiter_advance(FiraScal& s, FiraGate& gate, const FiraHp& hp, bool gram, bool calibrate, double acc, double accg, double sn,
                                                double c, int t) {
  if (calibrate) gate.gram_err = s.gram_err = (acc == accg) ? 0.0f : (float)fmin(fabs(accg - acc) / fmax(acc, 1e-300), 3.0e38);
  s.gram_now = gram ? (hp.fused ? 2 : 1) : 0;
  s.s_pre = sn;
  s.s_post = c * sn;
  s.s_prev = c * sn;        // the remembered norm is the limited one
  s.has_prev = 1;
  s.c = (float)c;
  s.t = t + 1;
}

// The limiter by itself: one factor per matrix (Eq. 9), which is worked out here and written over phi, a step without Z, or a long list.
__global__ __launch_bounds__(FIRA_LIMITER_THREADS) void fira_limiter_kernel(const FiraMat* __restrict__ mats,
                                                                            FiraScal* __restrict__ scal,
                                                                            const FiraEnt* __restrict__ ents,
                                                                            const float* __restrict__ partial, FiraGate* __restrict__ gate, FiraHp hp) {
  __shared__ double red[4];
  const FiraEnt ent = ents[blockIdx.x];
  const int tid = threadIdx.x;
  const FiraScal sc0 = scal[ent.mat];
  const FiraMat mt = mats[ent.mat];
  const bool gram = use_gram(hp, sc0);
  // On the residual route with the Gram data at hand (the first step after an install), also form the
  // Gram route's value and record how far it is from the exact one: the second gate of that route.
  const bool calibrate = !gram && calibrates_gram(hp, sc0);
  double acc = 0.0, accg = 0.0;
  if (hp.scaling == 1) {
    // Matrix-level factor (Eq. 9): k = ||N|| / (||R|| + eps) from the row sums the Adam kernel left in
    // phi and q; ||S||^2 = k^2 * (sum_i ||G_i - P R_i||^2), the sum taken with unit factors by either route.
    gptr<float> phi = as_global(mt.phi);
    gptr<const float> q = as_global<const float>(mt.q);
    gptr<const float> g2 = as_global<const float>(mt.g2);
    double nn = 0.0, rr = 0.0;
    for (int i = tid; i < mt.L; i += FIRA_LIMITER_THREADS) {
      nn += (double)phi[i];
      rr += (double)q[i];
      if (gram) acc += (double)residual_sq(hp, g2[i], q[i]);
      else if (calibrate) accg += (double)residual_sq(hp, g2[i], q[i]);
    }
    if (!gram)
      for (int i = tid; i < ent.npart; i += FIRA_LIMITER_THREADS) acc += (double)partial[ent.part0 + i];
    nn = limiter_block_sum(nn, red);     // (the barriers inside also order the reads of phi before its rewrite)
    rr = limiter_block_sum(rr, red);
    const float k = (float)(sqrt(nn) / (sqrt(rr) + hp.eps));
    acc *= (double)k * (double)k;
    accg *= (double)k * (double)k;
    for (int i = tid; i < mt.L; i += FIRA_LIMITER_THREADS) phi[i] = k;
    acc = limiter_block_sum(acc, red);
    if (calibrate) accg = limiter_block_sum(accg, red);
  } else {
    limiter_sums(mt, ent, partial, gram, calibrate, red, acc, accg);
  }
  if (tid == 0) {
    const double sn = sqrt(acc), c = limiter_factor(hp, sn, sc0.has_prev, sc0.s_prev);
    limiter_advance(scal[ent.mat], gate[ent.mat], hp, gram, calibrate, acc, accg, sn, c, sc0.t);
  }
}

// ------------------------------------------------------------------------------------------------
// Back-projection operand: Z_i = N_i - c k_i R_i, so that P N + c k (G - P R) = P Z + c k G.
// Overwrites N in place.  Matrices flagged zready hold Z for c = 1 already and skip this unless their limiter factor is below 1,
// but for those whose N and R were left as they are (leaves_n_and_r).
// ------------------------------------------------------------------------------------------------
// bf16 matrices: a wavefront takes sixteen rows, whose part of a K block is 1 KB of either operand, K blocks `first` and every step-th from there, two
// in flight.  c: the limiter's factor; k_i is read from phi (one value in all rows where there is a factor per matrix).
__device__ __forceinline__ void makez_block(const FiraMat& mt, float c, long long row0, int first, int step) {
  const int lane = threadIdx.x & 63, a8 = (lane & 3) * 8;
  const long long row = row0 + (lane >> 2);
  const int kblocks = (mt.r + 31) >> 5;
  if (row >= mt.L) return;
  gptr<char> Nb = reinterpret_cast<gptr<char>>(as_global(mt.Nb)) + row0 * 64 + lane * 16;
  gptr<const char> Rb = reinterpret_cast<gptr<const char>>(as_global<const bf16_raw>(mt.Rb)) + row0 * 64 + lane * 16;
  const float f = c * as_global<const float>(mt.phi)[row];
  for (int kb0 = first; kb0 < kblocks; kb0 += 2 * step) {
    u32x4 nv[2], rv[2];
#pragma unroll
    for (int u = 0; u < 2; ++u)
      if (kb0 + step * u < kblocks) {
        const long long at = (long long)(kb0 + step * u) * mt.Lq * 64;
        nv[u] = *reinterpret_cast<gptr<const u32x4>>(Nb + at);
        rv[u] = *reinterpret_cast<gptr<const u32x4>>(Rb + at);
      }
#pragma unroll
    for (int u = 0; u < 2; ++u)
      if (kb0 + step * u < kblocks) {
        const int left = mt.r - 32 * (kb0 + step * u) - a8;      // padding stays zero even for a non-finite factor
        const unsigned nw[4] = {nv[u].x, nv[u].y, nv[u].z, nv[u].w}, rw[4] = {rv[u].x, rv[u].y, rv[u].z, rv[u].w};
        unsigned zw[4];
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          const float z0 = __uint_as_float(nw[d] << 16) - f * __uint_as_float(rw[d] << 16);
          const float z1 = __uint_as_float(nw[d] & 0xffff0000u) - f * __uint_as_float(rw[d] & 0xffff0000u);
          zw[d] = pack_bf16x2(2 * d < left ? z0 : 0.0f, 2 * d + 1 < left ? z1 : 0.0f);
        }
        *reinterpret_cast<gptr<u32x4>>(Nb + (long long)(kb0 + step * u) * mt.Lq * 64) = u32x4{zw[0], zw[1], zw[2], zw[3]};
      }
  }
}
__device__ __forceinline__ void makez_row_split(const FiraMat& mt, float f, long long row) {
  const int lane = threadIdx.x & 63;
  gptr<bf16_raw> Nb = as_global(mt.Nb);
  gptr<const bf16_raw> Rb = as_global<const bf16_raw>(mt.Rb);
  for (int a = lane; a < mt.r; a += 64) {
    const float z = load_split_operand((gptr<const bf16_raw>)Nb, mt.Lq, row, mt.rp, a) - f * load_split_operand(Rb, mt.Lq, row, mt.rp, a);
    store_operand<FIRA_KX_SPLIT>(Nb, mt.Lq, row, mt.rp, a, z);
  }
}

// Sixteen rows of a bf16 matrix that already hold Z for c = 1 (N_i - k_i R_i): add back (1 - c) k_i R_i, with R in fp32.  Memory bound, by one
// wavefront: a lane takes eight values of a row, the sixteen rows of a K block are 1 KB of Z in one piece, and two K blocks, `first` and every
// step-th from there, are in flight.  Limited steps over the 350M shapes at r = 256, residual route and two planes: 1364 and 1286 us row by
// row with Z in scattered 8-byte pieces, 1334 and 1239 this way.
__device__ __forceinline__ void fixz_block(const FiraMat& mt, float n, long long row0, int first, int step, bool zsplit) {
  const int lane = threadIdx.x & 63, a8 = (lane & 3) * 8;
  const long long row = row0 + (lane >> 2);
  const int kblocks = (mt.r + 31) >> 5;
  if (row >= mt.L) return;
  gptr<char> Nb = reinterpret_cast<gptr<char>>(as_global(mt.Nb)) + row0 * 64 + lane * 16;
  gptr<const float> R = as_global<const float>(mt.Rt) + row * mt.r + a8;
  const long long plane = (long long)(mt.rp >> 5) * mt.Lq * 64;
  const float f = n * as_global<const float>(mt.phi)[row];
  const f32x4 zero = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int kb0 = first; kb0 < kblocks; kb0 += 2 * step) {
    u32x4 zv[2], lv[2];
    f32x4 rv[2][2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int kb = kb0 + step * u;
      if (kb < kblocks) {
        zv[u] = *reinterpret_cast<gptr<const u32x4>>(Nb + (long long)kb * mt.Lq * 64);
        if (zsplit) lv[u] = *reinterpret_cast<gptr<const u32x4>>(Nb + (long long)kb * mt.Lq * 64 + plane);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          rv[u][q] = 32 * kb + a8 + 4 * q < mt.r ? *reinterpret_cast<gptr<const f32x4>>(R + 32 * kb + 4 * q) : zero;   // r is a multiple of four
        }
      }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int kb = kb0 + step * u;
      if (kb < kblocks) {
        const unsigned w[4] = {zv[u].x, zv[u].y, zv[u].z, zv[u].w}, l[4] = {lv[u].x, lv[u].y, lv[u].z, lv[u].w};
        u32x2 h[2], lo[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          f32x4 z = f32x4{__uint_as_float(w[2 * q] << 16), __uint_as_float(w[2 * q] & 0xffff0000u), __uint_as_float(w[2 * q + 1] << 16),
                          __uint_as_float(w[2 * q + 1] & 0xffff0000u)};
          if (zsplit)
            z += f32x4{__uint_as_float(l[2 * q] << 16), __uint_as_float(l[2 * q] & 0xffff0000u), __uint_as_float(l[2 * q + 1] << 16),
                       __uint_as_float(l[2 * q + 1] & 0xffff0000u)};
          z += f * rv[u][q];
          if (32 * kb + a8 + 4 * q >= mt.r) z = zero;      // padding stays zero even for a non-finite factor
          h[q] = pack_bf16x4(z);
          lo[q] = split_remainder(z, h[q]);
        }
        *reinterpret_cast<gptr<u32x4>>(Nb + (long long)kb * mt.Lq * 64) = u32x4{h[0].x, h[0].y, h[1].x, h[1].y};
        if (zsplit) *reinterpret_cast<gptr<u32x4>>(Nb + (long long)kb * mt.Lq * 64 + plane) = u32x4{lo[0].x, lo[0].y, lo[1].x, lo[1].y};
      }
    }
  }
}

// The same correction without R (after the fused kernel): Z = N - c k R = c (N - k R) + (1 - c) N, with N
// formed again from the updated M and V.  c Z_1 carries Z_1's bf16 rounding, so Z is rounded twice
// here; that happens only on the steps on which the limiter is active.
// A block of 16 rows per workgroup; memory bound (12 bytes per element), so a lane takes eight elements of a row, a
// wavefront the 16 rows of one K block (1 KB of Z in one piece, whole 128-byte lines of M and V), and two K blocks are
// in flight.  168 matrices of the 1B shapes at r = 512: 765 us; 832 us row by row, with Z in scattered 64-byte pieces.
__device__ __forceinline__ void fixz_block_from_moments(const FiraMat& mt, const FiraHp& hp, float c, float bias, long long row0) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const long long row = row0 + (lane >> 2);
  const int kblocks = mt.rp >> 5, a8 = (lane & 3) * 8;
  if (row >= mt.L) return;
  gptr<char> Nb = reinterpret_cast<gptr<char>>(as_global(mt.Nb)) + row0 * 64 + lane * 16;
  gptr<const float> M = as_global<const float>(mt.M) + row * mt.r + a8;
  gptr<const float> V = as_global<const float>(mt.V) + row * mt.r + a8;
  const float n = 1.0f - c;
  const f32x4 zero = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int kb0 = wave; kb0 < kblocks; kb0 += 8) {
    u32x4 zv[2];
    f32x4 mv[2][2], vv[2][2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int kb = kb0 + 4 * u;
      if (kb < kblocks) {
        zv[u] = *reinterpret_cast<gptr<const u32x4>>(Nb + (long long)kb * mt.Lq * 64);
#pragma unroll
        for (int q = 0; q < 2; ++q) {          // r is a multiple of four; the operand's columns past it are zero
          const bool in = 32 * kb + a8 + 4 * q < mt.r;
          mv[u][q] = in ? *reinterpret_cast<gptr<const f32x4>>(M + 32 * kb + 4 * q) : zero;
          vv[u][q] = in ? *reinterpret_cast<gptr<const f32x4>>(V + 32 * kb + 4 * q) : zero;
        }
      }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int kb = kb0 + 4 * u;
      if (kb < kblocks) {
        const unsigned w[4] = {zv[u].x, zv[u].y, zv[u].z, zv[u].w};
        unsigned o[4];
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          float z[2] = {__uint_as_float(w[d] << 16), __uint_as_float(w[d] & 0xffff0000u)};
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int e = 2 * d + h;
            z[h] = c * z[h] + n * adam_direction(mv[u][e >> 2][e & 3], vv[u][e >> 2][e & 3], bias, hp.epsf);
            if (32 * kb + a8 + e >= mt.r) z[h] = 0.0f;       // padding stays zero even for a non-finite factor
          }
          o[d] = pack_bf16x2(z[0], z[1]);
        }
        *reinterpret_cast<gptr<u32x4>>(Nb + (long long)kb * mt.Lq * 64) = u32x4{o[0], o[1], o[2], o[3]};
      }
    }
  }
}

// The same for ranks that are no multiple of four (rounds_n_and_r): Z = N - c k R formed again from the updated M and V and from R, both rounded
// to bf16 first.  By one wavefront, K blocks `first` and every step-th from there (see fixz_block).
__device__ __forceinline__ void fixz_block_rounded(const FiraMat& mt, const FiraHp& hp, float c, float bias, long long row0, int first, int step) {
  const int lane = threadIdx.x & 63, a8 = (lane & 3) * 8;
  const long long row = row0 + (lane >> 2);
  const int kblocks = (mt.r + 31) >> 5;
  if (row >= mt.L) return;
  gptr<char> Nb = reinterpret_cast<gptr<char>>(as_global(mt.Nb)) + row0 * 64 + lane * 16;
  gptr<const float> M = as_global<const float>(mt.M) + row * mt.r + a8, V = as_global<const float>(mt.V) + row * mt.r + a8;
  gptr<const float> R = as_global<const float>(mt.Rt) + row * mt.r + a8;
  const float f = c * as_global<const float>(mt.phi)[row];
  for (int kb = first; kb < kblocks; kb += step) {
    f32x4 mv[2], vv[2], rv[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int at = 32 * kb + 4 * q, mine = max(mt.r - a8 - at, 0);
      mv[q] = load_row4(M + at, mine);
      vv[q] = load_row4(V + at, mine);
      rv[q] = load_row4(R + at, mine);
    }
    u32x2 h[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      f32x4 n;
#pragma unroll
      for (int e = 0; e < 4; ++e) n[e] = adam_direction(mv[q][e], vv[q][e], bias, hp.epsf);
      h[q] = pack_bf16x4(bf16_rounded(n) - f * bf16_rounded(rv[q])) & row4_mask(mt.r - a8 - 32 * kb - 4 * q);
    }
    *reinterpret_cast<gptr<u32x4>>(Nb + (long long)kb * mt.Lq * 64) = u32x4{h[0].x, h[0].y, h[1].x, h[1].y};
  }
}

// fp32 rows that hold Z for c = 1: Z = N - c k R formed again from the updated M and V and from R.
__device__ __forceinline__ void fixz_row_split(const FiraMat& mt, const FiraHp& hp, float f, float bias, long long row) {
  const int lane = threadIdx.x & 63;
  gptr<bf16_raw> Nb = as_global(mt.Nb);
  gptr<const float> R = as_global<const float>(mt.Rt) + row * mt.r;
  gptr<const float> M = as_global<const float>(mt.M) + row * mt.r;
  gptr<const float> V = as_global<const float>(mt.V) + row * mt.r;
  for (int a = lane * 4; a < mt.r; a += 256) {
    const f32x4 rv = load_row4(R + a, mt.r - a), mv = load_row4(M + a, mt.r - a), vv = load_row4(V + a, mt.r - a);
    const u32x2 mask = row4_mask(mt.r - a);
    f32x4 z;
#pragma unroll
    for (int e = 0; e < 4; ++e) z[e] = adam_direction(mv[e], vv[e], bias, hp.epsf) - f * rv[e];
    u32x2 zp[3];
    bf16_planes<FIRA_KX_SPLIT>(z, 3, zp);
#pragma unroll
    for (int p = 0; p < 3; ++p) *reinterpret_cast<gptr<u32x2>>(Nb + kblk_index(mt.Lq, row, p * mt.rp + a)) = zp[p] & mask;
  }
}

static_assert(FIRA_ZREADY_MAX_R_F32 == 512, "fira_adam_kernel's forms end there");
#define FIRA_MAKEZ_PARTS 32   // workgroups per listed matrix
// A matrix's Z for a limiter factor of c, by one of FIRA_MAKEZ_PARTS workgroups, which takes every FIRA_MAKEZ_PARTS-th block of 16 rows.
// t: the step count with this step in it; c_prev: the factor of the step before; fused_here: the fused kernel served the matrix and left no copy of R.
__device__ __forceinline__ void make_z(const FiraMat& mt, const FiraHp& hp, int part, float c, float c_prev, int t, bool fused_here) {
  const bool ready = mt.zready && hp.scaling != 1 && !leaves_n_and_r(mt, c_prev);
  if (ready && c == 1.0f) return;              // the Adam kernel already wrote Z for c = 1
  const int wave = threadIdx.x >> 6;
  const int rowblocks = (mt.L + FIRA_ROWS_PER_WG - 1) / FIRA_ROWS_PER_WG;
  const float bias = ready && (fused_here || mt.kx != 1 || rounds_n_and_r(mt)) ? bias_correction(hp, t) : 0.0f;
  if (mt.kx == 1) {
    // where a row is one or two K blocks, each wavefront has sixteen rows of its own
    const bool own = mt.r <= FIRA_PS;
    const int first = own ? 0 : wave, step = own ? 1 : 4;
    for (int rb = own ? 4 * part + wave : part; rb < rowblocks; rb += (own ? 4 : 1) * FIRA_MAKEZ_PARTS) {
      const long long row0 = (long long)rb * FIRA_ROWS_PER_WG;
      if (!ready) makez_block(mt, c, row0, first, step);
      else if (fused_here) fixz_block_from_moments(mt, hp, c, bias, row0);
      else if (rounds_n_and_r(mt)) fixz_block_rounded(mt, hp, c, bias, row0, first, step);
      else fixz_block(mt, 1.0f - c, row0, first, step, two_planes(hp, mt));
    }
    return;
  }
  for (int rb = part; rb < rowblocks; rb += FIRA_MAKEZ_PARTS) {
    const long long row_base = (long long)rb * FIRA_ROWS_PER_WG + wave * 4;
    for (int i = 0; i < 4; ++i) {
      const long long row = row_base + i;
      if (row >= mt.L) break;
      const float k = as_global<const float>(mt.phi)[row];
      if (ready) fixz_row_split(mt, hp, c * k, bias, row);
      else makez_row_split(mt, c * k, row);
    }
  }
}
// One workgroup per (listed matrix, part): it reads the matrix's c once and, in the common case, exits.
__global__ __launch_bounds__(256) void fira_makez_kernel(const FiraMat* __restrict__ mats,
                                                         const FiraScal* __restrict__ scal,
                                                         const FiraEnt* __restrict__ ents, FiraHp hp) {
  const FiraEnt ent = ents[blockIdx.x / FIRA_MAKEZ_PARTS];
  const FiraMat mt = mats[ent.mat];
  make_z(mt, hp, blockIdx.x % FIRA_MAKEZ_PARTS, scal[ent.mat].c, scal[ent.mat].c_in, scal[ent.mat].t, scal[ent.mat].gram_now == 2);
}
// The limiter and Z in one launch, for factors per row or none: every workgroup works the factor out for itself, from the values that the kernel
// with Adam set aside (set_limiter_inputs), and the first one of a matrix advances its state.  Two launches in turn are two latencies, and
// the second nearly always only reads c = 1.  What the repeated sums cost depends on how many workgroups there are, FIRA_MAKEZ_PARTS a matrix:
// up to 64 matrices all of them run at once, eight a CU, and beyond that the sums cost more than the launch.  Two launches and one, by matrices (21,
// 63, 84 and 168), a step of 256 x 688 at r = 64 29.8 and 28.2, 39.3 and 38.9, 45.8 and 46.1, 64.8 and 69.0 us; of 512 x 1376 at r = 128 61.5 and
// 59.9, 92.2 and 92.2, 113.5 and 114.9, 213 and 218, residual 76.1 and 74.1, 130.9 and 130.2, 168.1 and 169.3, 333 and 337; of 1024 x 2736 at
// r = 256, 63 matrices and 112, 351.5 and 351.6, 593.7 and 598.0, limited 352.8 and 352.6, 602.7 and 606.3; of 256 x 688 in fp32 47.2 and 45.2 (21),
// 84.5 and 83.8 (63), 119.6 and 121.5 (112).
__global__ __launch_bounds__(FIRA_LIMITER_THREADS) void fira_limit_and_makez_kernel(const FiraMat* __restrict__ mats, FiraScal* __restrict__ scal,
                                                                                    const FiraEnt* __restrict__ ents, const float* __restrict__ partial,
                                                                                    FiraGate* __restrict__ gate, FiraHp hp) {
  __shared__ double red[4];
  const FiraEnt ent = ents[blockIdx.x / FIRA_MAKEZ_PARTS];
  const int part = blockIdx.x % FIRA_MAKEZ_PARTS;
  const FiraMat mt = mats[ent.mat];
  FiraScal in;
  in.s_prev = scal[ent.mat].s_prev_in;
  in.has_prev = scal[ent.mat].has_prev_in;
  in.t = scal[ent.mat].t_in;
  in.ortho_err = scal[ent.mat].ortho_err_in;
  in.gram_err = scal[ent.mat].gram_err_in;
  const bool gram = use_gram(hp, in);
  // On the residual route with the Gram data at hand (the first step after an install), also form the
  // Gram route's value and record how far it is from the exact one: the second gate of that route.
  const bool calibrate = part == 0 && !gram && calibrates_gram(hp, in);
  double acc, accg;
  limiter_sums(mt, ent, partial, gram, calibrate, red, acc, accg);
  const double sn = sqrt(acc), c = limiter_factor(hp, sn, in.has_prev, in.s_prev);
  if (part == 0 && threadIdx.x == 0) limiter_advance(scal[ent.mat], gate[ent.mat], hp, gram, calibrate, acc, accg, sn, c, in.t);
  make_z(mt, hp, part, (float)c, scal[ent.mat].c_in, in.t + 1, gram && hp.fused);
}

// ------------------------------------------------------------------------------------------------
// "Fira-only-scaling" update: W -= lr*alpha * c * k_i * G over the tiles of the back-projection list
// (256 columns x 128 rows per workgroup), a pure stream: 16 bytes per lane, 512 contiguous bytes per
// row piece, factors per column (m <= n) or per row (m > n).
// ------------------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void fira_scale_update_kernel(const FiraMat* __restrict__ mats,
                                                                const FiraScal* __restrict__ scal,
                                                                const FiraEnt* __restrict__ ents,
                                                                const FiraTile* __restrict__ tiles, int ntiles, FiraHp hp) {
  const int ti = xcd_chunked_index(blockIdx.x, ntiles);
  if (ti < 0) return;
  const FiraTile tile = tiles[ti];
  const FiraEnt ent = ents[tile.ent];
  const FiraMat mt = mats[ent.mat];
  const float f = *hp.lr_alpha * scal[ent.mat].c;
  gptr<const T> G = as_global(reinterpret_cast<const T*>(ent.G));
  gptr<T> W = as_global(reinterpret_cast<T*>(ent.W));
  gptr<const float> phi = as_global<const float>(mt.phi);
  const int t = threadIdx.x;
  const long long j = (long long)tile.ta * 256 + 8 * (t & 31);
  if (j >= mt.n) return;
  float kc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) kc[e] = (mt.left && j + e < mt.n) ? f * phi[j + e] : 0.0f;
  for (int p = 0; p < 16; ++p) {
    const long long i = (long long)tile.tb * 128 + (t >> 5) + 8 * p;
    if (i >= mt.m) break;
    if (!mt.left) {
      const float fr = f * phi[i];
#pragma unroll
      for (int e = 0; e < 8; ++e) kc[e] = fr;
    }
    if (sizeof(T) == 2) {
      gptr<const bf16_raw> gr = reinterpret_cast<gptr<const bf16_raw>>(G) + i * mt.ld + j;
      gptr<bf16_raw> wr = reinterpret_cast<gptr<bf16_raw>>(W) + i * mt.ld + j;
      if (j + 8 <= mt.n) {       // rows may start at any element: 2-byte alignment only
        const u32x4 gv = __builtin_nontemporal_load(reinterpret_cast<gptr<const u32x4_a2>>(gr));
        const u32x4 wv = __builtin_nontemporal_load(reinterpret_cast<gptr<const u32x4_a2>>(wr));
        const unsigned gw[4] = {gv.x, gv.y, gv.z, gv.w}, ww[4] = {wv.x, wv.y, wv.z, wv.w};
        unsigned o[4];
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          const float w0 = __uint_as_float(ww[d] << 16) - kc[2 * d] * __uint_as_float(gw[d] << 16);
          const float w1 = __uint_as_float(ww[d] & 0xffff0000u) - kc[2 * d + 1] * __uint_as_float(gw[d] & 0xffff0000u);
          o[d] = pack_bf16x2(w0, w1);
        }
        __builtin_nontemporal_store(u32x4{o[0], o[1], o[2], o[3]}, reinterpret_cast<gptr<u32x4_a2>>(wr));
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (j + e < mt.n) wr[e] = f32_to_bf16(bf16_to_f32(wr[e]) - kc[e] * bf16_to_f32(gr[e]));
      }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (j + e < mt.n) {
          gptr<float> wp = reinterpret_cast<gptr<float>>(W) + i * mt.ld + j + e;
          *wp = *wp - kc[e] * reinterpret_cast<gptr<const float>>(G)[i * mt.ld + j + e];
        }
    }
  }
}

// ------------------------------------------------------------------------------------------------
// Operand preparation (outside the per-step hot loop)
// ------------------------------------------------------------------------------------------------

// Projector P[S][r] (fp32 or bf16) -> Pn[S][kx*rp] and PT[r][kx*Sp], both K-blocked; split planes follow sequence B.
// A memory-bound transposition: tiles of 32 (s) x 64 (a) go through LDS, so that both operands leave in 16-byte
// pieces of 2 and 4 KB contiguous runs (the operands' padding inside the last tile is written with its zeros).  All
// 168 projectors of the 1B shapes at r = 512: 344 us; 1039 us with one element per thread and 2-byte stores.
// value(idx): element idx of the projector, row-major.  BOTH: Pn as well as PT (the rounds of a refresh contract PT only).
template <bool BOTH, typename F>
__device__ __forceinline__ void prep_projector_tiles(const FiraMat& mt, F value) {
  __shared__ float tile[32][65];
  const int atiles = (mt.r + 63) / 64, tiles = ((mt.S + 31) / 32) * atiles;
  const int t = threadIdx.x;
  gptr<bf16_raw> pn = as_global(mt.Pn);
  gptr<bf16_raw> pt = as_global(mt.PT);
  for (int ti = blockIdx.x; ti < tiles; ti += gridDim.x) {
    const int s0 = (ti / atiles) * 32, a0 = (ti % atiles) * 64;
#pragma unroll
    for (int p = 0; p < 8; ++p) {
      const int sl = (t >> 6) + 4 * p, al = t & 63;
      const bool in = s0 + sl < mt.S && a0 + al < mt.r;
      const long long idx = (long long)(s0 + sl) * mt.r + a0 + al;
      tile[sl][al] = in ? value(idx) : 0.0f;
    }
    __syncthreads();
    // Pn: row s, eight a;  PT: row a, eight s
    const int sl = (t >> 2) & 31, na = (t >> 7) * 32 + (t & 3) * 8;
    const int al = t >> 2, ns = (t & 3) * 8;
    f32x4 n0, n1, t0, t1;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      n0[e] = tile[sl][na + e]; n1[e] = tile[sl][na + 4 + e];
      t0[e] = tile[ns + e][al]; t1[e] = tile[ns + 4 + e][al];
    }
    const int planes = mt.kx == 1 ? 1 : 3;
    u32x2 h0[3], h1[3];
#pragma unroll
    for (int side = BOTH ? 0 : 1; side < 2; ++side) {
      bf16_planes<FIRA_KX_SPLIT>(side ? t0 : n0, planes, h0);
      bf16_planes<FIRA_KX_SPLIT>(side ? t1 : n1, planes, h1);
#pragma unroll
      for (int q = 0; q < 6; ++q) {
        constexpr int seq[6] = {0, 1, 0, 2, 0, 1};     // h m h l h m
        if (q >= mt.kx) break;
        const u32x4 v = u32x4{h0[seq[q]].x, h0[seq[q]].y, h1[seq[q]].x, h1[seq[q]].y};
        if (side) *reinterpret_cast<gptr<u32x4>>(pt + kblk_index(mt.rq, a0 + al, q * mt.Sp + s0 + ns)) = v;
        else *reinterpret_cast<gptr<u32x4>>(pn + kblk_index(mt.Sq, s0 + sl, q * mt.rp + a0 + na)) = v;
      }
    }
    __syncthreads();
  }
}
template <bool BOTH, typename TP>
__device__ __forceinline__ void prep_projector_body(const FiraMat& mt, const TP* __restrict__ P) {
  prep_projector_tiles<BOTH>(mt, [&](long long idx) {
    if (sizeof(TP) == 2) return bf16_to_f32(as_global(reinterpret_cast<const bf16_raw*>(P))[idx]);
    return as_global(reinterpret_cast<const float*>(P))[idx];
  });
}
template <typename TP>
__global__ __launch_bounds__(256) void fira_prep_projector_kernel(FiraMat mt, const TP* __restrict__ P) { prep_projector_body<true, TP>(mt, P); }

// One float in device memory (the step size lr * alpha), written in stream order.
__global__ void fira_store_float_kernel(float* __restrict__ dst, float value) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *as_global(dst) = value;
}

// fp32 gradient -> its bf16 rounding (nearest even), rows of ldb elements (the projector refresh's way back).
__global__ void fira_round_gradient_kernel(const float* __restrict__ G, bf16_raw* __restrict__ Gb, int m, int n,
                                           long long ld, long long ldb) {
  const long long total = (long long)m * n;
  gptr<bf16_raw> out = as_global(Gb);
  for (long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (long long)gridDim.x * blockDim.x) {
    const long long i = idx / n;
    const long long j = idx - i * n;
    out[i * ldb + j] = f32_to_bf16(G[i * ld + j]);
  }
}

// ------------------------------------------------------------------------------------------------
// Gate of the Gram route, evaluated when a projector is installed: a randomized estimate of
// ||P^T P - I|| from 4 sign vectors x (err = max_t ||P^T (P x_t) - x_t|| / ||x_t||), on the bf16
// operand copy of P that the contractions use.  Two small kernels: y_t = P x_t (one wavefront per
// row of P), then z_t = P^T y_t - x_t (one workgroup, threads along the rank axis).
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ float ortho_sign(int a, int trial) {
  const unsigned h = ((unsigned)a * 2654435761u) ^ ((unsigned)trial * 2246822519u + 374761393u);
  return ((h >> 15) & 1u) ? 1.0f : -1.0f;
}

__device__ __forceinline__ void ortho_y_body(const FiraMat& mt, float* __restrict__ y /* [S][4] */) {
  gptr<const bf16_raw> Pn = as_global<const bf16_raw>(mt.Pn);
  const int lane = threadIdx.x & 63;
  const int s = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (s >= mt.S) return;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  for (int a = lane; a < mt.r; a += 64) {
    const float p = bf16_to_f32(Pn[kblk_index(mt.Sq, s, a)]);
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] += p * ortho_sign(a, t);
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) acc[t] = wave_sum(acc[t]);
  if (lane == 0) {
#pragma unroll
    for (int t = 0; t < 4; ++t) as_global(y)[(long long)s * 4 + t] = acc[t];
  }
}

__global__ __launch_bounds__(256) void fira_ortho_y_kernel(FiraMat mt, float* __restrict__ y) { ortho_y_body(mt, y); }

// z-partials: workgroup b sums rows [b*chunk, (b+1)*chunk) of P^T y for all four trials.
__device__ __forceinline__ void ortho_z_body(const FiraMat& mt, const float* __restrict__ y,
                                             float* __restrict__ zpart /* [splits][r][4] */) {
  gptr<const bf16_raw> Pn = as_global<const bf16_raw>(mt.Pn);
  gptr<const float> yy = as_global(y);
  const int chunk = (mt.S + FIRA_ORTHO_SPLITS - 1) / FIRA_ORTHO_SPLITS;
  const int s0 = blockIdx.x * chunk, s1 = min(mt.S, s0 + chunk);
  for (int a = threadIdx.x; a < mt.r; a += 256) {
    float z[4] = {0.f, 0.f, 0.f, 0.f};
    for (int s = s0; s < s1; ++s) {
      const float p = bf16_to_f32(Pn[kblk_index(mt.Sq, s, a)]);
#pragma unroll
      for (int k = 0; k < 4; ++k) z[k] += p * yy[(long long)s * 4 + k];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) as_global(zpart)[((long long)blockIdx.x * mt.r + a) * 4 + k] = z[k];
  }
}

__global__ __launch_bounds__(256) void fira_ortho_z_kernel(FiraMat mt, const float* __restrict__ y, float* __restrict__ zpart) {
  ortho_z_body(mt, y, zpart);
}

__device__ __forceinline__ void ortho_final_body(const FiraMat& mt, const float* __restrict__ zpart,
                                                 FiraScal* __restrict__ scal, FiraGate* __restrict__ gate, int mat, float (&red)[4][4]) {
  gptr<const float> zp = as_global(zpart);
  const int t = threadIdx.x;
  float zz[4] = {0.f, 0.f, 0.f, 0.f};
  for (int a = t; a < mt.r; a += 256) {
    // all trials of a split in one load, sixteen splits in flight: one value after the other, the splits were a chain of 256 loads
    f32x4 z = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 16
    for (int b = 0; b < FIRA_ORTHO_SPLITS; ++b) z += *reinterpret_cast<gptr<const f32x4>>(zp + ((long long)b * mt.r + a) * 4);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float d = z[k] - ortho_sign(a, k);
      zz[k] += d * d;
    }
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) zz[k] = wave_sum(zz[k]);
  if ((t & 63) == 0) {
#pragma unroll
    for (int k = 0; k < 4; ++k) red[t >> 6][k] = zz[k];
  }
  __syncthreads();
  if (t == 0) {
    float worst = 0.0f;
    for (int k = 0; k < 4; ++k)
      worst = fmaxf(worst, sqrtf(((red[0][k] + red[1][k]) + (red[2][k] + red[3][k])) / (float)mt.r));
    as_global(scal)[mat].ortho_err = worst;
    as_global(scal)[mat].gram_err = INFINITY;   // to be measured on the next step
    as_global(gate)[mat].ortho_err = worst;
    as_global(gate)[mat].gram_err = INFINITY;
  }
}
__global__ __launch_bounds__(256) void fira_ortho_final_kernel(FiraMat mt, const float* __restrict__ zpart,
                                                               FiraScal* __restrict__ scal, FiraGate* __restrict__ gate, int mat) {
  __shared__ float red[4][4];
  ortho_final_body(mt, zpart, scal, gate, mat, red);
}
