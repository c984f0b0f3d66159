// Integer LayerNorm of the Conformer block (Eq. 1 - 4: every module normalizes its input
// first, and the block ends with one; the paper takes LayerNorm's integer form from
// I-BERT).
//
// For a row z of d int8 values:
//   mu    = floor((2 sum z + d) / (2 d))                 mean, ties up
//   sigma = max(1, floor(sqrt(sum (z - mu)^2)))          integer square root
//   F     = floor(2^31 / sigma)
//   u_k   = floor((z_k - mu) F / 2)
//   x_k   = clamp8(floor((u_k g_k + c_k + 2^(n-1)) / 2^n))
// g and c fold gamma, beta and the move to the block's input grid into one
// fixed-point step per channel (the rounding term comes pre-added to c).
//
// The work is a few bytes per element, so the kernel is bound by moving the rows (HBM or
// L2) once the rest is kept off their way.  LPR lanes share a row (16 pieces of 16 bytes for
// d <= 256, 32 for d <= 512, else 64), each lane holding its pieces of R rows in registers:
//  * the per-channel constants (12 bytes a channel, twelve times a row's own bytes) are
//    loaded once for the R rows of a lane, and requested together with them;
//  * both sums of a row come from one pass, sum z and sum z^2 by v_dot4 against ones and
//    against z itself, sum (z - mu)^2 = sum z^2 - 2 mu sum z + d mu^2 exactly in integers,
//    and the lanes' sums are added by DPP and lane swaps;
//  * the mean (a multiplication by the reciprocal of 2 d), floor(sqrt(v)) (bit by bit) and
//    floor(2^31 / sigma) (restoring division) are integer sequences of about 220 dependent
//    instructions: lane r mod R runs them for row r, so one sequence serves the R rows
//    (as a scalar sequence per row they took most of the kernel's time over many rows);
//  * an element costs one 24-bit multiply-add (sigma > 256: F below 2^23, as of any row with a
//    spread of a few units), one 32 x 32 + 64-bit multiply-add and, for shifts of 32 and
//    more, a 32-bit shift and clamp of the sum's high word.
// 23000 rows of 1024: 31 -> 14.6 us (3.2 TB/s; a large copy reaches 4.9 TB/s), 6000 rows 9.0 ->
// 6.8 us, 2500 rows 7.0 -> 4.9 us, 125 rows 4.4 -> 3.4 us against one row per wave with scalar
// sequences and the constants in channel order.  What is left over many rows is the
// quarter-rate 64-bit multiply-add of each element.
// No floating-point instruction runs.
#include "ipk_internal.h"

namespace ipk {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef long long v2l __attribute__((ext_vector_type(2)));

struct LnArgs {
  const int8_t* z;
  int8_t* x;
  const v4i* g;  // multipliers, [4][d / 16]: entry (w, p) holds channels 16 p + 4 w .. + 3
  const v2l* c;  // bias plus 2^(shift-1), [8][d / 16]: entry (j, p) holds channels 16 p + 2 j, + 1
  long rows;
  int d, shift;
  uint32_t mean_m;  // floor(v / (2 d)) = v mean_m >> mean_s for 0 <= v < 2^24
  int mean_s;
};

constexpr int LN_WAVES = 4;  // waves per workgroup

// Sum over the LPR consecutive lanes that share a row, in each of them: DPP adds within 16
// lanes (quad_perm [1,0,3,2], quad_perm [2,3,0,1], row_half_mirror, row_mirror), then swaps
// of the 16-lane rows and of the halves.  Integer adds, so the order does not matter.
template <int LPR>
__device__ __forceinline__ int row_sum(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x140, 0xF, 0xF, false);
  if (LPR >= 32) {
    const auto r = __builtin_amdgcn_permlane16_swap((uint32_t)v, (uint32_t)v, false, false);
    v = (int)(r[0] + r[1]);
  }
  if (LPR >= 64) {
    const auto r = __builtin_amdgcn_permlane32_swap((uint32_t)v, (uint32_t)v, false, false);
    v = (int)(r[0] + r[1]);
  }
  return v;
}

// floor(sqrt(v)) for 0 <= v < 2^32, bit by bit
__device__ __forceinline__ uint32_t isqrt_u32(uint32_t v) {
  uint32_t res = 0, one = 1u << 30;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const uint32_t t = res + one;
    const bool c = v >= t;
    v -= c ? t : 0u;
    res = (res >> 1) + (c ? one : 0u);
    one >>= 2;
  }
  return res;
}

// floor(2^31 / s) for 1 <= s < 2^16 by restoring division (the remainder stays below s)
__device__ __forceinline__ uint32_t div_2p31(uint32_t s) {
  uint32_t r = 1, q = 0;  // the dividend's only one bit, bit 31, enters first
#pragma unroll
  for (int i = 31; i >= 0; --i) {
    const bool c = r >= s;
    r = (r - (c ? s : 0u)) << 1;
    q = (q << 1) | (c ? 1u : 0u);
  }
  return q;
}

// v_mad_i32_i24: a, b in the signed 24-bit range, the sum modulo 2^32
__device__ __forceinline__ int mad24(int a, int b, int c) {
  int r;
  asm("v_mad_i32_i24 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// LPR lanes per row, NP 16-byte pieces per lane and row (NP > 1 only with LPR = 64), R
// rows per lane.  HI: shift >= 32.  With NP <= 2 the lane's constants are loaded up front
// (at most 104 registers); wider rows load them per piece.
template <int LPR, int NP, int R, bool HI>
__global__ __launch_bounds__(64 * LN_WAVES) void layernorm_i8(LnArgs a) {
  static_assert(R <= LPR && (NP == 1 || (LPR == 64 && R == 1)), "row layout");
  constexpr bool PRE = NP <= 2;
  constexpr int GR = 64 / LPR;  // rows side by side in a wave
  const int lane = threadIdx.x & 63;
  const int sub = lane & (LPR - 1);
  const long row0 = ((long)blockIdx.x * LN_WAVES + (threadIdx.x >> 6)) * (R * GR) + lane / LPR;  // rows row0 + GR r
  if (row0 - lane / LPR >= a.rows) return;
  const int d = a.d, npieces = d >> 4;
  v4i zv[R][NP];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      const int p = sub + LPR * k;
      zv[r][k] = p < npieces && row0 + GR * r < a.rows ? *(const v4i*)(a.z + (row0 + GR * r) * d + 16 * p)
                                                       : (v4i){0, 0, 0, 0};
    }
  // the constants of the lane's 16 channels per piece: multipliers (4 x 16 bytes) and
  // biases (8 x 16 bytes), stored so that the lanes of a load walk 16-byte entries in
  // address order (in channel order a load touched 32 or 64 cache lines)
  v4i gv[PRE ? NP : 1][4];
  v2l cv[PRE ? NP : 1][8];
  auto load_consts = [&](int p, v4i (&g)[4], v2l (&c)[8]) {
#pragma unroll
    for (int w = 0; w < 4; ++w) g[w] = a.g[w * npieces + p];
#pragma unroll
    for (int j = 0; j < 8; ++j) c[j] = a.c[j * npieces + p];
  };
  if constexpr (PRE) {
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      const int p = sub + LPR * k;
      if (p < npieces) load_consts(p, gv[k], cv[k]);
    }
  }
  // |sum z| <= 128 d <= 2^21 and sum z^2 <= 2^14 d <= 2^28 for d <= 16384; the lane keeps the
  // sums of row sub mod R
  int s = 0, q = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    int sr = 0, qr = 0;
#pragma unroll
    for (int k = 0; k < NP; ++k)
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        sr = __builtin_amdgcn_sdot4(zv[r][k][w], 0x01010101, sr, false);
        qr = __builtin_amdgcn_sdot4(zv[r][k][w], zv[r][k][w], qr, false);
      }
    sr = row_sum<LPR>(sr);
    qr = row_sum<LPR>(qr);
    if ((sub & (R - 1)) == r) {
      s = sr;
      q = qr;
    }
  }
  // mean, ties up: floor((2 sum z + d) / (2 d)), shifted by 256 to stay positive
  const uint32_t mv = (uint32_t)(2 * s + d + 512 * d);  // below 2^24
  const int mu = (int)(((uint64_t)mv * a.mean_m) >> a.mean_s) - 256;
  const long long var = (long long)q - 2ll * mu * s + (long long)d * mu * mu;  // sum (z - mu)^2 < 2^31
  uint32_t sg = isqrt_u32((uint32_t)var);
  if (sg < 1) sg = 1;
  const uint32_t F = div_2p31(sg);  // floor(2^31 / sigma), sigma < 2^16
  const bool small = __all(F < (1u << 23));  // of every row of the wave
  const int shift = a.shift;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    uint32_t Fr = F;
    int mr = mu;
    if (R > 1) {  // from the lane that computed row r
      if (LPR == 64) {
        Fr = (uint32_t)__builtin_amdgcn_readlane((int)F, r);
        mr = __builtin_amdgcn_readlane(mu, r);
      } else {
        Fr = (uint32_t)__shfl((int)F, (lane & ~(LPR - 1)) | r);
        mr = __shfl(mu, (lane & ~(LPR - 1)) | r);
      }
    }
    const long row = row0 + GR * r;
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      const int p = sub + LPR * k;
      if (p >= npieces || row >= a.rows) continue;
      const int c0 = 16 * p;
      v4i g[4];
      v2l c[8];
      if constexpr (PRE) {
#pragma unroll
        for (int w = 0; w < 4; ++w) g[w] = gv[k][w];
#pragma unroll
        for (int j = 0; j < 8; ++j) c[j] = cv[k][j];
      } else {
        load_consts(p, g, c);
      }
      // u = floor(y F / 2), y = z - mu
      auto finish = [&](auto u_of) {
        v4i out;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          int o[4];
#pragma unroll
          for (int b = 0; b < 4; ++b) {
            const int zb = (zv[r][k][w] << (24 - 8 * b)) >> 24;
            const int e = 4 * w + b;
            const long long t = (long long)u_of(zb) * g[w][b] + c[e >> 1][e & 1];
            if (HI) {
              o[b] = min(max((int)(t >> 32) >> (shift - 32), -127), 127);
            } else {
              o[b] = (int)min(max(t >> shift, -127ll), 127ll);
            }
          }
          out[w] = (int)(__builtin_amdgcn_perm((uint32_t)o[1], (uint32_t)o[0], 0x0c0c0400u) |
                         __builtin_amdgcn_perm((uint32_t)o[3], (uint32_t)o[2], 0x04000c0cu));
        }
        *(v4i*)(a.x + row * d + c0) = out;
      };
      if (small) {
        // F < 2^23 (sigma > 256): |y F| < 255 2^23 fits 32 bits
        const int Fi = (int)Fr, mF = -mr * Fi;
        finish([&](int zb) { return mad24(zb, Fi, mF) >> 1; });
      } else {
        // with F = 2 Fh + Fo, u = y Fh + Fo floor(y / 2), and |y Fh| <= |y| F / 2 <= 2^30
        // since |y| <= sigma
        const int Fh = (int)(Fr >> 1), Fo = (Fr & 1) ? -1 : 0;
        finish([&](int zb) {
          const int y = zb - mr;
          return y * Fh + ((y >> 1) & Fo);
        });
      }
    }
  }
}

template <int LPR, int NP, int R>
static hipError_t launch_ln_shape(const LnArgs& a, hipStream_t st, const LaunchEv& ev) {
  const long per = (long)LN_WAVES * R * (64 / LPR);  // rows per workgroup
  const dim3 grid((unsigned)((a.rows + per - 1) / per)), block(64 * LN_WAVES);
  return a.shift >= 32 ? launch_kernel(layernorm_i8<LPR, NP, R, true>, grid, block, 0, st, ev, a)
                       : launch_kernel(layernorm_i8<LPR, NP, R, false>, grid, block, 0, st, ev, a);
}

// Four rows per lane once the rows give every SIMD two waves without it, one below that:
// 1000 rows of 1024 3.6 us against 4.6 us, 2500 rows 4.9 us against 5.4 us, 23000 rows 14.6 us
// against 21.0 us (two rows lie between the two, eight gain nothing).
template <int LPR>
static hipError_t launch_ln_rows(const LnArgs& a, hipStream_t st, const LaunchEv& ev) {
  return a.rows * LPR / 64 >= 2048 ? launch_ln_shape<LPR, 1, 4>(a, st, ev) : launch_ln_shape<LPR, 1, 1>(a, st, ev);
}

static hipError_t launch_ln(long rows, int d, const Residual& r, const int8_t* z, int8_t* out, hipStream_t st,
                            const LaunchEv& ev) {
  LnArgs a{};
  a.z = z;
  a.x = out;
  a.g = (const v4i*)r.ln_mult;
  a.c = (const v2l*)r.ln_bias;
  a.rows = rows;
  a.d = d;
  a.shift = r.ln_shift;
  if (d % 16) return hipErrorInvalidValue;
  int l = 0;  // ceil(log2(2 d))
  while ((1 << l) < 2 * d) ++l;
  a.mean_s = 24 + l;
  a.mean_m = (uint32_t)(((uint64_t)1 << a.mean_s) / (2 * (uint64_t)d) + 1);
  if (d <= 256) return launch_ln_rows<16>(a, st, ev);
  if (d <= 512) return launch_ln_rows<32>(a, st, ev);
  if (d <= 1024) return launch_ln_rows<64>(a, st, ev);
  const int np = (d + 1023) / 1024;
  if (np <= 2) return launch_ln_shape<64, 2, 1>(a, st, ev);
  if (np <= 4) return launch_ln_shape<64, 4, 1>(a, st, ev);
  if (np <= 8) return launch_ln_shape<64, 8, 1>(a, st, ev);
  if (np <= 16) return launch_ln_shape<64, 16, 1>(a, st, ev);
  return hipErrorInvalidValue;
}

hipError_t launch_layernorm(const RunShape& rs, const Residual& r, const int8_t* z, int8_t* out, hipStream_t st,
                            const LaunchEv& ev) {
  return launch_ln((long)rs.B * rs.T, rs.d, r, z, out, st, ev);
}

hipError_t launch_layernorm_rows(long rows, int d, const Residual& r, const int8_t* z, int8_t* out, hipStream_t st) {
  return launch_ln(rows, d, r, z, out, st, LaunchEv{});
}

}  // namespace ipk
