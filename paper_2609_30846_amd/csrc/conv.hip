// The element-wise and depthwise middle of the convolution module (Eq. 5):
// GLU -> depthwise convolution over time (K = 9, BatchNorm folded) -> INT16
// BatchNorm output -> Swish -> int8 input of PW2, in one pass over PW1's output.
//
// For utterance b, channel c and frame t (L = L_b, zero outside [0, L)):
//   g[t]  = clamp8(RS(a[t] sigma(b[t]), m_glu, n_glu))      a, b: the two halves of PW1's output
//   sigma = -(q_1 + sgn(b) L(b)),  L(q) = (min(|q|, q_c) - q_c)^2 + q_1   (Eq. 12's polynomial at x/2)
//   v[t]  = clamp16(RS(bias + sum_k w[k] g[t + k - 4], m_dw, n_dw))       the INT16 BatchNorm output
//   o[t]  = clamp8(RS(swish(v[t]), m_sw, n_sw)) for t < L, else 0        Eq. 12's Swish on v's grid
// Every product fits 64 bits: the host proves |a sigma| m_glu and |swish(v)| m_sw below
// 2^62 for every int8 pair and every int16 v before it accepts the constants.
//
// The GLU of every int8 pair (a, b) and the Swish of every int16 value with its
// requantization sit in tables computed once per handle with the formulas above
// (`glu_table`, `swish16_table`, 64 KB each), so a GLU costs one byte lookup and an output
// its taps, one requantization and one byte lookup.  The lookups are what bounds the kernel: 64
// lanes gather from as many cache lines, so from memory each took about a line per cycle
// of the CU's load path (that version, one channel per thread, took 33 us for 16 x 375
// frames of 1024 channels).  Here a workgroup of 16 waves owns its CU, copies both tables
// into LDS once (128 KB of the 160 KB) and walks over tiles of 256 channels x F frames:
//  * GLU: a lane forms 4 channels x 4 frames of the tile's window (F + 8 frames, one frame
//    quad per wave) from dword loads of a and b, and stores each channel's four frames
//    as one dword of the LDS tile, time-major within a channel (rows of 17 dwords, so both
//    sides are free of bank conflicts).  The next tile's loads are in flight meanwhile.
//  * taps: a lane takes 4 channels x 4 output frames; 12 consecutive frames of a channel are
//    three dwords, and an output is three v_dot4 against the taps shifted by its frame's place
//    in the quad (9 taps in 12 bytes, built once per tile);
//  * requantization to the int16 grid: the accumulator is clamped to the channel's bound
//    (past it the result saturates either way), so the shifted 64-bit product fits 32 bits.
// Loads and stores of a frame are 256 consecutive channels of a wave.  F is picked per
// launch (4 .. 56) so that the tiles fill whole rounds over the CUs.  16 x 375 frames of 1024
// channels: 33 -> 10.7 us, 20 x 1000 111 -> 29 us, 2500 15.8 -> 7.0 us, 125 9.6 -> 4.9 us; copying
// the tables takes about 1 us of each, and the lookups' bank conflicts are what is left.
// Per frame and channel the kernel reads 2 bytes of PW1's output (the halo twice) and writes
// the int8 Swish output; the int16 BatchNorm output is written only when the launch asks
// for it (an inspection of the intermediate, which reruns the kernel on the kept PW1
// output), not on a module run.
#include "ipk_internal.h"

namespace ipk {

constexpr int CONV_HALF = 4;      // frames on either side of the nine taps
constexpr int CONV_WAVES = 16;    // one workgroup per CU: frame quads of the window side by side
constexpr int CONV_CH = 256;      // channels per tile (four per lane)
constexpr int CONV_MAXF = 4 * CONV_WAVES - 2 * CONV_HALF;  // output frames per tile at most
constexpr int CONV_ROW = CONV_WAVES + 1;                   // dwords per channel row of the LDS tile
constexpr int CONV_TAB = 65536;                            // bytes of each table
constexpr int CONV_LDS = 2 * CONV_TAB + CONV_CH * CONV_ROW * 4;

struct ConvArgs {
  const int8_t* u;  // [B][T][2 d] PW1 output: a = channels [0, d), b = [d, 2 d)
  int8_t* o;        // [B][T][d]
  int16_t* v;       // [B][T][d] (only stored by the variant for inspection)
  const int32_t* w;    // [d][3]: the nine taps of a channel in 12 bytes
  const int32_t* bias;
  const int32_t* mult;
  const int32_t* lim;     // accumulator bound of each channel
  const uint8_t* swtab16;  // [65536]: Swish output of each int16 v, at (uint16) v
  const uint8_t* glutab;   // [256][256]: GLU output of (a, b), at (uint8) a 256 + (uint8) b
  Lengths lens;            // valid frames per utterance
  int T, d, shift_dw;
  int F, tiles;          // output frames per tile (a multiple of 4), tiles of the launch
  DivU dv_cg, dv_chunk;  // channel groups, frame chunks per utterance
};

__device__ __forceinline__ long long rs64(long long a, long long m, int n) {
  return (a * m + (1ll << (n - 1))) >> n;
}

__device__ __forceinline__ long long poly_l(long long aq, long long q_c, long long q_1) {
  const long long t = (aq < q_c ? aq : q_c) - q_c;
  return t * t + q_1;
}

// The Swish of Eq. 12 on every int16 input and its requantization to PW2's int8 grid,
// one thread per value (computed once per handle; the middle kernel looks it up).
__global__ __launch_bounds__(256) void swish16_table(uint8_t* tab, long long q_c, long long q_1, long long m,
                                                     int shift) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  const long long v = (int16_t)i;  // -32768 is never looked up
  const long long av = v < 0 ? -v : v;
  const long long q = -(av * poly_l(av, q_c, q_1) + v * q_1);
  const long long o = rs64(q, m, shift);
  tab[i] = (uint8_t)(int)(o < -127 ? -127 : (o > 127 ? 127 : o));
}

// The GLU of every int8 pair: g = clamp8(RS(a sigma(b), m_glu, n_glu)), one thread per
// (a, b), at (uint8) a 256 + (uint8) b (computed once per handle; the middle kernel looks
// it up).
__global__ __launch_bounds__(256) void glu_table(uint8_t* tab, long long q_c, long long q_1, long long m, int shift) {
  const long long av = (int8_t)blockIdx.x, bv = (int8_t)threadIdx.x;
  const long long ab = bv < 0 ? -bv : bv;
  const long long sg = bv > 0 ? 1 : (bv < 0 ? -1 : 0);
  const long long sig = -(q_1 + sg * poly_l(ab, q_c, q_1));
  const long long r = rs64(av * sig, m, shift);
  tab[blockIdx.x * 256 + threadIdx.x] = (uint8_t)(int)(r < -127 ? -127 : (r > 127 ? 127 : r));
}

typedef int v4i __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) uint8_t lds8;
typedef __attribute__((address_space(3))) uint32_t lds32;
typedef __attribute__((address_space(3))) v4i ldsv4;

// four bytes (in the low byte of each word) -> one dword
__device__ __forceinline__ uint32_t pack_b0(uint32_t b0, uint32_t b1, uint32_t b2, uint32_t b3) {
  return __builtin_amdgcn_perm(b3 << 8 | b2, b1 << 8 | b0, 0x05040100u);
}

template <bool STORE_V>
__global__ __launch_bounds__(64 * CONV_WAVES) void conv_glu_dw_swish(ConvArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  const uint32_t base = (uint32_t)(uintptr_t)(lds8*)smem;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int T = a.T, d = a.d, F = a.F;
  const uint32_t tile0 = base + 2 * CONV_TAB + (uint32_t)(lane * CONV_ROW) * 4;  // channel 4 lane's row
  constexpr uint32_t PLANE = 64 * CONV_ROW * 4;  // rows of channel 4 lane + j, j = 0 .. 3

  int c, b, t0, L;
  auto locate = [&](int tile) {
    const int k = (int)div_u((uint32_t)tile, a.dv_cg), cg = tile - k * (int)a.dv_cg.d;
    b = (int)div_u((uint32_t)k, a.dv_chunk);
    t0 = (k - b * (int)a.dv_chunk.d) * F;
    c = cg * CONV_CH + lane * 4;
    L = a.lens.len[b];
  };
  // a and b of this wave's frame quad of the window, frames t0 - 4 + 4 wave ..
  uint32_t ua[4], ub[4];
  auto fetch = [&]() {
    const int8_t* src = a.u + (size_t)b * T * 2 * d + c;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int t = t0 - CONV_HALF + 4 * wave + i;
      ua[i] = ub[i] = 0;
      if (4 * wave < F + 2 * CONV_HALF && t >= 0 && t < L && c < d) {
        ua[i] = *(const uint32_t*)(src + (size_t)t * 2 * d);
        ub[i] = *(const uint32_t*)(src + (size_t)t * 2 * d + d);
      }
    }
  };
  int tile = blockIdx.x;  // below the tile count: the grid is no larger
  locate(tile);
  fetch();
  {
    v4i tab[2 * CONV_TAB / (64 * CONV_WAVES * 16)];
    constexpr int N = 2 * CONV_TAB / (64 * CONV_WAVES * 16);
#pragma unroll
    for (int i = 0; i < N; ++i)
      tab[i] = ((const v4i*)(i < N / 2 ? a.glutab : a.swtab16))[(i % (N / 2)) * (64 * CONV_WAVES) + tid];
#pragma unroll
    for (int i = 0; i < N; ++i)
      *(ldsv4*)(uintptr_t)(base + (uint32_t)(i * 64 * CONV_WAVES + tid) * 16) = tab[i];
  }
  __syncthreads();
  for (;;) {
    const int cc = c, bb = b, tt0 = t0, LL = L;
    // GLU of the wave's frame quad
    if (4 * wave < F + 2 * CONV_HALF) {
      uint32_t g[4][4];  // [frame][channel]
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int t = tt0 - CONV_HALF + 4 * wave + i;
        // (b, a) byte pairs of channels 0, 1 and 2, 3: the table's 16-bit indexes
        const uint32_t p01 = __builtin_amdgcn_perm(ua[i], ub[i], 0x05010400u);
        const uint32_t p23 = __builtin_amdgcn_perm(ua[i], ub[i], 0x07030602u);
        if (t >= 0 && t < LL) {
          g[i][0] = *(const lds8*)(uintptr_t)(base + (p01 & 0xffffu));
          g[i][1] = *(const lds8*)(uintptr_t)(base + (p01 >> 16));
          g[i][2] = *(const lds8*)(uintptr_t)(base + (p23 & 0xffffu));
          g[i][3] = *(const lds8*)(uintptr_t)(base + (p23 >> 16));
        } else {
          g[i][0] = g[i][1] = g[i][2] = g[i][3] = 0;
        }
      }
#pragma unroll
      for (int j = 0; j < 4; ++j)
        *(lds32*)(uintptr_t)(tile0 + j * PLANE + wave * 4) = pack_b0(g[0][j], g[1][j], g[2][j], g[3][j]);
    }
    // the next tile's PW1 outputs arrive during the taps
    tile += gridDim.x;
    const bool more = tile < a.tiles;
    if (more) {
      locate(tile);
      fetch();
    }
    __syncthreads();
    if (4 * wave < F && cc < d) {
      const v4i bias = *(const v4i*)(a.bias + cc), mult = *(const v4i*)(a.mult + cc), lim = *(const v4i*)(a.lim + cc);
      v4i wt[3];  // 12 tap bytes of each of the four channels
#pragma unroll
      for (int i = 0; i < 3; ++i) wt[i] = *(const v4i*)(a.w + (size_t)cc * 3 + i * 4);
      const long long half = 1ll << (a.shift_dw - 1);
      uint32_t o[4][4];  // [frame][channel]
      int vv[4][4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        uint32_t gw[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) gw[i] = *(const lds32*)(uintptr_t)(tile0 + j * PLANE + (wave + i) * 4);
        const uint32_t w0 = (uint32_t)wt[(3 * j) / 4][(3 * j) % 4], w1 = (uint32_t)wt[(3 * j + 1) / 4][(3 * j + 1) % 4],
                       w2 = (uint32_t)wt[(3 * j + 2) / 4][(3 * j + 2) % 4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          // the taps moved k bytes up the 12-byte window
          const uint32_t s0 = w0 << (8 * k);
          const uint32_t s1 = k ? __builtin_amdgcn_alignbyte(w1, w0, 4 - k) : w1;
          const uint32_t s2 = k ? __builtin_amdgcn_alignbyte(w2, w1, 4 - k) : w2;
          int acc = __builtin_amdgcn_sdot4((int)gw[0], (int)s0, bias[j], false);
          acc = __builtin_amdgcn_sdot4((int)gw[1], (int)s1, acc, false);
          acc = __builtin_amdgcn_sdot4((int)gw[2], (int)s2, acc, false);
          acc = min(max(acc, -lim[j]), lim[j]);
          const int r = (int)(((long long)acc * mult[j] + half) >> a.shift_dw);
          vv[k][j] = min(max(r, -32767), 32767);
          o[k][j] = *(const lds8*)(uintptr_t)(base + CONV_TAB + ((uint32_t)vv[k][j] & 0xffffu));
        }
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int t = tt0 + 4 * wave + k;
        if (t >= T || 4 * wave + k >= F) continue;
        const size_t idx = ((size_t)bb * T + t) * d + cc;
        *(uint32_t*)(a.o + idx) = t < LL ? pack_b0(o[k][0], o[k][1], o[k][2], o[k][3]) : 0u;
        if (STORE_V) {
          *(uint32_t*)(a.v + idx) = ((uint32_t)vv[k][0] & 0xffffu) | ((uint32_t)vv[k][1] << 16);
          *(uint32_t*)(a.v + idx + 2) = ((uint32_t)vv[k][2] & 0xffffu) | ((uint32_t)vv[k][3] << 16);
        }
      }
    }
    if (!more) break;
    __syncthreads();
  }
}

hipError_t launch_swish16_table(uint8_t* tab, long long q_c, long long q_1, long long m, int shift, hipStream_t st) {
  hipLaunchKernelGGL(swish16_table, dim3(256), dim3(256), 0, st, tab, q_c, q_1, m, shift);
  return hipGetLastError();
}

hipError_t launch_glu_table(uint8_t* tab, long long q_c, long long q_1, long long m, int shift, hipStream_t st) {
  hipLaunchKernelGGL(glu_table, dim3(256), dim3(256), 0, st, tab, q_c, q_1, m, shift);
  return hipGetLastError();
}

// Output frames per tile: the tiles of a launch pass through the CUs in rounds, each taking
// about its frames plus 32 frames' worth of the halo, the loads' latency and the barriers.
static int pick_frames(long B, int T, int d) {
  constexpr long kCUs = 256;
  const long cgs = (d + CONV_CH - 1) / CONV_CH;
  int best = 4;
  long best_t = 0;
  for (int F = 4; F <= CONV_MAXF; F += 4) {
    const long tiles = B * ((T + F - 1) / F) * cgs;
    const long t = (tiles + kCUs - 1) / kCUs * (32 + F);
    if (best_t == 0 || t < best_t) {
      best = F;
      best_t = t;
    }
  }
  return best;
}

hipError_t launch_conv_middle(const ConvMiddle& m, const int8_t* u, const Lengths& lens, int B, int T, int d,
                              int8_t* o, int16_t* v, hipStream_t st) {
  ConvArgs a{};
  a.u = u;
  a.o = o;
  a.v = v;
  a.w = m.w_dw;
  a.bias = m.bias_dw;
  a.mult = m.mult_dw;
  a.lim = m.lim_dw;
  a.lens = lens;
  a.T = T;
  a.d = d;
  a.shift_dw = m.shift_dw;
  a.swtab16 = m.swtab16;
  a.glutab = m.glutab;
  a.F = pick_frames(B, T, d);
  const int cgs = (d + CONV_CH - 1) / CONV_CH, chunks = (T + a.F - 1) / a.F;
  a.tiles = B * chunks * cgs;
  a.dv_cg = make_div((uint32_t)cgs);
  a.dv_chunk = make_div((uint32_t)chunks);
  const auto kernel = v ? conv_glu_dw_swish<true> : conv_glu_dw_swish<false>;
  const hipError_t e = allow_lds((const void*)kernel, CONV_LDS);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kernel, dim3(a.tiles < 256 ? a.tiles : 256), dim3(64 * CONV_WAVES), CONV_LDS, st, a);
  return hipGetLastError();
}

}  // namespace ipk
