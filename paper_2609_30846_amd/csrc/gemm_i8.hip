// INT8 projection GEMMs with a fused fixed-point requantization epilogue.
//
// Every linear layer of the block (Q, K, V, the relative-position projection and
// the output projection) is Eq. 7: an int8 x int8 product accumulated in int32,
// rescaled by a per-output-channel multiplier m and a right shift n with round to
// nearest (ties up), and clamped to the symmetric int8 grid.
//
// Kernel shape: one workgroup of four (or eight) waves computes a TN (channels) x TM (tokens) tile with
// v_mfma_i32_32x32x32_i8; the waves form a WN x WM grid of (TN/WN) x (TM/WM) sub-tiles.  K
// advances in 128-byte steps, so every global row segment is a whole cache line.  The
// weights are stored in MFMA operand-fragment order (each 32-channel x 32-byte fragment a
// contiguous 1 KB block in lane order), so every wave loads its own weight fragments
// straight into registers with fully coalesced 16-byte loads, each slice's registers
// refilled for the next step as soon as its MFMAs have read them.  The token tile is
// fetched into registers one step ahead and staged in one of two LDS buffers, whose rows are
// 128 bytes with the eight 16-byte chunks XOR-swizzled by the row index, which keeps both
// the 16-byte stores of the fetch and the 16-byte MFMA operand reads free of bank
// conflicts.
//
// The step is one stream without branches: token fragments are read one 32-byte slice
// ahead of the MFMAs that use them, the next token tile is stored to LDS behind the first
// slice, and the step's only barrier sits ahead of the last slice, so that the first
// fragments of the next step are read under that slice's MFMAs.  Loads past the last step
// are sent out of their buffer's range (zeros, no traffic) instead of being branched
// around: with branches the compiler merged the wait counts of their paths and every
// other step waited for the loads issued just before it.
//
// A wave owns at most 64 x 128 outputs (accumulators in VGPRs, two waves per SIMD).  As
// 256 x 128 tiles of four waves two workgroups share a CU, and one's first fetch, epilogue
// and barriers run under the other's MFMAs: 23000 tokens x 1024 -> 4096 (with the Swish)
// take 103 us and 23000 x 4096 -> 1024 88 - 92 us, 1.9 - 2.1 POP/s (a library product of 8192^3
// random int8 reaches 2.3 POP/s on this card), where eight-wave 256 x 256 and 128 x 128 tiles
// under the branching loop took 127 and 122 us.  The 256 x 256 tile of eight waves moves a
// third less from L2 per product (two of its waves share each weight block): it is
// the faster one where one such tile per CU does the whole launch, and leaves the chip a
// higher clock for the kernel after it (2500 tokens, Q|K|V and position table: 15.1 us against
// 16.9 us from first to last workgroup, and the attention core after it at 2.20 GHz instead
// of 2.08 GHz on a card that runs into its power limit).
//
// Token tiles of Q|K|V never straddle two utterances (each is tiled on its own, and V^T is
// written in whole 64-key blocks); row-major products, the output projection among them, take
// all their rows as one sequence.  Every destination receives whole aligned 16-byte pieces.
// Tiles are dealt to the eight XCDs in contiguous, roughly square groups of the tile grid, so the
// operand rows one XCD touches fit its L2.
//
// Epilogue: the requantization y = clamp8(floor((acc m + 2^(n-1)) / 2^n)) in integers.
// When every channel of the matrix allows it (n <= 16, m' = m 2^(16-n) < 2^23 and
// one clamp bound A for all channels, at least ceil(2^23 / m') + 1 for each, with
// A m' + 2^15 < 2^31), the accumulator is first clamped to [-A, A] (beyond a channel's
// own bound the result saturates anyway), then one 24-bit multiply-add gives
// t = a m' + 2^15, whose clamp to [-127 2^16, 127 2^16 + 2^16 - 1] holds the int8
// result in byte 2: three full-rate instructions per value, one multiplier register per
// value, and a byte permute gathers four results into a dword.  Otherwise the value
// is evaluated in 64-bit integers, its constants read from LDS per value.  Each lane owns 4
// consecutive outputs per accumulator group; one exchange with the lane 32 away gives it 16
// consecutive bytes, stored with one 16-byte write.  Channel-major V^T is produced by swapping
// the MFMA operands in the waves whose channels are V, so that its 16-byte pieces run along
// tokens.
#include <type_traits>
#include <utility>

#include "gemm_tiles.h"
#include "ipk_internal.h"

namespace ipk {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

enum OutMode { OUT_QKV = 0, OUT_POS = 1, OUT_ROWMAJOR = 2 };

struct GemmProblem {
  const int8_t* x;      // [nb][rows][K] activations
  const int8_t* w;      // [N][K] weights
  const int32_t* req;   // [2][N] per output channel: multiplier, and shift in the wide form (Requant)
  int wide;             // 64-bit evaluation
  int clamp;            // the fast form's clamp bound
  int rows, N, K;
  int mode;
  int tile_begin;  // first logical tile of this problem
  TileGrid grid;
};

struct GemmArgs {
  GemmProblem prob[2];
  int nprob;
  int tiles_total;
  int per_xcd;  // logical tiles dealt to each XCD
  int8_t *q, *k, *vt, *p, *y;
  int T_al, H, dk_shift, d, p_rows, p_base;  // d_k = 2^dk_shift
  // residual add of the MHSA module (row-major outputs only): y := clamp8(RS(m_z z1 +
  // m_y y, 1, shift_r)) with z1 laid out as y
  const int8_t* z1;
  int m_z, m_y, shift_r;
  int res_wide;  // the residual add takes its 64-bit form
  const uint8_t* swtab;  // EPI_SWISH: output byte of each biased code h + 128
};

constexpr int BK = 128;  // bytes of K per step

// Byte offset of 16-byte chunk c of LDS row r.  Rows are 128 bytes; the chunk index
// is XORed with (r ^ r/8) mod 8, so any 16 consecutive rows (16-row aligned) that
// read one logical chunk touch 16 distinct (row parity, chunk) bank groups.
__device__ __forceinline__ int lds_off(int r, int c) { return r * BK + ((c ^ (r & 7) ^ ((r >> 3) & 3)) << 4); }

// f(integral_constant<int, 0>), ..., f(integral_constant<int, N - 1>), in order
template <typename F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// byte 2 of four words -> one dword (v_perm_b32 selector bytes: 0-3 pick the second
// operand's bytes, 4-7 the first's, 0x0c a zero byte)
__device__ __forceinline__ uint32_t pack_b2(uint32_t v0, uint32_t v1, uint32_t v2, uint32_t v3) {
  return __builtin_amdgcn_perm(v1, v0, 0x0c0c0602u) | __builtin_amdgcn_perm(v3, v2, 0x06020c0cu);
}

// v_med3_i32 with the low bound in a scalar register and the high one in a vector
// register (the compiler forms med3 from min/max only with constant bounds)
__device__ __forceinline__ int med3_sv(int x, int lo, int hi) {
  int r;
  asm("v_med3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(x), "s"(lo), "v"(hi));
  return r;
}

// a b + c for a, b in the signed 24-bit range (v_mad_i32_i24; the compiler cannot
// see the range of a clamp to runtime bounds and would sign-extend both first)
__device__ __forceinline__ int mad24_s(int a, int b, int c) {
  int r;
  asm("v_mad_i32_i24 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "s"(c));
  return r;
}

// Eq. 7 on the 16 accumulators of one MFMA output block, fast form: m[e] is element
// e's multiplier m', -A and A (negA, Av) the matrix's clamp bounds; v[e] receives the
// int8 result in byte 2.
__device__ __forceinline__ void requant16_fast(const v16i& a, const int (&m)[16], int negA, int Av, int (&v)[16]) {
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int c = med3_sv(a[e], negA, Av);
    v[e] = min(max(mad24_s(c, m[e], 1 << 15), -127 * 65536), 127 * 65536 + 65535);
  }
}

// The wide form: element e's multiplier and shift are sm[ch(e)], sn[ch(e)] (LDS).
template <typename CH>
__device__ __forceinline__ void requant16_wide(const v16i& a, const int* sm, const int* sn, CH ch, int (&v)[16]) {
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int m = sm[ch(e)], n = sn[ch(e)];
    const long long q = ((long long)a[e] * m + (1ll << (n - 1))) >> n;
    v[e] = (int)(q < -127 ? -127 : (q > 127 ? 127 : q)) << 16;
  }
}

// The 16 results (byte 2 of v[e]) packed four per dword: D[g] holds elements 4g .. 4g + 3.
// With SW, each int8 result h goes through the Swish table `stab` (LDS, indexed by h + 128).
template <bool SW = false>
__device__ __forceinline__ void pack16(const int (&v)[16], uint32_t (&D)[4], const uint8_t* stab = nullptr) {
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    if constexpr (SW) {
      uint32_t o[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = stab[(((uint32_t)v[4 * g + e] >> 16) & 0xffu) ^ 0x80u];
      D[g] = o[0] | (o[1] << 8) | (o[2] << 16) | (o[3] << 24);
    } else {
      D[g] = pack_b2((uint32_t)v[4 * g], (uint32_t)v[4 * g + 1], (uint32_t)v[4 * g + 2], (uint32_t)v[4 * g + 3]);
    }
  }
}

// The residual add of Eq. 2 on 16 int8 pairs: clamp8(floor((m_z z + m_y y + 2^(n-1)) / 2^n)).
// Narrow form (the host proves (m_z + m_y) 128 + 2^(n-1) < 2^31, n <= 31): two 24-bit
// multiply-adds, a shift and a clamp per value.
__device__ __forceinline__ v4i residual16(const v4i& y, const v4i& z, int m_z, int m_y, int shift) {
  const int half = (int)(1u << (shift - 1));
  v4i r;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    int q[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int yb = (y[w] << (24 - 8 * b)) >> 24, zb = (z[w] << (24 - 8 * b)) >> 24;
      const int t = mad24_s(zb, m_z, half);
      int u;
      asm("v_mad_i32_i24 %0, %1, %2, %3" : "=v"(u) : "v"(yb), "s"(m_y), "v"(t));
      q[b] = min(max(u >> shift, -127), 127);
    }
    r[w] = (int)(__builtin_amdgcn_perm((uint32_t)q[1], (uint32_t)q[0], 0x0c0c0400u) |
                 __builtin_amdgcn_perm((uint32_t)q[3], (uint32_t)q[2], 0x04000c0cu));
  }
  return r;
}

// The general form: m_z z + m_y y is exact in int32 (multipliers below 2^23, |z|, |y| <=
// 128); the rounding term and the shift (n <= 40) take 64 bits.
__device__ __forceinline__ v4i residual16_wide(const v4i& y, const v4i& z, int m_z, int m_y, int shift) {
  const long long half = 1ll << (shift - 1);
  v4i r;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    uint32_t o = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int yb = (y[w] << (24 - 8 * b)) >> 24, zb = (z[w] << (24 - 8 * b)) >> 24;
      const long long q = ((long long)(m_z * zb + m_y * yb) + half) >> shift;
      o |= ((uint32_t)(int)min(max(q, -127ll), 127ll) & 0xFFu) << (8 * b);
    }
    r[w] = (int)o;
  }
  return r;
}

// WN x WM waves (NWAVE = WN WM) each own a (TN/WN) x (TM/WM) sub-tile.  The weights
// come pre-packed in MFMA fragment order (wfrag_index): each wave streams its own
// fragments from memory straight into registers, one K step ahead, and only the token
// tile goes through LDS.  EPI: the epilogue of row-major outputs.  WIDE: some problem of
// the launch takes the wide form of Eq. 7 or of the residual add (its code costs registers
// even where unused, so launches in the fast forms alone leave it out).
template <int TN, int TM, int NWAVE, int WN, int EPI, bool WIDE>
__global__ __launch_bounds__(64 * NWAVE, NWAVE == 8 ? 1 : 2) void gemm_i8_requant(GemmArgs args) {
  constexpr int NTH = 64 * NWAVE;
  constexpr int WM = NWAVE / WN;            // waves along M
  constexpr int WTN = TN / WN;              // channels per wave
  constexpr int WTM = TM / WM;              // tokens per wave
  constexpr int FN = WTN / 32;              // 32-row MFMA tiles per wave along N
  constexpr int FM = WTM / 32;              // 32-col MFMA tiles per wave along M
  constexpr int LX = TM * (BK / 16) / NTH;  // 16-byte global loads per thread of the token tile
  constexpr int FROWS = NTH / 8;            // rows one pass of the fetch covers
  constexpr int KSL = BK / 32;              // 32-byte K slices per step
  static_assert(FN >= 1 && FM >= 1 && LX >= 1 && WTM % 32 == 0 && NTH >= TN && NWAVE % WN == 0, "tile shape");
  // two LDS buffers: the next K step is stored while the current one is multiplied
  __shared__ __align__(16) int8_t sx[2][TM * BK];
  __shared__ __align__(16) int sreq[2][TN];  // Eq. 7 constants of the tile's channels
  __shared__ uint32_t stab32[EPI == EPI_SWISH ? 64 : 1];  // the Swish table (read after the K loop)

  // XCD-aware deal: workgroup i runs on XCD i % 8; XCD x owns logical tiles
  // [x * per_xcd, (x + 1) * per_xcd)
  const int lin = blockIdx.x;
  const int tile = (lin & 7) * args.per_xcd + (lin >> 3);
  if (tile >= args.tiles_total) return;
  const int pi = (args.nprob > 1 && tile >= args.prob[1].tile_begin) ? 1 : 0;
  const GemmProblem& P = args.prob[pi];
  // the problem's scalars, all loaded at once: left alone the compiler loads each one
  // where it is first used, and every division below would wait for its own load
  TileGrid grid = P.grid;
  int tile_begin = P.tile_begin, K = P.K, rows = P.rows, N = P.N, mode = P.mode;
  asm volatile(""
               : "+s"(tile_begin), "+s"(grid.tiles_n), "+s"(grid.tiles_m), "+s"(grid.tiles_m_per), "+s"(grid.band),
                 "+s"(grid.span.m), "+s"(grid.span.s), "+s"(grid.full.m), "+s"(grid.full.s), "+s"(grid.last.m),
                 "+s"(grid.last.s), "+s"(grid.per.m), "+s"(grid.per.s), "+s"(K), "+s"(rows), "+s"(N), "+s"(mode));
  const TilePos pos = tile_at(grid, tile - tile_begin);
  const int n0 = pos.nt * TN;
  const int ub = pos.ub;       // utterance
  const int t0 = pos.mt * TM;  // first token

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wn = wave % WN, wm = wave / WN;

  // the tile's Eq. 7 constants and the Swish table: requested ahead of the first operands,
  // stored to LDS behind them (read after the K loop)
  int rq0, rq1 = 0;
  uint32_t swt = 0;
  {
    const int c = min(n0 + min(tid, TN - 1), N - 1);
    rq0 = P.req[c];
    if (WIDE) rq1 = P.req[N + c];
    if (EPI == EPI_SWISH) swt = ((const uint32_t*)args.swtab)[tid & 63];
  }
  const int rq_wide = WIDE ? __builtin_amdgcn_readfirstlane(P.wide) : 0, rq_clamp = __builtin_amdgcn_readfirstlane(P.clamp);

  // thread -> (row, chunk) of the fetch: 8 threads cover one 128-byte row segment.
  // Raw buffer loads: rows past the end of the operand (their whole offset is in the
  // per-lane operand, which the bounds check covers) read as zeros.
  const int fchunk = tid & 7, frow = tid >> 3;  // rows frow + FROWS r
  const __amdgpu_buffer_rsrc_t wres = __builtin_amdgcn_make_buffer_rsrc((void*)P.w, (short)0, N * K, BUF_WORD3);
  const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(P.x + ((size_t)ub * rows + t0) * K), (short)0, min(rows - t0, TM) * K, BUF_WORD3);
  const int foff = frow * K + fchunk * 16;

  // the next step's token tile in registers
  v4i rx[LX];
  // this wave's weight fragments of one K step (FN channel blocks x KSL slices, 1 KB
  // each, the slices of a block contiguous).  A slice past K (odd multiples of 64) meets
  // zero tokens, so its contents do not matter: block and slice are held inside the matrix,
  // and steps past the last are sent out of range by the per-lane offset.
  v4i wf[FN][KSL];
  const int nk = (K + BK - 1) / BK;
  const int cb0 = (n0 + wn * WTN) >> 5;  // first 32-channel block of this wave
  auto wfetch = [&](int kt, auto ks_tag) {
    constexpr int ks = decltype(ks_tag)::value;
    const int voff = lane * 16 + (kt < nk ? 0 : 0x7f000000);
    const int kc = min(kt * KSL + ks, (K >> 5) - 1);
#pragma unroll
    for (int i = 0; i < FN; ++i) {
      const int base = __builtin_amdgcn_readfirstlane((min(cb0 + i, (N >> 5) - 1) * (K >> 5) + kc) * 1024);
      wf[i][ks] = (v4i)__builtin_amdgcn_raw_buffer_load_b128(wres, voff, base, 0);
    }
  };
  // K is a multiple of 64: the last step of an odd multiple fills its upper half with zeros
  auto fetch = [&](int k0) {
    const int base = k0 + fchunk * 16 < K ? foff + k0 : 0x40000000;
#pragma unroll
    for (int r = 0; r < LX; ++r)
      rx[r] = (v4i)__builtin_amdgcn_raw_buffer_load_b128(xres, base + FROWS * r * K, 0, 0);
  };
  auto stash = [&](int buf) {
#pragma unroll
    for (int r = 0; r < LX; ++r) *(v4i*)(sx[buf] + lds_off(frow + FROWS * r, fchunk)) = rx[r];
  };

  // waves whose channels are V produce the transposed product (tokens along MFMA rows)
  const int nw0 = n0 + wn * WTN;
  const bool vwave = mode == OUT_QKV && nw0 >= 2 * args.d;

  v16i acc[FN][FM];
#pragma unroll
  for (int i = 0; i < FN; ++i)
#pragma unroll
    for (int j = 0; j < FM; ++j) acc[i][j] = (v16i){};

  // operand fragments: lane l reads row (l % 32), 16 bytes at k = 32 ks + 16 (l / 32)
  const int frag_row = lane & 31, half = lane >> 5;
  // the K loop, instantiated once per operand order so that the order is not a
  // branch inside it
  auto kloop = [&](auto swap_tag) {
    constexpr bool SWAP = decltype(swap_tag)::value;
    const int frag0 = lds_off(wm * WTM + frag_row, half);
    v4i bf[2][FM];
    auto rd = [&](const int buf, auto ks_tag, const int to) {
      const int8_t* fp = sx[buf] + (frag0 ^ (decltype(ks_tag)::value << 5));
#pragma unroll
      for (int j = 0; j < FM; ++j) bf[to][j] = *(const v4i*)(fp + j * 32 * BK);
    };
    auto step = [&](int kt, auto ph) {
      constexpr int P2 = decltype(ph)::value;
      static_for<KSL>([&](auto ks_tag) {
        constexpr int ks = decltype(ks_tag)::value;
        if constexpr (ks == KSL - 1) {
          __syncthreads();
          rd(P2 ^ 1, std::integral_constant<int, 0>{}, (ks + 1) & 1);
        } else {
          rd(P2, std::integral_constant<int, ks + 1>{}, (ks + 1) & 1);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < FN; ++i)
#pragma unroll
          for (int j = 0; j < FM; ++j)
            acc[i][j] = SWAP ? __builtin_amdgcn_mfma_i32_32x32x32_i8(bf[ks & 1][j], wf[i][ks], acc[i][j], 0, 0, 0)
                             : __builtin_amdgcn_mfma_i32_32x32x32_i8(wf[i][ks], bf[ks & 1][j], acc[i][j], 0, 0, 0);
        wfetch(kt + 1, ks_tag);
        if constexpr (ks == 0) {
          stash(P2 ^ 1);
          fetch((kt + 2) * BK);
        }
        __builtin_amdgcn_sched_barrier(0);
      });
    };
    constexpr std::integral_constant<int, 0> P0{};
    constexpr std::integral_constant<int, 1> P1{};
    // the scheduling barriers keep the loads in the loop's own order, so that the waits at
    // the loop's head count the same outstanding loads on entry as from its end
    fetch(0);
    __builtin_amdgcn_sched_barrier(0);
    wfetch(0, P0);
    __builtin_amdgcn_sched_barrier(0);
    stash(0);
    if (tid < TN) {
      sreq[0][tid] = rq0;
      if (WIDE) sreq[1][tid] = rq1;
    }
    if (EPI == EPI_SWISH && tid < 64) stab32[tid] = swt;
    __builtin_amdgcn_sched_barrier(0);
    fetch(BK);
    __builtin_amdgcn_sched_barrier(0);
    static_for<KSL - 1>([&](auto ks) { wfetch(0, std::integral_constant<int, decltype(ks)::value + 1>{}); });
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    rd(0, P0, 0);
    int kt = 0;
    for (; kt + 2 <= nk; kt += 2) {
      step(kt, P0);
      step(kt + 1, P1);
    }
    if (kt < nk) step(kt, P0);
  };
  if (vwave) kloop(std::true_type{});
  else kloop(std::false_type{});

  // Epilogue.  Accumulator g * 4 + e of a lane sits at MFMA row g * 8 + half * 4 + e
  // and column lane % 32.  After requantization each lane holds dwords D[g] (4 rows);
  // v_permlane32_swap trades the low half's D[2], D[3] for the high half's D[0], D[1],
  // which leaves the low half with rows 0..15 and the high half with rows 16..31 of
  // its column, 16 bytes each.  A 32-channel sub-tile never straddles N, a head or the
  // Q/K/V boundary (N and d_k are multiples of 64), so its destination is uniform.
  //
  // V^T is written up to T_al, so the padded keys hold zeros (a wave's WTM tokens are
  // WTM / 64 whole 64-key blocks of V^T, two 32-token MFMA columns each).
  const int col = lane & 31;
  const int tw0 = t0 + wm * WTM;
  // the epilogue's arguments, loaded together (one wait, not one per first use)
  int8_t *o_q = args.q, *o_k = args.k, *o_vt = args.vt, *o_p = args.p, *o_y = args.y;
  const int8_t* o_z1 = args.z1;
  int o_T_al = args.T_al, o_H = args.H, o_d = args.d, o_prows = args.p_rows, o_pbase = args.p_base, dks = args.dk_shift;
  asm volatile(""
               : "+s"(o_q), "+s"(o_k), "+s"(o_vt), "+s"(o_p), "+s"(o_y), "+s"(o_z1), "+s"(o_T_al), "+s"(o_H), "+s"(o_d),
                 "+s"(o_prows), "+s"(o_pbase), "+s"(dks));
  const int DK = 1 << dks, DKm = DK - 1;
  const size_t head_bytes = (size_t)o_T_al << dks;  // one (utterance, head) block of Q, K or V^T
  // frag_index / vt_index with d_k = 2^dks
  auto frag_off = [&](int row, int kk) {
    return ((size_t)(row >> 4) << (dks + 4)) + (size_t)((kk >> 6) << 10) + (((((kk >> 4) & 3) << 4) + (row & 15)) << 4) +
           (kk & 15);
  };
  auto vt_off = [&](int t, int kk) {
    return ((size_t)(t >> 6) << (dks + 6)) + (size_t)((kk >> 4) << 10) + (((((t >> 4) & 3) << 4) + (kk & 15)) << 4) +
           (t & 15);
  };
  // the residual input of the whole sub-tile, requested at once ahead of the requantization
  // (one trip to memory instead of one per output piece)
  v4i zv[EPI == EPI_RESID ? FN : 1][EPI == EPI_RESID ? FM : 1];
  if constexpr (EPI == EPI_RESID) {
#pragma unroll
    for (int i = 0; i < FN; ++i)
#pragma unroll
      for (int j = 0; j < FM; ++j) {
        const int nb = n0 + wn * WTN + i * 32, t = tw0 + j * 32 + col;
        if (nb < N && t < rows) zv[i][j] = *(const v4i*)(o_z1 + ((size_t)ub * rows + t) * N + nb + half * 16);
      }
  }
#pragma unroll
  for (int i = 0; i < FN; ++i) {
    const int nl = wn * WTN + i * 32;  // first channel of this sub-tile, tile-local
    const int nb = n0 + nl;
    if (nb >= N) continue;
    int8_t* dst;
    int kk = 0;  // channel of the sub-tile's first row inside its head
    int hd = 0;  // its head
    if (mode == OUT_QKV) {
      const int which = (nb >= o_d) + (nb >= 2 * o_d);
      const int c = nb - which * o_d;
      hd = c >> dks;
      dst = (which == 0 ? o_q : which == 1 ? o_k : o_vt) + ((size_t)ub * o_H + hd) * head_bytes;
      kk = c & DKm;
    } else if (mode == OUT_POS) {
      hd = nb >> dks;
      dst = o_p + ((size_t)hd * o_prows << dks);
      kk = nb & DKm;
    } else {
      dst = o_y + ((size_t)ub * rows + tw0) * N + nb;  // the token offset in 64 bits: an output may pass 4 GiB
    }
    // the tile-local channel of element e: with rows as tokens (V^T) the column, else
    // row g * 8 + half * 4 + e' of element e = 4g + e'
    auto chan = [&](int e) { return vwave ? nl + col : nl + (e >> 2) * 8 + half * 4 + (e & 3); };
    // the fast form's multipliers, the same for all the sub-tile's token columns
    int mc[16];
    if (vwave) {
      const int m1 = sreq[0][nl + col];
#pragma unroll
      for (int e = 0; e < 16; ++e) mc[e] = m1;
    } else {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const v4i q = *(const v4i*)&sreq[0][nl + g * 8 + half * 4];
#pragma unroll
        for (int e = 0; e < 4; ++e) mc[4 * g + e] = q[e];
      }
    }
    // this lane's destination for token column j = 0 (relative to dst, under 2^31),
    // the first token it stores and the bound on tokens: one 32-token column further
    // is a uniform step (jstep; for V^T, 512 bytes within a 64-key block, and the
    // next block at even columns)
    int tl, tmax;
    uint32_t off0;
    if (vwave) {
      tl = tw0 + half * 16;
      tmax = o_T_al;
      off0 = (uint32_t)vt_off(tl, kk + col);
    } else {
      tl = tw0 + col;
      tmax = rows;
      off0 = mode == OUT_ROWMAJOR ? (uint32_t)(col * N + half * 16)
                                  : (uint32_t)frag_off((mode == OUT_POS ? o_pbase : 0) + tl, kk + half * 16);
    }
    const uint32_t jstep = mode == OUT_ROWMAJOR ? 32u * (uint32_t)N : 2u << (dks + 4);
#pragma unroll
    for (int j = 0; j < FM; ++j) {
      int v[16];
      if (rq_wide) {
        // a compiler barrier keeps the wide form's LDS reads here instead of letting
        // them be hoisted into live registers next to the fast form's
        asm volatile("" ::: "memory");
        requant16_wide(acc[i][j], sreq[0], sreq[1], chan, v);
      } else {
        requant16_fast(acc[i][j], mc, -rq_clamp, rq_clamp, v);
      }
      uint32_t D[4];
      pack16<EPI == EPI_SWISH>(v, D, (const uint8_t*)stab32);
      const auto x02 = __builtin_amdgcn_permlane32_swap(D[0], D[2], false, false);
      const auto x13 = __builtin_amdgcn_permlane32_swap(D[1], D[3], false, false);
      v4i out = (v4i){(int)x02[0], (int)x02[1], (int)x13[0], (int)x13[1]};

      // V^T: 16 consecutive tokens of one channel, stored up to T_al (zeros past the
      // utterance: the operand rows there read as zeros); otherwise 16 consecutive
      // channels of one token
      const uint32_t joff = vwave ? ((uint32_t)(j >> 1) << (dks + 6)) + (uint32_t)(j & 1) * 512u : (uint32_t)j * jstep;
      if (tl + j * 32 < tmax) {
        if constexpr (EPI == EPI_RESID) {
          out = WIDE && args.res_wide ? residual16_wide(out, zv[i][j], args.m_z, args.m_y, args.shift_r)
                                      : residual16(out, zv[i][j], args.m_z, args.m_y, args.shift_r);
        }
        *(v4i*)(dst + (off0 + joff)) = out;
      }
    }
  }
}

static int add_problem(GemmArgs& a, int idx, const int8_t* x, const int8_t* w, const Requant& rq, int nb,
                       int rows, int N, int K, int mode, int tile_begin, int TN, int TM) {
  GemmProblem& p = a.prob[idx];
  p.x = x;
  p.w = w;
  p.req = rq.req;
  p.wide = rq.wide;
  p.clamp = rq.clamp;
  p.rows = rows;
  p.N = N;
  p.K = K;
  p.mode = mode;
  p.tile_begin = tile_begin;
  p.grid = tile_grid(nb, rows, N, TN, TM);
  return p.grid.tiles_n * p.grid.tiles_m;
}

static void fill_dest(GemmArgs& a, const RunShape& rs, const Workspace& ws, int8_t* y) {
  a.q = ws.q;
  a.k = ws.k;
  a.vt = ws.vt;
  a.p = ws.p;
  a.z1 = nullptr;
  a.y = y;
  a.T_al = rs.T_al;
  a.H = rs.H;
  a.dk_shift = rs.DK == 128 ? 7 : 6;  // d_k is 64 or 128
  a.d = rs.d;
  a.p_rows = rs.p_rows;
  a.p_base = rs.p_base;
}

template <int TN, int TM, int NWAVE, int WN, int EPI>
static hipError_t launch_gemm(GemmArgs& a, int tiles, hipStream_t st, const LaunchEv& ev) {
  a.tiles_total = tiles;
  a.per_xcd = (tiles + 7) / 8;
  const bool wide = a.prob[0].wide || (a.nprob > 1 && a.prob[1].wide) || (EPI == EPI_RESID && a.res_wide);
  return wide ? launch_kernel(gemm_i8_requant<TN, TM, NWAVE, WN, EPI, true>, dim3(8 * a.per_xcd), dim3(64 * NWAVE), 0,
                              st, ev, a)
              : launch_kernel(gemm_i8_requant<TN, TM, NWAVE, WN, EPI, false>, dim3(8 * a.per_xcd), dim3(64 * NWAVE), 0,
                              st, ev, a);
}

template <int I, int EPI>
static hipError_t launch_shape(GemmArgs& a, int tiles, hipStream_t st, const LaunchEv& ev) {
  return launch_gemm<kTiles[I].tn, kTiles[I].tm, kTiles[I].tm == 256 ? 8 : 4, kTiles[I].tn == 64 ? 2 : 4, EPI>(a, tiles, st,
                                                                                                               ev);
}

// Launches the products of `dims` (all of contraction length K) with the shape that
// pick_shape takes; fill(args, tn, tm) adds them and returns their tiles.  min_tm: 64 where V^T
// is written (whole 64-key blocks).
template <int EPI, typename Fill>
static hipError_t launch_best(const GemmDims* dims, int n, int K, int min_tm, Fill fill, hipStream_t st,
                              const LaunchEv& ev) {
  const int best = pick_shape(dims, n, K, min_tm, EPI);
  GemmArgs a{};
  const int tiles = fill(a, kTiles[best].tn, kTiles[best].tm);
  switch (best) {
    case 0: return launch_shape<0, EPI>(a, tiles, st, ev);
    case 1: return launch_shape<1, EPI>(a, tiles, st, ev);
    case 2: return launch_shape<2, EPI>(a, tiles, st, ev);
    case 3: return launch_shape<3, EPI>(a, tiles, st, ev);
    case 4: return launch_shape<4, EPI>(a, tiles, st, ev);
    default: return launch_shape<5, EPI>(a, tiles, st, ev);
  }
}

hipError_t launch_projections(const RunShape& rs, const Weights& w, const Workspace& ws, const int8_t* x,
                              const int8_t* pos_table, hipStream_t st, const LaunchEv& ev) {
  const GemmDims dims[2] = {{rs.B, rs.T, 3 * rs.d}, {1, 2 * rs.T - 1, rs.d}};
  auto fill = [&](GemmArgs& a, int tn, int tm) {
    fill_dest(a, rs, ws, nullptr);
    int tiles = add_problem(a, 0, x, w.w_qkv, w.rq_qkv, rs.B, rs.T, 3 * rs.d, rs.d, OUT_QKV, 0, tn, tm);
    a.nprob = 1;
    if (pos_table) {
      tiles += add_problem(a, 1, pos_table, w.w_pos, w.rq_pos, 1, 2 * rs.T - 1, rs.d, rs.d, OUT_POS, tiles, tn, tm);
      a.nprob = 2;
    }
    return tiles;
  };
  return launch_best<EPI_PLAIN>(dims, pos_table ? 2 : 1, rs.d, KCHUNK, fill, st, ev);
}

hipError_t launch_pos_projection(const RunShape& rs, const Weights& w, int8_t* p, const int8_t* pos_table,
                                 hipStream_t st) {
  Workspace ws{};
  ws.p = p;
  const int rows = 2 * rs.T - 1;
  const GemmDims dims{1, rows, rs.d};
  auto fill = [&](GemmArgs& a, int tn, int tm) {
    fill_dest(a, rs, ws, nullptr);
    a.nprob = 1;
    return add_problem(a, 0, pos_table, w.w_pos, w.rq_pos, 1, rows, rs.d, rs.d, OUT_POS, 0, tn, tm);
  };
  return launch_best<EPI_PLAIN>(&dims, 1, rs.d, 32, fill, st, LaunchEv{});
}

// A row-major product of `rows` tokens (K -> N), `setup` filling the epilogue's arguments.
template <int EPI, typename Setup>
static hipError_t launch_rowmajor(const int8_t* x, int rows, int N, int K, const int8_t* w, const Requant& rq,
                                  int8_t* y, Setup setup, hipStream_t st, const LaunchEv& ev) {
  const GemmDims dims{1, rows, N};
  auto fill = [&](GemmArgs& a, int tn, int tm) {
    a.y = y;
    a.nprob = 1;
    setup(a);
    return add_problem(a, 0, x, w, rq, 1, rows, N, K, OUT_ROWMAJOR, 0, tn, tm);
  };
  return launch_best<EPI>(&dims, 1, K, 32, fill, st, ev);
}

static void set_residual(GemmArgs& a, const int8_t* z, int m_z, int m_y, int shift_r) {
  a.z1 = z;
  a.m_z = m_z;
  a.m_y = m_y;
  a.shift_r = shift_r;
  a.res_wide = shift_r > 31 || ((int64_t)m_z + m_y) * 128 + ((int64_t)1 << (shift_r - 1)) >= ((int64_t)1 << 31);
}

hipError_t launch_out_projection(const RunShape& rs, const Weights& w, const Workspace& ws, int8_t* y,
                                 hipStream_t st, const LaunchEv& ev, const Residual* res, const int8_t* z1) {
  // the utterances' rows are contiguous on both sides, so tiles may straddle them
  const int rows = rs.B * rs.T;
  if (res)
    return launch_rowmajor<EPI_RESID>(
        ws.ctx, rows, rs.d, rs.d, w.w_out, w.rq_out, y,
        [&](GemmArgs& a) { set_residual(a, z1, res->m_z, res->m_y, res->shift_r); }, st, ev);
  return launch_rowmajor<EPI_PLAIN>(ws.ctx, rows, rs.d, rs.d, w.w_out, w.rq_out, y, [](GemmArgs&) {}, st, ev);
}

// ---------------------------------------------------------------------------
// The feed-forward module of Eq. 1: W1 with the integer Swish in its epilogue, W2
// with the residual add in its epilogue.

// The integer Swish of Eq. 12 and its requantization to FFN2's input grid, for every
// int8 input h (one thread per biased code h + 128; code 0 is never looked up):
//   L = (min(|h|, q_c) - q_c)^2 + q_1,  q = -(|h| L + h q_1),  o = clamp8(RS(q, m, n)).
// The host checks that |q m| + 2^(n-1) stays below 2^62 for every h.
__global__ __launch_bounds__(256) void swish_table(uint8_t* tab, long long q_c, long long q_1, long long m,
                                                   int shift) {
  const long long h = (long long)threadIdx.x - 128;
  const long long ah = h < 0 ? -h : h;
  const long long t = (ah < q_c ? ah : q_c) - q_c;
  const long long L = t * t + q_1;
  const long long q = -(ah * L + h * q_1);
  const long long o = (q * m + (1ll << (shift - 1))) >> shift;
  tab[threadIdx.x] = (uint8_t)(int)(o < -127 ? -127 : (o > 127 ? 127 : o));
}

hipError_t launch_swish_table(uint8_t* tab, long long q_c, long long q_1, long long m, int shift, hipStream_t st) {
  hipLaunchKernelGGL(swish_table, dim3(1), dim3(256), 0, st, tab, q_c, q_1, m, shift);
  return hipGetLastError();
}

hipError_t launch_ffn_up(const int8_t* x, int rows, int d, int d_ff, const int8_t* w1, const Requant& rq1,
                         const uint8_t* swtab, int8_t* o, hipStream_t st) {
  return launch_rowmajor<EPI_SWISH>(x, rows, d_ff, d, w1, rq1, o, [&](GemmArgs& a) { a.swtab = swtab; }, st,
                                    LaunchEv{});
}

hipError_t launch_linear_resid(const int8_t* x, int rows, int N, int K, const int8_t* w, const Requant& rq,
                               const int8_t* z, int m_z, int m_y, int shift_r, int8_t* z_out, hipStream_t st) {
  return launch_rowmajor<EPI_RESID>(x, rows, N, K, w, rq, z_out,
                                    [&](GemmArgs& a) { set_residual(a, z, m_z, m_y, shift_r); }, st, LaunchEv{});
}

hipError_t launch_linear(const int8_t* x, int rows, int K, int N, const int8_t* w, const Requant& rq, int8_t* y,
                         hipStream_t st) {
  return launch_rowmajor<EPI_PLAIN>(x, rows, N, K, w, rq, y, [](GemmArgs&) {}, st, LaunchEv{});
}

// one thread per 16-byte piece of the destination
__global__ __launch_bounds__(256) void pack_wfrag(const int8_t* __restrict__ w, int8_t* __restrict__ dst, int N,
                                                  int K, DivU dv_ksl) {
  const long p = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= (long)N * K / 16) return;
  const int l = (int)(p & 63);
  const int frag = (int)(p >> 6);
  const int cb = (int)div_u((uint32_t)frag, dv_ksl), ks = frag - cb * (int)dv_ksl.d;
  const int8_t* src = w + (size_t)(cb * 32 + (l & 31)) * K + ks * 32 + (l >> 5) * 16;
  *(uint4*)(dst + p * 16) = *(const uint4*)src;
}

hipError_t pack_weight_fragments(const int8_t* w, int8_t* dst, int N, int K, hipStream_t st) {
  if (N % 32 || K % 32) return hipErrorInvalidValue;
  const long pieces = (long)N * K / 16;
  hipLaunchKernelGGL(pack_wfrag, dim3((unsigned)((pieces + 255) / 256)), dim3(256), 0, st, w, dst, N, K,
                     make_div((uint32_t)(K >> 5)));
  return hipGetLastError();
}

}  // namespace ipk
